// The staging of per-step tables (smat_staging.h) against a runtime that this program plays itself: the
// "kernels" are the places below that write a slot's words.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <thread>
#include <vector>

#include "smat_staging.h"

#define EXPECT(cond)                                               \
  do {                                                             \
    if (!(cond)) {                                                 \
      std::printf("FAIL line %d: %s\n", __LINE__, #cond);          \
      std::exit(1);                                                \
    }                                                              \
  } while (0)

struct Fake {
  using Error = int;
  using Stream = int;
  static constexpr Error kOk = 0;
  static inline int queries = 0, query_error = 0, queried = -1, frees = 0, drain_error = 0;
  static inline std::atomic<int> answer_after{-1};  // queries until `finish` runs
  static inline void (*finish)() = nullptr;
  static inline std::vector<int> drains;
  static Error alloc(void** p, size_t bytes) {
    *p = std::aligned_alloc(256, (bytes + 255) / 256 * 256);
    return kOk;
  }
  static void free(void* p) {
    ++frees;
    std::free(p);
  }
  static int device_of(Stream s) { return s / 10; }
  static Error failed(Stream s) {
    ++queries;
    queried = s;
    if (finish && queries == answer_after) finish();
    return query_error;
  }
  static Error drain(int device) {
    drains.push_back(device);
    if (finish) finish();
    return drain_error;
  }
  static std::chrono::microseconds patience() { return std::chrono::microseconds(200); }
  static void reset() {
    queries = query_error = frees = drain_error = 0;
    queried = answer_after = -1;
    finish = nullptr;
    drains.clear();
  }
};
using Staging = smat::StagingOf<Fake>;

// what the upload kernel of `sig` does once it has read its part: block b of `blocks`
static void signal_block(smat::UploadSignal sig, uint32_t b) { __atomic_store_n(sig.done + b, sig.seq, __ATOMIC_RELEASE); }

static smat::UploadSignal g_sig;

int main() {
  // slots: eight up to 1 MB, two above; the words lie behind the slots and differ between slots
  for (size_t bytes : {size_t(0), size_t(1), size_t(1) << 20, (size_t(1) << 20) + 1}) {
    Staging st;
    EXPECT(st.init(bytes) == 0 && st.init(bytes) == 0);
    const uint32_t slots = bytes <= (size_t(1) << 20) ? 8 : 2;
    EXPECT(st.slots == slots && st.slot_bytes >= bytes && st.slot_bytes % 256 == 0);
    std::vector<smat::UploadSignal> sent;
    std::vector<char*> place;
    for (uint32_t k = 0; k < slots; ++k) {
      EXPECT(st.take(10) == 0 && Fake::queries == 0);  // a fresh slot is never waited for
      sent.push_back(st.signal());
      place.push_back(st.data());
      st.sent(smat::kUploadBlocks, 10);
    }
    for (uint32_t k = 0; k < slots; ++k) {
      EXPECT(sent[k].seq == 1 && place[k] == place[0] + k * st.slot_bytes);
      EXPECT(reinterpret_cast<char*>(sent[k].done) == place[0] + slots * st.slot_bytes + k * smat::kUploadBlocks * 4);
    }
    // three more turns: each slot is free only once all blocks of its own upload have signalled, in
    // whatever order, and other slots' uploads don't matter
    for (uint32_t turn = 0; turn < 3; ++turn)
      for (uint32_t k = 0; k < slots; ++k) {
        EXPECT(st.next == k && !st.read(k));
        for (uint32_t b = smat::kUploadBlocks; b-- > 0;) {
          EXPECT(!st.read(k));
          signal_block(sent[k], b);
        }
        EXPECT(st.read(k) && st.take(10) == 0 && Fake::queries == 0);
        EXPECT(slots == 2 || !st.read((k + 1) % slots));
        sent[k] = st.signal();
        EXPECT(sent[k].seq == turn + 2);
        st.sent(smat::kUploadBlocks, 10);
      }
    for (auto& s : sent)
      for (uint32_t b = 0; b < smat::kUploadBlocks; ++b) signal_block(s, b);
    st.release();
    EXPECT(Fake::frees == 1 && Fake::drains.empty() && st.mem == nullptr);
    st.release();
    EXPECT(Fake::frees == 1);
    Fake::reset();
  }

  // an upload of fewer blocks than the slot's last one waits for those alone
  {
    Staging st;
    st.init(256);
    for (uint32_t k = 0; k < 8; ++k) {
      const smat::UploadSignal s = st.signal();
      st.sent(3, 10);
      for (uint32_t b = 0; b < 3; ++b) signal_block(s, b);
    }
    EXPECT(st.take(10) == 0);
    const smat::UploadSignal s = st.signal();
    st.sent(1, 10);
    signal_block(s, 0);
    EXPECT(st.read(0));
    st.release();
    Fake::reset();
  }

  // a full turn with the first upload still unread: take() waits for it, another thread's "kernel" ends the wait
  {
    Staging st;
    st.init(256);
    std::vector<smat::UploadSignal> sent;
    for (uint32_t k = 0; k < 8; ++k) {
      EXPECT(st.take(10) == 0);
      sent.push_back(st.signal());
      st.sent(1, 10);
    }
    std::atomic<bool> signalled{false};
    std::thread kernel([&] {
      std::this_thread::sleep_for(std::chrono::milliseconds(30));
      signalled = true;
      signal_block(sent[0], 0);
    });
    EXPECT(st.take(20) == 0 && signalled);
    kernel.join();
    // it asked about the calling stream meanwhile, which waits for nothing, and drained no device
    EXPECT(Fake::queries > 1 && Fake::queried == 20 && Fake::drains.empty());

    // a device that has failed ends the wait with its error, at the first question
    Fake::reset();
    st.sent(1, 20);
    Fake::query_error = 700;
    EXPECT(st.take(20) == 700 && Fake::queries == 1 && Fake::drains.empty());
    EXPECT(st.next == 1 && !st.read(1));  // nothing was taken
    Fake::query_error = 0;
    signal_block(sent[1], 0);
    EXPECT(st.take(20) == 0);

    // release: an unread slot's own device is drained (20 / 10), and then it is read
    Fake::reset();
    for (uint32_t k = 2; k < 8; ++k) signal_block(sent[k], 0);
    g_sig = {st.words(0), st.seq[0]};
    Fake::finish = [] { signal_block(g_sig, 0); };
    st.release();
    EXPECT(Fake::drains.size() == 1 && Fake::drains[0] == 2 && Fake::frees == 1 && Fake::queries == 0);
    Fake::reset();
  }

  // release on a device that cannot be drained ends, and leaves the memory that a kernel may still read
  for (int error : {700, 0}) {
    Staging st;
    st.init(256);
    st.sent(1, 30);
    Fake::drain_error = error;
    char* mem = st.mem;
    st.release();
    EXPECT(Fake::drains.size() == 1 && Fake::drains[0] == 3 && Fake::frees == 0 && st.mem == nullptr);
    std::free(mem);
    Fake::reset();
  }
  std::printf("ok\n");
  return 0;
}
