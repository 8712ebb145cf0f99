// Pinned staging of a plan's per-step tables: up to eight slots, used in turn, that upload kernels read
// in place.  Each kernel writes its slot's sequence number to the slot's words once it has read it, so
// reuse waits for exactly the upload that used the slot, whatever streams the calls name, and the
// stream carries no event for it.  Eight slots let the host issue that many steps ahead of the GPU;
// tables over 1 MB get two.
//
// The runtime's calls come through RT, so that the protocol runs without a GPU too:
//   Stream, Error, kOk     the runtime's types and its success code
//   alloc(&p, bytes)       pinned memory that every device can read and write; free(p)
//   device_of(stream)      the device of a stream
//   failed(stream)         kOk unless the stream's device has failed; never waits
//   drain(device)          waits for everything queued on a device
//   patience()             how long a wait polls before it asks one of the two above
#pragma once

#include <stdint.h>

#include <algorithm>
#include <chrono>
#include <cstddef>
#include <cstring>
#include <thread>

namespace smat {

// What an upload kernel writes once it has read its staging: block b stores seq to done[b] (pinned host
// memory).
struct UploadSignal {
  uint32_t* done;
  uint32_t seq;
};
// Blocks of an upload of n items (16 blocks of 256 threads saturate the host link with 8-byte loads).
constexpr uint32_t kUploadBlocks = 16;
inline uint32_t upload_blocks(uint64_t n) {
  return (uint32_t)(n >= kUploadBlocks * 256u ? kUploadBlocks : n ? (n + 255) / 256 : 1);
}

template <typename RT>
struct StagingOf {
  using Error = typename RT::Error;
  using Stream = typename RT::Stream;
  static constexpr uint32_t kMaxSlots = 8;
  char* mem = nullptr;
  size_t slot_bytes = 0;
  uint32_t slots = 0, next = 0;
  uint32_t seq[kMaxSlots] = {}, blocks[kMaxSlots] = {};
  int device[kMaxSlots] = {};

  Error init(size_t bytes) {
    if (mem) return RT::kOk;
    slot_bytes = (std::max<size_t>(bytes, 256) + 255) & ~size_t(255);
    slots = slot_bytes <= (size_t(1) << 20) ? kMaxSlots : 2;
    const size_t words = slots * kUploadBlocks * sizeof(uint32_t);
    char* p = nullptr;
    const Error e = RT::alloc((void**)&p, slots * slot_bytes + words);
    if (e != RT::kOk) return e;
    std::memset(p + slots * slot_bytes, 0, words);
    mem = p;
    return RT::kOk;
  }
  char* data() const { return mem + next * slot_bytes; }
  uint32_t* words(uint32_t slot) const {
    return reinterpret_cast<uint32_t*>(mem + slots * slot_bytes) + slot * kUploadBlocks;
  }
  // Whether the slot's last upload has read it.
  bool read(uint32_t slot) const {
    for (uint32_t b = 0; b < blocks[slot]; ++b)
      if (__atomic_load_n(words(slot) + b, __ATOMIC_ACQUIRE) != seq[slot]) return false;
    return true;
  }
  // The next slot, free to be written, for an upload on `stream`: fill data(), launch the upload with
  // signal(), then sent().  The wait is for the slot alone; one that lasts asks now and then whether the
  // device has failed, and returns its error, so that it ends there too.
  Error take(Stream stream) const {
    while (!poll(next))
      if (const Error e = RT::failed(stream); e != RT::kOk) return e;
    return RT::kOk;
  }
  UploadSignal signal() const { return {words(next), seq[next] + 1}; }
  void sent(uint32_t used_blocks, Stream stream) {
    ++seq[next];
    blocks[next] = used_blocks;
    device[next] = RT::device_of(stream);
    next = (next + 1) % slots;
  }
  // Waits for the uploads, then frees the memory.  Where a slot stays unread on a device that cannot be
  // drained, nothing tells whether a kernel still reads it: the memory is left to the process's end.
  void release() {
    if (!mem) return;
    bool all = true;
    for (uint32_t k = 0; k < slots; ++k)
      if (!poll(k)) all = RT::drain(device[k]) == RT::kOk && read(k) && all;
    if (all) RT::free(mem);
    mem = nullptr;
  }

 private:
  // read(slot), waited for up to the runtime's patience.
  bool poll(uint32_t slot) const {
    using clock = std::chrono::steady_clock;
    const auto until = clock::now() + RT::patience();
    for (uint32_t k = 1; !read(slot); ++k) {
      if (k % 1024) continue;
      std::this_thread::yield();
      if (clock::now() >= until) return read(slot);
    }
    return true;
  }
};

}  // namespace smat
