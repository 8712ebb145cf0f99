// Host-side launchers of the SMAT kernels (internal to libsmat).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "smat_device.h"
#include "smat_staging.h"

namespace smat {

// ---------------------------------------------------------------- resident blocks
// HBM streams fastest when the loads in flight on a compute unit hold about 50 KB: with less the
// memory system idles between requests, with more the waves of many tiles compete for open DRAM rows.
// A CU holds up to 32 one-wave blocks, so a kernel whose waves load much each passes that mark; it
// reserves LDS it never touches, which bounds the blocks that are resident together (LDS is granted
// in 1,280-byte granules out of 160 KB).  Arrays of a few times the 256 MB Infinity Cache and less are
// partly served from there, where more requests only help: the fused optimizer step of 9.6e6
// parameters (251 MB) took 53.4 us capped and 52.4 us uncapped, of 31.5e6 (820 MB) 147.1 and 148.8 us.
// So a launch is capped from 512 MB up.
constexpr uint32_t kLdsBytes = 160u * 1024u, kLdsGranule = 1280u, kBytesInFlight = 50u * 1024u;
constexpr uint64_t kCapFromBytes = 512ull << 20;
constexpr uint32_t lds_for_blocks(uint32_t blocks) {
  return blocks >= 32u ? 0u : kLdsBytes / blocks / kLdsGranule * kLdsGranule;
}
// LDS to reserve per block of a kernel whose one-wave blocks each keep wave_bytes of loads in flight
// and whose launch streams `bytes` in all.
constexpr uint32_t lds_for_loads(uint32_t wave_bytes, uint64_t bytes) {
  return bytes < kCapFromBytes ? 0u : lds_for_blocks(kBytesInFlight / wave_bytes);
}

// fn(first, count) over consecutive pieces [first, first + count) of `total` units, count <= per,
// stopping at the first launch error.
template <typename F>
hipError_t for_pieces(uint64_t total, uint64_t per, F&& fn) {
  for (uint64_t first = 0; first < total; first += per) {
    fn(first, total - first < per ? total - first : per);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

// fn called with the storage type of a dtype code (0 = fp32, 1 = bf16) or with a flag, as a type.
template <typename T>
struct TypeTag {
  using type = T;
};
template <typename F>
void with_type(int dtype, F&& fn) {
  if (dtype == 1)
    fn(TypeTag<Bf16>());
  else
    fn(TypeTag<float>());
}
template <typename F>
void with_flag(bool flag, F&& fn) {
  if (flag)
    fn(std::true_type());
  else
    fn(std::false_type());
}

// fn(entries, chunks, grid, order, first segment) for the launches of a list's table with tiles of Q
// quads (table_pieces), stopping at the first launch error.
template <int Q, typename F>
hipError_t for_table(const ChunkTable& t, bool runs, F&& fn) {
  hipError_t e = hipSuccess;
  table_pieces(t.chunks, t.segments, Q, runs, max_grid_blocks(kBlock), [&](const TablePiece& p) {
    const uint2* entries = t.entries + p.entry;
    if (p.order == kMixed)
      fn(entries, p.chunks, dim3(p.blocks), std::integral_constant<int, kMixed>(), p.segment);
    else if (p.order == kRuns)
      fn(entries, p.chunks, dim3(p.blocks), std::integral_constant<int, kRuns>(), p.segment);
    else
      fn(entries, p.chunks, dim3(p.blocks), std::integral_constant<int, kLinear>(), p.segment);
    return (e = hipGetLastError()) == hipSuccess;
  });
  return e != hipSuccess ? e : hipGetLastError();
}
// Segments, and elements up to the padding of tensors' ends, that a table covers.
inline uint64_t table_segments(const ChunkTable& t) { return (uint64_t)t.chunks * kChunkSegments + t.segments; }
inline uint64_t table_elems(const ChunkTable& t) { return table_segments(t) * (uint64_t)kSegment; }

// Whether an array's tiles begin inside a 128-byte line (its address as device_rec gives it; tiles are
// multiples of 512 bytes).
inline bool off_line(const void* p) { return reinterpret_cast<uintptr_t>(p) % 128 != 0; }

// Storage bytes of a dtype code (0 = fp32, 1 = bf16).
inline size_t storage_bytes(int dtype) { return dtype == 1 ? 2 : 4; }

// p advanced by `elems` elements of `bytes` each (a null pointer stays null).
template <typename P>
inline P* step_ptr(P* p, uint64_t elems, size_t bytes) {
  return p ? reinterpret_cast<P*>(reinterpret_cast<uintptr_t>(p) + elems * bytes) : p;
}

// p moved back by `elems` elements of `bytes` each (a null pointer stays null).
template <typename P>
inline P* back_ptr(P* p, uint64_t elems, size_t bytes) {
  return p ? reinterpret_cast<P*>(reinterpret_cast<uintptr_t>(p) - elems * bytes) : p;
}

// Elements before a tensor's first one in its first Philox group.
inline uint32_t group_head(uint64_t elem_offset) { return (uint32_t)elem_offset & 3u; }

// A tensor's record as the kernels read it: from the start of its first Philox group, with the head and
// the sector bits in sflags (see TensorRec::sflags in smat_device.h).
inline TensorRec device_rec(const TensorRec& R, int t0_dtype, int out_dtype, int g_dtype) {
  const uint32_t head = R.n > 0 ? group_head(R.elem_offset) : 0u;
  TensorRec r = R;
  r.theta = back_ptr(R.theta, head, 4);
  r.theta0 = back_ptr(R.theta0, head, storage_bytes(t0_dtype));
  r.out = back_ptr(R.out, head, storage_bytes(out_dtype));
  r.grad_sim = back_ptr(R.grad_sim, head, storage_bytes(g_dtype));
  r.grad_theta = back_ptr(R.grad_theta, head, 4);
  r.n = R.n + head;
  r.elem_offset = R.elem_offset - head;
  r.sflags = R.sflags | (head << kHeadShift) | (reinterpret_cast<uintptr_t>(r.theta) % 64 ? 0u : kSectorSim) |
             (reinterpret_cast<uintptr_t>(r.grad_theta) % 64 ? 0u : kSectorBwd);
  if ((R.sflags & kVecBwd) && R.n % 4 == 0 && R.elem_offset % (uint64_t)kSegment == 0) r.sflags |= kBwdWhole;
  return r;
}
inline AdamRec device_adam(const AdamRec& A, const TensorRec& R) {
  const uint32_t head = R.n > 0 ? group_head(R.elem_offset) : 0u;
  return AdamRec{back_ptr(A.exp_avg, head, 4), back_ptr(A.exp_avg_sq, head, 4)};
}

// Elements [off, off + len) of a one-tensor record (as device_rec gives it) as a record of its own.  off
// is a multiple of the tile, hence of 4 elements, so every pointer keeps its alignment, the flags still
// hold and only the first piece has the head.
inline TensorRec rec_piece(const TensorRec& R, uint64_t off, uint64_t len, int t0_dtype, int out_dtype,
                           int g_dtype) {
  TensorRec r = R;
  r.theta = step_ptr(R.theta, off, 4);
  r.theta0 = step_ptr(R.theta0, off, storage_bytes(t0_dtype));
  r.out = step_ptr(R.out, off, storage_bytes(out_dtype));
  r.grad_sim = step_ptr(R.grad_sim, off, storage_bytes(g_dtype));
  r.grad_theta = step_ptr(R.grad_theta, off, 4);
  r.n = (int64_t)len;
  r.elem_offset = R.elem_offset + off;
  if (off) r.sflags &= (1u << kHeadShift) - 1u;
  return r;
}

// Storage codes match smat_dtype: 0 = fp32, 1 = bf16.  `runs`: the block order of tiles that begin inside
// a line (block_order in smat_tile.h).
hipError_t launch_simulate_one(const TensorRec& rec, const ParamRec& prm, int theta0_dtype, int out_dtype,
                               uint64_t seed, uint32_t step, bool runs, hipStream_t stream);
hipError_t launch_backward_one(const TensorRec& rec, const ParamRec& prm, int grad_dtype, float lambda,
                               uint64_t seed, uint32_t step, bool runs, hipStream_t stream);
hipError_t launch_simulate_multi(const TensorRec* recs, const ParamRec* prms, const ChunkTable& table,
                                 int theta0_dtype, int out_dtype, uint64_t seed, uint32_t step, bool runs,
                                 hipStream_t stream);
hipError_t launch_backward_multi(const TensorRec* recs, const ParamRec* prms, const ChunkTable& table,
                                 int grad_dtype, bool accumulate, float lambda, uint64_t seed, uint32_t step,
                                 bool runs, hipStream_t stream);
// Graph-capturable forms: seed, step and scale read from `state` in device memory, each tensor's
// coefficient formed from the scale and its ScaleRec.
hipError_t launch_simulate_multi_dev(const TensorRec* recs, const ParamRec* prms, const ScaleRec* scales,
                                     const ChunkTable& table, int theta0_dtype, int out_dtype,
                                     const StepState* state, bool runs, hipStream_t stream);
hipError_t launch_backward_multi_dev(const TensorRec* recs, const ParamRec* prms, const ScaleRec* scales,
                                     const ChunkTable& table, int grad_dtype, bool accumulate,
                                     float lambda, const StepState* state, bool runs, hipStream_t stream);
// step += increment and the scale of that step, in place (one thread).
hipError_t launch_step_advance(StepState* state, uint32_t increment, float alpha_min, hipStream_t stream);
hipError_t launch_adamw_one(const TensorRec& rec, const AdamRec& st, const ParamRec& prm, const AdamConsts& A,
                            int grad_dtype, bool accumulate, float lambda, uint64_t seed, uint32_t step,
                            const float* dev_scale, bool runs, hipStream_t stream);
hipError_t launch_adamw_multi(const TensorRec* recs, const AdamRec* states, const ParamRec* prms,
                              const ChunkTable& table, const AdamConsts& A, int grad_dtype, bool accumulate,
                              float lambda, uint64_t seed, uint32_t step, const float* dev_scale, bool runs,
                              hipStream_t stream);
// Squared norm of the simulated step's expert gradient over the list: one fp32 partial per
// one-wave block of kNormQuads quads per thread (one segment), their fp64 block
// sums (at most kNormSums doubles), then sumsq and/or the clipping factor.
constexpr int kNormQuads = 8;
static_assert(tile_elems(kNormQuads) == kSegment, "one norm partial per segment");
constexpr uint32_t kNormSums = 256;
hipError_t launch_sqnorm_multi(const TensorRec* recs, const ParamRec* prms, const ChunkTable& table,
                               float* partials, double* sums, int grad_dtype, bool accumulate, float lambda,
                               uint64_t seed, uint32_t step, double* sumsq, float* clip_coef, float max_norm,
                               hipStream_t stream);
// Graph-capturable forms of the list optimizer step and gradient norm: seed, step and scale from
// `state`; the optimizer's learning rate and step count from `adam_state`, turned into the step's
// constants in `consts` (device memory of the plan) by a one-thread launch ahead of the update.
hipError_t launch_sqnorm_multi_dev(const TensorRec* recs, const ParamRec* prms, const ScaleRec* scales,
                                   const ChunkTable& table, float* partials, double* sums,
                                   int grad_dtype, bool accumulate, float lambda, const StepState* state,
                                   double* sumsq, float* clip_coef, float max_norm, hipStream_t stream);
hipError_t launch_adamw_multi_dev(const TensorRec* recs, const AdamRec* states, const ParamRec* prms,
                                  const ScaleRec* scales, const ChunkTable& table, const AdamHyper& h,
                                  const AdamStepState* adam_state, AdamConsts* consts, int grad_dtype,
                                  bool accumulate, float lambda, const StepState* state, const float* dev_scale,
                                  bool runs, hipStream_t stream);
// ---------------------------------------------------------------- table uploads
// Per-step tables from pinned host memory (`staged`, device-accessible) into a workspace; bytes is a
// multiple of 8.
hipError_t launch_upload(const void* staged, void* dst, size_t bytes, UploadSignal sig, hipStream_t stream);

// ---------------------------------------------------------------- N-expert merge
// One expert's term on one tensor: its mask key (seed, step), threshold and coefficient
// t = gamma/keep (rescaled) or gamma, and kFlagMask / kFlagDropAll, plus the ten Philox round keys of
// the seed, formed once per term so that no wave adds them up again for every expert.
struct alignas(8) MergeRec {
  uint64_t seed;
  uint32_t step;
  uint32_t thr;
  float t;
  uint32_t flags;
  uint32_t rk0[10];
  uint32_t rk1[10];
};
static_assert(sizeof(MergeRec) == 104, "MergeRec layout");
// A term without its round keys: what the host hands to launch_upload_terms.
struct alignas(8) MergeTerm {
  uint64_t seed;
  uint32_t step;
  uint32_t thr;
  float t;
  uint32_t flags;
};
static_assert(sizeof(MergeTerm) == 24, "MergeTerm layout");
__host__ __device__ inline MergeRec merge_rec(const MergeTerm& m) {
  const PhiloxKeys K = philox_keys(m.seed);
  MergeRec r{m.seed, m.step, m.thr, m.t, m.flags, {}, {}};
#pragma unroll
  for (int k = 0; k < 10; ++k) {
    r.rk0[k] = K.k0[k];
    r.rk1[k] = K.k1[k];
  }
  return r;
}
// dst[i] = merge_rec(staged[i]) for `cells` terms in pinned host memory.
hipError_t launch_upload_terms(const MergeTerm* staged, MergeRec* dst, uint64_t cells, UploadSignal sig,
                               hipStream_t stream);
constexpr int kMaxExperts = 16;
constexpr uint32_t kVecMerge = 16u;  // TensorRec::sflags: theta0, out and every expert aligned to their elements
// Arguments of the one-tensor merge, passed by value (no device tables).
struct MergeArgs {
  const void* x[kMaxExperts];
  MergeRec r[kMaxExperts];
};
// `plain`: no term draws a mask or leaves its expert out.
hipError_t launch_merge_one(const TensorRec& rec, const MergeArgs& args, int nexp, int expert_dtype, int theta0_dtype,
                            int out_dtype, bool plain, bool runs, hipStream_t stream);
hipError_t launch_merge_multi(const TensorRec* recs, const void* const* experts, const MergeRec* terms,
                              const ChunkTable& table, int nexp, int expert_dtype, int theta0_dtype,
                              int out_dtype, bool plain, bool runs, hipStream_t stream);

// Plain streaming copy of n16 16-byte vectors (the measured HBM reference).
constexpr int kCopyVecs = 1;  // 16-byte vectors per thread of the reference copy
hipError_t launch_stream_copy(const void* src, void* dst, uint64_t n16, hipStream_t stream);

hipError_t launch_debug_draws(uint64_t seed, uint32_t step, uint32_t tensor_id, uint64_t elem_offset,
                              int64_t n, const ParamRec& prm, uint32_t* mask_words, uint32_t* noise_words,
                              uint8_t* kept, float* z, hipStream_t stream);

}  // namespace smat
