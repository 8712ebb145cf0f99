// A plain streaming copy for gfx950, built like the library's kernels (one-wave blocks, 16-byte
// nontemporal loads and stores, consecutive blocks on consecutive spans): the achievable HBM
// stream rate that the benchmark states its kernels against.  It computes nothing of the method.
// One vector per thread: measured on MI355X over 60-135 GB, it streams 7-10 % faster than two or
// four vectors per thread (fewer bytes in flight per wave keep more DRAM rows open to reuse).
//
// Also here: the upload of a plan's small per-step tables by a kernel that reads the pinned staging over
// the host link and says itself when it has.  A copy command costs the stream a switch to the copy
// engine and back, and an event after it a gap of 5 us before the next kernel: 46 KB of parameters (1,454
// tensors) kept the GPU idle for 43 us of a 956 us step, 118 KB of merge terms for 41 us, and a few KB
// through the runtime's copy kernel for 10 us.  The kernel takes 3-5 us in line with the others.
#include "smat_launch.h"

namespace smat {

// The staging is written by the host between launches: system-scope loads read it past the caches.
constexpr int kUploadBlock = 256;
__device__ __forceinline__ uint64_t load_host(const uint64_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The block has read its part of the staging: every wave's stores, which carry the loaded values, are
// issued before the barrier, so the staging is free once the word is written.
__device__ __forceinline__ void signal_read(UploadSignal sig) {
  __syncthreads();
  if (threadIdx.x == 0)
    __hip_atomic_store(sig.done + blockIdx.x, sig.seq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__global__ __launch_bounds__(kUploadBlock) void k_upload(const uint64_t* __restrict__ staged,
                                                         uint64_t* __restrict__ dst, uint64_t n8, UploadSignal sig) {
#pragma unroll 4
  for (uint64_t i = (uint64_t)blockIdx.x * kUploadBlock + threadIdx.x; i < n8; i += (uint64_t)gridDim.x * kUploadBlock)
    dst[i] = load_host(staged + i);
  signal_read(sig);
}

hipError_t launch_upload(const void* staged, void* dst, size_t bytes, UploadSignal sig, hipStream_t stream) {
  const uint64_t n8 = bytes / 8;
  k_upload<<<dim3(upload_blocks(n8)), dim3(kUploadBlock), 0, stream>>>(static_cast<const uint64_t*>(staged),
                                                                       static_cast<uint64_t*>(dst), n8, sig);
  return hipGetLastError();
}

// One thread per term: 24 bytes over the host link, the 104-byte record with its round keys written out.
__global__ __launch_bounds__(kUploadBlock) void k_upload_terms(const MergeTerm* __restrict__ staged,
                                                               MergeRec* __restrict__ dst, uint64_t cells,
                                                               UploadSignal sig) {
  for (uint64_t i = (uint64_t)blockIdx.x * kUploadBlock + threadIdx.x; i < cells;
       i += (uint64_t)gridDim.x * kUploadBlock) {
    const uint64_t* p = reinterpret_cast<const uint64_t*>(staged + i);
    const uint64_t w[3] = {load_host(p), load_host(p + 1), load_host(p + 2)};
    dst[i] = merge_rec(MergeTerm{w[0], (uint32_t)w[1], (uint32_t)(w[1] >> 32), __uint_as_float((uint32_t)w[2]),
                                 (uint32_t)(w[2] >> 32)});
  }
  signal_read(sig);
}

hipError_t launch_upload_terms(const MergeTerm* staged, MergeRec* dst, uint64_t cells, UploadSignal sig,
                               hipStream_t stream) {
  k_upload_terms<<<dim3(upload_blocks(cells)), dim3(kUploadBlock), 0, stream>>>(staged, dst, cells, sig);
  return hipGetLastError();
}

__global__ __launch_bounds__(kBlock) void k_stream_copy(const f32x4* __restrict__ src, f32x4* __restrict__ dst,
                                                        uint64_t n16) {
  const uint64_t base = (uint64_t)blockIdx.x * (kBlock * kCopyVecs) + threadIdx.x;
  f32x4 v[kCopyVecs];
#pragma unroll
  for (int u = 0; u < kCopyVecs; ++u) {
    const uint64_t i = base + (uint64_t)u * kBlock;
    if (i < n16) v[u] = __builtin_nontemporal_load(src + i);
  }
#pragma unroll
  for (int u = 0; u < kCopyVecs; ++u) {
    const uint64_t i = base + (uint64_t)u * kBlock;
    if (i < n16) __builtin_nontemporal_store(v[u], dst + i);
  }
}

// Copies past max_grid_blocks blocks run as several launches over consecutive ranges.
hipError_t launch_stream_copy(const void* src, void* dst, uint64_t n16, hipStream_t stream) {
  const uint64_t per_block = (uint64_t)kBlock * kCopyVecs;
  return for_pieces(n16, (uint64_t)max_grid_blocks(kBlock) * per_block, [&](uint64_t first, uint64_t count) {
    const dim3 grid((uint32_t)((count + per_block - 1) / per_block)), block(kBlock);
    k_stream_copy<<<grid, block, 0, stream>>>(static_cast<const f32x4*>(src) + first, static_cast<f32x4*>(dst) + first,
                                              count);
  });
}

}  // namespace smat
