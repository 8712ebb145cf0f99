// Tile addressing shared by the SMAT kernels: a tile is a run of consecutive elements of one
// tensor handed to the element code, with its pointers already advanced to the tile's start.
#pragma once

#include "smat_device.h"

namespace smat {

template <typename T>
struct StorageBytes;
template <>
struct StorageBytes<float> {
  static constexpr int value = 4;
};
template <>
struct StorageBytes<Bf16> {
  static constexpr int value = 2;
};

// A tile: pointers at the tile's first element, its global index e0 (a multiple of 4), its length, the
// tensor id and the static flags.  Thread x of the block owns quads x + u * (block size) of the tile.
// The first `head` elements of a tensor's first tile are not the tensor's (see TensorRec::sflags).
struct Tile {
  const float* theta;
  const void* theta0;
  void* out;
  const void* grad_sim;
  float* grad_theta;
  uint64_t e0;
  uint32_t len;
  uint32_t tensor_id;
  uint32_t sflags;
  uint32_t head;
};

template <typename T>
__device__ __forceinline__ const void* advance(const void* p, int64_t elems) {
  return static_cast<const char*>(p) + elems * StorageBytes<T>::value;
}

__device__ __forceinline__ uint32_t tile_len(int64_t n, int64_t begin, int64_t tile) {
  return (uint32_t)(n - begin < tile ? n - begin : tile);
}

template <typename T0, typename TO>
__device__ __forceinline__ Tile tensor_tile(const TensorRec& R, int64_t begin, int64_t tile) {
  return Tile{R.theta + begin, advance<T0>(R.theta0, begin), const_cast<void*>(advance<TO>(R.out, begin)),
              R.grad_sim, R.grad_theta, R.elem_offset + (uint64_t)begin, tile_len(R.n, begin, tile), R.tensor_id,
              R.sflags, begin == 0 ? R.sflags >> kHeadShift : 0u};
}

// Record i of a per-tensor table, addressed with a 32-bit byte offset that the scalar unit forms in
// one shift (plans hold at most kMaxListTensors tensors, so i * 64 stays below 2^32).
template <typename R>
__device__ __forceinline__ const R& rec_at(const R* base, uint32_t i) {
  return *reinterpret_cast<const R*>(reinterpret_cast<const char*>(base) + i * (uint32_t)sizeof(R));
}

// The tensor and tile of a block of a list launch; `chunks` is read by kMixed only.  The table (8 B per
// entry) and the tensor records (64 B per tensor) are small enough to stay in L2 while the kernel
// streams the tensors.
struct ListBlock {
  uint32_t tensor, tile;
};
template <int Q, int ORDER>
__device__ __forceinline__ ListBlock list_block(const uint2* entries, uint32_t chunks) {
  const EntryTile t = entry_tile<Q, ORDER>(blockIdx.x, gridDim.x, chunks);
  const uint2 e = entries[t.entry];
  return {e.x, e.y * tiles_per_segment(Q) + t.tile};
}

// What a block of a device-driven list launch reads about its tensor and its step.  All of it is fetched in
// one round of scalar loads (the empty asm needs every field at once): left to itself the compiler reads
// the fields where branches first use them, in five rounds one after the other, before the wave's first
// vector load.
struct DeviceRecs {
  TensorRec R;
  ParamRec P;
  ScaleRec C;
  StepState S;
};
__device__ __forceinline__ DeviceRecs device_recs(const TensorRec* recs, const ParamRec* prms, const ScaleRec* scales,
                                                  const StepState* state, uint32_t tensor, float lambda) {
  DeviceRecs D{rec_at(recs, tensor), rec_at(prms, tensor), rec_at(scales, tensor), *state};
  asm volatile("" ::"s"(D.R.theta), "s"(D.R.theta0), "s"(D.R.out), "s"(D.R.grad_sim), "s"(D.R.grad_theta),
               "s"(D.R.n), "s"(D.R.elem_offset), "s"(D.R.tensor_id), "s"(D.R.sflags), "s"(D.P.thr), "s"(D.P.sigma),
               "s"(D.P.flags), "s"(D.C.s), "s"(D.C.keep), "s"(D.C.divide), "s"(D.S.seed), "s"(D.S.step),
               "s"(D.S.scale), "s"(lambda));
  return D;
}

// Tile ti of a list's tensor.  len is 0 when the tile lies past the end of the tensor.  It comes from
// 32-bit scalar arithmetic: a plan holds fewer than 2^31 one-quad tiles in all, so a tile's index
// within its tensor and the tensor's count of whole tiles stay below 2^31.
template <typename T0, typename TO, typename TG>
__device__ __forceinline__ Tile list_tile(const TensorRec& R, uint32_t ti, int64_t tile) {
  const uint64_t n = (uint64_t)R.n;
  const uint32_t whole = (uint32_t)(n / (uint64_t)tile), tail = (uint32_t)n % (uint32_t)tile;
  const int64_t begin = (int64_t)ti * tile;
  return Tile{R.theta + begin,
              advance<T0>(R.theta0, begin),
              const_cast<void*>(advance<TO>(R.out, begin)),
              advance<TG>(R.grad_sim, begin),
              R.grad_theta + begin,
              R.elem_offset + (uint64_t)begin,
              ti < whole ? (uint32_t)tile : (ti == whole ? tail : 0u),
              R.tensor_id,
              R.sflags,
              ti == 0u ? R.sflags >> kHeadShift : 0u};
}

// Where a tile takes its Philox keys and its tensor's coefficient t from.  A launch whose step the host
// knows has both in its arguments; a device-driven one forms them per wave, LATE: once the tile has issued
// its loads.
struct HostStep {
  static constexpr bool LATE = false;
  const PhiloxKeys& K;
  uint32_t step;
  __device__ __forceinline__ const PhiloxKeys& keys() const { return K; }
  __device__ __forceinline__ float coefficient(const ParamRec& P) const { return P.t; }
};
struct DeviceStep {
  static constexpr bool LATE = true;
  uint64_t seed;
  uint32_t step;
  float scale;
  ScaleRec C;
  __device__ __forceinline__ PhiloxKeys keys() const { return philox_keys(seed); }
  __device__ __forceinline__ float coefficient(const ParamRec&) const { return device_coefficient(scale, C); }
};

// The whole quads [first, end) of a tile, which move as vectors, and edge(q) for the partial ones: the
// first quad of a tensor with a head, and the quad that holds a tensor's last 1-3 elements, each given
// to the thread that owns it.
struct WholeQuads {
  uint32_t first, end;
  __device__ __forceinline__ bool any() const { return first < end; }
  __device__ __forceinline__ bool has(uint32_t q) const { return q >= first && q < end; }
  __device__ __forceinline__ uint32_t clamp(uint32_t q) const { return max(min(q, end - 1u), first); }
};
__device__ __forceinline__ WholeQuads whole_quads(uint32_t len, uint32_t head) { return {head ? 1u : 0u, len >> 2}; }

template <typename F>
__device__ __forceinline__ void for_edges(uint32_t len, uint32_t head, F&& edge) {
  const uint32_t nq = len >> 2;
  if (head && threadIdx.x == 0) edge(0u);
  if ((len & 3u) && (nq > 0 || !head) && threadIdx.x == (nq & (kBlock - 1))) edge(nq);
}

}  // namespace smat
