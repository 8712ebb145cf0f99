// HIP kernels of the N-expert merge for gfx950 (Eq. merged-state, evaluation side):
//   theta_merge = theta0 + sum_j alpha_j m_j (.) (theta_j - theta0)
// with a scalar weight per expert (Task Arithmetic, weight averaging) and DARE masks m_j drawn like
// the training masks: Philox4x32-10 keyed by expert j's seed, counter (group, tensor_id,
// 4 step_j + mask stream), kept iff word < floor(keep_j 2^32), kept entries scaled by 1/keep_j.
// The accumulation acc = fma(t_j, theta_j, fma(-t_j, theta0, acc)) starting from theta0 is the
// simulate's exact-endpoint lerp for one expert, so a one-expert merge reproduces the simulated
// state without noise bit for bit.  A pure HBM stream (N + 2 arrays), built like the other
// kernels: one-wave blocks over tiles of one or two quads per thread (merge_form), loads issued before
// the mask draws and at raised wave priority, the list form mapping blocks to (tensor, chunk) through
// the chunk table.
#include "smat_launch.h"
#include "smat_tile.h"

namespace smat {

// Thread x owns quads x + u kBlock, u < Q, of the tile.  AHEAD: for terms without masks, the loads run
// one expert ahead of the sums.
template <typename TE, typename T0, typename TO, int Q, bool AHEAD, typename XAT, typename RAT>
__device__ __forceinline__ void merge_tile(const void* t0p, void* outp, uint64_t e0, uint32_t len, uint32_t head,
                                           uint32_t tensor_id, bool vec, int nexp, XAT expert_at, RAT rec_at) {
  // the elements of quad q that are the tensor's, one at a time within each expert
  auto edge = [&](uint32_t q) {
    const uint32_t lo = max(4u * q, head), hi = min(4u * q + 4u, len);
    if (lo >= hi) return;
    float b[4], acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t i = 4u * q + j;
      acc[j] = b[j] = i >= lo && i < hi ? QuadIO<T0>::load1(t0p, i) : 0.0f;
    }
    for (int x = 0; x < nexp; ++x) {
      const MergeRec R = rec_at(x);
      if (R.flags & kFlagDropAll) continue;
      const void* xp = expert_at(x);
      Words w{};
      if (R.flags & kFlagMask)
        w = group_words((e0 >> 2) + q, tensor_id, (R.step << 2) | kStreamMask, (uint32_t)R.seed,
                        (uint32_t)(R.seed >> 32));
      const uint32_t mw[4] = {w.w0, w.w1, w.w2, w.w3};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const uint32_t i = 4u * q + j;
        const bool kept = i >= lo && i < hi && (!(R.flags & kFlagMask) || mw[j] < R.thr);
        if (kept) acc[j] = __builtin_fmaf(R.t, QuadIO<TE>::load1(xp, i), __builtin_fmaf(-R.t, b[j], acc[j]));
      }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t i = 4u * q + j;
      if (i >= lo && i < hi) QuadIO<TO>::store1(outp, i, acc[j]);
    }
  };

  if (!vec || groups_wrap(e0, Q * kBlock)) {
    normal_priority();
#pragma unroll 1
    for (int u = 0; u < Q; ++u) edge(u * kBlock + threadIdx.x);
    return;
  }
  const WholeQuads W = whole_quads(len, head);
  if (W.any()) {
    float b[Q][4], acc[Q][4];
    // the experts' masks of a group differ only in the key, so they share round 1's product
    const TileGroups G = tile_groups(e0);
    uint64_t p0[Q];
#pragma unroll
    for (int u = 0; u < Q; ++u) p0[u] = philox_p0(G.lo + u * kBlock + threadIdx.x);
    typename QuadIO<TE>::Raw rx[Q];
    auto load = [&](const void* xp) {
#pragma unroll
      for (int u = 0; u < Q; ++u)
        rx[u] = QuadIO<TE>::load_raw(xp, W.clamp(u * kBlock + threadIdx.x));
    };
    {
      typename QuadIO<T0>::Raw r0[Q];
#pragma unroll
      for (int u = 0; u < Q; ++u) r0[u] = QuadIO<T0>::load_raw(t0p, W.clamp(u * kBlock + threadIdx.x));
      if (AHEAD) load(expert_at(0));
      normal_priority();
#pragma unroll
      for (int u = 0; u < Q; ++u) {
        QuadIO<T0>::unpack(r0[u], b[u]);
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[u][j] = b[u][j];
      }
    }
    auto fold = [&](const typename QuadIO<TE>::Raw* r, const bool(*kept)[4], float t) {
#pragma unroll
      for (int u = 0; u < Q; ++u) {
        float v[4];
        QuadIO<TE>::unpack(r[u], v);
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (!kept || kept[u][j]) acc[u][j] = __builtin_fmaf(t, v[j], __builtin_fmaf(-t, b[u][j], acc[u][j]));
      }
    };
    if (AHEAD) {
      // no expert draws a mask or is left out: the next expert's loads are in flight during this one's sum
      for (int x = 0; x < nexp; ++x) {
        const float t = rec_at(x).t;
        typename QuadIO<TE>::Raw now[Q];
#pragma unroll
        for (int u = 0; u < Q; ++u) now[u] = rx[u];
        if (x + 1 < nexp) load(expert_at(x + 1));
        fold(now, nullptr, t);
      }
    } else {
      for (int x = 0; x < nexp; ++x) {
        const MergeRec R = rec_at(x);
        const void* xp = expert_at(x);
        // the expert's pointer and its term's fields in one round of scalar loads, before any branch
        asm volatile("" ::"s"(xp), "s"(R.t), "s"(R.flags), "s"(R.thr), "s"(R.step));
        if (R.flags & kFlagDropAll) continue;
        // each expert's loads go out at raised priority, ahead of other waves' draws (as in the simulate)
        raise_priority();
        load(xp);
        normal_priority();
        bool kept[Q][4];
#pragma unroll
        for (int u = 0; u < Q; ++u) {
#pragma unroll
          for (int j = 0; j < 4; ++j) kept[u][j] = true;
          if (R.flags & kFlagMask) {
            const Words w = philox_tile_rk(p0[u], G.hi, tensor_id, (R.step << 2) | kStreamMask, R.rk0, R.rk1);
            kept[u][0] = w.w0 < R.thr;
            kept[u][1] = w.w1 < R.thr;
            kept[u][2] = w.w2 < R.thr;
            kept[u][3] = w.w3 < R.thr;
          }
        }
        fold(rx, kept, R.t);
      }
    }
#pragma unroll
    for (int u = 0; u < Q; ++u) {
      const uint32_t q = u * kBlock + threadIdx.x;
      if (W.has(q)) QuadIO<TO>::store(outp, q, acc[u]);
    }
  }
  for_edges(len, head, edge);
}

template <typename TE, typename T0, typename TO, int Q, bool AHEAD, bool RUNS>
__global__ __launch_bounds__(kBlock) void k_merge_one(TensorRec R, MergeArgs A, int nexp) {
  raise_priority();
  constexpr int64_t tile = tile_elems(Q);
  const int64_t begin = (int64_t)block_order<RUNS>(blockIdx.x, gridDim.x, tiles_per_chunk(Q)) * tile;
  merge_tile<TE, T0, TO, Q, AHEAD>(
      advance<T0>(R.theta0, begin), const_cast<void*>(advance<TO>(R.out, begin)), R.elem_offset + (uint64_t)begin,
      tile_len(R.n, begin, tile), begin == 0 ? R.sflags >> kHeadShift : 0u, R.tensor_id, (R.sflags & kVecMerge) != 0,
      nexp, [&](int j) { return advance<TE>(A.x[j], begin); }, [&](int j) { return A.r[j]; });
}

template <typename TE, typename T0, typename TO, int Q, bool AHEAD, int ORDER>
__global__ __launch_bounds__(kBlock) void k_merge_multi(const TensorRec* __restrict__ recs,
                                                        const void* const* __restrict__ experts,
                                                        const MergeRec* __restrict__ terms,
                                                        const uint2* __restrict__ entries, uint32_t chunks,
                                                        int nexp) {
  raise_priority();
  constexpr int64_t tile = tile_elems(Q);
  const ListBlock B = list_block<Q, ORDER>(entries, chunks);
  const TensorRec R = recs[B.tensor];
  const int64_t begin = (int64_t)B.tile * tile;
  if (begin >= R.n) return;  // unused tile of a tensor's last segment
  const size_t row = (size_t)B.tensor * (size_t)nexp;
  merge_tile<TE, T0, TO, Q, AHEAD>(
      advance<T0>(R.theta0, begin), const_cast<void*>(advance<TO>(R.out, begin)), R.elem_offset + (uint64_t)begin,
      tile_len(R.n, begin, tile), begin == 0 ? R.sflags >> kHeadShift : 0u, R.tensor_id, (R.sflags & kVecMerge) != 0,
      nexp, [&](int j) { return advance<TE>(experts[row + j], begin); }, [&](int j) { return terms[row + j]; });
}

// ---------------------------------------------------------------- launchers
// Jobs whose grid would pass max_grid_blocks run as several launches (element ranges of one tensor,
// ranges of a list's chunk table).
template <typename TE, typename T0, typename TO, int Q, bool AHEAD>
static hipError_t merge_one_as(const TensorRec& rec, const MergeArgs& args, int nexp, uint32_t lds,
                               bool runs, hipStream_t stream) {
  constexpr int64_t tile = tile_elems(Q);
  constexpr int e_dt = std::is_same<TE, Bf16>::value ? 1 : 0, t0_dt = std::is_same<T0, Bf16>::value ? 1 : 0,
                o_dt = std::is_same<TO, Bf16>::value ? 1 : 0;
  return for_pieces((uint64_t)rec.n, (uint64_t)max_grid_blocks(kBlock) * tile, [&](uint64_t off, uint64_t len) {
    const TensorRec r = rec_piece(rec, off, len, t0_dt, o_dt, 0);
    MergeArgs a = args;
    for (int j = 0; j < nexp; ++j) a.x[j] = step_ptr(args.x[j], off, storage_bytes(e_dt));
    const dim3 grid((uint32_t)((len + tile - 1) / tile)), block(kBlock);
    with_flag(runs, [&](auto rn) {
      k_merge_one<TE, T0, TO, Q, AHEAD, decltype(rn)::value><<<grid, block, lds, stream>>>(r, a, nexp);
    });
  });
}

template <typename TE, typename T0, typename TO, int Q, bool AHEAD>
static hipError_t merge_multi_as(const TensorRec* recs, const void* const* experts, const MergeRec* terms,
                                 const ChunkTable& table, int nexp, uint32_t lds, bool runs,
                                 hipStream_t stream) {
  return for_table<Q>(table, runs, [&](const uint2* entries, uint32_t chunks, dim3 grid, auto order, uint64_t) {
    const dim3 block(kBlock);
    k_merge_multi<TE, T0, TO, Q, AHEAD, decltype(order)::value>
        <<<grid, block, lds, stream>>>(recs, experts, terms, entries, chunks, nexp);
  });
}

// The form a merge of `bytes` in all takes: go(quads per thread, experts loaded ahead, LDS to reserve).
// A merge's waves live long (one round of loads per expert), so which tiles are open together decides
// how well its N + 2 streams use the DRAM rows.  Measured on lists of 0.1-1.5e9 parameters:
//   - fp32 experts, one quad per thread with 25 resident blocks: 3 experts 2.12 -> 1.77 ms (fp32 out),
//     1.81 -> 1.65 (bf16 out), 8 experts 4.31 -> 3.75, with masks 2.11 -> 1.76; two quads at their best
//     cap (12) 1.83.  Below 128 MB two quads are as fast or faster (2M parameters 15.0 against 15.7 us).
//   - bf16 experts, two quads, none masked: the next expert's loads issued ahead with 25 resident
//     blocks take 7 experts from 4.37 to 4.25 ms, 16 from 2.43 to 2.40, 4 from 1.134 to 1.115; with 3
//     the gain is gone, with 2 it loses 1 %, and lists under 1 GB lose 1-4 %.
//   - masked bf16 experts are bound by their draws and want every block resident (5.10 ms; 5.39 with
//     25 blocks and loads ahead).
template <typename TE, typename F>
static hipError_t merge_form(int nexp, bool plain, uint64_t bytes, F&& go) {
  using std::integral_constant;
  constexpr uint32_t lds = lds_for_blocks(25);
  if constexpr (std::is_same<TE, float>::value) {
    if (bytes >= (128ull << 20))
      return go(integral_constant<int, 1>(), std::false_type(), bytes >= kCapFromBytes ? lds : 0u);
  } else {
    if (plain && nexp >= 4 && bytes >= (1ull << 30)) return go(integral_constant<int, 2>(), std::true_type(), lds);
  }
  return go(integral_constant<int, 2>(), std::false_type(), 0u);
}

template <typename TE, typename T0, typename TO>
constexpr uint64_t merge_bytes(uint64_t elems, int nexp) {
  return elems * (uint64_t)(nexp * StorageBytes<TE>::value + StorageBytes<T0>::value + StorageBytes<TO>::value);
}

template <typename TE, typename T0, typename TO>
static hipError_t merge_one(const TensorRec& rec, const MergeArgs& args, int nexp, bool plain, bool runs,
                            hipStream_t stream) {
  const uint64_t bytes = merge_bytes<TE, T0, TO>((uint64_t)rec.n, nexp);
  return merge_form<TE>(nexp, plain, bytes, [&](auto q, auto ahead, uint32_t lds) {
    return merge_one_as<TE, T0, TO, q(), ahead()>(rec, args, nexp, lds, runs, stream);
  });
}

template <typename TE, typename T0, typename TO>
static hipError_t merge_multi(const TensorRec* recs, const void* const* experts, const MergeRec* terms,
                              const ChunkTable& table, int nexp, bool plain, bool runs,
                              hipStream_t stream) {
  const uint64_t bytes = merge_bytes<TE, T0, TO>(table_elems(table), nexp);
  return merge_form<TE>(nexp, plain, bytes, [&](auto q, auto ahead, uint32_t lds) {
    return merge_multi_as<TE, T0, TO, q(), ahead()>(recs, experts, terms, table, nexp, lds, runs, stream);
  });
}

// Storage codes: 0 = fp32, 1 = bf16, for (expert, theta0, out).
#define SMAT_MERGE_DISPATCH(FN, ...)                                                               \
  switch (expert_dtype * 4 + theta0_dtype * 2 + out_dtype) {                                        \
    case 0: return FN<float, float, float>(__VA_ARGS__);                                           \
    case 1: return FN<float, float, Bf16>(__VA_ARGS__);                                            \
    case 2: return FN<float, Bf16, float>(__VA_ARGS__);                                            \
    case 3: return FN<float, Bf16, Bf16>(__VA_ARGS__);                                             \
    case 4: return FN<Bf16, float, float>(__VA_ARGS__);                                            \
    case 5: return FN<Bf16, float, Bf16>(__VA_ARGS__);                                             \
    case 6: return FN<Bf16, Bf16, float>(__VA_ARGS__);                                             \
    default: return FN<Bf16, Bf16, Bf16>(__VA_ARGS__);                                             \
  }

hipError_t launch_merge_one(const TensorRec& rec, const MergeArgs& args, int nexp, int expert_dtype, int theta0_dtype,
                            int out_dtype, bool plain, bool runs, hipStream_t stream) {
  SMAT_MERGE_DISPATCH(merge_one, rec, args, nexp, plain, runs, stream)
}

hipError_t launch_merge_multi(const TensorRec* recs, const void* const* experts, const MergeRec* terms,
                              const ChunkTable& table, int nexp, int expert_dtype, int theta0_dtype,
                              int out_dtype, bool plain, bool runs, hipStream_t stream) {
  SMAT_MERGE_DISPATCH(merge_multi, recs, experts, terms, table, nexp, plain, runs, stream)
}

#undef SMAT_MERGE_DISPATCH

}  // namespace smat
