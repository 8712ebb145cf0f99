// How a list is cut into tiles and launches: sizes, the pieces of a list's table that each fit one launch,
// and the tile that a block of a piece takes.  Plain integer code, the same on the host and the device.
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define SMAT_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define SMAT_HOST_DEVICE inline
#endif

namespace smat {

// Work decomposition: a block of kBlock threads (one wave) handles one tile of Q quads per
// thread (tile = 4 * kBlock * Q elements); thread x owns quads x, x + kBlock, ... of the tile,
// so every load/store instruction of the wave covers one contiguous span and consecutive blocks
// stream consecutive memory.  A list is cut into chunks of kChunk elements
// through a table that keeps its entries few; where many small tensors would leave most blocks of
// their chunks without a tile, the remainders go in segments of kSegment elements instead (ChunkTable).
// The simulate, the backward and the fused optimizer step take one
// quad per thread: each wave then keeps one 64-lane piece of every array in flight, the access shape
// that streams fastest on MI355X.
constexpr int kBlock = 64;
constexpr int64_t kChunk = 16384;
constexpr int64_t kSegment = 2048;
constexpr uint32_t kChunkSegments = (uint32_t)(kChunk / kSegment);
constexpr int64_t tile_elems(int quads) { return 4 * kBlock * quads; }
constexpr uint32_t tiles_per_segment(int quads) { return (uint32_t)(kSegment / tile_elems(quads)); }
constexpr uint32_t tiles_per_chunk(int quads) { return kChunkSegments * tiles_per_segment(quads); }

// A dispatch packet holds the grid's total work-items (blocks x threads per block) in 32 bits, and a
// grid past that wraps without an error.  The launchers split larger jobs into several launches of
// at most this many blocks each (for one-wave blocks 2^26 - 1, i.e. 17.2e9 elements at one quad per
// thread).
constexpr uint32_t max_grid_blocks(int threads) { return 0xFFFFFFFFu / (uint32_t)threads; }

// How a list launch finds its tiles: chunks in linear block order or in runs per XCD (block_order), or a
// table that also has segments.
enum TableOrder : int { kLinear = 0, kRuns = 1, kMixed = 2 };
constexpr uint32_t kMixedRuns = 1u << 31;  // on the chunk count of a kMixed launch: its chunks in runs

// One launch over consecutive entries of a table (`chunks` entries for chunks, then `segments` for single
// segments): its first entry, the chunk count that the kernel gets (read by kMixed only), its blocks and
// the segments of the table that lie before it.
struct TablePiece {
  uint64_t entry;
  uint32_t chunks, blocks;
  TableOrder order;
  uint64_t segment;
};

// fn(piece) for the launches of a table with tiles of `quads` quads, each of at most max_blocks blocks
// (at least a chunk's), until it returns false.  One launch where the table fits it; else its chunks, then
// its segments, each in as many as it takes.
template <typename F>
void table_pieces(uint32_t chunks, uint32_t segments, int quads, bool runs, uint32_t max_blocks, F&& fn) {
  const uint32_t tps = tiles_per_segment(quads), tpc = tiles_per_chunk(quads);
  const uint64_t blocks = (uint64_t)chunks * tpc + (uint64_t)segments * tps;
  if (segments > 0 && blocks <= max_blocks) {
    fn(TablePiece{0, chunks | (runs ? kMixedRuns : 0u), (uint32_t)blocks, kMixed, 0});
    return;
  }
  for (uint64_t first = 0, per = max_blocks / tpc; first < chunks; first += per) {
    const uint32_t count = (uint32_t)(chunks - first < per ? chunks - first : per);
    if (!fn(TablePiece{first, 0, count * tpc, runs ? kRuns : kLinear, first * kChunkSegments})) return;
  }
  for (uint64_t first = 0, per = max_blocks / tps; first < segments; first += per) {
    const uint32_t count = (uint32_t)(segments - first < per ? segments - first : per);
    if (!fn(TablePiece{chunks + first, 0, count * tps, kMixed, (uint64_t)chunks * kChunkSegments + first})) return;
  }
}

// Block order.  Consecutive blocks go to the eight XCDs in turn, each with an L2 of its own.  With tiles
// that begin on a 128-byte line that is the best order: the chip streams one contiguous window of every
// array.  Where tiles begin inside a line (tensors packed end to end), neighbouring tiles share a line at
// their border, which two XCDs then fetch, and write in part, each for itself.  RUNS gives an XCD whole
// runs of tpc tiles (16,384 elements) of eight runs at a time, so that borders meet in one L2.  Step of
// six 67M-element tensors in one buffer, linear order -> runs: 1.37 -> 1.16 ms when the tensors begin 2
// to 32 bytes off a line, 1.30 -> 1.13 ms 64 off, but 1.088 -> 1.115 on it (the 1.5B list: 3-7 % slower);
// optimizer step 2.65 -> 2.35, 3-expert merge 0.74 -> 0.67.
template <bool RUNS>
SMAT_HOST_DEVICE uint32_t block_order(uint32_t b, uint32_t blocks, uint32_t tpc) {
  const uint32_t group = 8u * tpc;
  if (!RUNS || b >= blocks / group * group) return b;
  return b / group * group + (b % 8u) * tpc + b / 8u % tpc;
}

// The entry of a piece (counted from its first) that block b of `blocks` takes, and the tile of that entry;
// `chunks` is read by kMixed only.
struct EntryTile {
  uint32_t entry, tile;
};
template <int Q, int ORDER>
SMAT_HOST_DEVICE EntryTile entry_tile(uint32_t b, uint32_t blocks, uint32_t chunks) {
  constexpr uint32_t tps = tiles_per_segment(Q), tpc = tiles_per_chunk(Q);
  if (ORDER == kMixed) {
    const uint32_t count = chunks & ~kMixedRuns, chunk_blocks = count * tpc;
    if (b >= chunk_blocks) {
      b -= chunk_blocks;
      return {count + b / tps, b % tps};
    }
    if (chunks & kMixedRuns) b = block_order<true>(b, chunk_blocks, tpc);
  } else {
    b = block_order<ORDER == kRuns>(b, blocks, tpc);
  }
  return {b / tpc, b % tpc};
}

}  // namespace smat
