// A list's table in launches and blocks (smat_table.h), walked block by block on the host: over all launches
// every tile of every chunk and segment is taken exactly once, the norm's partials land in table order, and
// no launch is larger than it may be, with a limit small enough that tables take many launches.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "smat_table.h"

using namespace smat;

#define EXPECT(cond)                                                                        \
  do {                                                                                      \
    if (!(cond)) {                                                                          \
      std::printf("FAIL line %d: %s\n", __LINE__, #cond);                                   \
      std::exit(1);                                                                         \
    }                                                                                       \
  } while (0)

static uint64_t g_launches[3];

template <int Q>
static EntryTile at(const TablePiece& p, uint32_t b) {
  if (p.order == kLinear) return entry_tile<Q, kLinear>(b, p.blocks, p.chunks);
  if (p.order == kRuns) return entry_tile<Q, kRuns>(b, p.blocks, p.chunks);
  return entry_tile<Q, kMixed>(b, p.blocks, p.chunks);
}

template <int Q>
static int walk(uint32_t chunks, uint32_t segments, bool runs, uint32_t max_blocks) {
  const uint32_t tps = tiles_per_segment(Q), tpc = tiles_per_chunk(Q);
  const uint64_t tiles = (uint64_t)chunks * tpc + (uint64_t)segments * tps;
  std::vector<unsigned char> seen(tiles, 0);
  int launches = 0;
  table_pieces(chunks, segments, Q, runs, max_blocks, [&](const TablePiece& p) {
    ++launches;
    ++g_launches[p.order];
    EXPECT(p.blocks > 0 && p.blocks <= max_blocks);
    for (uint32_t b = 0; b < p.blocks; ++b) {
      const EntryTile t = at<Q>(p, b);
      const uint64_t e = p.entry + t.entry;
      EXPECT(e < (uint64_t)chunks + segments);
      EXPECT(t.tile < (e < chunks ? tpc : tps));
      const uint64_t tile = e < chunks ? e * tpc + t.tile : (uint64_t)chunks * tpc + (e - chunks) * tps + t.tile;
      EXPECT(!seen[tile]);
      seen[tile] = 1;
      // the gradient norm (one tile a segment, linear order): block b of a launch writes partial segment + b
      if (tps == 1 && !runs) EXPECT(p.segment + b == tile);
    }
    return true;
  });
  for (unsigned char s : seen) EXPECT(s);
  return launches;
}

template <int Q>
static void walk_all() {
  const uint32_t tpc = tiles_per_chunk(Q);
  for (uint32_t chunks : {0u, 1u, 2u, 7u, 8u, 9u, 17u, 41u})
    for (uint32_t segments : {0u, 1u, 3u, 8u, 50u})
      for (int runs = 0; runs < 2; ++runs) {
        const uint64_t all = (uint64_t)chunks * tpc + (uint64_t)segments * tiles_per_segment(Q);
        // from one chunk a launch up to all of them, and one block more or less than a whole table
        for (uint64_t limit : std::vector<uint64_t>{tpc, tpc + 1, 3 * tpc - 1, 16 * tpc, all - 1, all, all + 1}) {
          if (limit < tpc || limit > 1u << 30) continue;
          const int launches = walk<Q>(chunks, segments, runs != 0, (uint32_t)limit);
          if (segments > 0 && all <= limit) EXPECT(launches == 1);
          if (all > limit) EXPECT(launches > 1);
        }
      }
}

// The same arithmetic at the real limit, by counts: tables up to the 2^31 one-quad tiles a plan may have.
static void real_limit(uint32_t chunks, uint32_t segments, int quads, int want) {
  const uint32_t limit = max_grid_blocks(kBlock);
  EXPECT(limit == (1u << 26) - 1);
  uint64_t entry = 0, segment = 0;
  int launches = 0;
  table_pieces(chunks, segments, quads, false, limit, [&](const TablePiece& p) {
    ++launches;
    EXPECT(p.entry == entry && p.segment == segment && p.blocks > 0 && p.blocks <= limit);
    const uint64_t in_chunks = p.order == kMixed ? (uint64_t)p.chunks * tiles_per_chunk(quads) : p.blocks;
    entry += in_chunks / tiles_per_chunk(quads) + (p.blocks - in_chunks) / tiles_per_segment(quads);
    segment += in_chunks / tiles_per_chunk(quads) * kChunkSegments + (p.blocks - in_chunks) / tiles_per_segment(quads);
    return true;
  });
  EXPECT(entry == (uint64_t)chunks + segments && segment == (uint64_t)chunks * kChunkSegments + segments);
  EXPECT(launches == want);
}

int main() {
  walk_all<1>();
  walk_all<2>();
  walk_all<8>();
  for (uint64_t n : g_launches) EXPECT(n > 100);
  const uint32_t per_chunk = ((1u << 26) - 1) / 64, per_segment = ((1u << 26) - 1) / 8;  // chunks, segments a launch
  real_limit(per_chunk, 0, 1, 1);
  real_limit(per_chunk + 1, 0, 1, 2);
  real_limit((1u << 31) / 64 - 1, 0, 1, 33);
  real_limit(0, per_segment, 1, 1);
  real_limit(0, per_segment + 1, 1, 2);
  real_limit(1, per_segment, 1, 2);
  real_limit(per_chunk + 1, per_segment + 1, 1, 4);
  real_limit(per_chunk + 1, per_segment + 1, 8, 1);
  real_limit(1u << 23, 1u << 23, 8, 3);
  // a launch that fails is the last one, among the chunks (9 launches) and among the segments after them
  for (int stop : {1, 3, 9, 10}) {
    int calls = 0;
    table_pieces(9, 25, 1, false, 64, [&](const TablePiece&) { return ++calls < stop; });
    EXPECT(calls == stop);
  }
  std::printf("ok\n");
  return 0;
}
