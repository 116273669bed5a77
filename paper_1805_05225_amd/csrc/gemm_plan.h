// How gemm_tile.hip cuts K into ranges: plain functions of sizes (no HIP here, so that a host program can check them).
#pragma once
#include <algorithm>
#include <cstddef>

namespace lstm {

constexpr int kTileEdge = 128, kTileK = 64;      // rows and columns of a tile of C; k per stage
inline long tile_count(long M, long N, int nz) { return (M + kTileEdge - 1) / kTileEdge * ((N + kTileEdge - 1) / kTileEdge) * nz; }
inline long tile_stages(long K, int nseg) { return (K + kTileK - 1) / kTileK * nseg; }
// Ranges of a product by itself (`others`: tiles of the product that shares its launch): as many as run at a time, at least four stages each.
inline int tile_ranges(long tiles, long others, long stages) {
  return (int)std::max(1L, std::min(std::min(512 / std::max(tiles + others, 1L), stages / 4), 16L));
}
// Bytes of the parts of `ks` ranges; as they lie behind one another.
inline size_t tile_part_bytes(long M, long N, int nz, int ks) { return ks > 1 ? (size_t)ks * nz * M * ((N + 3) / 4 * 4) * 4 : 0; }
inline size_t tile_part_room(long M, long N, int nz, int ks) { return (tile_part_bytes(M, N, nz, ks) + 255) / 256 * 256; }

struct TileProduct { long M, N, K; int nz, nseg; };
// Ranges of three products in one launch, one behind the other in this order, whose parts lie in `room` bytes: about the same number of stages in all three; how many by what the launch is
// expected to take, in stages: a work-group costs 8 more than it has, 512 run at a time (up to 256 have a compute unit each and take 0.6 of the time), a megabyte of parts is half a stage.
// Behind a full device one of the last two products' work-groups ends alone; the first product's, the longest, have begun before.  Of 1500 layers of 60 to 5000 frames measured with each of
// their choices (two to nine), this one is 1.02 times the fastest in the mean and at most 1.05 in nine of ten; with half of the longest work-group at the end instead, and no look at the room, it
// asked for ranges of dX that did not fit and ran it whole, or cut it where whole is faster (1620 frames, n_in = 1733, n = 833, both directions: three products 142 us whole, 154 in two ranges).
// -> that cost
inline double tile_ranges3(const TileProduct (&p)[3], size_t room, int (&ks)[3]) {
  long tiles[3], stages[3], most = 4;
  for (int i = 0; i < 3; ++i) {
    tiles[i] = tile_count(p[i].M, p[i].N, p[i].nz);
    stages[i] = tile_stages(p[i].K, p[i].nseg);
    most = std::max(most, stages[i]);
  }
  double least = 0.;
  for (long per = most; per >= 4; per -= std::max(1L, per / 32)) {
    double groups = 0., work = 0., longest = 0., parts = 0.;
    size_t used = 0;
    int k[3];
    for (int i = 0; i < 3; ++i) {
      k[i] = (int)std::max(1L, std::min({(stages[i] + per - 1) / per, stages[i] / 4, 16L}));
      const double each = (double)stages[i] / k[i] + 8.;
      groups += (double)tiles[i] * k[i];
      work += tiles[i] * k[i] * each;
      longest = std::max(longest, each);
      parts += 5e-7 * tile_part_bytes(p[i].M, p[i].N, p[i].nz, k[i]);
      used += tile_part_room(p[i].M, p[i].N, p[i].nz, k[i]);
    }
    if (used > room) continue;                   // (per = most: no ranges, which always fit)
    const double last = std::max((double)stages[1] / k[1], (double)stages[2] / k[2]) + 8.;
    const double cost = parts + (groups <= 256. ? 0.6 * longest : groups <= 512. ? longest : std::max(longest, work / 512. + last));
    if (per == most || cost < least) { least = cost; std::copy(k, k + 3, ks); }
  }
  return least;
}

}  // namespace lstm
