// Which tile of the result a workgroup computes: integer arithmetic only, the same on the host and on the device.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstddef>

namespace mq {

// Block index -> tile.  Workgroups are dealt round-robin to the 8 XCDs, each
// with its own L2; giving every XCD one contiguous run of tiles (n fastest)
// makes the blocks that run together on an XCD share A row panels and the
// parameter in that XCD's L2.
__host__ __device__ __forceinline__ unsigned xcd_remap(unsigned bid, unsigned total) {
  const unsigned q = total / 8, r = total % 8, x = bid % 8, idx = bid / 8;
  return x * q + (x < r ? x : r) + idx;
}

// Tile coordinates of a block.  After the XCD remap, consecutive tile numbers
// walk down a band of GM tile rows before moving to the next tile column, so
// the ~32 blocks resident on one XCD cover a GM x (32 / GM) patch of the
// result: each A row panel and each parameter panel they stream is then shared
// by several of them in that XCD's L2 instead of being fetched once per block.
// GM * tiles_n must fit 32 bits.
__host__ __device__ __forceinline__ void tile_at(unsigned bid, unsigned total, unsigned tiles_m, unsigned tiles_n, unsigned GM,
                                                 unsigned& tile_m, unsigned& tile_n) {
  const unsigned t = xcd_remap(bid, total);
  const unsigned band = t / (GM * tiles_n), in_band = t % (GM * tiles_n);
  const unsigned first = band * GM;
  const unsigned rows = tiles_m - first < GM ? tiles_m - first : GM;
  tile_m = first + in_band % rows;
  tile_n = in_band / rows;
}

// The same for kernels that last a few microseconds, where four integer divisions (100 clocks and more each, one after the
// other) in front of the first load show: reciprocals from the host.  t / d = high half of t ceil(2^32 / d) for t, d < 2^16.
struct Tiles {
  unsigned total, m, n, band, by_band, by_rows, by_last;
};

// Which tiles an XCD's share of the grid covers: a band of tile rows and as many columns as its workgroups fill, so that the
// rows and columns its L2 has to take in are the fewest bytes (a tile has `aspect` times as many rows as columns).  With the
// columns of a row of tiles dealt over the XCDs instead, every L2 took in all of A: 1001 x 512 x 2048 in 8 bit, quantizer
// included, 10.4 -> 9.3 us, in 16 bit 18.2 -> 15.4, 2000 x 300 x 1800 in 8 bit 15.2 -> 11.9.
// No band has more rows than there are: of one row of five million tiles the square root would be 800 rows, and that many
// times the columns does not fit 32 bits.  (band * tiles_n is at most the number of tiles, below 2^31.)
inline unsigned band_rows(size_t tiles_m, size_t tiles_n, int aspect) {
  const double rows = std::sqrt((double)((tiles_m * tiles_n + 7) / 8) / aspect);
  const unsigned band = rows < 1.5 ? 1u : (unsigned)(rows + 0.5);
  return band < tiles_m ? band : (unsigned)tiles_m;
}

inline Tiles tiles_of(size_t tiles_m, size_t tiles_n, int aspect) {
  auto inverse = [](size_t d) { return d <= 1 ? 0u : (unsigned)((((unsigned long long)1 << 32) + d - 1) / d); };
  const unsigned band = band_rows(tiles_m, tiles_n, aspect);
  const size_t last = tiles_m % band;
  return {(unsigned)(tiles_m * tiles_n), (unsigned)tiles_m, (unsigned)tiles_n, band, inverse(band * tiles_n), inverse(band),
          inverse(last == 0 ? band : last)};
}

__host__ __device__ __forceinline__ void tile_at(unsigned bid, const Tiles& c, unsigned& tile_m, unsigned& tile_n) {
  if (c.total >= 1u << 16) return tile_at(bid, c.total, c.m, c.n, c.band, tile_m, tile_n);
  auto over = [](unsigned t, unsigned inverse) { return inverse == 0u ? t : (unsigned)(((unsigned long long)t * inverse) >> 32); };
  const unsigned t = xcd_remap(bid, c.total);
  const unsigned band = over(t, c.by_band), in_band = t - band * c.band * c.n, first = band * c.band;
  const bool whole = first + c.band <= c.m;
  tile_n = over(in_band, whole ? c.by_rows : c.by_last);
  tile_m = first + in_band - tile_n * (whole ? c.band : c.m - first);
}

}  // namespace mq
