// How the step kernels cut the rows of a grid: plain arithmetic, shared by
// the launches, the kernels, and a check that runs on the host alone.
#ifndef LBM_TILING_H
#define LBM_TILING_H

#include <algorithm>
#include <cmath>

#ifdef __HIPCC__
#define LBM_HD __host__ __device__
#else
#define LBM_HD
#endif

namespace {

// Workgroups of a launch per XCD: the hardware deals workgroups out to the
// eight XCDs round-robin (workgroup b runs on XCD b % 8).
constexpr int kXcds = 8;

// The rows one XCD walks in a single-grid step, cut into chunks: `rows`
// high (the last one possibly lower) up to the band's last tail_rows rows,
// then short chunks (tail_h high, the last one possibly lower) over those.
// Band x holds rows [x ny / 8, (x + 1) ny / 8).
struct Band {
  int y0, y1;    // the band's rows
  int ys;        // first row of the short chunks
  int nlong;     // chunks of at most `rows` rows in [y0, ys)
  int nchunks;   // long and short
};

LBM_HD inline Band band_of(int x, int ny, int rows, int tail_rows, int tail_h) {
  Band b;
  b.y0 = int((long long)x * ny / kXcds);
  b.y1 = int((long long)(x + 1) * ny / kXcds);
  const int t = tail_rows < b.y1 - b.y0 ? tail_rows : b.y1 - b.y0;
  b.ys = b.y1 - t;
  b.nlong = (b.ys - b.y0 + rows - 1) / rows;
  b.nchunks = b.nlong + (t + tail_h - 1) / tail_h;
  return b;
}

// The two-step kernel's strips: 64 columns of which 56 are stored.
constexpr int kPairHalo = 4;                   // columns on each side
constexpr int kPairCols = 64 - 2 * kPairHalo;  // columns stored
inline int pair_strips(int nx) { return (nx + kPairCols - 1) / kPairCols; }

// Mean tile height from which the two-step kernel is faster than
// lbm_step_kernel: below it the four rows a tile walks beyond its own outweigh
// the gain.  us per step, lbm_step_kernel -> this:
//  * float32 600^2 (3.2 rows) 20.6 -> 20.9, 640^2 (3.75) 23.7 -> 21.2, 720^2
//    (4.6) 26.3 -> 24.0.  With odd nx lbm_step_kernel, one column per lane, is
//    faster itself, and the variants whose sites take most arithmetic gain less
//    (GENR: r != 1, HAS_S: rho_A != rho_B).  HAS_S alone: 633x640
//    (3.75) 20.3 -> 20.5, 661^2 (3.9) 20.7 -> 20.6, 671x690 (4.0) 22.7 -> 22.3;
//    both: 641x660 (3.9) 21.0 -> 21.4, 685x720 (4.6) 23.5 -> 24.1, 783x740
//    (5.06) 27.0 -> 26.6;
//  * float64 450^2 (3.9) 22.5 -> 23.4, 512^2 (5.0) 27.0 -> 26.1; both: 512^2
//    27.6 -> 28.4, 526^2 (5.14) 28.6 -> 28.7, 534^2 (5.21) 29.2 -> 28.8.
inline double pair_least_rows(bool f32, bool odd_nx, bool genr, bool has_s) {
  if (!f32) return genr && has_s ? 5.2 : 4.7;
  if (!odd_nx || !has_s) return 3.7;
  return genr ? 5.0 : 3.85;
}

// Tiles per XCD of the two-step kernel, 0 where its tiles would be lower than
// `least` rows.  All wavefront slots take one tile (slots: per XCD), or as many
// as keep the tiles at 40 rows or fewer: 4096^2 float32 with tiles of 148, 74,
// 37 rows 523, 497, 485 us per step; 2048^2 with 37 and 18 rows 134.0 and 134.2.
inline int pair_tiles_of(int nx, int ny, int slots, double least) {
  if (slots <= 0 || ny < 16) return 0;  // the rows a tile reaches past the grid wrap once
  const double rows = double(pair_strips(nx)) * ny / kXcds / slots;  // mean tile height
  if (rows < least) return 0;
  const long long tiles = (long long)slots * (long long)std::ceil(rows / 40.0);
  return int(std::max<long long>(tiles, pair_strips(nx)));  // a chunk per strip at least
}

// Tile `tile` of XCD xcd in the two-step kernel: each strip of the band is
// cut into tiles / nstrips chunks, one more in the first tiles % nstrips
// strips, so that the band makes exactly `tiles` tiles.  May be empty.
struct PairTile {
  int strip, y0, y1;
};

LBM_HD inline PairTile pair_tile_of(int xcd, int tile, int ny, int tiles, int nstrips) {
  PairTile t;
  const int chunk = tile / nstrips;
  t.strip = tile - chunk * nstrips;
  const int full = tiles / nstrips;
  const int chunks = full + (t.strip < tiles - full * nstrips ? 1 : 0);
  const Band b = band_of(xcd, ny, 1, 0, 1);
  // b.y0 + rows c / chunks, rounded down, for c = chunk, chunk + 1.  rows c
  // itself can pass 2^31 (a band of 300000 rows in 7500 chunks); without the
  // whole rows per chunk what is left stays below chunks^2, and a strip has
  // at most 45000 chunks: one per 40 rows of the highest grid that fits, and
  // one per wavefront slot.
  const unsigned rows = unsigned(b.y1 - b.y0), n = unsigned(chunks), c = unsigned(chunk);
  const unsigned whole = rows / n, part = rows % n;
  t.y0 = b.y0 + int(whole * c + part * c / n);
  t.y1 = b.y0 + int(whole * (c + 1) + part * (c + 1) / n);
  return t;
}

}  // namespace

#endif  // LBM_TILING_H
