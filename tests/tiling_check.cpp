// Check of the step kernels' tilings on the host: over grids up to the
// largest that are accepted, the tiles of the two-step kernel cover every
// band of rows once, in order, and the bands cover the grid.  Built and run
// by test_tiling.py.
#include <cstdio>

#include "tiling.h"

// 0 if the tiles of an nx x ny grid on `slots` wavefronts per XCD are right.
static int check(int nx, int ny, bool f32, int slots) {
  const int tiles = pair_tiles_of(nx, ny, slots, f32 ? 3.7 : 4.7), strips = pair_strips(nx);
  if (tiles == 0) return 0;
  if (tiles < strips) return 1;
  int rows_done = 0;
  for (int x = 0; x < kXcds; ++x) {
    const Band b = band_of(x, ny, 1, 0, 1);
    if (b.y0 != rows_done) return 2;
    rows_done = b.y1;
    for (int s = 0; s < strips; ++s) {
      int y = b.y0;
      for (int t = s; t < tiles; t += strips) {
        const PairTile p = pair_tile_of(x, t, ny, tiles, strips);
        if (p.strip != s || p.y0 != y || p.y1 < p.y0) return 3;
        y = p.y1;
      }
      if (y != b.y1) return 4;
    }
  }
  return rows_done == ny ? 0 : 5;
}

int main() {
  int bad = 0;
  for (const bool f32 : {false, true}) {
    const long long most = 0xFFFFFF00LL / 26 / (f32 ? 4 : 8);  // sites accepted
    for (const int slots : {32, 64, 128, 256, 512, 1024})
      for (const int nx : {3, 8, 16, 17, 56, 57, 64, 113, 1024, 6000, 100000, 2500000})
        for (const long long part : {1LL, 2LL, 7LL, 64LL, 1000LL}) {
          const int ny = int(most / nx / part);
          const int e = check(nx, ny, f32, slots);
          if (e) {
            std::printf("%s %d x %d, %d slots: error %d\n", f32 ? "float32" : "float64", nx, ny,
                        slots, e);
            ++bad;
          }
        }
  }
  if (!bad) std::puts("tiling ok");
  return bad ? 1 : 0;
}
