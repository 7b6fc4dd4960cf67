// Host check of the sixteen-bit pixel coordinates of the input transform on the matrix pipe: for every image
// edge that input_fits_matrix_pipe admits, each row and column of each tile is inside the image exactly where
// plain integers say so.  Prints the largest height and width admitted.
#include <cstdio>

#include "wino_kernels.hpp"

static bool edge_ok(int size, int tiles) {
  const wino::PixelPair last = {(unsigned short)(size - 1), (unsigned short)(size - 1)};
  for (int t = 0; t < tiles; ++t)
    for (int a = 0; a < 6; ++a) {
      const int at = 4 * t - 1 + a;
      const wino::PixelPair corner = {(unsigned short)(4 * t - 1), (unsigned short)(4 * t - 1)};
      // one coordinate at the edge under test, the other one at pixel 0
      const wino::PixelPair row = corner + wino::PixelPair{(unsigned short)a, (unsigned short)(1 - 4 * t)};
      const wino::PixelPair column = corner + wino::PixelPair{(unsigned short)(1 - 4 * t), (unsigned short)a};
      const bool want = at >= 0 && at < size;
      if (wino::inside_image(row, last) != want || wino::inside_image(column, last) != want)
        return std::printf("size %d, pixel %d\n", size, at), false;
    }
  return true;
}

int main() {
  int tallest = 0, widest = 0;
  for (int side = 0; side < 2; ++side)
    for (int size = 1; size < 65700; size = size == 70 ? 4000 : size == 4200 ? 65500 : size + 1) {
      wino::Geometry g{};
      g.N = 2, g.m = 4, g.C = g.K = 16;
      g.H = side ? 4 : size, g.W = side ? size : 4;
      g.TH = (g.H + 3) / 4, g.TW = (g.W + 3) / 4, g.T = g.N * g.TH * g.TW;
      if (!wino::input_fits_matrix_pipe(g, 1)) continue;
      (side ? widest : tallest) = size;
      if (!edge_ok(g.H, g.TH) || !edge_ok(g.W, g.TW)) return 1;
    }
  std::printf("ok %d %d\n", tallest, widest);
  return 0;
}
