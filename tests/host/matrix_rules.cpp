// Prints, for each layer given as "N H W K bits", the tiles of a work group of the single kernel
// with its brackets on the matrix pipe (fused_matrix_tiles).
#include <cstdio>
#include <cstdlib>

#include "wino_kernels.hpp"

int main(int argc, char** argv) {
  for (int i = 1; i + 4 < argc; i += 5) {
    wino::Geometry g{};
    int v[5];
    for (int j = 0; j < 5; ++j) v[j] = std::atoi(argv[i + j]);
    g.m = 4, g.N = v[0], g.H = v[1], g.W = v[2], g.K = v[3];
    g.TH = (g.H + 3) / 4, g.TW = (g.W + 3) / 4, g.T = g.N * g.TH * g.TW;
    std::printf("%d\n", wino::fused_matrix_tiles(g, wino::fused_channels(v[4])));
  }
  return 0;
}
