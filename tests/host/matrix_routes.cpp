// Prints, for each F(4,3) Legendre layer given as "N H W C K", whether the matrix pipe takes its input transform alone,
// its input transform beside its filters, its output transform to fp32 and to int8 (int8 M).
#include <cstdio>
#include <cstdlib>

#include "wino_kernels.hpp"

int main(int argc, char** argv) {
  for (int i = 1; i + 4 < argc; i += 5) {
    wino::Geometry g{};
    int v[5];
    for (int j = 0; j < 5; ++j) v[j] = std::atoi(argv[i + j]);
    g.m = 4, g.N = v[0], g.H = v[1], g.W = v[2], g.C = v[3], g.K = v[4];
    g.TH = (g.H + 3) / 4, g.TW = (g.W + 3) / 4, g.T = g.N * g.TH * g.TW;
    std::printf("%d%d%d%d\n", wino::input_on_matrix_pipe(g, 1, 0), wino::input_on_matrix_pipe(g, 1, (long)g.K * g.C),
                wino::output_on_matrix_pipe(g, 0), wino::output_on_matrix_pipe(g, 2));
  }
  return 0;
}
