// Prints, for each layer given as "m N H W C K bits", the launch shapes that the library's rules choose
// for it: tile rows of a work group of the contraction (contract_tile_rows), tiles of a work group of
// the single kernel (fused_tiles), blocks per wave of the fp32 contraction (f32_contract_blocks),
// whether dV and dU read dM into registers (backward_from_registers).
#include <cstdio>
#include <cstdlib>

#include "wino_kernels.hpp"

int main(int argc, char** argv) {
  for (int i = 1; i + 6 < argc; i += 7) {
    int v[7];
    for (int j = 0; j < 7; ++j) v[j] = std::atoi(argv[i + j]);
    wino::Geometry g{};
    g.m = v[0], g.N = v[1], g.H = v[2], g.W = v[3], g.C = v[4], g.K = v[5];
    g.TH = (g.H + g.m - 1) / g.m, g.TW = (g.W + g.m - 1) / g.m, g.T = g.N * g.TH * g.TW;
    const wino::F32Blocks w = wino::f32_contract_blocks(g);
    const wino::FromRegisters r = wino::backward_from_registers(g);
    std::printf("%d %d %d%d %d%d\n", wino::contract_tile_rows(g),
                wino::fused_tiles(g, wino::fused_channels(v[6])), w.t, w.k, r.dv, r.du);
  }
  return 0;
}
