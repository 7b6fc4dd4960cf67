// fp32 path (bits_in = 32): the same four stages of eq. 3 / eq. 4 without any
// cast, on float tensors with the layouts of the int8 path (x NHWC, w KCRS,
// U [n*n][T][C], V [n*n][K][C], M [n*n][T][K], y NHWC), checked against fp64.
// One lane per item in the transforms, which are bound by the bytes of U, M and
// y; the contraction runs on the matrix cores.
#include <cfloat>

#include "wino_kernels.hpp"
#include "wino_real_brackets.hpp"

namespace wino {

// The pair of brackets of eq. 2 / eq. 4 multiplies out to one canonical bracket (asserted at compile
// time in wino_tables.hpp).  In the Legendre base that product is evaluated in double between its fp32
// input and its fp32 result, so nothing of the pair's cancelling terms is lost; the canonical base
// keeps plain fp32.
template <bool LEG, const RMat& T>
__device__ __forceinline__ void bracket(const float (&x)[T.cols][T.cols], float (&out)[T.rows][T.rows]) {
  if constexpr (LEG)
    bracket_d<T>(x, out);
  else
    bracket_f<T>(x, out);
}

template <int M, bool LEG>
__device__ __forceinline__ void weight_f32_body(const float* __restrict__ w, float* __restrict__ V,
                                                const Geometry& g, unsigned block) {
  constexpr int n = M + 2;
  using TB = TabF<M>;
  const long gid = (long)block * 256 + threadIdx.x;
  const long KC = (long)g.K * g.C;
  if (gid >= KC) return;
  float wi[3][3];
  rfor<0, 3>([&](auto a) {
    rfor<0, 3>([&](auto b) { wi[a][b] = w[gid * 9 + decltype(a)::value * 3 + decltype(b)::value]; });
  });
  float v[n][n];
  bracket<LEG, TB::G>(wi, v);
  rfor<0, n>([&](auto i) {
    rfor<0, n>([&](auto j) {
      V[(long)(decltype(i)::value * n + decltype(j)::value) * KC + gid] = v[i][j];
    });
  });
}

template <int M, bool LEG>
__device__ __forceinline__ void input_f32_body(const float* __restrict__ x, float* __restrict__ U,
                                               const Geometry& g, Divider by_c, unsigned block) {
  constexpr int n = M + 2;
  using TB = TabF<M>;
  const long total = (long)g.T * g.C;
  int t, c;
  item_of_lane(block, g.C, by_c, t, c);
  if (t >= g.T) return;
  int b, ty, tx;
  tile_coords(g, t, b, ty, tx);
  const float* xb = x + (long)b * g.H * g.W * g.C + c;
  float xi[n][n];
  rfor<0, n>([&](auto a) {
    rfor<0, n>([&](auto bb) {
      const int h = ty * M - 1 + decltype(a)::value;
      const int ww = tx * M - 1 + decltype(bb)::value;
      float v = 0.f;
      if ((unsigned)h < (unsigned)g.H && (unsigned)ww < (unsigned)g.W)
        v = xb[((long)h * g.W + ww) * g.C];
      xi[a][bb] = v;
    });
  });
  float u[n][n];
  bracket<LEG, TB::BT>(xi, u);
  float* ub = U + (long)t * g.C + c;
  rfor<0, n>([&](auto i) {
    rfor<0, n>([&](auto j) {
      __builtin_nontemporal_store(u[i][j], ub + (long)(decltype(i)::value * n + decltype(j)::value) * total);
    });
  });
}

// The two operand transforms are independent of each other: one launch, the first nb_w work groups
// take filters, the rest (tile, channel) items.  Either part may be empty.  Bound by the bytes of U:
// 2048 tiles of 128 channels (46 MB with x) 12.7 us; 5.2 + 15.6 us as two launches with run-time
// divisions per lane and both brackets of a Legendre pair evaluated one after the other in double.
template <int M, bool LEG>
__global__ __launch_bounds__(256) void k_operands_f32(const float* __restrict__ x,
                                                      float* __restrict__ U,
                                                      const float* __restrict__ w,
                                                      float* __restrict__ V, Geometry g,
                                                      Divider by_c, unsigned nb_w) {
  if (blockIdx.x < nb_w)
    weight_f32_body<M, LEG>(w, V, g, blockIdx.x);
  else
    input_f32_body<M, LEG>(x, U, g, by_c, blockIdx.x - nb_w);
}

// ---------------------------------------------------------------------------
// Contraction: M[p][t][k] = sum_c U[p][t][c] V[p][k][c], n*n fp32 GEMMs on the bf16 matrix pipe
// without giving up fp32 accuracy.  Both operands are scaled by 2^24 and cut, while they are staged,
// into three bf16 pieces, each rounded to nearest: x = h + m + l exactly, |m| <= 2^-8 |x|,
// |l| <= 2^-17 |x|.  The scale keeps every piece of every fp32 number, subnormals included, a normal
// bf16 (a piece is a multiple of the last bit of x, at least 2^-149): unscaled, l is lost below 2^-110
// and m below 2^-118, and results of such operands had a relative error of up to 3e-3.  Six of the nine
// piece products are accumulated in fp32 (exact products, smallest first), and the sums are scaled by
// 2^-48; the three that are left out (ml, lm, ll) are together at most 2^-24 of |x y|, what rounding
// one fp32 product may lose.  Error against 64 bits (2-norm), C = 16, 128, 512: 3.3e-8, 1.6e-7, 3.4e-7; plain
// fp32 sums 7.4e-8, 2.0e-7, 4.1e-7.  Infinities, NaNs, operands from 2^103 and sums from 2^80 on leave that
// range: work groups in which a result is not finite sum again in plain fp32.
//
// Work group = 4 waves (2 x 2) = (64 MB) tiles x (64 NB) output channels, a wave MB x NB blocks of
// 32 x 32 (f32_contract_blocks).  The channels run in chunks of 32 staged through LDS ([row][channel] per
// piece), the next chunk's global loads in flight during the 12 MB NB MFMAs of a wave.
// What bounds it: at C = 128 the bytes of U and M.  2048 tiles, C = K = 128 (78 MB, 2.4 GFLOP): 160 us
// with one lane per output and both panels in LDS as fp32, 23.3 us here (3.3 TB/s), both repeated on
// their own; 28.9 us between the other kernels of a layer.  Before the scale, 23.9 us; with 64-row or 64-column
// blocks 25.4; with padded rows (61 KB of LDS, two groups per compute unit instead of three, so that
// the 576 groups run in two rounds) 28.8 us.
// ---------------------------------------------------------------------------
using v2f = __attribute__((ext_vector_type(2))) float;
using v4f = __attribute__((ext_vector_type(4))) float;
// The same in a tensor that may start at any float.
typedef v4f v4f_any __attribute__((aligned(4)));
using v2u = __attribute__((ext_vector_type(2))) unsigned;
using v16f = __attribute__((ext_vector_type(16))) float;
using bf16x2 = __attribute__((ext_vector_type(2))) __bf16;
using bf16x8 = __attribute__((ext_vector_type(8))) __bf16;

constexpr int kF32Chunk = 32;  // channels staged at a time
constexpr int kF32Row = kF32Chunk;   // bf16 per staged row
// Position of 16-byte segment q (channels 8 q .. 8 q + 7) in a staged row: four rows cover all banks,
// so the segment index is XOR-ed with the row's bits 2 and 3 and the 16 rows of a fragment-read
// phase fall on distinct banks.
__device__ __forceinline__ int f32_seg(int row, int q) { return row * kF32Row + 8 * (q ^ ((row >> 2) & 3)); }

constexpr float kF32Up = 0x1p24f, kF32Down = 0x1p-48f;   // scale of the operands, of the sums
// Two values as bf16 pieces, the first at the lower address of each packed pair.
__device__ __forceinline__ void split3_rne(float a, float b, unsigned& h, unsigned& m, unsigned& l) {
  auto pack = [](float u, float v) {
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v2f{u, v}, bf16x2));
  };
  h = pack(a, b);
  a -= __uint_as_float(h << 16), b -= __uint_as_float(h & 0xffff0000u);
  m = pack(a, b);
  l = pack(a - __uint_as_float(m << 16), b - __uint_as_float(m & 0xffff0000u));
}

constexpr int f32_lds_floats(int mb, int nb) {
  const int staged = 3 * (mb + nb) * 64 * kF32Row / 2, out = 4 * 32 * (32 * nb + 4);
  return staged > out ? staged : out;
}

// STREAM: M leaves in nontemporal stores.
template <int MB, int NB, bool STREAM>
__global__ __launch_bounds__(256, 3) void k_contract_f32(const float* __restrict__ U,
                                                         const float* __restrict__ V,
                                                         float* __restrict__ Mo, int T, int C, int K,
                                                         int tblocks, int kblocks, int units) {
  constexpr int TR = 64 * MB, TC = 64 * NB;
  __shared__ __attribute__((aligned(16))) float smem[f32_lds_floats(MB, NB)];
  unsigned short* As = reinterpret_cast<unsigned short*>(smem);      // [piece][tile][channel]
  unsigned short* Bs = As + 3 * TR * kF32Row;                        // [piece][k][channel]
  // Work-group ids go round-robin over the 8 XCDs.  A unit is (point, tile block); an XCD takes a
  // contiguous eighth of the units with all their k blocks, so that a point's V enters one or two
  // L2s and a tile block's U exactly one.
  const unsigned xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int unit = (int)(xcd * ((unsigned)(units + 7) / 8) + slot / (unsigned)kblocks);
  // padding slots: past the last unit, or past this XCD's eighth (uniform exit, no barrier yet)
  if (unit >= units) return;
  const int p = unit / tblocks, row0 = (unit - p * tblocks) * TR;
  const int col0 = (int)(slot % (unsigned)kblocks) * TC;
  const float* Up = U + ((long)p * T + row0) * C;
  const float* Vp = V + ((long)p * K + col0) * C;
  const int trows = T - row0, krows = K - col0;                      // rows that exist (>= 1)
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int srow = tid >> 3, sq = 4 * (tid & 7);                     // staging: 8 lanes per row

  v4f ra[2 * MB], rb[2 * NB];
  auto fetch = [&](int c0) {
    const bool cok = c0 + sq < C;                                    // C is a multiple of 16
#pragma unroll
    for (int it = 0; it < 2 * MB; ++it) {
      ra[it] = v4f{0.f, 0.f, 0.f, 0.f};
      if (cok && srow + 32 * it < trows)
        ra[it] = *reinterpret_cast<const v4f_any*>(Up + (long)(srow + 32 * it) * C + c0 + sq);
    }
#pragma unroll
    for (int it = 0; it < 2 * NB; ++it) {
      rb[it] = v4f{0.f, 0.f, 0.f, 0.f};
      if (cok && srow + 32 * it < krows)
        rb[it] = *reinterpret_cast<const v4f_any*>(Vp + (long)(srow + 32 * it) * C + c0 + sq);
    }
  };
  auto put = [&](unsigned short* base, int rows, int row, const v4f& v) {
    unsigned h[2], m[2], l[2];
    split3_rne(v[0] * kF32Up, v[1] * kF32Up, h[0], m[0], l[0]);
    split3_rne(v[2] * kF32Up, v[3] * kF32Up, h[1], m[1], l[1]);
    unsigned short* at = base + f32_seg(row, sq >> 3) + (sq & 4);
    *reinterpret_cast<v2u*>(at) = v2u{h[0], h[1]};
    *reinterpret_cast<v2u*>(at + rows * kF32Row) = v2u{m[0], m[1]};
    *reinterpret_cast<v2u*>(at + 2 * rows * kF32Row) = v2u{l[0], l[1]};
  };

  v16f acc[MB][NB];
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;
  const int wr = (wave >> 1) * 32 * MB, wc = (wave & 1) * 32 * NB;
  const int l32 = lane & 31, lk = lane >> 5;
  // MFMA operands: lane -> row lane % 32, channels 8 (lane / 32) .. + 7 of each 16

  fetch(0);
  for (int c0 = 0; c0 < C; c0 += kF32Chunk) {
    __syncthreads();                  // the previous chunk's fragment reads are done
#pragma unroll
    for (int it = 0; it < 2 * MB; ++it) put(As, TR, srow + 32 * it, ra[it]);
#pragma unroll
    for (int it = 0; it < 2 * NB; ++it) put(Bs, TC, srow + 32 * it, rb[it]);
    __syncthreads();
    if (c0 + kF32Chunk < C) fetch(c0 + kF32Chunk);
#pragma unroll
    for (int kk = 0; kk < kF32Chunk; kk += 16) {
      if (kk && c0 + kk >= C) break;   // uniform: half a chunk
      bf16x8 fA[3][MB], fB[3][NB];
#pragma unroll
      for (int q = 0; q < 3; ++q) {
#pragma unroll
        for (int a = 0; a < MB; ++a)
          fA[q][a] = *reinterpret_cast<const bf16x8*>(As + (q * TR + a * 32) * kF32Row + f32_seg(wr + l32, (kk >> 3) + lk));
#pragma unroll
        for (int b = 0; b < NB; ++b)
          fB[q][b] = *reinterpret_cast<const bf16x8*>(Bs + (q * TC + b * 32) * kF32Row + f32_seg(wc + l32, (kk >> 3) + lk));
      }
      // (piece of U, piece of V), smallest products first
      constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
      for (int q = 0; q < 6; ++q)
#pragma unroll
        for (int a = 0; a < MB; ++a)
#pragma unroll
          for (int b = 0; b < NB; ++b)
            acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fA[pa[q]][a], fB[pb[q]][b], acc[a][b], 0, 0, 0);
    }
  }

  float inf_or_nan = 0.f;             // turns NaN where a sum is not finite
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        acc[a][b][i] *= kF32Down;
        inf_or_nan = __builtin_fmaf(acc[a][b][i], 0.f, inf_or_nan);
      }
  float* Mp = Mo + ((long)p * T + row0) * K + col0;
  // acc[a][b][i] holds (tile = 32 a + (i / 4) * 8 + (lane / 32) * 4 + i % 4, k = 32 b + lane % 32) of
  // the wave's block.  A work group with a sum that is not finite forms all of its sums in plain fp32
  // instead, channel by channel, one 32 x 32 block of each wave at a time from panels in LDS.  2048
  // tiles, C = K = 128, all NaN: 120 us (2842 with every such sum on its own from memory).
  if (__builtin_expect(__syncthreads_or(inf_or_nan != 0.f), 0)) {
    constexpr int kRowF = kF32Chunk + 4;
    float* Af = smem;
    float* Bf = smem + TR * kRowF;
    static_assert((TR + TC) * kRowF <= f32_lds_floats(MB, NB));
#pragma unroll 1
    for (int ab = 0; ab < MB * NB; ++ab) {
      const int r32 = wr + 32 * (ab / NB) + lk * 4, k32 = wc + 32 * (ab % NB) + l32;
      float sum[16] = {};
#pragma unroll 1
      for (int c0 = 0; c0 < C; c0 += kF32Chunk) {
        fetch(c0);                    // zeros past C, the last tile and the last output channel
        __syncthreads();
#pragma unroll
        for (int it = 0; it < 2 * MB; ++it) *reinterpret_cast<v4f*>(Af + (srow + 32 * it) * kRowF + sq) = ra[it];
#pragma unroll
        for (int it = 0; it < 2 * NB; ++it) *reinterpret_cast<v4f*>(Bf + (srow + 32 * it) * kRowF + sq) = rb[it];
        __syncthreads();
        const int cend = min(kF32Chunk, C - c0);
#pragma unroll 1
        for (int c = 0; c < cend; c += 4) {
          const v4f v = *reinterpret_cast<const v4f*>(Bf + k32 * kRowF + c);
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const v4f u = *reinterpret_cast<const v4f*>(Af + (r32 + (i >> 2) * 8 + (i & 3)) * kRowF + c);
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[i] = __builtin_fmaf(u[e], v[e], sum[i]);
          }
        }
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int row = r32 + (i >> 2) * 8 + (i & 3);
        if (row < trows && k32 < krows) Mp[(long)row * K + k32] = sum[i];
      }
    }
    return;
  }

  // 32 tiles at a time leave through the wave's own part of LDS in 16-byte stores.
  constexpr int kLdC = 32 * NB + 4;
  float* Cs = smem + wave * 32 * kLdC;
#pragma unroll
  for (int a = 0; a < MB; ++a) {
    __syncthreads();                  // the fragments (a = 0) resp. the previous rows have been read
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i)
        Cs[((i >> 2) * 8 + lk * 4 + (i & 3)) * kLdC + 32 * b + l32] = acc[a][b][i];
    __syncthreads();
#pragma unroll
    for (int it = 0; it < 4 * NB; ++it) {
      const int idx = lane + it * 64;
      const int r = idx / (8 * NB), q = 4 * (idx % (8 * NB));
      const int row = wr + 32 * a + r, col = wc + q;
      if (row < trows && col < krows) { // K is a multiple of 16: a quad is inside or outside
        const v4f v = *reinterpret_cast<const v4f*>(Cs + r * kLdC + q);
        v4f_any* at = reinterpret_cast<v4f_any*>(Mp + (long)row * K + col);
        if constexpr (STREAM)
          __builtin_nontemporal_store(v, at);
        else
          *at = v;
      }
    }
  }
}

// STREAM: M is read in nontemporal loads.
template <int M, bool LEG, bool STREAM>
__global__ __launch_bounds__(256) void k_output_f32(const float* __restrict__ Mq,
                                                    float* __restrict__ y, Geometry g,
                                                    Divider by_k, int relu) {
  constexpr int n = M + 2;
  using TB = TabF<M>;
  const long total = (long)g.T * g.K;
  int t, k;
  item_of_lane(blockIdx.x, g.K, by_k, t, k);
  if (t >= g.T) return;
  int b, ty, tx;
  tile_coords(g, t, b, ty, tx);
  const float* mb = Mq + (long)t * g.K + k;
  float mi[n][n];
  rfor<0, n>([&](auto i) {
    rfor<0, n>([&](auto j) {
      const float* at = mb + (long)(decltype(i)::value * n + decltype(j)::value) * total;
      mi[i][j] = STREAM ? __builtin_nontemporal_load(at) : *at;
    });
  });
  float out[M][M];
  bracket<LEG, TB::AT>(mi, out);
  float* yb = y + (((long)b * g.H + ty * M) * g.W + tx * M) * g.K + k;
  rfor<0, M>([&](auto i) {
    rfor<0, M>([&](auto j) {
      constexpr int I = decltype(i)::value, J = decltype(j)::value;
      if (ty * M + I < g.H && tx * M + J < g.W) {
        const float v = out[i][j];
        __builtin_nontemporal_store(relu ? fmaxf(v, 0.f) : v, yb + ((long)I * g.W + J) * g.K);
      }
    });
  });
}

// M passes by the L2s (nontemporal) where it and U do not fit them (32 MB).  Layer us, nontemporal /
// plain, the same tensors over and over: F(2,3), 16384 tiles, C = K = 16 (32 MB) 29.8 / 28.2, F(6,3), 512
// tiles, C = K = 128 (32 MB) 37.7 / 30.6; four sets of tensors in turn: 23.5 / 23.1 and 29.1 / 29.1.  Past
// that it depends on what else the caches hold: F(4,3), 2048 tiles, C = K = 128 (72 MB) 50.6 / 47.8 over and
// over, 50.3 / 50.7 in turn.
static bool f32_streams_m(const Geometry& g) {
  return 4L * (g.m + 2) * (g.m + 2) * g.T * ((long)g.C + g.K) > (32L << 20);
}

template <int MB, int NB>
static hipError_t contract_f32_shape(const Geometry& g, const float* U, const float* V, float* Mo,
                                     hipStream_t st) {
  const int tblocks = (g.T + 64 * MB - 1) / (64 * MB), kblocks = (g.K + 64 * NB - 1) / (64 * NB);
  const long units = (long)(g.m + 2) * (g.m + 2) * tblocks;
  const long blocks = (units + 7) / 8 * 8 * kblocks;
  if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks), bs(256);
  if (f32_streams_m(g))
    wino_launch((k_contract_f32<MB, NB, true>), grid, bs, st, U, V, Mo, g.T, g.C, g.K, tblocks, kblocks, (int)units);
  else
    wino_launch((k_contract_f32<MB, NB, false>), grid, bs, st, U, V, Mo, g.T, g.C, g.K, tblocks, kblocks, (int)units);
  return hipGetLastError();
}

static hipError_t contract_f32(const Geometry& g, const float* U, const float* V, float* Mo,
                               hipStream_t st) {
  const F32Blocks w = f32_contract_blocks(g);
  if (w.t == 2)
    return w.k == 2 ? contract_f32_shape<2, 2>(g, U, V, Mo, st) : contract_f32_shape<2, 1>(g, U, V, Mo, st);
  return w.k == 2 ? contract_f32_shape<1, 2>(g, U, V, Mo, st) : contract_f32_shape<1, 1>(g, U, V, Mo, st);
}

static inline unsigned nblk(long items) { return (unsigned)((items + 255) / 256); }

template <int M>
static hipError_t operands_f32(const Geometry& g, bool leg, const float* x, float* U, const float* w,
                               float* V, hipStream_t st) {
  const unsigned nb_in = x ? nblk((long)g.T * g.C) : 0, nb_w = w ? nblk((long)g.K * g.C) : 0;
  if (nb_in + nb_w == 0) return hipSuccess;
  if (leg)
    wino_launch((k_operands_f32<M, true>), dim3(nb_in + nb_w), dim3(256), st, x, U, w, V, g,
                divider_of(g.C), nb_w);
  else
    wino_launch((k_operands_f32<M, false>), dim3(nb_in + nb_w), dim3(256), st, x, U, w, V, g,
                divider_of(g.C), nb_w);
  return hipGetLastError();
}

template <int M, bool LEG>
static hipError_t output_f32_base(const Geometry& g, const float* Mq, float* y, bool relu, hipStream_t st) {
  const dim3 grid(nblk((long)g.T * g.K)), bs(256);
  if (f32_streams_m(g))
    wino_launch((k_output_f32<M, LEG, true>), grid, bs, st, Mq, y, g, divider_of(g.K), relu ? 1 : 0);
  else
    wino_launch((k_output_f32<M, LEG, false>), grid, bs, st, Mq, y, g, divider_of(g.K), relu ? 1 : 0);
  return hipGetLastError();
}

template <int M>
static hipError_t output_f32(const Geometry& g, bool leg, const float* Mq, float* y, bool relu,
                             hipStream_t st) {
  return leg ? output_f32_base<M, true>(g, Mq, y, relu, st) : output_f32_base<M, false>(g, Mq, y, relu, st);
}

hipError_t launch_operands_f32(const Geometry& g, bool legendre, const float* x, float* U,
                               const float* w, float* V, hipStream_t st) {
  switch (g.m) {
    case 2: return operands_f32<2>(g, legendre, x, U, w, V, st);
    case 4: return operands_f32<4>(g, legendre, x, U, w, V, st);
    case 6: return operands_f32<6>(g, legendre, x, U, w, V, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_contract_f32(const Geometry& g, const float* U, const float* V, float* Mo,
                               hipStream_t st) {
  return (long)g.T * g.K == 0 ? hipSuccess : contract_f32(g, U, V, Mo, st);
}

hipError_t launch_output_f32(const Geometry& g, bool legendre, const float* Mq, float* y, bool relu,
                             hipStream_t st) {
  if ((long)g.T * g.K == 0) return hipSuccess;
  switch (g.m) {
    case 2: return output_f32<2>(g, legendre, Mq, y, relu, st);
    case 4: return output_f32<4>(g, legendre, Mq, y, relu, st);
    case 6: return output_f32<6>(g, legendre, Mq, y, relu, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace wino
