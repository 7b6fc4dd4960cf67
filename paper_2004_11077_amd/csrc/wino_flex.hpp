// "Flex" layer (Section 4.2): the brackets with G_P, B_P, A_P (G, B, A in the
// canonical base) use fp32 matrices supplied at run time -- trained parameters
// -- while the brackets with the fixed P^{-1} keep the exact integer arithmetic
// of the static kernels.  A run-time bracket T x T^T is evaluated on the
// integer codes in fp32 in one fixed order,
//     left[i][b] = ((T[i][0] x[0][b] + T[i][1] x[1][b]) + ...)
//     out[i][j]  = ((left[i][0] T[j][0] + left[i][1] T[j][1]) + ...)
// every product and every sum rounded to fp32, never fused, so that a CPU
// reference can follow it bit for bit; its cast uses one multiplier for the
// whole tensor.  Trained matrices have no zeros or powers of two to exploit: a bracket is dense.
#pragma once
#include "wino_transforms.hpp"

namespace wino {

// x: integer codes held as floats.
template <int ROWS, int COLS>
__device__ __forceinline__ void fsandwich(const float* __restrict__ Tm,
                                          const float (&x)[COLS][COLS], float (&out)[ROWS][ROWS]) {
#pragma clang fp contract(off)
  float left[ROWS][COLS];
  static_for<0, ROWS>([&](auto i) {
    static_for<0, COLS>([&](auto b) {
      float acc = Tm[decltype(i)::value * COLS] * x[0][b];
      static_for<1, COLS>([&](auto a) {
        const float prod = Tm[decltype(i)::value * COLS + decltype(a)::value] * x[a][b];
        acc = acc + prod;
      });
      left[i][b] = acc;
    });
  });
  static_for<0, ROWS>([&](auto i) {
    static_for<0, ROWS>([&](auto j) {
      float acc = left[i][0] * Tm[decltype(j)::value * COLS];
      static_for<1, COLS>([&](auto b) {
        const float prod = left[i][b] * Tm[decltype(j)::value * COLS + decltype(b)::value];
        acc = acc + prod;
      });
      out[i][j] = acc;
    });
  });
}

template <int R>
__device__ __forceinline__ void to_floats(const int (&x)[R][R], float (&f)[R][R]) {
  static_for<0, R>([&](auto i) { static_for<0, R>([&](auto j) { f[i][j] = (float)x[i][j]; }); });
}

// The input of a run-time bracket as floats: the codes themselves (canonical base) or the codes of
// the cast after the integer bracket T = P^{-T}, |x| <= IN_MAX (Legendre).  A cast's biased float
// 1.5 * 2^23 + q becomes q by one exact subtraction.
template <const IMat& T, int64_t IN_MAX, bool LEG>
__device__ __forceinline__ void flex_input(const int (&x)[T.cols][T.cols], const MultTable& inner,
                                           float (&f)[T.rows][T.rows]) {
  if constexpr (LEG) {
    acc_t<T, IN_MAX> num[T.rows][T.rows];
    sandwich<T, IN_MAX>(x, num);
    uint32_t bits[T.rows][T.rows];
    cast_result_biased<T, IN_MAX, true>(num, inner, 127.f, bits);
    static_for<0, T.rows>([&](auto i) {
      static_for<0, T.rows>([&](auto j) { f[i][j] = __uint_as_float(bits[i][j]) - kMagic; });
    });
  } else {
    to_floats<T.cols>(x, f);
  }
}

// The stages proper: the fetches and stores of the fixed-matrix transforms (weight_items,
// input_items, fetch_m: 16-byte accesses through LDS) around the run-time brackets.  Bound by the
// vector ALU: a dense bracket is 2 n^3 separately rounded products and as many sums (F(4,3): 829
// instructions of an input item's 1200, 8 us at full issue rate for 262144 items and their filters).
// 1024 tiles, C = K = 256: operand transforms 21.0 us with a byte load per pixel and a byte store per
// code, 14.8 us with 16-byte accesses through LDS; output transform 11.3 -> 9.8 us.  The dealing to
// XCDs takes the contraction between them from 9.5 to 8.4 us.  That is for the same tensors call after
// call (layer 36.4 -> 30.5 us), where part of what the dealing saves are lines that the call before left in
// the L2s; the first call on new tensors takes 55 to 58 us against 58 to 59.
template <int M, bool LEG>
__device__ __forceinline__ void flex_weight_body(const int8_t* __restrict__ w, int8_t* __restrict__ V,
                                                 const Geometry& g, const FlexMats& fm,
                                                 const StageMults& mu, float mult_first,
                                                 unsigned block) {
  constexpr int n = M + 2;
  using TB = Tab<M>;
  weight_items<M>(w, V, g, block, [&](const int (&wi)[3][3], int (&q)[n][n]) {
    float wf[3][3], val[n][n];
    to_floats<3>(wi, wf);
    fsandwich<n, 3>(fm.GP, wf, val);
    uint32_t w1[n][n];
    static_for<0, n>([&](auto i) {
      static_for<0, n>([&](auto j) { w1[i][j] = cast_biased(val[i][j], mult_first, 127.f); });
    });
    if constexpr (LEG) {
      acc_t<TB::Pinv, 127> num2[n][n];
      sandwich_codes<TB::Pinv, 127>(w1, num2);
      cast_result<TB::Pinv, 127, true>(num2, mu.outer, 127.f, q);
    } else {
      static_for<0, n>([&](auto i) { static_for<0, n>([&](auto j) { q[i][j] = (int)w1[i][j]; }); });
    }
  });
}

template <int M, bool LEG, bool WHOLE>
__device__ __forceinline__ void flex_input_body(const int8_t* __restrict__ x, int8_t* __restrict__ U,
                                                const Geometry& g, const FlexMats& fm,
                                                const StageMults& mu, float mult_u,
                                                unsigned block) {
  constexpr int n = M + 2;
  using TB = Tab<M>;
  input_items<M, WHOLE>(x, U, g, block, [&](const int (&xi)[n][n], int (&q)[n][n]) {
    float xf[n][n], val[n][n];
    flex_input<TB::PinvT, 127, LEG>(xi, mu.inner, xf);
    fsandwich<n, n>(fm.BPT, xf, val);
    static_for<0, n>([&](auto i) {
      static_for<0, n>([&](auto j) { q[i][j] = (int)cast_biased(val[i][j], mult_u, 127.f); });
    });
  });
}

template <int M, bool LEG>
__global__ __launch_bounds__(256) void k_flex_weight(const int8_t* __restrict__ w,
                                                     int8_t* __restrict__ V, Geometry g, FlexMats fm,
                                                     StageMults mu, float mult_first) {
  flex_weight_body<M, LEG>(w, V, g, fm, mu, mult_first, blockIdx.x);
}

template <int M, bool LEG, bool WHOLE>
__global__ __launch_bounds__(256) void k_flex_input(const int8_t* __restrict__ x,
                                                    int8_t* __restrict__ U, Geometry g, FlexMats fm,
                                                    StageMults mu, float mult_u) {
  flex_input_body<M, LEG, WHOLE>(x, U, g, fm, mu, mult_u, image_on_one_xcd(g, blockIdx.x));
}

// Both operand transforms of a layer in one launch: the slots, the padding and the dealing to XCDs
// are those of k_operand_transforms.
template <int M, bool LEG, bool WHOLE>
__global__ __launch_bounds__(256) void k_flex_operands(const int8_t* __restrict__ x,
                                                       int8_t* __restrict__ U,
                                                       const int8_t* __restrict__ w,
                                                       int8_t* __restrict__ V, Geometry g,
                                                       FlexMats fm, StageMults mu_in, float mult_u,
                                                       StageMults mu_w, float mult_first,
                                                       unsigned nb_in) {
  const unsigned wslots = gridDim.x - nb_in;          // a multiple of 8
  if (blockIdx.x >= wslots)
    flex_input_body<M, LEG, WHOLE>(x, U, g, fm, mu_in, mult_u, image_on_one_xcd(g, blockIdx.x - wslots));
  else if (blockIdx.x < weight_blocks(g))             // the padding slots have nothing to do
    flex_weight_body<M, LEG>(w, V, g, fm, mu_w, mult_first, blockIdx.x);
}

// OUT: 0 fp32 (mult_out = scale of the bracket's input), 2 int8 codes
// (mult_out = that scale / s_y).  WHOLE, addresses and dealing as in k_output_transform.
template <int M, bool LEG, typename MT, int OUT, bool WHOLE>
__global__ __launch_bounds__(256) void k_flex_output(const MT* __restrict__ Mq, void* __restrict__ yv,
                                                     Geometry g, Divider by_k, FlexMats fm,
                                                     StageMults mu, float mult_out, int relu) {
  constexpr int n = M + 2;
  const int tid = threadIdx.x;
  const unsigned block = WHOLE ? image_on_one_xcd(g, blockIdx.x) : blockIdx.x;
  const long total = (long)g.T * g.K;
  int t, k;
  if constexpr (WHOLE) {
    t = (int)fast_div(block, g.mul_kg, g.sh_kg);
    k = (int)(block - (unsigned)t * (unsigned)(g.K >> 8)) * 256 + tid;
  } else {
    item_of_lane(block, g.K, by_k, t, k);
  }
  const bool active = WHOLE || t < g.T;
  int xi[n][n];
  fetch_m<n, WHOLE>(Mq, total, (long)block * 256, active, t, k, g.K, xi);
  if (!active) return;
  int tx, ty, b;
  tile_coords(g, t, b, ty, tx);
  float xf[n][n], val[M][M];
  flex_input<Tab<M>::PinvT, MTraits<MT>::in_max, LEG>(xi, mu.inner, xf);
  fsandwich<M, n>(fm.APT, xf, val);
  // ReLU as a lower bound on the bit pattern (none: below every value)
  const int lo = relu ? 0 : (int)0x80000000;
  constexpr int YB = OUT == 2 ? 1 : 4;               // bytes of one output
  const long ytile = (((long)b * g.H + ty * M) * g.W + tx * M) * g.K;
  char* ybase = static_cast<char*>(yv) + (ytile + (WHOLE ? k - tid : k)) * YB;
  unsigned lane_off = WHOLE ? (unsigned)tid * YB : 0u;
  const int wk = g.W * g.K;
  static_for<0, M>([&](auto i) {
    static_for<0, M>([&](auto j) {
      if (ty * M + decltype(i)::value < g.H && tx * M + decltype(j)::value < g.W) {
        const int rel = decltype(i)::value * wk + decltype(j)::value * g.K;
        if constexpr (WHOLE) asm("" : "+v"(lane_off));
        char* at = ybase + (long)rel * YB + lane_off;
        if constexpr (OUT == 0) {
          const float v = val[i][j] * mult_out;
          __builtin_nontemporal_store(max(__float_as_int(v), lo), reinterpret_cast<int*>(at));
        } else {
          const int v = cast_code(val[i][j], mult_out, 127.f);
          __builtin_nontemporal_store((int8_t)max(v, lo), reinterpret_cast<int8_t*>(at));
        }
      }
    });
  });
}

template <int M>
hipError_t PerMFlex<M>::weight(const Geometry& g, bool leg, const int8_t* w, int8_t* V,
                               const FlexMats& fm, const StageMults& mu, float mult_first,
                               hipStream_t st) {
  const dim3 nb(blocks_for((long)g.K * g.C)), bs(256);
  if (leg) wino_launch((k_flex_weight<M, true>), nb, bs, st, w, V, g, fm, mu, mult_first);
  else wino_launch((k_flex_weight<M, false>), nb, bs, st, w, V, g, fm, mu, mult_first);
  return hipGetLastError();
}

template <int M>
hipError_t PerMFlex<M>::input(const Geometry& g0, bool leg, const int8_t* x, int8_t* U,
                              const FlexMats& fm, const StageMults& mu, float mult_u, hipStream_t st) {
  const dim3 nb(blocks_for((long)g0.T * g0.C)), bs(256);
  const bool whole = whole_tiles(g0.C, g0.H, g0.W);
  const Geometry g = with_image_groups(g0, whole);
  if (leg && whole) wino_launch((k_flex_input<M, true, true>), nb, bs, st, x, U, g, fm, mu, mult_u);
  else if (leg) wino_launch((k_flex_input<M, true, false>), nb, bs, st, x, U, g, fm, mu, mult_u);
  else if (whole) wino_launch((k_flex_input<M, false, true>), nb, bs, st, x, U, g, fm, mu, mult_u);
  else wino_launch((k_flex_input<M, false, false>), nb, bs, st, x, U, g, fm, mu, mult_u);
  return hipGetLastError();
}

template <int M>
hipError_t PerMFlex<M>::operands(const Geometry& g0, bool leg, const int8_t* x, int8_t* U,
                                 const int8_t* w, int8_t* V, const FlexMats& fm,
                                 const StageMults& mu_in, float mult_u, const StageMults& mu_w,
                                 float mult_first, hipStream_t st) {
  const unsigned nb_in = input_blocks(g0), nb_w = weight_blocks(g0);
  const bool whole = whole_tiles(g0.C, g0.H, g0.W);
  const Geometry g = with_image_groups(g0, whole);
  const dim3 grid(nb_in + (nb_w + 7) / 8 * 8), bs(256);   // filter slots padded to whole sets of XCDs
#define WINO_FLEX_OPS(LEG_, WHOLE_)                                                              \
  wino_launch((k_flex_operands<M, LEG_, WHOLE_>), grid, bs, st, x, U, w, V, g, fm, mu_in, mult_u, \
              mu_w, mult_first, nb_in)
  if (leg && whole) WINO_FLEX_OPS(true, true);
  else if (leg) WINO_FLEX_OPS(true, false);
  else if (whole) WINO_FLEX_OPS(false, true);
  else WINO_FLEX_OPS(false, false);
#undef WINO_FLEX_OPS
  return hipGetLastError();
}

template <int M, bool LEG, typename MT, bool WHOLE>
static hipError_t flex_output_mtw(const Geometry& g, const MT* mp, void* y, int out_type, bool relu,
                                  const FlexMats& fm, const StageMults& mu, float mult_out,
                                  hipStream_t st) {
  const dim3 nb(blocks_for((long)g.T * g.K)), bs(256);
  const Divider by_k = divider_of(g.K);
  const int r = relu ? 1 : 0;
  if (out_type == 0)
    wino_launch((k_flex_output<M, LEG, MT, 0, WHOLE>), nb, bs, st, mp, y, g, by_k, fm, mu, mult_out, r);
  else
    wino_launch((k_flex_output<M, LEG, MT, 2, WHOLE>), nb, bs, st, mp, y, g, by_k, fm, mu, mult_out, r);
  return hipGetLastError();
}

template <int M, bool LEG, typename MT>
static hipError_t flex_output_mt(const Geometry& g, const void* Mq, void* y, int out_type, bool relu,
                                 const FlexMats& fm, const StageMults& mu, float mult_out,
                                 hipStream_t st) {
  const MT* mp = static_cast<const MT*>(Mq);
  // the block-uniform form for the int8 M, as in the fixed-matrix output transform
  if constexpr (sizeof(MT) == 1)
    if (whole_tiles(g.K, g.H, g.W))
      return flex_output_mtw<M, LEG, MT, true>(with_output_groups(g), mp, y, out_type, relu, fm, mu, mult_out, st);
  return flex_output_mtw<M, LEG, MT, false>(g, mp, y, out_type, relu, fm, mu, mult_out, st);
}

template <int M>
hipError_t PerMFlex<M>::output(const Geometry& g, bool leg, const void* Mq, int m_bits, void* y,
                               int out_type, bool relu, const FlexMats& fm, const StageMults& mu,
                               float mult_out, hipStream_t st) {
#define WINO_FLEX_O(LEG_)                                                                        \
  (m_bits == 8   ? flex_output_mt<M, LEG_, int8_t>(g, Mq, y, out_type, relu, fm, mu, mult_out, st)  \
   : m_bits == 9 ? flex_output_mt<M, LEG_, int16_t>(g, Mq, y, out_type, relu, fm, mu, mult_out, st) \
                 : flex_output_mt<M, LEG_, int32_t>(g, Mq, y, out_type, relu, fm, mu, mult_out, st))
  return leg ? WINO_FLEX_O(true) : WINO_FLEX_O(false);
#undef WINO_FLEX_O
}

}  // namespace wino
