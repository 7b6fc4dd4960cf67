// Calibration of a flex layer: the scale of every cast is chosen on the device, each kernel deriving
// the scales it needs from the maxima that the kernels before it left in scratch memory, so that the
// host waits once, at the end.  The arithmetic is the host's, in double:
//     scale = float( max_ij( amax_ij s_prev / (rho_i rho_j) ) / qmax ),   multipliers as in fill_mults.
// Launches (w and x share theirs; the canonical base has no second bracket):
//   k_fcal_first     maxima of the first brackets
//   k_fcal_second    maxima of the second brackets, behind the cast that the first ones call for
//   k_fcal_operands  V and U
//   contraction      its maxima, then M (launch_contract_cal)
//   k_fcal_m_inner, k_fcal_output   maxima of the brackets of M
// 2048 tiles, C = K = 128, 9-bit M: about 100 us for the call; with the host choosing each scale in turn
// (seven read-backs), one atomic per wave and entry on a single location and the exact contraction
// result written and read once more it took 450 us.  Each launch is now bound by its bracket's
// arithmetic or, for M, by its loads (7 to 14 us).
// Entries whose row denominators have equal products share one maximum (shared_mult_index): their
// real values differ by one factor, so the largest is the largest integer.
#pragma once
#include "wino_flex.hpp"

namespace wino {

// rho_i rho_j of entry lane (1 past the last entry).
template <const IMat& T>
struct RhoProducts {
  double v[kMaxPts];
  constexpr RhoProducts() : v{} {
    for (int q = 0; q < kMaxPts; ++q)
      v[q] = q < T.rows * T.rows ? (double)(T.rho[q / T.rows] * T.rho[q % T.rows]) : 1.0;
  }
};
template <const IMat& T>
__device__ const RhoProducts<T> kRhoProducts{};

__device__ __forceinline__ float cal_positive_scale(double real, double qmax) {
  return real > 0.0 ? (float)(real / qmax) : 1.0f;
}
// Scale of the cast after an fp32 bracket.
__device__ __forceinline__ float cal_float_scale(const unsigned long long* amax, double s_prev) {
  return cal_positive_scale((double)__uint_as_float((unsigned)amax[0]) * s_prev, 127.0);
}
// Scale of the cast after the integer bracket T (every lane of the wave returns it).
template <const IMat& T>
__device__ __forceinline__ float cal_int_scale(const unsigned long long* amax, double s_prev) {
  const int lane = threadIdx.x & 63;
  const unsigned long long a = lane < T.rows * T.rows ? amax[lane] : 0;
  double best = ((double)a * s_prev) / kRhoProducts<T>.v[lane];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) best = fmax(best, __shfl_xor(best, off));
  return cal_positive_scale(best, 127.0);
}
// Multipliers of that cast, one entry per lane, spread to a table of scalar registers (entries that
// nothing reads cost nothing).
template <const IMat& T>
__device__ __forceinline__ void cal_mults(double s_prev, float s_next, MultTable& mu) {
  const float v = (float)(s_prev / (kRhoProducts<T>.v[threadIdx.x & 63] * (double)s_next));
  static_for<0, T.rows * T.rows>([&](auto q) {
    mu.v[decltype(q)::value] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), decltype(q)::value));
  });
}

// Maximum over the work group of a non-negative float, merged into amax[0].
__device__ __forceinline__ void group_max_float(float v, unsigned long long* __restrict__ amax) {
  __shared__ unsigned s_max[4];
  const unsigned top = wave_max_u32(__float_as_uint(v));
  if ((threadIdx.x & 63) == 63) s_max[threadIdx.x >> 6] = top;
  __syncthreads();
  if (threadIdx.x == 0) raise_max(amax, max(max(s_max[0], s_max[1]), max(s_max[2], s_max[3])));
}

template <int R>
__device__ __forceinline__ float tile_absmax(const float (&v)[R][R]) {
  float best = 0.f;
  static_for<0, R>([&](auto i) {
    static_for<0, R>([&](auto j) { best = fmaxf(best, fabsf(v[i][j])); });
  });
  return best;
}

// Maxima over the work group of |entry| of a result of sandwich<T, IN_MAX>, merged into amax.
template <const IMat& T, int64_t IN_MAX, typename AccT>
__device__ __forceinline__ void group_max_int(const AccT (&num)[T.rows][T.rows],
                                              unsigned long long* __restrict__ amax) {
  constexpr int R = T.rows;
  __shared__ unsigned long long s_max[4][R * R];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  static_for<0, R * R>([&](auto lead) {
    constexpr int L = decltype(lead)::value;
    if constexpr (shared_mult_index<T, L / R, L % R>() == L) {
      unsigned long long top = 0;
      constexpr bool narrow = sizeof(AccT) == 4;
      static_for<0, R * R>([&](auto q) {
        constexpr int I = decltype(q)::value / R, J = decltype(q)::value % R;
        if constexpr (shared_mult_index<T, I, J>() == L) {
          const long long v = (long long)entry<T, IN_MAX, I, J>(num[I][J]);
          top = max(top, (unsigned long long)(v < 0 ? -v : v));
        }
      });
      if constexpr (narrow) {
        top = wave_max_u32((unsigned)top);
      } else {
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) top = max(top, (unsigned long long)__shfl_xor(top, off));
      }
      if (lane == 63) s_max[wave][L] = top;
    } else if (lane == 63) {
      s_max[wave][L] = 0;
    }
  });
  __syncthreads();
  if (threadIdx.x < R * R) {
    const int q = threadIdx.x;
    const unsigned long long top = max(max(s_max[0][q], s_max[1][q]), max(s_max[2][q], s_max[3][q]));
    if (top != 0) raise_max(amax + q, top);
  }
}

// First brackets: the fp32 one of w; the integer one of x (Legendre) or its fp32 one.
template <int M, bool LEG>
__global__ __launch_bounds__(256) void k_fcal_first(const int8_t* __restrict__ x,
                                                    const int8_t* __restrict__ w, CalScratch cal,
                                                    Geometry g, FlexMats fm, unsigned nb_w) {
  constexpr int n = M + 2;
  using TB = Tab<M>;
  if (blockIdx.x < nb_w) {
    weight_items<M, false>(w, nullptr, g, blockIdx.x, [&](const int (&wi)[3][3], int (&)[n][n]) {
      float wf[3][3], val[n][n];
      to_floats<3>(wi, wf);
      fsandwich<n, 3>(fm.GP, wf, val);
      group_max_float(tile_absmax<n>(val), cal.array(kCalW1));
    });
  } else {
    input_items<M, false, false>(x, nullptr, g, blockIdx.x - nb_w, [&](const int (&xi)[n][n], int (&)[n][n]) {
      if constexpr (LEG) {
        acc_t<TB::PinvT, 127> num[n][n];
        sandwich<TB::PinvT, 127>(xi, num);
        group_max_int<TB::PinvT, 127>(num, cal.array(kCalX1));
      } else {
        float xf[n][n], val[n][n];
        to_floats<n>(xi, xf);
        fsandwich<n, n>(fm.BPT, xf, val);
        group_max_float(tile_absmax<n>(val), cal.array(kCalX2));
      }
    });
  }
}

// Second brackets (Legendre): the integer one of w, the fp32 one of x.
template <int M>
__global__ __launch_bounds__(256) void k_fcal_second(const int8_t* __restrict__ x,
                                                     const int8_t* __restrict__ w, CalScratch cal,
                                                     Geometry g, FlexMats fm, float s_x, float s_w,
                                                     unsigned nb_w) {
  constexpr int n = M + 2;
  using TB = Tab<M>;
  if (blockIdx.x < nb_w) {
    const float s_w1 = cal_float_scale(cal.array(kCalW1), s_w);
    const float first = (float)((double)s_w / (double)s_w1);
    weight_items<M, false>(w, nullptr, g, blockIdx.x, [&](const int (&wi)[3][3], int (&)[n][n]) {
      float wf[3][3], val[n][n];
      to_floats<3>(wi, wf);
      fsandwich<n, 3>(fm.GP, wf, val);
      uint32_t w1[n][n];
      static_for<0, n>([&](auto i) {
        static_for<0, n>([&](auto j) { w1[i][j] = cast_biased(val[i][j], first, 127.f); });
      });
      acc_t<TB::Pinv, 127> num[n][n];
      sandwich_codes<TB::Pinv, 127>(w1, num);
      group_max_int<TB::Pinv, 127>(num, cal.array(kCalW2));
    });
  } else {
    const float s_x1 = cal_int_scale<TB::PinvT>(cal.array(kCalX1), s_x);
    MultTable inner;
    cal_mults<TB::PinvT>(s_x, s_x1, inner);
    input_items<M, false, false>(x, nullptr, g, blockIdx.x - nb_w, [&](const int (&xi)[n][n], int (&)[n][n]) {
      float xf[n][n], val[n][n];
      flex_input<TB::PinvT, 127, true>(xi, inner, xf);
      fsandwich<n, n>(fm.BPT, xf, val);
      group_max_float(tile_absmax<n>(val), cal.array(kCalX2));
    });
  }
}

// V and U with the scales that the maxima call for; the scales go to scratch memory.
template <int M, bool LEG>
__global__ __launch_bounds__(256) void k_fcal_operands(const int8_t* __restrict__ x,
                                                       int8_t* __restrict__ U,
                                                       const int8_t* __restrict__ w,
                                                       int8_t* __restrict__ V, CalScratch cal,
                                                       Geometry g, FlexMats fm, float s_x, float s_w,
                                                       unsigned nb_w) {
  using TB = Tab<M>;
  const bool first = threadIdx.x == 0 && (blockIdx.x == 0 || blockIdx.x == nb_w);
  StageMults mu;
  if (blockIdx.x < nb_w) {
    float s_w1 = s_w, s_v = cal_float_scale(cal.array(kCalW1), s_w);
    float mult = (float)((double)s_w / (double)s_v);
    if constexpr (LEG) {
      s_w1 = s_v;
      s_v = cal_int_scale<TB::Pinv>(cal.array(kCalW2), s_w1);
      cal_mults<TB::Pinv>(s_w1, s_v, mu.outer);
    }
    if (first) cal.scales()[kCalSW1] = s_w1, cal.scales()[kCalSV] = s_v;
    flex_weight_body<M, LEG>(w, V, g, fm, mu, mult, blockIdx.x);
  } else {
    float s_x1 = s_x;
    if constexpr (LEG) {
      s_x1 = cal_int_scale<TB::PinvT>(cal.array(kCalX1), s_x);
      cal_mults<TB::PinvT>(s_x, s_x1, mu.inner);
    }
    const float s_u = cal_float_scale(cal.array(kCalX2), s_x1);
    if (first) cal.scales()[kCalSX1] = s_x1, cal.scales()[kCalSU] = s_u;
    flex_input_body<M, LEG, false>(x, U, g, fm, mu, (float)((double)s_x1 / (double)s_u), blockIdx.x - nb_w);
  }
}

// What one code of M stands for.
template <typename MT>
__device__ __forceinline__ double cal_m_scale(const CalScratch& cal) {
  return sizeof(MT) == 4 ? (double)cal.scales()[kCalSU] * (double)cal.scales()[kCalSV]
                         : (double)cal.scales()[kCalSM];
}

// Integer bracket of M (Legendre).
template <int M, typename MT>
__global__ __launch_bounds__(256) void k_fcal_m_inner(const MT* __restrict__ Mq, CalScratch cal,
                                                      Geometry g, Divider by_k) {
  constexpr int n = M + 2;
  constexpr int64_t IN_MAX = MTraits<MT>::in_max;
  using TB = Tab<M>;
  int t, k;
  item_of_lane(blockIdx.x, g.K, by_k, t, k);
  int xi[n][n] = {};
  fetch_m<n, false>(Mq, (long)g.T * g.K, (long)blockIdx.x * 256, t < g.T, t, k, g.K, xi);
  acc_t<TB::PinvT, IN_MAX> num[n][n];
  sandwich<TB::PinvT, IN_MAX>(xi, num);
  group_max_int<TB::PinvT, IN_MAX>(num, cal.array(kCalM1));
}

// fp32 bracket of M: positions cropped from partial tiles do not count; with relu only the positive
// part has to be covered.
template <int M, bool LEG, typename MT>
__global__ __launch_bounds__(256) void k_fcal_output(const MT* __restrict__ Mq, CalScratch cal,
                                                     Geometry g, Divider by_k, FlexMats fm, int relu) {
  constexpr int n = M + 2;
  using TB = Tab<M>;
  MultTable inner;
  if constexpr (LEG) {
    const double s_m = cal_m_scale<MT>(cal);
    const float s_m1 = cal_int_scale<TB::PinvT>(cal.array(kCalM1), s_m);
    if (blockIdx.x == 0 && threadIdx.x == 0) cal.scales()[kCalSM1] = s_m1;
    cal_mults<TB::PinvT>(s_m, s_m1, inner);
  }
  int t, k;
  item_of_lane(blockIdx.x, g.K, by_k, t, k);
  const bool active = t < g.T;
  int xi[n][n] = {};
  fetch_m<n, false>(Mq, (long)g.T * g.K, (long)blockIdx.x * 256, active, t, k, g.K, xi);
  int b, ty, tx;
  tile_coords(g, active ? t : 0, b, ty, tx);
  float xf[n][n], val[M][M];
  flex_input<TB::PinvT, MTraits<MT>::in_max, LEG>(xi, inner, xf);
  fsandwich<M, n>(fm.APT, xf, val);
  float best = 0.f;
  static_for<0, M>([&](auto i) {
    static_for<0, M>([&](auto j) {
      const bool inside = ty * M + decltype(i)::value < g.H && tx * M + decltype(j)::value < g.W;
      const float v = relu ? fmaxf(val[i][j], 0.f) : fabsf(val[i][j]);
      best = fmaxf(best, active && inside ? v : 0.f);
    });
  });
  group_max_float(best, cal.array(kCalY));
}

template <int M, bool LEG, typename MT>
static hipError_t fcal_output(const Geometry& g, const void* Mq, bool relu, CalScratch cal,
                              const FlexMats& fm, hipStream_t st) {
  const dim3 nb(blocks_for((long)g.T * g.K)), bs(256);
  const Divider by_k = divider_of(g.K);
  const MT* mp = static_cast<const MT*>(Mq);
  if constexpr (LEG) wino_launch((k_fcal_m_inner<M, MT>), nb, bs, st, mp, cal, g, by_k);
  wino_launch((k_fcal_output<M, LEG, MT>), nb, bs, st, mp, cal, g, by_k, fm, relu ? 1 : 0);
  return hipGetLastError();
}

template <int M>
hipError_t PerMFlex<M>::calibrate(const Geometry& g, bool leg, const int8_t* x, int8_t* U,
                                  const int8_t* w, int8_t* V, void* Mq, int m_bits, bool relu,
                                  float s_x, float s_w, CalScratch cal, const FlexMats& fm,
                                  hipStream_t st) {
  const unsigned nb_w = weight_blocks(g), nb_x = input_blocks(g);
  const dim3 grid(nb_w + nb_x), bs(256);
  hipError_t e = launch_fill_zero(cal.base, (long)kCalArrays * cal.n2 * 8, st);
  if (e != hipSuccess) return e;
  if (leg) {
    wino_launch((k_fcal_first<M, true>), grid, bs, st, x, w, cal, g, fm, nb_w);
    wino_launch((k_fcal_second<M>), grid, bs, st, x, w, cal, g, fm, s_x, s_w, nb_w);
    wino_launch((k_fcal_operands<M, true>), grid, bs, st, x, U, w, V, cal, g, fm, s_x, s_w, nb_w);
  } else {
    wino_launch((k_fcal_first<M, false>), grid, bs, st, x, w, cal, g, fm, nb_w);
    wino_launch((k_fcal_operands<M, false>), grid, bs, st, x, U, w, V, cal, g, fm, s_x, s_w, nb_w);
  }
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (m_bits == 32) {                                  // no cast: the exact result is M
    const MultTable unused{};
    e = launch_contract(g, U, V, Mq, 32, unused, st);
  } else {
    e = launch_contract_cal(g, U, V, Mq, m_bits, cal, st);
  }
  if (e != hipSuccess) return e;
#define WINO_FCAL_OUT(LEG_)                                                     \
  (m_bits == 8   ? fcal_output<M, LEG_, int8_t>(g, Mq, relu, cal, fm, st)       \
   : m_bits == 9 ? fcal_output<M, LEG_, int16_t>(g, Mq, relu, cal, fm, st)      \
                 : fcal_output<M, LEG_, int32_t>(g, Mq, relu, cal, fm, st))
  return leg ? WINO_FCAL_OUT(true) : WINO_FCAL_OUT(false);
#undef WINO_FCAL_OUT
}

}  // namespace wino
