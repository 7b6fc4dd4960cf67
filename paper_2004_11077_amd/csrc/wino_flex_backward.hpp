// Backward pass of the flex layer (Section 4.2: G_P, B_P, A_P are trained, P and
// P^{-1} stay fixed), fp32, casts passing their gradient on unchanged.
// For a bracket R = T S T^T with a trained matrix T:
//     dT = sum over items of  dR (T S^T) + dR^T (T S),      dS = T^T (dR T),
// and through a fixed bracket S1 = L S L^T:  dS = L^T dS1 L.  The inputs S of the
// trained brackets are recomputed from the forward pass's integer tensors with the
// forward pass's exact arithmetic (X1 from x, M1 from M) and dequantised.
//
//   k_fbwd_output   dY, M  -> dM, per-block partial sums of dA_P^T
//   fbwd_input_body   dU, x  -> per-tile dX, per-block partial sums of dB_P^T   \ one launch,
//   fbwd_weight_body  dV, w  -> dw, per-block partial sums of dG_P              / k_fbwd_input_weight
//                     (dx itself where a work group takes whole images, flex_backward_takes_images)
//   k_bwd_tile_sum  per-tile dX -> dx elsewhere (fixed order over the <= 4 covering tiles)
//   k_sum_partials  partial sums -> the three matrix gradients (fixed order)
// The two contraction gradients between them are those of the static layer.
// Bound by vector arithmetic (about 2400 instructions per (tile, channel) item of the input bracket) and
// by the bytes of dM, dU and dX.  2048 tiles, C = K = 128, F(4,3): input and filter brackets 38.1 us with
// sums over lanes by LDS permutes, 64-bit divisions and all of T S, T S^T and dT held at once (128
// registers, now 95), then 27.5; output bracket 23.7, now 19.8.
#pragma once
#include "wino_flex.hpp"
#include "wino_real_brackets.hpp"

namespace wino {

// With a run-time T (ROWS x COLS, row-major): A = dR T, from which dS = T^T A follows (flex_input_grad).
template <int ROWS, int COLS>
__device__ __forceinline__ void flex_right(const float* __restrict__ Tm, const float (&dR)[ROWS][ROWS],
                                           float (&A)[ROWS][COLS]) {
  static_for<0, ROWS>([&](auto i) {
    static_for<0, COLS>([&](auto k) {
      float acc = 0.f;
      static_for<0, ROWS>([&](auto j) {
        acc = __builtin_fmaf(dR[i][j], Tm[decltype(j)::value * COLS + decltype(k)::value], acc);
      });
      A[i][k] = acc;
    });
  });
}

// The same for G_P (COLS = 3, S the taps of a filter) as A S^T + (dR^T T) S: its error per item is 0.9 times that
// of the other order.
template <int ROWS>
__device__ __forceinline__ void flex_filter_grad(const float* __restrict__ Tm, const float (&S)[3][3],
                                                 const float (&dR)[ROWS][ROWS],
                                                 const float (&A)[ROWS][3], float (&dT)[ROWS * 3]) {
  static_for<0, ROWS>([&](auto i) {
    float B[3];                                  // row i of dR^T T
    static_for<0, 3>([&](auto k) {
      float acc = 0.f;
      static_for<0, ROWS>([&](auto j) {
        acc = __builtin_fmaf(dR[j][i], Tm[decltype(j)::value * 3 + decltype(k)::value], acc);
      });
      B[k] = acc;
    });
    static_for<0, 3>([&](auto b) {
      float acc = 0.f;
      static_for<0, 3>([&](auto k) { acc = __builtin_fmaf(B[k], S[k][b], acc); });
      static_for<0, 3>([&](auto k) { acc = __builtin_fmaf(A[i][k], S[b][k], acc); });
      dT[decltype(i)::value * 3 + decltype(b)::value] = acc;
    });
  });
}

// dS = T^T A.
template <int ROWS, int COLS>
__device__ __forceinline__ void flex_input_grad(const float* __restrict__ Tm,
                                                const float (&A)[ROWS][COLS], float (&dS)[COLS][COLS]) {
  static_for<0, COLS>([&](auto b) {
    static_for<0, COLS>([&](auto a) {
      float acc = 0.f;
      static_for<0, ROWS>([&](auto i) {
        acc = __builtin_fmaf(Tm[decltype(i)::value * COLS + decltype(a)::value], A[i][b], acc);
      });
      dS[a][b] = acc;
    });
  });
}

// a's two halves added in lanes 0 .. 31, b's in lanes 32 .. 63.
__device__ __forceinline__ float add_halves(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Rows 0 + 1 and 2 + 3 (of 16 lanes) of a in rows 0 and 2, those of b in rows 1 and 3.
__device__ __forceinline__ float add_rows(float a, float b) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Sums of v[i] over the 256 lanes of the work group, in a fixed order: a tree inside a wave
// (wave_sums), then wave 0 + 1 + 2 + 3, written to row[i] by lane i (store_sums).  Four values share a
// register from the second step on, a row of 16 lanes each: 7 adds for four values instead of
// 24, and no LDS before the last step.
template <int CNT>
struct WaveSums {
  static constexpr int regs = (CNT + 3) / 4;
  float of[4][4 * regs];
};
// Values 4 Q .. 4 Q + 3 (those that exist).
template <int Q, int CNT>
__device__ __forceinline__ void wave_sum_of_four(const float (&v)[CNT], WaveSums<CNT>& sums) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // value 4 Q in row 0, 4 Q + 2 in row 1, 4 Q + 1 in row 2, 4 Q + 3 in row 3
  const int mine = ((lane >> 4) & 1) * 2 + (lane >> 5);
  auto value = [&](auto i) { return 4 * Q + decltype(i)::value < CNT ? v[min(4 * Q + decltype(i)::value, CNT - 1)] : 0.f; };
  using std::integral_constant;
  float x = add_rows(add_halves(value(integral_constant<int, 0>{}), value(integral_constant<int, 1>{})),
                     add_halves(value(integral_constant<int, 2>{}), value(integral_constant<int, 3>{})));
#define WINO_DPP_ADD(CTRL) \
  x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, false))
  WINO_DPP_ADD(0x128);   // row_ror:8, 4, 2, 1: every lane of a row has the row's sum
  WINO_DPP_ADD(0x124);
  WINO_DPP_ADD(0x122);
  WINO_DPP_ADD(0x121);
#undef WINO_DPP_ADD
  if ((lane & 15) == 0) sums.of[wave][4 * Q + mine] = x;
}
template <int CNT>
__device__ __forceinline__ void wave_sums(const float (&v)[CNT], WaveSums<CNT>& sums) {
  static_for<0, WaveSums<CNT>::regs>([&](auto q) { wave_sum_of_four<decltype(q)::value>(v, sums); });
}
// COLUMN > 0: the values are a matrix column by column, COLUMN values each, stored row by row.
template <int COLUMN = 0, int CNT>
__device__ __forceinline__ void store_sums(const WaveSums<CNT>& sums, float* __restrict__ row) {
  __syncthreads();
  if (threadIdx.x < CNT) {
    const int i = threadIdx.x;
    const float sum = ((sums.of[0][i] + sums.of[1][i]) + sums.of[2][i]) + sums.of[3][i];
    row[COLUMN ? i % COLUMN * (CNT / COLUMN) + i / COLUMN : i] = sum;
  }
}

// This lane's share of dT = dR (T S^T) + dR^T (T S), a column at a time, summed over the wave as soon as four
// values are there (values column by column: store_sums<CNT, ROWS>).  The products with S come first: T S is
// where the bracket's large terms cancel, and S holds codes.  dT = A S^T + (dR^T T) S takes a sixth
// fewer multiply-adds with dS = T^T A, but cancels after the rounding of A: its error per item was 1.1 to
// 1.4 times as large for A_P and 1.1 to 1.7 times for B_P.
template <int ROWS, int COLS>
__device__ __forceinline__ void flex_matrix_grad(const float* __restrict__ Tm,
                                                 const float (&S)[COLS][COLS],
                                                 const float (&dR)[ROWS][ROWS],
                                                 WaveSums<ROWS * COLS>& sums) {
  static_assert(ROWS * COLS % 4 == 0);
  float dT[ROWS * COLS];
  static_for<0, COLS>([&](auto b) {
    constexpr int V = decltype(b)::value * ROWS;
    static_for<0, ROWS>([&](auto i) { dT[V + decltype(i)::value] = 0.f; });
    static_for<0, ROWS>([&](auto j) {
      float ts = 0.f, tst = 0.f;                 // entries (j, b) of T S and T S^T
      static_for<0, COLS>([&](auto a) {
        const float c = Tm[decltype(j)::value * COLS + decltype(a)::value];
        ts = __builtin_fmaf(c, S[a][b], ts);
        tst = __builtin_fmaf(c, S[b][a], tst);
      });
      static_for<0, ROWS>([&](auto i) {
        float& acc = dT[V + decltype(i)::value];
        acc = __builtin_fmaf(dR[i][j], tst, acc);
        acc = __builtin_fmaf(dR[j][i], ts, acc);
      });
    });
    static_for<V / 4, (V + ROWS) / 4>([&](auto q) { wave_sum_of_four<decltype(q)::value>(dT, sums); });
  });
}

constexpr int kPartialStride = 64;   // floats per work group in the partial-sum arrays

// dY, M -> dM and the partial sums of dAPT (m x n).  s_in: what one code of the
// A_P bracket's input stands for (s_m1, or the scale of M in the canonical base).
template <int M, bool LEG, typename MT>
__global__ __launch_bounds__(256) void k_fbwd_output(const MT* __restrict__ Mq,
                                                     const float* __restrict__ dy,
                                                     float* __restrict__ dM,
                                                     float* __restrict__ part, Geometry g,
                                                     FlexMats fm, StageMults mu, float s_in,
                                                     Divider by_k) {
  constexpr int n = M + 2;
  constexpr int64_t IN_MAX = MTraits<MT>::in_max;
  using TB = Tab<M>;
  const long total = (long)g.T * g.K;
  const long gid = (long)blockIdx.x * 256 + threadIdx.x;
  const bool active = gid < total;
  int t, k, b, ty, tx;
  item_of_lane(blockIdx.x, g.K, by_k, t, k);
  if (!active) t = 0, k = 0;
  tile_coords(g, t, b, ty, tx);
  int xi[n][n];
  static_for<0, n>([&](auto i) {
    static_for<0, n>([&](auto j) {
      xi[i][j] = active ? (int)Mq[(long)(decltype(i)::value * n + decltype(j)::value) * total + gid] : 0;
    });
  });
  if constexpr (LEG) {
    acc_t<TB::PinvT, IN_MAX> num1[n][n];
    sandwich<TB::PinvT, IN_MAX>(xi, num1);
    cast_result<TB::PinvT, IN_MAX>(num1, mu.inner, 127.f, xi);
  }
  float S[n][n];
  static_for<0, n>([&](auto i) { static_for<0, n>([&](auto j) { S[i][j] = (float)xi[i][j] * s_in; }); });
  float dR[M][M];
  static_for<0, M>([&](auto i) {
    static_for<0, M>([&](auto j) {
      const int h = ty * M + decltype(i)::value, w = tx * M + decltype(j)::value;
      dR[i][j] = (active && h < g.H && w < g.W) ? dy[(((long)b * g.H + h) * g.W + w) * g.K + k] : 0.f;
    });
  });
  __shared__ WaveSums<M * n> s_sums;
  flex_matrix_grad<M, n>(fm.APT, S, dR, s_sums);
  float A[M][n];
  flex_right<M, n>(fm.APT, dR, A);
  float dS[n][n];
  flex_input_grad<M, n>(fm.APT, A, dS);
  if (active) {
    if constexpr (LEG) {
      float out[n][n];
      adjoint_bracket_f<TabF<M>::PinvT>(dS, out);
      static_for<0, n>([&](auto i) {
        static_for<0, n>([&](auto j) {
          dM[(long)(decltype(i)::value * n + decltype(j)::value) * total + gid] = out[i][j];
        });
      });
    } else {
      static_for<0, n>([&](auto i) {
        static_for<0, n>([&](auto j) {
          dM[(long)(decltype(i)::value * n + decltype(j)::value) * total + gid] = dS[i][j];
        });
      });
    }
  }
  store_sums<M>(s_sums, part + (long)blockIdx.x * kPartialStride);
}

// dU, x -> per-tile dX [a*n+b][t][c] (IMAGES: dx) and the partial sums of dBPT (n x n).
// s_in: what one code of the B_P bracket's input stands for (s_x1, or s_x).
template <int M, bool LEG, bool IMAGES>
__device__ __forceinline__ void fbwd_input_body(const int8_t* __restrict__ x,
                                                const float* __restrict__ dU,
                                                float* __restrict__ dXt, float* __restrict__ part,
                                                const Geometry& g, const FlexMats& fm,
                                                const StageMults& mu, float s_in, Divider by_c,
                                                Divider by_w, unsigned block) {
  constexpr int n = M + 2;
  using TB = Tab<M>;
  const long total = (long)g.T * g.C;
  int t, c, b, ty, tx;
  const int tiles = g.TH * g.TW, cw = IMAGES ? 256 / tiles : 0;      // powers of two
  const int cw_bits = IMAGES ? 31 - __clz(cw) : 0;
  if constexpr (IMAGES) {
    const int chunks = g.C >> cw_bits;
    block = image_on_one_xcd(g, block);            // the channel chunks of an image share its lines
    const int image = (int)(block / (unsigned)chunks);
    t = image * tiles + ((int)threadIdx.x >> cw_bits);
    c = ((int)block - image * chunks) * cw + ((int)threadIdx.x & (cw - 1));
  } else {
    item_of_lane(block, g.C, by_c, t, c);
  }
  const long gid = IMAGES ? (long)t * g.C + c : (long)block * 256 + threadIdx.x;
  const bool active = IMAGES || gid < total;
  if (!active) t = 0, c = 0;
  tile_coords(g, t, b, ty, tx);
  int xi[n][n];
  static_for<0, n>([&](auto a) {
    static_for<0, n>([&](auto bb) {
      const int h = ty * M - 1 + decltype(a)::value;
      const int ww = tx * M - 1 + decltype(bb)::value;
      int v = 0;
      if (active && h >= 0 && h < g.H && ww >= 0 && ww < g.W)
        v = x[(((long)b * g.H + h) * g.W + ww) * g.C + c];
      xi[a][bb] = v;
    });
  });
  if constexpr (LEG) {
    acc_t<TB::PinvT, 127> num1[n][n];
    sandwich<TB::PinvT, 127>(xi, num1);
    cast_result<TB::PinvT, 127>(num1, mu.inner, 127.f, xi);
  }
  float S[n][n], dR[n][n];
  static_for<0, n>([&](auto i) {
    static_for<0, n>([&](auto j) {
      S[i][j] = (float)xi[i][j] * s_in;
      dR[i][j] = active ? dU[(long)(decltype(i)::value * n + decltype(j)::value) * total + gid] : 0.f;
    });
  });
  __shared__ WaveSums<n * n> s_sums;
  flex_matrix_grad<n, n>(fm.BPT, S, dR, s_sums);
  float A[n][n];
  flex_right<n, n>(fm.BPT, dR, A);
  float dS[n][n];
  flex_input_grad<n, n>(fm.BPT, A, dS);
  __shared__ __attribute__((aligned(16))) float s_dx[IMAGES ? n * n * 256 : 4];
  if (active) {
    auto put = [&](int p, float v) {
      if constexpr (IMAGES)
        s_dx[p * 256 + threadIdx.x] = v;
      else
        dXt[(long)p * total + gid] = v;
    };
    if constexpr (LEG) {
      float out[n][n];
      adjoint_bracket_f<TabF<M>::PinvT>(dS, out);
      static_for<0, n>([&](auto i) { static_for<0, n>([&](auto j) { put(decltype(i)::value * n + decltype(j)::value, out[i][j]); }); });
    } else {
      static_for<0, n>([&](auto i) { static_for<0, n>([&](auto j) { put(decltype(i)::value * n + decltype(j)::value, dS[i][j]); }); });
    }
  }
  store_sums<n>(s_sums, part + (long)block * kPartialStride);      // (a barrier first)
  if constexpr (IMAGES) {
    // the pixels of the image, four channels per lane; contributions in the order of k_bwd_tile_sum
    using v4f = __attribute__((ext_vector_type(4))) float;
    const int c0 = c & ~(cw - 1);
    float* dx = dXt + (long)b * g.H * g.W * g.C + c0;
    for (int e = threadIdx.x; e < (g.H * g.W << cw_bits >> 2); e += 256) {
      const int pix = e >> (cw_bits - 2), c4 = (4 * e) & (cw - 1);
      const int h = (int)fast_div((uint32_t)pix, by_w.mul, by_w.sh), w = pix - h * g.W;
      v4f acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int dyv = 0; dyv < 2; ++dyv) {
        const int ty1 = (h + 1) / M - dyv, i = (h + 1) % M + dyv * M;
        if (ty1 < 0 || ty1 >= g.TH || i >= n) continue;
#pragma unroll
        for (int dxv = 0; dxv < 2; ++dxv) {
          const int tx1 = (w + 1) / M - dxv, j = (w + 1) % M + dxv * M;
          if (tx1 < 0 || tx1 >= g.TW || j >= n) continue;
          acc += *reinterpret_cast<const v4f*>(s_dx + (i * n + j) * 256 + (ty1 * g.TW + tx1) * cw + c4);
        }
      }
      *reinterpret_cast<v4f*>(dx + (long)pix * g.C + c4) = acc;
    }
  }
}

// dV, w -> dw [k][c][3][3] and the partial sums of dGP (n x 3).
template <int M, bool LEG>
__device__ __forceinline__ void fbwd_weight_body(const int8_t* __restrict__ w,
                                                 float* __restrict__ dV,
                                                 float* __restrict__ dw, float* __restrict__ part,
                                                 const Geometry& g, const FlexMats& fm, float s_w,
                                                 unsigned block, int parts) {
  constexpr int n = M + 2;
  const long total = (long)g.K * g.C;
  const long gid = (long)block * 256 + threadIdx.x;
  const bool active = gid < total;
  float S[3][3];
  static_for<0, 3>([&](auto a) {
    static_for<0, 3>([&](auto bb) {
      S[a][bb] = active ? (float)w[gid * 9 + decltype(a)::value * 3 + decltype(bb)::value] * s_w : 0.f;
    });
  });
  float dR[n][n];
  {
    float v[n][n];
    load_summed_dv<n>(dV, total, gid, parts, active, v);
    if constexpr (LEG) {
      adjoint_bracket_f<TabF<M>::Pinv>(v, dR);      // V = P^{-1} W1 P^{-T}
    } else {
      static_for<0, n>([&](auto i) { static_for<0, n>([&](auto j) { dR[i][j] = v[i][j]; }); });
    }
  }
  __shared__ WaveSums<n * 3> s_sums;
  float A[n][3];
  flex_right<n, 3>(fm.GP, dR, A);
  {
    float dT[n * 3];
    flex_filter_grad<n>(fm.GP, S, dR, A, dT);
    wave_sums(dT, s_sums);
  }
  float dS[3][3];
  flex_input_grad<n, 3>(fm.GP, A, dS);
  if (active) {
    static_for<0, 3>([&](auto a) {
      static_for<0, 3>([&](auto bb) {
        dw[gid * 9 + decltype(a)::value * 3 + decltype(bb)::value] = dS[a][bb];
      });
    });
  }
  store_sums(s_sums, part + (long)block * kPartialStride);
}

// The input and the filter bracket are independent of each other: one launch, the first
// nb_w work groups take filters (few, and the longer chain of loads where dV comes in
// parts: they start first), the rest (tile, channel) items.
// dXt: dx itself where IMAGES.
template <int M, bool LEG, bool IMAGES>
__global__ __launch_bounds__(256, (M <= 4 ? 4 : 1)) void k_fbwd_input_weight(
    const int8_t* __restrict__ x, const float* __restrict__ dU, float* __restrict__ dXt,
    float* __restrict__ part_in, const int8_t* __restrict__ w, float* __restrict__ dV,
    float* __restrict__ dw, float* __restrict__ part_w, Geometry g, FlexMats fm, StageMults mu,
    float s_in, float s_w, Divider by_c, Divider by_w, unsigned nb_w, int parts) {
  if (blockIdx.x < nb_w)
    fbwd_weight_body<M, LEG>(w, dV, dw, part_w, g, fm, s_w, blockIdx.x, parts);
  else
    fbwd_input_body<M, LEG, IMAGES>(x, dU, dXt, part_in, g, fm, mu, s_in, by_c, by_w, blockIdx.x - nb_w);
}

// dx[b][h][w][c] from per-tile gradients: tile ty reads input rows ty*M - 1 ... ty*M + M,
// so pixel row h is local row (h+1) % M of tile (h+1) / M and, when that is 0 or 1,
// also local row M + (h+1) % M of the tile above; columns alike.  The (at most four)
// contributions are added in a fixed order.
template <int M>
__global__ __launch_bounds__(256) void k_bwd_tile_sum(const float* __restrict__ dXt,
                                                      float* __restrict__ dx, Geometry g) {
  using v4f = __attribute__((ext_vector_type(4))) float;
  constexpr int n = M + 2;
  // one lane per four channels of a pixel (C is a multiple of 16); blockIdx.y = image row
  const int c4s = g.C / 4;
  const unsigned e = blockIdx.x * 256 + threadIdx.x;       // index in the row: w * c4s + c4
  if (e >= (unsigned)(g.W * c4s)) return;
  const int w = (int)(e / (unsigned)c4s), c = 4 * (int)(e - (unsigned)w * c4s);
  const long row = (long)blockIdx.y + (long)blockIdx.z * 65535;   // b * H + h
  if (row >= (long)g.N * g.H) return;
  const int b = (int)(row / g.H), h = (int)(row - (long)b * g.H);
  const long TC = (long)g.T * g.C;
  const int ty1 = (h + 1) / M, i1 = (h + 1) % M;
  const int tx1 = (w + 1) / M, j1 = (w + 1) % M;
  v4f acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int dyv = 0; dyv < 2; ++dyv) {
    const int ty = ty1 - dyv, i = i1 + dyv * M;
    if (ty < 0 || ty >= g.TH || i >= n) continue;
#pragma unroll
    for (int dxv = 0; dxv < 2; ++dxv) {
      const int tx = tx1 - dxv, j = j1 + dxv * M;
      if (tx < 0 || tx >= g.TW || j >= n) continue;
      const long t = ((long)b * g.TH + ty) * g.TW + tx;
      acc += *reinterpret_cast<const v4f*>(dXt + (long)(i * n + j) * TC + t * g.C + c);
    }
  }
  *reinterpret_cast<v4f*>(dx + (row * g.W + w) * g.C + c) = acc;
}

template <int M>
hipError_t PerMFlexBwd<M>::output(const Geometry& g, bool leg, const void* Mq, int m_bits,
                                  const float* dy, float* dM, float* part, const FlexMats& fm,
                                  const StageMults& mu, float s_in, hipStream_t st) {
  const dim3 grid((unsigned)(((long)g.T * g.K + 255) / 256)), bs(256);
#define WINO_FBWD_OUT(LEGV, MTV)                                                                 \
  wino_launch((k_fbwd_output<M, LEGV, MTV>), grid, bs, st, static_cast<const MTV*>(Mq), dy, dM, \
              part, g, fm, mu, s_in, divider_of(g.K))
  if (leg) {
    if (m_bits == 8) WINO_FBWD_OUT(true, int8_t);
    else if (m_bits == 9) WINO_FBWD_OUT(true, int16_t);
    else WINO_FBWD_OUT(true, int32_t);
  } else {
    if (m_bits == 8) WINO_FBWD_OUT(false, int8_t);
    else if (m_bits == 9) WINO_FBWD_OUT(false, int16_t);
    else WINO_FBWD_OUT(false, int32_t);
  }
#undef WINO_FBWD_OUT
  return hipGetLastError();
}

template <int M>
hipError_t PerMFlexBwd<M>::input_weight(const Geometry& g, bool leg, const int8_t* x,
                                        const float* dU, float* dXt, float* dx, float* part_in,
                                        const int8_t* w, float* dV, float* dw,
                                        float* part_w, const FlexMats& fm, const StageMults& mu,
                                        float s_in, float s_w, hipStream_t st) {
  const unsigned nb_in = (unsigned)(((long)g.T * g.C + 255) / 256);
  const unsigned nb_w = (unsigned)(((long)g.K * g.C + 255) / 256);
  const dim3 grid(nb_in + nb_w), bs(256);
  const int parts = backward_dv_reader_parts(g);
  const bool images = flex_backward_takes_images(g);
  const Geometry gi = images ? with_dealt_units(g, (long)g.C * g.TH * g.TW / 256, g.N) : g;
  float* out = images ? dx : dXt;
#define WINO_FBWD_IN(LEGV, IMGV)                                                                              \
  wino_launch((k_fbwd_input_weight<M, LEGV, IMGV>), grid, bs, st, x, dU, out, part_in, w, dV, dw, part_w, gi, \
              fm, mu, s_in, s_w, divider_of(g.C), divider_of(g.W), nb_w, parts)
  if (leg) {
    if (images) WINO_FBWD_IN(true, true);
    else WINO_FBWD_IN(true, false);
  } else {
    if (images) WINO_FBWD_IN(false, true);
    else WINO_FBWD_IN(false, false);
  }
#undef WINO_FBWD_IN
  return hipGetLastError();
}

// dXt -> dx where the brackets did not leave dx.
template <int M>
hipError_t PerMFlexBwd<M>::tile_sum(const Geometry& g, const float* dXt, float* dx,
                                    hipStream_t st) {
  const long rows = (long)g.N * g.H, per_row = (long)g.W * (g.C / 4);
  if (rows == 0 || per_row == 0 || flex_backward_takes_images(g)) return hipSuccess;
  // grid: x over a row's (pixel, 4 channels) items, y and z over the image rows
  const long zs = (rows + 65534) / 65535;
  if (zs > 65535 || per_row >= (1L << 31)) return hipErrorInvalidValue;
  const dim3 grid((unsigned)((per_row + 255) / 256), (unsigned)(rows < 65535 ? rows : 65535), (unsigned)zs);
  wino_launch((k_bwd_tile_sum<M>), grid, dim3(256), st, dXt, dx, g);
  return hipGetLastError();
}

}  // namespace wino
