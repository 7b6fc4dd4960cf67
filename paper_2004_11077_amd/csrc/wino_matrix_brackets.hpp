// The integer brackets of F(4,3) on the matrix pipe (gfx950): the input bracket pair
// B_P^T [P^-T X P^-1] B_P and the output bracket pair A_P^T [P^-T M P^-1] A_P of eq. 4, with the same
// exact integer numerators and the same casts as the vector-ALU form in wino_transforms.hpp.
//
// A bracket N X N^T is the matrix N (x) N applied to the 36 entries of X, a product with the
// 36 entries of 16 items as columns: v_mfma_f32_16x16x32_f16, four sets of 16 per wave of 64 items.
// The sums are exact: coefficients are integers that fit the 11 significant bits of an f16 (larger
// ones are cut in two, c = 4096 H + L, with an accumulator each), codes enter as unsigned integers
// below 2^10 in units of 2^-24, which is what their bits mean as a subnormal f16, and every
// partial sum stays below 2^24 units (checked at compile time).  num = 4096 H + L is rounded once
// by a fused multiply-add, exactly as the conversion of an integer numerator to fp32 would be.
// The offset that makes the codes unsigned is taken back by two constant entries of the reduction.
//
// Why: the brackets are bound by vector issue.  Of the F(4,3) Legendre input transform 608 vector instructions
// per 64 items become 310 in its loop (casts: two operations per code of X1, three per code of U; pairs; addresses), and
// 48 matrix instructions run beside them on their own pipe.  Operand transforms of 16384 images, 8x8, C = K =
// 256: 352 -> 272 us; of 128 images, 16x16, C = K = 128: 10.0 -> 8.6 us.  Its stores (604 MB) take 50 of the
// 272 us (measured without them), vector issue 180.
//
// Layout.  Of a 16x16x32 product lane (g, n) = (lane / 16, lane % 16) holds operand entries
// 8 g ... 8 g + 7 of column n and results 4 g ... 4 g + 3 of column n, so the results of the first
// product are operand entries of the second without moving between lanes, whatever order the
// reduction takes: the order of the second reduction IS the order of the first one's results.
// A column is an item; a lane works on four consecutive channels (a dword of codes) per entry,
// so set j of four holds channels 4 n + j.
//
// The first bracket (P^-T: lower triangular, even and odd rows apart) has the rows 0 and 1 of the
// identity: the four entries (0|1, 0|1) need no product.  The other 32 are 16 with even row index and 16
// with odd, each fed by the 18 entries of its own row parity: one product each.  A lane fetches
// nine entries: four of even rows (registers 0-3), four of odd rows (4-7) and one of the four
// identity entries (8).  Which entry lane group g has in which register: kPixel.
#pragma once
#include "wino_kernels.hpp"
#include "wino_tables.hpp"

namespace wino {
namespace mb {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v4h __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));

// Entry 6 a + b of register s in lane group g.  Every group has each of its entries' columns such that
// g = (b ^ x_a) mod 4 with x = 0 3 0 0 3 3 (group_of): staging an entry's dwords rotated by its
// group spreads the four groups' reads over all LDS banks.
constexpr int kPixel[9][4] = {{4, 5, 2, 3},     {12, 13, 14, 15}, {27, 26, 25, 24},
                              {16, 17, 29, 28}, {9, 8, 11, 10},   {18, 19, 20, 21},
                              {22, 32, 31, 30}, {33, 23, 35, 34}, {0, 1, 7, 6}};
WINO_HOST_DEVICE constexpr int group_of(int a, int b) { return (b ^ (((0x32 >> a) & 1) * 3)) & 3; }
// Lane group that holds result p of a second bracket with 36 of them.
WINO_HOST_DEVICE constexpr int out_group(int p) { return (p < 32 ? p >> 2 : p) & 3; }
constexpr bool pixels_ok() {
  long seen = 0;
  for (int s = 0; s < 9; ++s)
    for (int g = 0; g < 4; ++g) {
      const int p = kPixel[s][g], a = p / 6, b = p % 6;
      if ((seen >> p) & 1) return false;
      seen |= 1L << p;
      if (group_of(a, b) != g) return false;
      if (s < 8 && ((a & 1) != (s >= 4))) return false;
      if (s == 8 && (a > 1 || b > 1)) return false;
    }
  return seen == (1L << 36) - 1;
}
static_assert(pixels_ok());
// Register s of the lane's group: entry index, from a constant with one byte per group.
template <int S>
__device__ __forceinline__ int pixel(int group) {
  constexpr uint32_t k = kPixel[S][0] | kPixel[S][1] << 8 | kPixel[S][2] << 16 | kPixel[S][3] << 24;
  return (k >> (8 * group)) & 255;
}
template <int S>
__device__ __forceinline__ int pixel_row(int group) {
  constexpr uint32_t k = kPixel[S][0] / 6 | kPixel[S][1] / 6 << 8 | kPixel[S][2] / 6 << 16 | kPixel[S][3] / 6 << 24;
  return (k >> (8 * group)) & 255;
}
template <int S>
__device__ __forceinline__ int pixel_col(int group) {
  constexpr uint32_t k = kPixel[S][0] % 6 | kPixel[S][1] % 6 << 8 | kPixel[S][2] % 6 << 16 | kPixel[S][3] % 6 << 24;
  return (k >> (8 * group)) & 255;
}

// Row m of the first product of parity e: entry (i, j) with i = e (mod 2), identity entries left out.
struct Entry {
  int i, j;
};
constexpr Entry first_row(int e, int m) {
  for (int i = e, at = 0; i < 6; i += 2)
    for (int j = i < 2 ? 2 : 0; j < 6; ++j)
      if (at++ == m) return {i, j};
  return {-1, -1};
}
// Entry of X1 that reduction position (lane group g, register s) of the second bracket holds.
constexpr Entry second_in(int g, int s) {
  return s < 8 ? first_row(s >> 2, 4 * g + (s & 3)) : Entry{kPixel[8][g] / 6, kPixel[8][g] % 6};
}

// The f16 of an integer with at most 11 significant bits.
constexpr bool f16_exact(long v) {
  if (v < 0) v = -v;
  while (v > 2047 && v % 2 == 0) v /= 2;
  return v <= 2047;
}
constexpr uint16_t f16_bits(long v) {
  if (v == 0) return 0;
  const uint16_t sign = v < 0 ? 0x8000 : 0;
  if (v < 0) v = -v;
  int e = 0;
  while ((v >> (e + 1)) != 0) ++e;                   // 2^e <= v < 2^(e + 1)
  const long man = e >= 10 ? v >> (e - 10) : v << (10 - e);
  return (uint16_t)(sign | ((e + 15) << 10) | (man & 1023));
}

// The two constant reduction entries, f16 bits and value in units of 2^-24: k1 = 128, k2 = 128 * 64.
constexpr uint32_t kConst1 = 0x0080u, kConst2 = 0x1000u;
constexpr long kRatio = 64;

// Every partial sum, in any order, of terms c u with 0 <= u < 2 bias and the offset -bias sum(c): the
// positive coefficients add up to `plus`, the negative ones to -`minus`.
constexpr bool sums_exact(long plus, long minus, long bias) {
  const long off = (plus - minus) * bias, slack = kRatio * 128;
  return plus * (2 * bias - 1) + (off < 0 ? -off : 0) + slack < (1L << 24) &&
         minus * (2 * bias - 1) + (off > 0 ? off : 0) + slack < (1L << 24);
}

// One operand of the matrix instruction: 64 lanes x 8 (or 4) halves.
struct Operand8 {
  uint32_t w[64][4];
};
struct Operand4 {
  uint32_t w[64][2];
};
constexpr void put8(Operand8& o, int m, int k, long v) {
  const int lane = (k / 8) * 16 + m, i = k % 8;
  o.w[lane][i / 2] |= (uint32_t)f16_bits(v) << (16 * (i % 2));
}
constexpr void put4(Operand4& o, int m, int k, long v) {
  const int lane = (k / 4) * 16 + m, i = k % 4;
  o.w[lane][i / 2] |= (uint32_t)f16_bits(v) << (16 * (i % 2));
}

// ---- first bracket: operand of parity e -------------------------------------------------
// Reduction entries of lane group g: registers 4 e ... 4 e + 3, the identity entry, a constant, the last of
// the four again (coefficients of more than 11 significant bits are cut into two terms), a constant.
struct FirstOps {
  Operand8 op[2];
  bool ok;
};
template <const IMat& T, int BIAS>
constexpr FirstOps first_ops() {
  FirstOps f{};
  f.ok = T.rows == 6 && T.cols == 6;
  for (int e = 0; e < 2; ++e)
    for (int m = 0; m < 16; ++m) {
      const Entry r = first_row(e, m);
      long plus = 0, minus = 0;
      for (int g = 0; g < 4; ++g)
        for (int s = 0; s < 5; ++s) {
          const int p = kPixel[s == 4 ? 8 : 4 * e + s][g];
          const long c = (long)T.N[r.i][p / 6] * T.N[r.j][p % 6];
          (c < 0 ? minus : plus) += c < 0 ? -c : c;
          long first = c;
          if (!f16_exact(c)) {
            if (s != 3) f.ok = false;
            first = c < 0 ? -2048 : 2048;
            if (!f16_exact(c - first)) f.ok = false;
            put8(f.op[e], m, 8 * g + 6, c - first);
          }
          put8(f.op[e], m, 8 * g + s, first);
        }
      // every entry of the other parity must be out of this row's reach
      for (int p = 0; p < 36; ++p)
        if (((p / 6) & 1) != e && T.N[r.i][p / 6] * T.N[r.j][p % 6] != 0) f.ok = false;
      const long off = (minus - plus) * (BIAS / 128), hi = off / kRatio, lo = off - hi * kRatio;
      if (!f16_exact(hi) || !f16_exact(lo)) f.ok = false;
      put8(f.op[e], m, 5, lo);
      put8(f.op[e], m, 7, hi);
      if (!sums_exact(plus, minus, BIAS)) f.ok = false;
    }
  for (int i = 0; i < 2; ++i)
    for (int a = 0; a < 6; ++a)
      if (T.N[i][a] != (i == a) || T.rho[i] != 1) f.ok = false;
  return f;
}

// ---- second bracket -----------------------------------------------------------------
// Results: 36 (input transform) in three blocks of 16 rows: entries 0-15, 16-31 and 32-35, the
// last one with both digits in one block (row 4 g: L, row 4 g + 1: H of entry 32 + g); or 16
// (output transform) in one block.  Products of a block: digit L, digit H.
constexpr long digit(long c, int d) {
  const long h = (c + 2048) >> 12;
  return d ? h : c - h * 4096;
}
template <int NOP>
struct SecondOps {
  Operand8 op[NOP];
  Operand4 opk[NOP];     // reduction entries: identity entry's code, two constants, none
  bool ok;
};
template <const IMat& T>
constexpr int second_count() {
  return T.rows == 6 ? 5 : 2;
}
template <const IMat& T, int BIAS>
constexpr SecondOps<second_count<T>()> second_ops() {
  constexpr int NOP = second_count<T>(), R = T.rows;
  SecondOps<NOP> f{};
  f.ok = T.cols == 6 && (R == 6 || R == 4);
  for (int op = 0; op < NOP; ++op)
    for (int m = 0; m < 16; ++m) {
      int p = m + 16 * (op / 2), d = op % 2;
      if (op == 4) {
        if (m % 4 > 1) continue;
        p = 32 + m / 4, d = m % 4;
      }
      long plus = 0, minus = 0;
      for (int g = 0; g < 4; ++g)
        for (int s = 0; s < 9; ++s) {
          const Entry q = second_in(g, s);
          const long c = digit((long)T.N[p / R][q.i] * T.N[p % R][q.j], d);
          (c < 0 ? minus : plus) += c < 0 ? -c : c;
          if (!f16_exact(c)) f.ok = false;
          if (s < 8)
            put8(f.op[op], m, 8 * g + s, c);
          else
            put4(f.opk[op], m, 4 * g, c);
        }
      const long off = (minus - plus) * (BIAS / 128), hi = off / kRatio, lo = off - hi * kRatio;
      if (!f16_exact(hi) || !f16_exact(lo)) f.ok = false;
      put4(f.opk[op], m, 1, lo);
      put4(f.opk[op], m, 2, hi);
      if (!sums_exact(plus, minus, BIAS)) f.ok = false;
    }
  return f;
}

// The operands of one bracket pair in device memory, read once per wave.
template <const IMat& T1, const IMat& T2, int BIAS>
struct PairOps {
  FirstOps first;
  SecondOps<second_count<T2>()> second;
};
template <const IMat& T1, const IMat& T2, int BIAS>
constexpr PairOps<T1, T2, BIAS> make_pair_ops() {
  return {first_ops<T1, BIAS>(), second_ops<T2, 128>()};
}
template <const IMat& T1, const IMat& T2, int BIAS>
__device__ constexpr PairOps<T1, T2, BIAS> kPairOps = make_pair_ops<T1, T2, BIAS>();

// Multipliers of a launch in the order the lanes take them, all but the identity entries' times 2^24
// (numerators come in units of 2^-24).
struct PairMults {
  float inner[36];    // rows 0-15 of the even product, 0-15 of the odd one, identity entry of group 0-3
  float outer[36];    // entries of the second bracket in their own order
};
// v * 2^24 for a cast: kept finite, where it saturates every non-zero numerator all the same.
inline float scaled_mult(float v) {
  const float s = v * 16777216.f;
  return s <= 3.4028234663852886e38f ? s : 3.4028234663852886e38f;
}
template <const IMat& T2>
inline PairMults pair_mults(const StageMults& mu) {
  PairMults r{};
  for (int e = 0; e < 2; ++e)
    for (int m = 0; m < 16; ++m) {
      const Entry q = first_row(e, m);
      r.inner[16 * e + m] = scaled_mult(mu.inner.v[q.i * 6 + q.j]);
    }
  for (int g = 0; g < 4; ++g) r.inner[32 + g] = mu.inner.v[kPixel[8][g]];
  for (int p = 0; p < T2.rows * T2.rows; ++p) r.outer[p] = scaled_mult(mu.outer.v[p]);
  return r;
}

// 1.5 * 2^23 + 128: a cast on top of it (cast_biased) leaves code + 128 in the low half of its pattern.
constexpr float kMagicU = 12583040.f;

// Sixteen-bit pair {low half of lo, low half of hi}.
__device__ __forceinline__ uint32_t low_halves(uint32_t hi, uint32_t lo) {
  return __builtin_amdgcn_perm(hi, lo, 0x05040100u);
}

// One bracket pair for a wave: 64 items, four channels per lane.
// IN_BYTES: bytes of a code of X (1: int8; 2: int16 codes of 9 bits).
template <const IMat& T1, const IMat& T2, int IN_BYTES>
struct Pair {
  static constexpr int kInBytes = IN_BYTES;
  static constexpr int BIAS = IN_BYTES == 1 ? 128 : 256;
  static constexpr int NOP = second_count<T2>();
  static constexpr int NV = T2.rows == 6 ? 9 : 4;    // results of a lane and item
  using Ops = PairOps<T1, T2, BIAS>;
  static constexpr Ops check = make_pair_ops<T1, T2, BIAS>();
  static_assert(check.first.ok && check.second.ok);

  v8h a1[2], a2[NOP];
  v4h a2k[NOP];
  float inner[9], outer[NV];

  __device__ __forceinline__ void load(const PairMults& mu, int lane) {
    const Ops& t = kPairOps<T1, T2, BIAS>;
    const int g = lane >> 4;
#pragma unroll
    for (int e = 0; e < 2; ++e) a1[e] = __builtin_bit_cast(v8h, *reinterpret_cast<const v4u*>(t.first.op[e].w[lane]));
#pragma unroll
    for (int o = 0; o < NOP; ++o) {
      a2[o] = __builtin_bit_cast(v8h, *reinterpret_cast<const v4u*>(t.second.op[o].w[lane]));
      a2k[o] = __builtin_bit_cast(v4h, *reinterpret_cast<const v2u*>(t.second.opk[o].w[lane]));
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) inner[i] = mu.inner[16 * (i >> 2) + 4 * g + (i & 3)];
    inner[8] = mu.inner[32 + g];
#pragma unroll
    for (int i = 0; i < NV; ++i) outer[i] = mu.outer[i < 8 ? 16 * (i >> 2) + 4 * g + (i & 3) : 32 + g];
  }

  // The codes of four channels at the lane's nine entries, offset to unsigned.
  struct In {
    uint32_t u[9][IN_BYTES];
  };
  __device__ __forceinline__ static void put(In& in, int s, uint32_t codes) {
    static_assert(IN_BYTES == 1);
    in.u[s][0] = codes ^ 0x80808080u;
  }
  __device__ __forceinline__ static void put(In& in, int s, uint32_t lo, uint32_t hi) {
    static_assert(IN_BYTES == 2);
    typedef unsigned short v2us __attribute__((ext_vector_type(2)));
    const v2us off = {256, 256};
    in.u[s][0] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(v2us, lo) + off);
    in.u[s][1] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(v2us, hi) + off);
  }
  // {code of channel J in register s0, code of channel J in register s1} as 16-bit integers
  template <int J>
  __device__ __forceinline__ static uint32_t two(const In& in, int s1, int s0) {
    if constexpr (IN_BYTES == 1)
      return __builtin_amdgcn_perm(in.u[s1][0], in.u[s0][0], 0x0c000c00u | (4u + J) << 16 | J);
    else
      return __builtin_amdgcn_perm(in.u[s1][J / 2], in.u[s0][J / 2],
                                   J & 1 ? 0x07060302u : 0x05040100u);
  }
  // {code of channel J in register s, low half of k}
  template <int J>
  __device__ __forceinline__ static uint32_t with(const In& in, int s, uint32_t k) {
    if constexpr (IN_BYTES == 1)
      return __builtin_amdgcn_perm(k, in.u[s][0], 0x05040c00u | J);
    else
      return __builtin_amdgcn_perm(k, in.u[s][J / 2], J & 1 ? 0x05040302u : 0x05040100u);
  }
  template <int J>
  __device__ __forceinline__ static float single(const In& in, int s) {
    if constexpr (IN_BYTES == 1)
      return (float)((in.u[s][0] >> (8 * J)) & 255u) - 128.f;
    else
      return (float)((in.u[s][J / 2] >> (16 * (J & 1))) & 0xffffu) - 256.f;
  }

  // Numerators of the second bracket, channel J, in units of 2^-24, rounded to fp32 once.
  template <int J>
  __device__ __forceinline__ void numerators(const In& in, float (&num)[NV]) const {
    constexpr v4f zero = {0.f, 0.f, 0.f, 0.f};
    const uint32_t w8 = with<J>(in, 8, kConst1);
    const v4u be = {two<J>(in, 1, 0), two<J>(in, 3, 2), w8, with<J>(in, 3, kConst2)};
    const v4u bo = {two<J>(in, 5, 4), two<J>(in, 7, 6), w8, with<J>(in, 7, kConst2)};
    const v4f de = __builtin_amdgcn_mfma_f32_16x16x32_f16(a1[0], __builtin_bit_cast(v8h, be), zero, 0, 0, 0);
    const v4f dd = __builtin_amdgcn_mfma_f32_16x16x32_f16(a1[1], __builtin_bit_cast(v8h, bo), zero, 0, 0, 0);
    uint32_t t[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
      const float v = i < 4 ? de[i & 3] : i < 8 ? dd[i & 3] : single<J>(in, 8);
      const float q = __builtin_fmaf(v, inner[i], kMagicU);
      t[i] = __float_as_uint(__builtin_amdgcn_fmed3f(q, kMagicU - 127.f, kMagicU + 127.f));
    }
    const v4u b2 = {low_halves(t[1], t[0]), low_halves(t[3], t[2]), low_halves(t[5], t[4]),
                    low_halves(t[7], t[6])};
    const v2u b2k = {low_halves(kConst1, t[8]), kConst2};
    v4f d[NOP];
#pragma unroll
    for (int o = 0; o < NOP; ++o)
      d[o] = __builtin_amdgcn_mfma_f32_16x16x16f16(a2k[o], __builtin_bit_cast(v4h, b2k), zero, 0, 0, 0);
#pragma unroll
    for (int o = 0; o < NOP; ++o)
      d[o] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a2[o], __builtin_bit_cast(v8h, b2), d[o], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      if (i < 8)
        num[i] = __builtin_fmaf(d[2 * (i >> 2) + 1][i & 3], 4096.f, d[2 * (i >> 2)][i & 3]);
      else
        num[i] = __builtin_fmaf(d[NOP - 1][1], 4096.f, d[NOP - 1][0]);
    }
  }
};

// Codes of four channels from their biased casts, as a dword.
__device__ __forceinline__ uint32_t pack_codes(const uint32_t (&t)[4]) {
  return __builtin_amdgcn_perm(t[1], t[0], 0x0c0c0400u) | __builtin_amdgcn_perm(t[3], t[2], 0x04000c0cu);
}

constexpr float kMagic0 = kMagicU - 128.f;       // low byte of a cast on top of it: the code
// `codes` with the low byte of a biased cast put in as byte J (the bytes above it are not yet used).
template <int J>
__device__ __forceinline__ uint32_t add_code(uint32_t codes, float biased) {
  const uint32_t t = __float_as_uint(biased);
  if constexpr (J == 0)
    return t;
  else
    return __builtin_amdgcn_perm(t, codes, J == 1 ? 0x0c0c0400u : J == 2 ? 0x0c040100u : 0x04020100u);
}
// NJ sets of channels (four, or the first two), one at a time: scheduled together, they need twice the
// registers.
template <int NJ, class F>
__device__ __forceinline__ void each_set(F&& set) {
  set(std::integral_constant<int, 0>{});
  __builtin_amdgcn_sched_barrier(0);
  set(std::integral_constant<int, 1>{});
  if constexpr (NJ == 4) {
    __builtin_amdgcn_sched_barrier(0);
    set(std::integral_constant<int, 2>{});
    __builtin_amdgcn_sched_barrier(0);
    set(std::integral_constant<int, 3>{});
  }
}

// Input bracket pair: the lane's nine results (input_result) as dwords of NJ channels' codes.
template <int NJ, const IMat& T1, const IMat& T2, int IN_BYTES>
__device__ __forceinline__ void input_codes(const Pair<T1, T2, IN_BYTES>& ops,
                                            const typename Pair<T1, T2, IN_BYTES>::In& in, uint32_t (&out)[9]) {
  each_set<NJ>([&](auto j) {
    constexpr int J = decltype(j)::value;
    float num[9];
    ops.template numerators<J>(in, num);
#pragma unroll
    for (int i = 0; i < 9; ++i)
      out[i] = add_code<J>(out[i], __builtin_amdgcn_fmed3f(__builtin_fmaf(num[i], ops.outer[i], kMagic0),
                                                           kMagic0 - 127.f, kMagic0 + 127.f));
  });
}
// Entry of a lane's result i.
__device__ __forceinline__ int input_result(int i, int group) {
  return i < 8 ? 16 * (i >> 2) + 4 * group + (i & 3) : 32 + group;
}

// Output bracket pair.  A lane has row `group` of the item's 4 x 4 outputs, NJ channels: their codes (int8,
// OUT = 2) or floats (OUT = 0) at output column r go to put(r, value).
// Multipliers of a dequantised output must stay finite in these units.
inline bool output_mults_fit(const StageMults& mu) {
  for (int p = 0; p < 16; ++p)
    if (!(mu.outer.v[p] <= 0x1p103f)) return false;
  return true;
}
template <int NJ, int OUT, const IMat& T1, const IMat& T2, int IN_BYTES, class Put>
__device__ __forceinline__ void finish_outputs(const Pair<T1, T2, IN_BYTES>& ops,
                                               const typename Pair<T1, T2, IN_BYTES>::In& in, int relu,
                                               Put&& put) {
  typedef int vni __attribute__((ext_vector_type(NJ)));
  // ReLU as a lower bound (none: below every value): of a float through its bit pattern, negative values
  // being negative integers, of a code by the clamp of its cast.
  const int lo_f = relu ? 0 : (int)0x80000000;
  const float lo_q = relu ? kMagic0 : kMagic0 - 127.f;
  vni f[4];
  uint32_t q[4];
  each_set<NJ>([&](auto j) {
    constexpr int J = decltype(j)::value;
    float num[4];
    ops.template numerators<J>(in, num);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if constexpr (OUT == 0)
        f[r][J] = max(__float_as_int(num[r] * ops.outer[r]), lo_f);
      else
        q[r] = add_code<J>(q[r], __builtin_amdgcn_fmed3f(__builtin_fmaf(num[r], ops.outer[r], kMagic0), lo_q,
                                                         kMagic0 + 127.f));
    }
  });
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if constexpr (OUT == 0)
      put(r, f[r]);
    else if constexpr (NJ == 4)
      put(r, (int)q[r]);
    else
      put(r, (short)q[r]);
  }
}

}  // namespace mb
}  // namespace wino
