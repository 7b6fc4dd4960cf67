// Internal launcher interface between the C ABI (wino_api.cpp) and the HIP
// kernels (wino_kernels.hip).  Not part of the public boundary.
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <cstdint>

namespace wino {

// Optional per-launch timing: a pair of HIP events handed over with
// set_profile_events() is attached to the NEXT kernel this thread launches
// through wino_launch (the events then carry that dispatch's own begin and
// end timestamps); the pair is consumed by that launch.  Pairs queue up (at
// most 8 pending): the k-th pending pair goes to the k-th launch from now.
struct ProfileEvents {
  hipEvent_t start, stop;
};
void set_profile_events(hipEvent_t start, hipEvent_t stop);
ProfileEvents take_profile_events();

template <class K, class... Args>
inline void wino_launch(K kernel, dim3 grid, dim3 block, hipStream_t st, Args... args) {
  const ProfileEvents p = take_profile_events();
  if (p.start || p.stop)
    hipExtLaunchKernelGGL(kernel, grid, block, 0, st, p.start, p.stop, 0, args...);
  else
    hipLaunchKernelGGL(kernel, grid, block, 0, st, args...);
}

// Records the text of a failure for wino_last_error() on this thread and returns `code`
// (for the parts of the C ABI that live outside wino_api.cpp).
int report_error(int code, const char* fmt, ...);

constexpr int kMaxPts = 64;   // n*n for n = 8

// fp32 multipliers of one cast, indexed [i*cols + j] (Section 4.2 cast after a
// bracket; value = s_prev / (rho_i rho_j s_next), rounded to fp32 on the host).
struct MultTable {
  float v[kMaxPts];
};

// Left shifts applied to the codes of M before the output bracket when M has
// per-point power-of-two scales (entry p = i*n + j; all zero otherwise).  Four bits per
// entry (a shift is at most kMaxMShift = 8), eight entries per word: a kernel keeps the whole
// table in 8 scalar registers and extracts an entry where it is used, instead of holding up
// to 64 registers live across its loops.
struct ShiftTable {
  uint32_t w[kMaxPts / 8];
  void set(int p, int shift) {
    w[p >> 3] = (w[p >> 3] & ~(15u << ((p & 7) * 4))) | ((uint32_t)shift << ((p & 7) * 4));
  }
#if defined(__HIPCC__)
  // Entry P as a wave-uniform value.  The extraction is kept where it is written (volatile):
  // moved out of a loop, the entries would again occupy one scalar register each.
  template <int P>
  __device__ __forceinline__ int at() const {
    uint32_t r;
    asm volatile("s_bfe_u32 %0, %1, %2" : "=s"(r) : "s"(w[P >> 3]), "n"(((P & 7) * 4) | (4 << 16)) : "scc");
    return (int)r;
  }
#endif
};
constexpr int kMaxMShift = 8;

struct Geometry {
  int N, H, W, C, K;
  int m;        // output tile edge
  int TH, TW;   // tiles per image
  int T;        // total tiles
  int frag;     // 1: U and V are in MFMA-fragment order (below), 0: rows [n*n][T or K][C]
  // division of a tile index (< 2^30) by TW and by TW * TH as multiply-high and shift
  uint32_t mul_tw, sh_tw, mul_im, sh_im;
  // division of a work-group index (< 2^30) by the groups per tile of the one-tile-per-group
  // transform kernels: C / 256 (input), K / 256 (output); 1 where that is not a whole number
  uint32_t mul_cg, sh_cg, mul_kg, sh_kg;
  // division of a work-group index by the 64-channel chunks of a row, ceil(C / 64): the groups
  // of the fragment-order transforms are (four rows, one chunk)
  uint32_t mul_ch, sh_ch;
  // input and output transform: work groups per unit (an image or a run of tiles) when every
  // unit's groups are to run on one XCD (0 = work groups in plain order), and the number of
  // groups covered by that order; set per launch (with_image_groups, with_output_groups)
  int img_blocks, img_blocks_end;
};

// Work-group ids go round-robin over the 8 XCDs, each with a private L2 that keeps its lines
// from one kernel to the next.  A line that one XCD wrote and another one read is expensive to
// write again (the other L2's copy has to be found and dropped), and tiles of an image share
// input lines.  The transforms therefore deal their work groups to XCDs in units: launch slot
// b = 8 q + x (XCD x) takes group (q % G) of unit 8 (q / G) + x, G = groups per unit; the slots
// past the last full set of eight units keep their plain order.  A unit is
//   * fragment order: 32 consecutive tiles, the tile block of the contraction + output kernel,
//     which takes tile block j on XCD j % 8: U is read, and written again by the next call, on
//     the XCD that wrote it;
//   * rows, small layers: an eighth of the tiles, which the contraction kernel and the output
//     transform then give to the same XCD (xcd_chunk_tiles), so that U and M stay in one L2;
//   * rows otherwise: one image (shared input lines enter one L2 once).
#if defined(__HIPCC__)
#define WINO_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define WINO_HOST_DEVICE inline
#endif
WINO_HOST_DEVICE unsigned image_on_one_xcd(const Geometry& g, unsigned b) {
  if (g.img_blocks == 0 || b >= (unsigned)g.img_blocks_end) return b;
  const unsigned x = b & 7, q = b >> 3, G = (unsigned)g.img_blocks;
  const unsigned set = q / G, within = q - set * G;
  return (set * 8 + x) * G + within;
}

// Work groups of 256 lanes for `items` lanes' worth of work.
WINO_HOST_DEVICE unsigned blocks_for(long items) { return (unsigned)((items + 255) / 256); }
// A work group's 256 items are the channels of one tile (and offsets inside one
// image fit 32 bits): the kernels then keep the tile arithmetic in scalar registers.
inline bool whole_tiles(int channels, int H, int W) {
  return channels > 0 && channels % 256 == 0 && (long)H * W * channels < (1L << 31);
}
// Work groups of the operand transforms: 256 consecutive items each in row order; in
// fragment order one per (4 rows, 64-channel chunk).
WINO_HOST_DEVICE unsigned weight_blocks(const Geometry& g) {
  return g.frag ? (unsigned)(((long)g.K >> 2) * ((g.C + 63) >> 6)) : blocks_for((long)g.K * g.C);
}
inline unsigned input_blocks(const Geometry& g) {
  return g.frag ? (unsigned)((((long)g.T + 3) >> 2) * ((g.C + 63) >> 6)) : blocks_for((long)g.T * g.C);
}
// Tile rows of a work group of the contraction kernel: 128, or 64 where fewer than two
// 128-row blocks per compute unit would exist (measured: 7 % on a 4x4 x 512-channel layer with
// 256 tiles; no gain from about two blocks per compute unit on).
inline int contract_tile_rows(const Geometry& g) {
  const int n = g.m + 2;
  const long big_tiles = (long)n * n * ((g.T + 127) / 128) * ((g.K + 127) / 128);
  return big_tiles < 2 * 256 ? 64 : 128;
}
// Row order, one kernel per stage: tiles per XCD when input transform, contraction and output
// transform all give the same eighth of the tiles to an XCD, 0 when they do not.  They do when
// the eighths are whole contraction blocks, both transforms run their one-tile-per-group
// kernels (the ones that can be dealt) and U and M together (n*n T (C + K) bytes) fit the eight
// 4 MiB L2s with room to spare: measured on 8x8 images with 256 channels, 26.9 -> 25.8 us per
// layer at N = 256 (19 MB); but 45.9 -> 47.6 us for F(6,3) on the same images (32 MiB), and
// 229 -> 240 us at N = 4096, where nothing stays in an L2 and the output transform loses by
// reading and writing one long run per XCD.  With the contraction alone renumbered (a
// 128-channel layer, whose transforms keep their plain order) a layer lost 10 %.
constexpr long kAlignedXcdBytes = 24L << 20;
inline long xcd_chunk_tiles(const Geometry& g) {
  const int tt = contract_tile_rows(g), n = g.m + 2;
  if (g.frag || g.T <= 0 || g.T % (8L * tt) != 0) return 0;
  if (!whole_tiles(g.C, g.H, g.W) || !whole_tiles(g.K, g.H, g.W)) return 0;
  return (long)n * n * g.T * ((long)g.C + g.K) <= kAlignedXcdBytes ? g.T / 8 : 0;
}
// Groups of tile rows of the contraction kernel: a unit of its block numbering is (point,
// group), and unit u runs on XCD u % 8.  Aligned with the transforms: 8 groups, group j on XCD j.
// Otherwise the smallest split that spreads n*n points over the 8 XCDs evenly.
inline int contract_tile_groups(const Geometry& g, int tile_rows) {
  const int n = g.m + 2, tblocks = (g.T + tile_rows - 1) / tile_rows;
  if (tile_rows == contract_tile_rows(g) && xcd_chunk_tiles(g) > 0) return 8;
  int tgroups = 1;
  while (tgroups < 8 && (n * n * tgroups) % 8 != 0 && tgroups * 2 <= tblocks) tgroups *= 2;
  return tgroups;
}
// Sets the dealing of `per_unit` work groups per unit over `units` units (off when there are
// fewer than eight units or the numbers do not fit).
inline Geometry with_dealt_units(Geometry g, long per_unit, long units) {
  g.img_blocks = 0, g.img_blocks_end = 0;
  const long end = (units / 8) * 8 * per_unit;
  if (per_unit > 0 && per_unit < (1L << 20) && units >= 8 && end < 0x7fffffffL)
    g.img_blocks = (int)per_unit, g.img_blocks_end = (int)end;
  return g;
}
// Work for a group of four waves of 128 items each (input_pairs): two blocks, in fragment order eight tiles and a
// 64-channel chunk.
inline unsigned input_pair_count(const Geometry& g) {
  return g.frag ? (unsigned)((((long)g.T + 7) >> 3) * ((g.C + 63) >> 6)) : (input_blocks(g) + 1) / 2;
}
// Geometry for the input transform's launch (whole: the block-uniform row-order kernel, one
// work group per tile and 256 channels).
// per: 256-item blocks per work group (1 or 2; an image of an odd number of blocks is then dealt
// together with the next one).
inline Geometry with_image_groups(const Geometry& g, bool whole, int per = 1) {
  const long nch = (g.C + 63) >> 6;
  if (g.frag) return with_dealt_units(g, 8 * nch / per, g.T / 32);
  if (!whole) return with_dealt_units(g, 0, 0);
  if (const long chunk = xcd_chunk_tiles(g)) return with_dealt_units(g, chunk * (g.C / 256) / per, 8);
  const long blocks = (long)g.TH * g.TW * (g.C / 256);
  return blocks % per ? with_dealt_units(g, blocks, g.N / per) : with_dealt_units(g, blocks / per, g.N);
}
// Geometry for the launch of the block-uniform output transform (one work group per tile and
// 256 output channels; per as above).
inline Geometry with_output_groups(const Geometry& g, int per = 1) {
  return with_dealt_units(g, xcd_chunk_tiles(g) * (g.K / 256) / per, 8);
}

// q = n / d for n < 2^30.  d a power of two: a shift (mul = 0).  Otherwise, with f = floor(log2 d),
// q = (n * mul) >> (32 + f), mul = floor(2^(32 + f) / d) + 1 < 2^32: the excess
// mul d - 2^(32 + f) is at most d < 2^(f + 1), so n times it stays below 2^(32 + f).
inline void fast_div_setup(uint32_t d, uint32_t* mul, uint32_t* sh) {
  uint32_t f = 0;
  while ((2u << f) <= d) ++f;                      // f = floor(log2 d), d >= 1
  *sh = f;
  *mul = (d & (d - 1)) == 0 ? 0u : (uint32_t)((((unsigned long long)1 << (32 + f)) / d) + 1);
}
inline void geometry_set_divisors(Geometry& g) {
  fast_div_setup((uint32_t)(g.TW > 0 ? g.TW : 1), &g.mul_tw, &g.sh_tw);
  fast_div_setup((uint32_t)(g.TW * g.TH > 0 ? g.TW * g.TH : 1), &g.mul_im, &g.sh_im);
  fast_div_setup((uint32_t)(g.C >= 256 && g.C % 256 == 0 ? g.C / 256 : 1), &g.mul_cg, &g.sh_cg);
  fast_div_setup((uint32_t)(g.K >= 256 && g.K % 256 == 0 ? g.K / 256 : 1), &g.mul_kg, &g.sh_kg);
  fast_div_setup((uint32_t)(g.C > 64 ? (g.C + 63) / 64 : 1), &g.mul_ch, &g.sh_ch);
}
// A prepared divider as a kernel argument of its own (kernels that need one the Geometry does not hold).
struct Divider {
  uint32_t mul, sh;
};
inline Divider divider_of(int d) {
  Divider r;
  fast_div_setup((uint32_t)(d > 0 ? d : 1), &r.mul, &r.sh);
  return r;
}
#if defined(__HIPCC__)
// n / d with the pair prepared by fast_div_setup for d (n < 2^30).
__device__ __forceinline__ uint32_t fast_div(uint32_t n, uint32_t mul, uint32_t sh) {
  return (mul ? __umulhi(n, mul) : n) >> sh;
}
#endif
#if defined(__HIPCC__)
// tile t -> (image b, tile row ty, tile column tx) with t = (b TH + ty) TW + tx, t < 2^30.
__device__ __forceinline__ void tile_coords(const Geometry& g, int t, int& b, int& ty, int& tx) {
  const uint32_t im = (uint32_t)(g.TW * g.TH);
  b = (int)((g.mul_im ? __umulhi((uint32_t)t, g.mul_im) : (uint32_t)t) >> g.sh_im);
  const uint32_t r = (uint32_t)t - (uint32_t)b * im;
  ty = (int)((g.mul_tw ? __umulhi(r, g.mul_tw) : r) >> g.sh_tw);
  tx = (int)(r - (uint32_t)ty * (uint32_t)g.TW);
}
// Item 256 * block + lane of the (tile, channel) items, `channels` (C or K) per tile with its
// divider: the division of the group's first item is block-uniform (scalar), the lane's, of an
// offset below channels + 256, is a multiply-high.  Items past the last one get a tile index >= T.
__device__ __forceinline__ void item_of_lane(unsigned block, int channels, Divider d, int& t, int& c) {
  const unsigned long long first = (unsigned long long)block * 256;
  const unsigned t0 = (first >> 30) == 0 ? fast_div((uint32_t)first, d.mul, d.sh)
                                         : (unsigned)(first / (unsigned)channels);
  const unsigned r = (unsigned)(first - (unsigned long long)t0 * (unsigned)channels) + threadIdx.x;
  const unsigned q = fast_div(r, d.mul, d.sh);
  t = (int)(t0 + q);
  c = (int)(r - q * (unsigned)channels);
}
#endif

// Fragment order of a transformed operand X[p][row][c] (rows = tiles for U, output channels
// for V): rows in groups of 16 (RG = ceil(rows / 16) groups), channels in chunks of 64
// (NCH = ceil(C / 64) chunks); the 16 x 64 block of (group, chunk) is one contiguous KiB laid
// out [c % 64 / 16][row % 16][c % 16], which is exactly the register layout of a 16x16x64
// int8 MFMA operand: lane l of a wave reads bytes [16 l, 16 l + 16) of the block.
//   offset(p, row, c) = ((p RG + row / 16) NCH + c / 64) 1024 + (c % 64 / 16) 256 + (row % 16) 16 + c % 16
// Rows past the last one are never written (they only feed results that are discarded);
// channels past C hold zeros in V (and anything in U).
inline long frag_bytes(long n2, long rows, long C) {
  return n2 * ((rows + 15) / 16) * ((C + 63) / 64) * 1024;
}

struct StageMults {
  MultTable inner;   // inner bracket of eq. 2 / eq. 4 (unused when !inner)
  MultTable outer;   // outer bracket, or the only one for the canonical base
};

// Per-M launchers of the transform stages (defined in wino_transforms.hpp and
// instantiated once per M in its own translation unit).
// brackets: 0 = one bracket per stage (canonical matrices); 1, 2, 3 = the two-bracket form of
// eq. 2 / eq. 4 in the monic Legendre, Chebyshev, Hermite base.
template <int M>
struct PerM {
  static hipError_t weight(const Geometry& g, int brackets, const int8_t* w, int8_t* V,
                           const StageMults& mu, hipStream_t st);
  static hipError_t input(const Geometry& g, int brackets, const int8_t* x, int8_t* U,
                          const StageMults& mu, hipStream_t st);
  static hipError_t operands(const Geometry& g, int brackets, const int8_t* x, int8_t* U,
                             const int8_t* w, int8_t* V, const StageMults& mu_in,
                             const StageMults& mu_w, hipStream_t st);
  // sh != nullptr: M carries per-point shifts (8- or 9-bit M only)
  static hipError_t output(const Geometry& g, int brackets, const void* M_, int m_bits,
                           void* y, int out_type, bool relu, const StageMults& mu,
                           const ShiftTable* sh, hipStream_t st);
};
extern template struct PerM<2>;
extern template struct PerM<4>;
extern template struct PerM<6>;

// Calibration launchers (wino_calibrate.hpp): per-(i, j) maxima of the integer
// numerators of one bracket, merged into amax[64] (device, zeroed by the caller).
template <int M>
struct PerMCal {
  static hipError_t weight(const Geometry& g, bool legendre_inner, int phase, const int8_t* w,
                           unsigned long long* amax, const StageMults& mu, hipStream_t st);
  static hipError_t input(const Geometry& g, bool legendre_inner, int phase, const int8_t* x,
                          unsigned long long* amax, const StageMults& mu, hipStream_t st);
  static hipError_t output(const Geometry& g, bool legendre_inner, int phase, const void* M_,
                           int m_bits, unsigned long long* amax, const StageMults& mu, bool relu,
                           const ShiftTable* sh, hipStream_t st);
};
extern template struct PerMCal<2>;
extern template struct PerMCal<4>;
extern template struct PerMCal<6>;

// Run-time fp32 matrices of the trainable brackets (Section 4.2, "flex"),
// row-major with their own column counts: GP n x 3, BPT n x n, APT m x n.
struct FlexMats {
  float GP[8 * 3];
  float BPT[8 * 8];
  float APT[6 * 8];
};

// Scratch memory of a calibration that chooses its scales on the device: one array of n*n maxima per
// cast (zero at the start), then the scales that later kernels need.  A maximum is an integer
// numerator or the bit pattern of a non-negative float.
enum { kCalW1, kCalW2, kCalX1, kCalX2, kCalM, kCalM1, kCalY, kCalArrays };   // maxima: first and second bracket of w and x, M, brackets of M
enum { kCalSX1, kCalSU, kCalSW1, kCalSV, kCalSM, kCalSM1, kCalScales };      // scales
struct CalScratch {
  unsigned long long* base;
  int n2;
  WINO_HOST_DEVICE unsigned long long* array(int which) const { return base + which * n2; }
  WINO_HOST_DEVICE float* scales() const { return reinterpret_cast<float*>(base + kCalArrays * n2); }
  static constexpr size_t bytes(int n2) { return (size_t)kCalArrays * n2 * 8 + kCalScales * 4; }
};
#if defined(__HIPCC__)
// Maximum over the wave, in lane 63.
__device__ __forceinline__ unsigned wave_max_u32(unsigned v) {
#define WINO_DPP_MAX(CTRL) v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false))
  WINO_DPP_MAX(0x111);   // row_shr:1, 2, 4, 8: lane 15 of a row of 16 has the row's maximum
  WINO_DPP_MAX(0x112);
  WINO_DPP_MAX(0x114);
  WINO_DPP_MAX(0x118);
  WINO_DPP_MAX(0x142);   // row_bcast:15, row_bcast:31
  WINO_DPP_MAX(0x143);
#undef WINO_DPP_MAX
  return v;
}
// *at = max(*at, v).  The plain read first: once the maximum has been met most groups find nothing to
// raise, and the memory location sees a few atomics instead of one per group.
__device__ __forceinline__ void raise_max(unsigned long long* at, unsigned long long v) {
  if (v > __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(at, v);
}
#endif

// Launchers of the flex kernels (wino_flex.hpp, wino_flex_calibrate.hpp).
template <int M>
struct PerMFlex {
  static hipError_t weight(const Geometry& g, bool legendre, const int8_t* w, int8_t* V,
                           const FlexMats& fm, const StageMults& mu, float mult_first, hipStream_t st);
  static hipError_t input(const Geometry& g, bool legendre, const int8_t* x, int8_t* U,
                          const FlexMats& fm, const StageMults& mu, float mult_u, hipStream_t st);
  static hipError_t output(const Geometry& g, bool legendre, const void* M_, int m_bits, void* y,
                           int out_type, bool relu, const FlexMats& fm, const StageMults& mu,
                           float mult_out, hipStream_t st);
  // input and weight stage in one launch
  static hipError_t operands(const Geometry& g, bool legendre, const int8_t* x, int8_t* U,
                             const int8_t* w, int8_t* V, const FlexMats& fm,
                             const StageMults& mu_in, float mult_u, const StageMults& mu_w,
                             float mult_first, hipStream_t st);
  // every launch of a calibration
  static hipError_t calibrate(const Geometry& g, bool legendre, const int8_t* x, int8_t* U,
                              const int8_t* w, int8_t* V, void* M_, int m_bits, bool relu, float s_x,
                              float s_w, CalScratch cal, const FlexMats& fm, hipStream_t st);
};
extern template struct PerMFlex<2>;
extern template struct PerMFlex<4>;
extern template struct PerMFlex<6>;

// stage 0 weight, 1 input, 2 output, dispatched on g.m.
hipError_t launch_flex_stage(int stage, const Geometry& g, bool legendre, const void* in, int m_bits,
                             void* out, int out_type, bool relu, const FlexMats& fm,
                             const StageMults& mu, float mult, hipStream_t st);

// Runs a flex layer up to M and chooses its scales on the device: when the stream has got there,
// U, V, M hold the layer's tensors, cal the scales of all casts but the last and the maximum
// (kCalY) that s_y follows from.  cal may overlap nothing the layer writes.
hipError_t launch_flex_calibrate(const Geometry& g, bool legendre, const int8_t* x, int8_t* U,
                                 const int8_t* w, int8_t* V, void* M_, int m_bits, bool relu,
                                 float s_x, float s_w, CalScratch cal, const FlexMats& fm,
                                 hipStream_t st);
// Contraction of a calibration (m_bits 8 or 9): maxima of the exact result into cal, then the
// contraction again with the cast that they call for.
hipError_t launch_contract_cal(const Geometry& g, const int8_t* U, const int8_t* V, void* M_, int m_bits,
                               CalScratch cal, hipStream_t st);

// Input and weight stage of a flex layer in one launch (both outputs non-empty).
hipError_t launch_flex_operands(const Geometry& g, bool legendre, const int8_t* x, int8_t* U,
                                const int8_t* w, int8_t* V, const FlexMats& fm,
                                const StageMults& mu_in, float mult_u, const StageMults& mu_w,
                                float mult_first, hipStream_t st);

// stage: 0 weight, 1 input, 2 output; phase 1 = inner bracket, 2 = outer bracket.
hipError_t launch_calibrate_stage(int stage, const Geometry& g, bool legendre_inner, int phase,
                                  const void* in, int m_bits, unsigned long long* amax,
                                  const StageMults& mu, bool relu, const ShiftTable* sh,
                                  hipStream_t st);
// amax[s] = max |v[s * count + i]|, i < count, for each of `segments` consecutive
// int32 arrays (device pointers).
hipError_t launch_absmax_i32(const int32_t* v, long count, int segments,
                             unsigned long long* amax, hipStream_t st);

// brackets: 0 = the single-bracket form (canonical, or a base with its brackets multiplied
// out); 1 / 2 / 3 = the two-bracket pipeline in the Legendre / Chebyshev / Hermite base.
hipError_t launch_weight_transform(const Geometry& g, int brackets, const int8_t* w,
                                   int8_t* V, const StageMults& mu, hipStream_t st);
hipError_t launch_input_transform(const Geometry& g, int brackets, const int8_t* x,
                                  int8_t* U, const StageMults& mu, hipStream_t st);
// Input and weight transform in one launch (both outputs non-empty).
hipError_t launch_operand_transforms(const Geometry& g, int brackets, const int8_t* x,
                                     int8_t* U, const int8_t* w, int8_t* V,
                                     const StageMults& mu_in, const StageMults& mu_w,
                                     hipStream_t st);
// m_bits: 8 -> int8 M, 9 -> int16 M, 32 -> int32 M (no cast).
// mult.v[p]: multiplier of the cast of point p (unused for m_bits = 32).
hipError_t launch_contract(const Geometry& g, const int8_t* U, const int8_t* V, void* M,
                           int m_bits, const MultTable& mult, hipStream_t st);
// out_type: 0 fp32 (outer table = dequantisation factors), 1 int32 numerators,
// 2 int8 codes (outer table = cast multipliers).
hipError_t launch_output_transform(const Geometry& g, int brackets, const void* M,
                                   int m_bits, void* y, int out_type, bool relu,
                                   const StageMults& mu, const ShiftTable* sh, hipStream_t st);

// Contraction and output transform in one kernel, M kept in LDS (wino_conout.hpp);
// m_bits 8 or 9, out_type 0 or 2, C > 0; U and V in rows or fragment order (g.frag).
template <int M>
struct PerMCO {
  static hipError_t run(const Geometry& g, bool legendre_inner, const int8_t* U, const int8_t* V,
                        void* y, int m_bits, int out_type, bool relu, const StageMults& out_mu,
                        const MultTable& mm, const ShiftTable* sh, hipStream_t st);
  static long blocks(const Geometry& g, int m_bits);
};
// Work groups launch_contract_output would start for this geometry.
long contract_output_blocks(const Geometry& g, int m_bits);
extern template struct PerMCO<2>;
extern template struct PerMCO<4>;
extern template struct PerMCO<6>;
hipError_t launch_contract_output(const Geometry& g, bool legendre_inner, const int8_t* U,
                                  const int8_t* V, void* y, int m_bits, int out_type, bool relu,
                                  const StageMults& out_mu, const MultTable& mm,
                                  const ShiftTable* sh, hipStream_t st);
// Zero fill of `bytes` (a multiple of 16) at a 16-byte aligned device address, by a kernel.
hipError_t launch_fill_zero(void* dst, long bytes, hipStream_t st);

// Fused variant (input transform + contraction + output transform in one kernel);
// V is the transformed filter tensor.  m = 2 or 4, m_bits 8 or 9, out_type 0 or 2.
// mm: cast multiplier of the contraction per point; sh: per-point shifts or null.  w_mu not null: V is
// the filter tensor itself, transformed with these multipliers (fused_takes_raw_filters); the
// transformed filters are also left in Vout.
hipError_t launch_fused(const Geometry& g, bool legendre_inner, const int8_t* x, const int8_t* V,
                        void* y, int m_bits, int out_type, bool relu, const StageMults& in_mu,
                        const StageMults& out_mu, const MultTable& mm, const ShiftTable* sh,
                        const StageMults* w_mu, int8_t* Vout, hipStream_t st);
// Output channels per work group of the fused kernel.
inline int fused_channels(int m_bits) { return m_bits == 8 ? 64 : 32; }
// Tiles per work group of the fused kernel (kb = fused_channels).  A launch takes about (first + each *
// rounds) / 10 us, rounds = work groups over 256 compute units: smaller groups have the shorter chain of
// phases, larger ones waste less of the matrix instruction's 16 columns and of phase B.  Measured, C = K
// = 64, us per layer with transformed filters, int8 M and output:
//   tiles             1024   2048   3072   4096   6144   8192  10240  12288  16384  32768
//   F(4,3)  16        15.7   15.8   15.9   16.0   23.7   23.8   31.8   31.8   40.7   77.9
//            8        10.2   10.2   15.0   15.1   19.9   25.1   30.7   35.8   46.0   88.3
//            4         8.4   10.8   13.8   16.8   23.4   30.2   36.5   43.0   55.9  106.8
//   F(2,3)  16         7.4    7.4    7.5    7.5   10.2   10.2   11.8   11.9   15.2   27.0
//            8         5.5    5.5    6.8    6.9    8.5   10.0   12.4   14.0   18.2   33.1
//            4         5.5    5.9    6.8    8.3   10.8   13.5   16.2   18.9   24.3   45.9
// The third round of 16-tile groups is cheap in F(2,3) with full blocks of 64 channels (at 10240 tiles and
// K = 48 12.2 against 11.9 us with 8 tiles, K = 16 12.1 against 11.7): a dearer round of 8 there.  9-bit M (blocks of
// 32), C = K = 64, F(4,3): 13.4, 8.9, 9.7 at 1024 tiles, 19.1, 19.9, 25.3 at 4096; F(2,3): 6.7, 5.6, 5.5 and
// 8.9, 8.3, 10.9.  The choice is within 3 % of the best of the three over these shapes and C, K down
// to 16, but for F(2,3) with a 9-bit M and C = K = 64 at 4096 tiles (8 %).
inline int fused_tiles(const Geometry& g, int kb) {
  struct Cost { int tiles; long first, each; };
  constexpr Cost kCost[3] = {{16, 80, 78}, {8, 53, 49}, {4, 54, 30}};
  constexpr Cost kCostFullBlocks2[3] = {{16, 80, 78}, {8, 50, 53}, {4, 54, 30}};
  int best = 16;
  long best_cost = 0;
  for (const Cost& c : g.m == 2 && kb == 64 && g.K >= 64 ? kCostFullBlocks2 : kCost) {
    const long groups = ((long)g.T + c.tiles - 1) / c.tiles * ((g.K + kb - 1) / kb);
    const long cost = c.first + c.each * ((groups + 255) / 256);
    if (best_cost == 0 || cost < best_cost) best = c.tiles, best_cost = cost;
  }
  return best;
}
// The same for the single kernel with its brackets on the matrix pipe (F(4,3), Legendre base, one scale per
// tensor): the smallest groups of which there is at most one per compute unit, else the largest.  us per layer with
// transformed filters, C = K = 64, int8 output, against the kernel above ("vector", in groups of its own rule):
//   tiles              256   1024   1536   2048   3072   4096   6144   8192  10240  12288  16384  32768
//   8-bit M   4        7.3    8.1   11.1   11.2   16.2   20.1   28.9   38.0   47.0   56.2   74.4  148.1
//             8        8.7    8.7    8.8    8.7   12.3   12.4   18.3   23.3   28.6   34.0   44.9   90.0
//            16       11.6   11.6   11.8   11.6   11.8   11.9   17.1   17.3   24.8   25.0   32.6   65.3
//        vector        8.2    8.5          10.2   13.8   15.0   19.9   23.8   30.5   31.6   40.7   77.8
//   9-bit M   4        6.6    9.2   12.7   15.5   21.9   28.4   41.5   54.4   67.2   80.2  105.9  214.0
//             8        8.0    8.6   10.9   11.2   16.1   19.8   28.4   36.3   44.1   52.0   67.6  137.8
//            16       10.0   10.4   10.4   10.6   14.8   15.0   20.8   26.7   32.8   39.1   50.8  101.3
//        vector        7.3    8.8          12.2   15.9   19.3   26.1   33.8   40.8   47.3   62.1  124.1
// (9 bits: two blocks of 32 channels.)  C = K = 32, C = 16 and K = 48, and fp32 output have the same order.
inline int fused_matrix_tiles(const Geometry& g, int kb) {
  for (int tiles : {4, 8})
    if (((long)g.T + tiles - 1) / tiles * ((g.K + kb - 1) / kb) <= 256) return tiles;
  return 16;
}
// Row and column of a pixel as input_pairs holds them, sixteen bits each (-1 is 65535).
typedef unsigned short PixelPair __attribute__((ext_vector_type(2)));
WINO_HOST_DEVICE bool inside_image(PixelPair pixel, PixelPair last) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(pixel, last)) == __builtin_bit_cast(uint32_t, pixel);
}
// The input transform of F(4,3) in the Legendre base runs on the matrix pipe (input_pairs) where every pixel of
// a tile has sixteen-bit coordinates and an image's offsets fit thirty bits.  Tiles reach row 4 TH and column
// 4 TW, past the image's edge: those, not H and W, must stay below 2^16, or a row of padding would wrap round
// to row 0.
inline bool input_fits_matrix_pipe(const Geometry& g, int brackets) {
  return g.m == 4 && brackets == 1 && 4L * g.TH < 65536 && 4L * g.TW < 65536 && (long)g.W * g.C < 65536 &&
         (long)g.H * g.W * g.C < (1L << 30);
}
// And where it is the faster form.  Each wave reads 10 KB of matrix operands first and takes its 128 items
// one half after the other, a longer chain than the vector form's, which only pays once there are enough
// waves; beside filters in one launch, once the items are twice the filters.  us of the launch, vector -> matrix,
// F(4,3) on 8x8 images, by (tile, channel) items:
//   items                       32768         65536         98304        131072        262144        524288
//   C = K = 64,  input     4.32 -> 4.84  4.72 -> 5.24  5.96 -> 5.72  6.40 -> 6.48  8.30 -> 8.60  12.6 -> 12.6
//   C = K = 256, input     4.20 -> 4.72  4.48 -> 5.04  5.60 -> 5.42  5.76 -> 5.10  7.80 -> 6.76  11.8 -> 11.2
//   C = K = 256, both      5.76 -> 6.16  6.24 -> 6.64  7.00 -> 7.04  7.36 -> 7.00  8.96 -> 7.98  13.6 -> 12.9
//   C = K = 512, both      9.40 -> 10.5  9.72 -> 10.6  10.4 -> 11.1  10.5 -> 11.3  11.5 -> 12.2  16.2 -> 15.2
//   C = K = 256, fragments 7.36 -> 8.18  6.48 -> 6.98  7.76 -> 7.40  7.36 -> 7.16  9.08 -> 7.96  13.8 -> 11.8
// filters: how many the launch transforms as well (0: the input transform alone).
constexpr long kMatrixInputItems = 3L << 15;
inline bool input_on_matrix_pipe(const Geometry& g, int brackets, long filters) {
  const long items = (long)g.T * g.C;
  return input_fits_matrix_pipe(g, brackets) && items >= kMatrixInputItems && items >= 2 * filters;
}
// Output transform of F(4,3) in the Legendre base from an int8 M: on the matrix pipe (k_output_pairs) where
// offsets into M and into a few images of y fit 32 bits and it is the faster form, by the items of a point's
// plane, T K.  us in a layer with one kernel per stage, vector -> matrix (8x8 images):
//   items            2^16          2^18          2^19       3 * 2^18       2^20       3 * 2^19       2^21       3 * 2^20
//   fp32 K = 64   5.5 ->  4.8   8.0 ->  6.0  12.2 -> 14.8  18.1 -> 18.4  24.9 -> 25.1  35.7 -> 32.9  45.4 -> 49.4
//        K = 128                8.2 ->  6.3  12.4 -> 14.7                25.2 -> 23.8  35.5 -> 34.8  45.2 -> 49.0  67.3 -> 62.7
//        K = 256  5.3 ->  4.7   7.8 ->  6.4  11.4 -> 14.6                22.6 -> 24.1                39.3 -> 49.7  56.8 -> 63.0
//   int8 K = 64   5.4 ->  4.5   8.3 ->  5.7  12.9 -> 10.6  18.4 -> 13.6  24.3 -> 19.5  34.7 -> 22.5  43.7 -> 34.6
//        K = 256  5.2 ->  4.6   8.1 ->  6.1  12.2 -> 11.2                18.8 -> 19.0                32.3 -> 36.1  45.6 -> 41.7
// So: int8 y everywhere but on whole tiles (K a multiple of 256, which have a vector form of their own) whose planes are
// a multiple of 2 MiB apart, which puts the nine planes a lane reads on the same channels; fp32 y up to 3 * 2^17 items
// (layers of 6 * 2^16: -2 to -5 %, of 7 * 2^16: +1 to +2.6 % up to K = 64), and from 2^20 where neither holds (a store
// of whole tiles is a KiB of a pixel there, 256 bytes here).  Beyond
// 192 MB of M, more than the last-level cache keeps of it, never: loads of 64 bytes then cost more than the
// arithmetic saves (2^24 items, K = 256: 285 / 240 us, fp32 / int8 y, against 348 at best).
constexpr long kMatrixOutputBytes = 192L << 20;
inline bool output_on_matrix_pipe(const Geometry& g, int out_type) {
  const long items = (long)g.T * g.K;
  if (36 * items > kMatrixOutputBytes || (long)g.H * g.W * g.K * 4 >= (1L << 30)) return false;
  const bool whole = whole_tiles(g.K, g.H, g.W), same_channels = items % (1L << 21) == 0;
  if (out_type == 2) return !(whole && same_channels);
  return items <= 3L << 17 || (!whole && !same_channels && items >= 1L << 20);
}
// A work group of the input bracket of the flex backward pass can take all tiles of an image, 1, 2, 4, 8 or 16, for
// 256 / tiles channels: the sum over the tiles that cover a pixel then needs no tensor of per-tile gradients (written
// and read, 38 MB each for 128 images of 16x16, C = 128) and no launch of its own: 27.5 + 9.6 -> 32.4 us there, the
// training step 9 us less.  Whole backward passes, us, per-tile gradients -> whole images, Legendre, C = K = 128 unless
// said otherwise:
//   tiles                        1 (64 images)      2 (64)         4 (256)          8 (64)         16 (128)
//   F(2,3)  C = K = 512 at 1     41.8 ->  39.0   23.1 -> 20.6   37.6 ->  35.5   29.8 -> 26.2    47.3 ->  41.6
//   F(4,3)  C = K = 512 at 1     54.3 ->  53.6   32.6 -> 29.8   57.3 ->  51.9   45.2 -> 43.9    88.5 ->  82.7
//   F(6,3)  C = K = 512 at 1     93.4 ->  89.6   53.4 -> 51.8  107.6 ->  96.8   70.8 -> 65.9   187.6 -> 156.1
// (one or two images of C = K = 64: 18.6 -> 16.1, 26.2 -> 24.1, 42.8 -> 43.0 for F(2,3), F(4,3), F(6,3).)
inline bool flex_backward_takes_images(const Geometry& g) {
  const int tiles = g.TH * g.TW;
  return tiles >= 1 && tiles <= 16 && (tiles & (tiles - 1)) == 0 && g.C % (256 / tiles) == 0 &&
         (long)g.H * g.W * g.C < (1L << 29);
}
// Few enough filters (and tiles) for every work group of the fused kernel to transform its own.
inline bool fused_takes_raw_filters(const Geometry& g) {
  return (long)g.K * g.C <= 1024 && g.T <= 1024;
}

// Backward pass (wino_backward.hip), fp32.  which: 0 dY -> dM, 1 dU -> dx.
hipError_t launch_backward_transform(int which, const Geometry& g, const float* in, float* out,
                                     hipStream_t st);
// Tiles of the two contractions: 64 wide along a dimension of up to 64 channels, else 128 (two 64-wide
// blocks); along the tiles always 128.
inline int backward_row_blocks(const Geometry& g) { return g.K > 64 ? 2 : 1; }
inline int backward_col_blocks(const Geometry& g) { return g.C > 64 ? 2 : 1; }
// Number of partial sums (a power of two, 1 ... 32) the dV contraction leaves for this
// shape; the dV buffer holds that many [n*n][K][C] tensors.  Up to eight are added, into the
// first one, by whichever kernel reads dV next (backward_dv_reader_parts says how many it
// will find); more are added by launch_backward_sum_splits, which launches nothing otherwise.
// The dV contraction has few outputs (n*n x K x C) and a long reduction (all tiles): while it
// has fewer tiles than the chip has compute units, the reduction is cut into 2^j ranges that
// run as separate work groups.  Ranges hold at least four chunks of 32; at most 32, and at most
// 64 MB of partial sums.
inline int backward_dv_splits(const Geometry& g) {
  const long n2 = (long)(g.m + 2) * (g.m + 2);
  const int tr = 64 * backward_row_blocks(g), tc = 64 * backward_col_blocks(g);
  const long tiles = n2 * ((g.K + tr - 1) / tr) * ((g.C + tc - 1) / tc);
  const long chunks = ((long)g.T + 31) / 32;
  const long bytes = n2 * g.K * g.C * 4;
  int s = 1;
  while (tiles * s < 256 && (long)s * 2 * 4 <= chunks && s < 32 && (long)s * 2 * bytes <= (64L << 20))
    s *= 2;
  return s;
}
// Which of the two contractions read dM straight into registers (gemm_reg_body), the other way being
// through LDS (gemm_lds_body).  Registers keep a whole stage of 64 in flight per wave, which wins while a
// compute unit has one or two work groups to hide its waits with, and on long reductions; LDS
// coalesces the loads and shares them among waves, which wins once the chip is full and the reduction is
// short.  Whole backward pass in us, both from registers / only dV / neither:
//   F(4,3)    100 tiles, C = K = 128 (80 work groups)     21.2 /  21.8 /  22.4
//            1000 tiles, C = 112, K = 96 (608)            38.7 /  37.1 /  35.5
//            1000 tiles, C = K = 256 (864)                68.5 /  72.2 /  69.6
//             512 tiles, C = K = 512 (1152)               99.4 / 100.2 / 107.9
//            2048 tiles, C = K = 256 (1728)              120.1 / 123.1 / 134.0
//           16384 tiles, C = K = 64 (5248)               225.2 / 208.7 / 230.6
// Over 574 shapes (F(2,3), F(4,3), F(6,3), 16 to 16384 tiles, 16 to 512 channels) the choice takes 95.2 % of the
// time of neither, 98.4 % of that of both and 100.4 % of that of the best of the three.  The narrowest
// layers, one sixteenth of a tile of outputs: F(2,3), 512 tiles, C = K = 16: 14.9 / 15.1 / 14.0; F(4,3), 16384
// tiles: 80.2 / 79.9 / 75.5, but F(2,3), 16384 tiles: 45.0 / 44.9 / 47.2.
struct FromRegisters {
  bool dv, du;
};
inline FromRegisters backward_from_registers(const Geometry& g) {
  const long n2 = (long)(g.m + 2) * (g.m + 2);
  const int tr = 64 * backward_row_blocks(g), tc = 64 * backward_col_blocks(g), splits = backward_dv_splits(g);
  const long cols = (g.C + tc - 1) / tc;
  const long groups = cols * ((n2 * ((g.K + tr - 1) / tr) + 7) / 8 * 8 * splits + (n2 * ((g.T + 127) / 128) + 7) / 8 * 8);
  const long range = ((g.T + 31) / 32 + splits - 1) / splits * 32;    // of dV's reduction per work group
  if (g.C + g.K <= 32 && (g.m == 4 || range <= 512)) return {false, false};
  const bool few = groups <= 384;
  return {few || g.K >= 256 || range >= 256, few || (g.K >= 256 && groups <= 5L * g.K)};
}
int backward_dv_reader_parts(const Geometry& g);
hipError_t launch_backward_sum_splits(const Geometry& g, float* dV, hipStream_t st);
// dV -> dw alone, and dU -> dx with dV -> dw in one launch (both non-empty).
hipError_t launch_backward_dw(const Geometry& g, float* dV, float* dw, hipStream_t st);
hipError_t launch_backward_dx_dw(const Geometry& g, const float* dU, float* dx, float* dV,
                                 float* dw, hipStream_t st);
// for_weights = false: out = dU[p][t][c] = scale[p] sum_k dM[p][t][k] codes[p][k][c] (codes = V);
// for_weights = true:  out = dV[p][k][c] = scale[p] sum_t dM[p][t][k] codes[p][t][c] (codes = U).
hipError_t launch_backward_gemm(bool for_weights, const Geometry& g, const float* dM,
                                const int8_t* codes, float* out, const MultTable& scale,
                                hipStream_t st);

// Backward pass of the flex layer (wino_flex_backward.hpp).  `part` receives one row
// of 64 floats per work group (the group's share of the matrix gradient).
template <int M>
struct PerMFlexBwd {
  static hipError_t output(const Geometry& g, bool legendre, const void* M_, int m_bits,
                           const float* dy, float* dM, float* part, const FlexMats& fm,
                           const StageMults& mu, float s_in, hipStream_t st);
  static hipError_t input_weight(const Geometry& g, bool legendre, const int8_t* x,
                                 const float* dU, float* dXt, float* dx, float* part_in, const int8_t* w,
                                 float* dV, float* dw, float* part_w, const FlexMats& fm,
                                 const StageMults& mu, float s_in, float s_w, hipStream_t st);
  static hipError_t tile_sum(const Geometry& g, const float* dXt, float* dx, hipStream_t st);
};
extern template struct PerMFlexBwd<2>;
extern template struct PerMFlexBwd<4>;
extern template struct PerMFlexBwd<6>;
// The launches of the flex backward pass besides the contractions, dispatched on g.m.
hipError_t launch_flex_backward_output(const Geometry& g, bool legendre, const void* M_, int m_bits,
                                       const float* dy, float* dM, float* part, const FlexMats& fm,
                                       const StageMults& mu, float s_in, hipStream_t st);
hipError_t launch_flex_backward_input_weight(const Geometry& g, bool legendre, const int8_t* x,
                                             const float* dU, float* dXt, float* dx, float* part_in,
                                             const int8_t* w, float* dV, float* dw,
                                             float* part_w, const FlexMats& fm,
                                             const StageMults& mu, float s_in, float s_w,
                                             hipStream_t st);
hipError_t launch_flex_backward_tile_sum(const Geometry& g, const float* dXt, float* dx,
                                         hipStream_t st);
// For each of three arrays: out[i][v] = sum over r < rows[i] of part[i][r * 64 + v],
// v < count[i], in a fixed order; one launch.
hipError_t launch_sum_partials(const float* const part[3], const long rows[3], const int count[3],
                               float* const out[3], hipStream_t st);

// Both contraction gradients in one launch (falls back to two when one is empty).
hipError_t launch_backward_gemms(const Geometry& g, const float* dM, const int8_t* U,
                                 const int8_t* V, float* dU, float* dV, const MultTable& s_u,
                                 const MultTable& s_v, hipStream_t st);

// Peak probes: kind 0 = int8 MFMA loop (blocks * 4 waves * iters * 4 MFMAs of
// 32x32x32), kind 1 = 24-bit multiply-add loop (blocks * 256 lanes * iters * 8),
// kind 2 = bf16 MFMA loop (blocks * 4 waves * iters * 4 MFMAs of 32x32x16).
hipError_t launch_probe(int kind, int blocks, int iters, int* sink, hipStream_t st);

// Blocks of 32 x 32 per wave of the fp32 contraction along the tiles and the output channels (a work
// group: 64 t tiles x 64 k channels): two along a dimension longer than 64, but one along both where two
// leave no more than one work group per compute unit.  Layer us, two / one: F(2,3), 4 tiles, C = K = 512
// (64 / 128 groups) 38.1 / 33.5; 512 tiles, C = K = 128 (64 / 256) 21.0 / 17.5; 2048 tiles (256 / 1024) 30.7 /
// 29.4; F(4,3), 1000 tiles, C = 112, K = 96 (288 / 1152) 32.6 / 33.1; 2048 tiles, C = K = 128 (576 / 2304)
// 48.9 / 51.1.
struct F32Blocks {
  int t, k;
};
inline F32Blocks f32_contract_blocks(const Geometry& g) {
  const F32Blocks w{g.T > 64 ? 2 : 1, g.K > 64 ? 2 : 1};
  const long groups = (long)(g.m + 2) * (g.m + 2) * ((g.T + 64 * w.t - 1) / (64 * w.t)) *
                      ((g.K + 64 * w.k - 1) / (64 * w.k));
  return groups <= 256 ? F32Blocks{1, 1} : w;
}

// fp32 path (wino_fp32.hip): no casts, float tensors in the int8 path's layouts.
// Operand transforms in one launch; x or w null leaves that one out.
hipError_t launch_operands_f32(const Geometry& g, bool legendre, const float* x, float* U,
                               const float* w, float* V, hipStream_t st);
hipError_t launch_contract_f32(const Geometry& g, const float* U, const float* V, float* M,
                               hipStream_t st);
hipError_t launch_output_f32(const Geometry& g, bool legendre, const float* M, float* y, bool relu,
                             hipStream_t st);

}  // namespace wino
