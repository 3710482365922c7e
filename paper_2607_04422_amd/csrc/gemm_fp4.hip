// Matrix products of the Newton-Schulz step on gfx950 MFMA.
//
// All three products of a step (Section 3.4 display equation) have both
// operands contiguous along the contraction index:
//   A = qX qX^T        (K = n, symmetric: upper tiles only, mirrored)
//   B = b A + c qA qA^T (K = m, symmetric; epilogue reads A, may overwrite it)
//   X <- a X + qB qXt^T (K = m; epilogue reads X_k and writes X_{k+1} in place)
//
// NVFP4 operands (exact bridge): codes and E4M3 scales are decoded to f16 in
// registers (q * s needs at most 6 significant bits and lies in [2^-10, 2688], so it
// is exact in f16).  One MFMA 32x32x16 covers exactly one 16-element block: all its
// products are integer multiples of s_a s_b / 4 with |sum| < 2^19 of those units, so
// the MFMA result (accumulator input 0) is the exact block sum.  Block sums are
// accumulated in binary64 and the epilogue forms the output in binary64 and rounds
// once to binary32, so every product equals the binary32 rounding of its exact value
// whenever the binary64 running sums are exact (every partial sum within 53 bits of
// the smallest product unit, which holds unless the block exponents of a row span
// more than about 20 binades).
//
// Chained blocks.  Element values are q s with q = k/2 (|k| <= 12) and
// s = M 2^(E-10) (E4M3: M <= 15, E >= 1; subnormal scales as M = m, E = 1).  With
// e = E + (trailing zero bits of M), every product of a row i of the first operand and
// a row j of the second over a group G of blocks is a multiple of
// u = 2^(ea_min(i) + eb_min(j) - 22), the minima over G.  Any partial sum of those
// products, in any order, is at most their sum of magnitudes, and by Cauchy-Schwarz at
// most sqrt(S_a(i) S_b(j)), S the sum of squared values over G.  With
// rho_i = S_a(i) 2^(22 - 2 ea_min(i)) = sum_b n2_b 4^(E_b - ea_min(i)) (n2 = sum (2q)^2
// M^2 per block; sigma_j alike) the bound is below 2^24 u whenever rho_i sigma_j <
// 2^48; then every partial sum is exactly representable in binary32, and the MFMAs of
// the group may accumulate into one binary32 register, folded into binary64 once.  A
// group is an aligned run of four or two 64-element stages where the bound of the run
// holds, one stage, or (where a stage's own bound fails) single blocks.  Each wave
// tests the largest rho and sigma of its own rows (diagonal tiles of symmetric
// products test tile-wide maxima, so that (i, j) and (j, i) add the same binary32
// values in the same order and the product stays exactly symmetric).
//
// What bounds the kernel: vector instruction issue.  Per MFMA (32 cycles of the matrix
// core, 4 of the issue port) a 64 x 64 wave tile decodes 8.5 instructions' worth of
// operands and folds 8 per group and stage (one conversion and one binary64 add per
// output), at about 4.4 cycles each; the matrix cores and vector instructions of the
// two waves of a SIMD overlap when they alternate finely, so each MFMA is followed by
// decode instructions of the next block.  Groups of more than one stage cut the folds
// to 0.24 (Gram of qX), 0.8-1.0 (Gram of qA) and 0.55-0.8 (update) per stage and output
// on Student-t momentum, against 1.0, 1.4 and 1.2 with one-stage groups.  Measured
// against shared decoded operands in LDS with one barrier per stage and one-stage
// groups (28-matrix 3B set, same box): Gram of qX 683 -> 816, Gram of qA 607 -> 678,
// update product 662 -> 795 TFLOP/s, call 37.7 -> 33.6 ms.
//
// Work per wave: a 64 x 64 output tile (2 x 2 MFMA tiles), 64 binary64 accumulators and
// 64 binary32 chain registers per lane (249-251 VGPRs, two waves per SIMD); four
// waves share a 128 x 128 workgroup tile.  Small launches run 32 x 32 per wave, 64 x
// 64 per workgroup.
//
// Binary32 accumulation (GemmFp4Args::acc32, the library's FP4ROOT_F_FP32_ACCUM):
// the same loop with one chain over the whole contraction (zeroed once, never
// folded, no chain bounds), as tensor-core NVFP4 products accumulate in FP32.
// Each product is then within the binary32 accumulation bound of its exact value
// rather than equal to its rounding.
#include "device.h"
#include "internal.h"

#include <atomic>
#include <type_traits>
#include <utility>

namespace fp4r {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Tile forms of the NVFP4 products: WM x WN waves, each owning TM x TN MFMA 32x32
// tiles, WPE waves per SIMD.  Wide decodes half as much per MFMA; Narrow has four
// times the workgroups and a shorter chain per stage, so it wins while a launch does
// not fill the chip with wide workgroups.
template <int WM_, int WN_, int TM_, int TN_, int WPE_>
struct Fp4Tiling {
  static constexpr int WM = WM_, WN = WN_, TM = TM_, TN = TN_, WPE = WPE_, NW = WM_ * WN_;
  static constexpr int kTile = WM_ * TM_ * 32;
  static_assert(kTile == WN_ * TN_ * 32, "square workgroup tiles (symmetric products)");
};
constexpr int kFp4Waves = 4;
using Fp4Wide = Fp4Tiling<2, 2, 2, 2, 2>;
using Fp4Narrow = Fp4Tiling<2, 2, 1, 1, 4>;
static_assert(Fp4Wide::NW == kFp4Waves && Fp4Narrow::NW == kFp4Waves && Fp4Wide::kTile == 2 * Fp4Narrow::kTile,
              "a wide tile is four narrow ones of as many threads");

// Output tile coordinates.  Symmetric products enumerate the upper triangle
// row by row; others are row-major over (tiles_m x tiles_n).
FP4R_DEV void tile_coords(int64_t t, int tiles_m, int tiles_n, bool sym, int& tm, int& tn) {
  if (!sym) {
    tm = (int)(t / tiles_n);
    tn = (int)(t % tiles_n);
    return;
  }
  int r = 0;
  int64_t left = t;
  while (left >= tiles_n - r) {
    left -= tiles_n - r;
    ++r;
  }
  tm = r;
  tn = r + (int)left;
}

// ---------------------------------------------------------------------------
// NVFP4 operand staging.  A lane of a 32x32x16 MFMA holds eight consecutive
// contraction elements of one row: half h = lane / 32 of a 16-element block.  The
// operands are stage-major with the code words of a row's four blocks ordered by
// half (see OperandOut), so the 16 bytes at half h are the lane's codes of a whole
// stage, one word per block.  Each wave copies the rows it multiplies into a ring of
// its own in LDS, straight from memory (global_load_lds, no registers), and decodes
// the words in registers just before their MFMAs: no data passes between waves, so
// the main loop has no barrier.

// Copies one stage of a wave's operand rows into its ring slot at LDS byte `lds`:
// 16 code bytes per lane for each of TM + TN row tiles (lane i to slot byte 512 +
// 1024 t + 16 i) and the scale words of up to 64 rows per operand (4 bytes per lane, A
// at slot byte 0, B at 256).  An instruction offset moves both addresses, so one M0
// value serves them all and the code bases are 4096 bytes low: the lane offsets
// `co` (64-byte granules of rows, + 4096 - 512 - 1024 t) make up for it.  The loads are
// counted by vmcnt only: the caller waits (wait_loads) before reading the slot.
template <int TM, int TN>
FP4R_DEV void load_stage(uint32_t lds, const uint32_t (&co)[TM + TN], uint32_t so_a, uint32_t so_b,
                         const uint8_t* ca, const uint8_t* cb, const uint8_t* sa, const uint8_t* sb) {
  static_assert((TM == 2 && TN == 2) || (TM == 1 && TN == 1), "row tiles per wave");
  if constexpr (TM == 2) {
    asm volatile(
        "s_mov_b32 m0, %0\n\ts_nop 0\n\t"
        "global_load_lds_dword %5, %9\n\t"
        "global_load_lds_dword %6, %10 offset:256\n\t"
        "global_load_lds_dwordx4 %1, %7 offset:512\n\t"
        "global_load_lds_dwordx4 %2, %7 offset:1536\n\t"
        "global_load_lds_dwordx4 %3, %8 offset:2560\n\t"
        "global_load_lds_dwordx4 %4, %8 offset:3584" ::"s"(lds),
        "v"(co[0]), "v"(co[1]), "v"(co[2]), "v"(co[3]), "v"(so_a), "v"(so_b), "s"(ca), "s"(cb), "s"(sa), "s"(sb)
        : "memory", "m0");
  } else {
    asm volatile(
        "s_mov_b32 m0, %0\n\ts_nop 0\n\t"
        "global_load_lds_dword %3, %7\n\t"
        "global_load_lds_dword %4, %8 offset:256\n\t"
        "global_load_lds_dwordx4 %1, %5 offset:512\n\t"
        "global_load_lds_dwordx4 %2, %6 offset:1536" ::"s"(lds),
        "v"(co[0]), "v"(co[1]), "v"(so_a), "v"(so_b), "s"(ca), "s"(cb), "s"(sa), "s"(sb)
        : "memory", "m0");
  }
}
// Waits until at most N of this wave's vector memory operations are outstanding.
template <int N>
FP4R_DEV void wait_loads() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

constexpr int kBufWord3 = 0x00020000;          // raw 32-bit data format, no swizzle
constexpr uint32_t kBufOutOfRange = 0x7FFFFFF0u;

constexpr int kSchedValu = 0x2, kSchedMfma = 0x8;   // masks of sched_group_barrier

template <int SEL>
FP4R_DEV f16x2 fp4_pair(uint32_t w, f16x2 s2) {
  // two E2M1 codes (low nibble first) -> two f16, then the exact product with the block scale
  const f16x2 q = __builtin_amdgcn_cvt_scalef32_pk_f16_fp4(w, 1.0f, SEL);
  return q * s2;
}
// Eight codes times their block scale: an MFMA operand of one lane.
FP4R_DEV f16x8 fp4_decode(uint32_t w, _Float16 s) {
  const f16x2 s2 = {s, s};
  const f16x2 p0 = fp4_pair<0>(w, s2), p1 = fp4_pair<1>(w, s2);
  const f16x2 p2 = fp4_pair<2>(w, s2), p3 = fp4_pair<3>(w, s2);
  f16x8 v;
  v[0] = p0[0]; v[1] = p0[1]; v[2] = p1[0]; v[3] = p1[1];
  v[4] = p2[0]; v[5] = p2[1]; v[6] = p3[0]; v[7] = p3[1];
  return v;
}

// Stages whose chain decisions a wave prepares (K up to 64 kChainStages); later stages
// fold every block.
constexpr int kChainWindows = 8, kChainStages = 64 * kChainWindows;

// ---------------------------------------------------------------------------
// Rotated amaxes of an output, for the tensor scale of the operand encoded from
// it next (Section 3.2: the scale follows the largest magnitude after the 16-point
// rotation).  The rotation is the encoder's binary32 butterfly (signs, strides 1,
// 2, 4, 8, factor 1/4); only the largest magnitude is wanted, which permits three
// exact shortcuts:
// * the signs enter the stride-1 stage: fl(s_i u_i +- s_j u_j) is one fma of exact
//   products;
// * a stage across lanes may produce the difference with its sign flipped in the
//   lane holding the higher position: the later stages pair positions that agree
//   in that bit, so the flip reaches the final value unchanged (a sign only);
// * of the last stage's pair fl(p + q), fl(p - q) the larger magnitude is
//   fl(|p| + |q|), and the factor 1/4 commutes with the maximum (rounding is
//   monotone), so it is applied once to the final maximum.

template <int CTRL>
FP4R_DEV float dpp_f(float v) {
  // every source lane of the patterns used here exists (bound_ctrl only spares the old value)
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true));
}
constexpr int kDppXor1 = 0xB1, kDppXor2 = 0x4E, kDppHalfMirror = 0x141, kDppMirror = 0x140;

// Row direction, four consecutive elements per lane: lane p = lane % 4 of a quad
// holds positions 4p .. 4p + 3 of a 16-element block; sg = their signs (+-1),
// s4 = +1 for even p, -1 for odd p.  Returns the unscaled maximum magnitude of
// the quad's block (every lane of the quad gets the same value).  All lanes of
// the wave must be active.
FP4R_DEV float rot_rows_max4(float4 u, const float (&sg)[4], float s4) {
  const float t1 = sg[1] * u.y, t3 = sg[3] * u.w;
  const float a0 = __builtin_fmaf(sg[0], u.x, t1), a1 = __builtin_fmaf(sg[0], u.x, -t1);
  const float a2 = __builtin_fmaf(sg[2], u.z, t3), a3 = __builtin_fmaf(sg[2], u.z, -t3);
  const float b0 = a0 + a2, b2 = a0 - a2, b1 = a1 + a3, b3 = a1 - a3;
  // stride 4: partner p ^ 1
  const float c0 = __builtin_fmaf(dpp_f<kDppXor1>(b0), s4, b0);
  const float c1 = __builtin_fmaf(dpp_f<kDppXor1>(b1), s4, b1);
  const float c2 = __builtin_fmaf(dpp_f<kDppXor1>(b2), s4, b2);
  const float c3 = __builtin_fmaf(dpp_f<kDppXor1>(b3), s4, b3);
  // stride 8: partner p ^ 2
  const float m0 = fabsf(c0) + fabsf(dpp_f<kDppXor2>(c0));
  const float m1 = fabsf(c1) + fabsf(dpp_f<kDppXor2>(c1));
  const float m2 = fabsf(c2) + fabsf(dpp_f<kDppXor2>(c2));
  const float m3 = fabsf(c3) + fabsf(dpp_f<kDppXor2>(c3));
  return fmaxf(fmaxf(m0, m1), fmaxf(m2, m3));
}

// Column direction, on the MFMA 32x32 output layout: v[B .. B + 7] of a lane are
// rows (e & 3) + 4 hb + 8 (e >> 2), e = 0 .. 7, of a 16-row block of its column
// (hb = lane / 32); sg = the signs of those rows, s4 = +1 (hb = 0) or -1.
// Returns the unscaled maximum magnitude over the lane's 8 outputs.  All lanes of
// the wave must be active.
template <int B>
FP4R_DEV float rot_cols_max8(const float (&v)[16], const float (&sg)[8], float s4) {
  float a[8], b[8], c[8];
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    const float t = sg[e + 1] * v[B + e + 1];
    a[e] = __builtin_fmaf(sg[e], v[B + e], t);
    a[e + 1] = __builtin_fmaf(sg[e], v[B + e], -t);
  }
#pragma unroll
  for (int e = 0; e < 8; e += 4) {
    b[e] = a[e] + a[e + 2];
    b[e + 2] = a[e] - a[e + 2];
    b[e + 1] = a[e + 1] + a[e + 3];
    b[e + 3] = a[e + 1] - a[e + 3];
  }
  // stride 4: both halves' values of the pair in every lane
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const auto lh = __builtin_amdgcn_permlane32_swap(__float_as_uint(b[e]), __float_as_uint(b[e]), false, false);
    c[e] = __builtin_fmaf(__uint_as_float(lh[1]), s4, __uint_as_float(lh[0]));
  }
  float m = 0.0f;
#pragma unroll
  for (int e = 0; e < 4; ++e) m = fmaxf(m, fabsf(c[e]) + fabsf(c[e + 4]));
  return m;
}

// Maximum of a non-negative value over the wave (bit pattern, uniform).
FP4R_DEV uint32_t wave_max_bits(float v) {
  v = fmaxf(v, dpp_f<kDppXor1>(v));
  v = fmaxf(v, dpp_f<kDppXor2>(v));
  v = fmaxf(v, dpp_f<kDppHalfMirror>(v));
  v = fmaxf(v, dpp_f<kDppMirror>(v));
  const uint32_t b = __float_as_uint(v);
  const uint32_t r0 = __builtin_amdgcn_readlane(b, 0), r1 = __builtin_amdgcn_readlane(b, 16);
  const uint32_t r2 = __builtin_amdgcn_readlane(b, 32), r3 = __builtin_amdgcn_readlane(b, 48);
  const uint32_t m01 = r0 > r1 ? r0 : r1, m23 = r2 > r3 ? r2 : r3;
  return m01 > m23 ? m01 : m23;
}

// ---------------------------------------------------------------------------
// Exact NVFP4 product.

// Zeroes a chain register with eight 64-bit moves (sixteen 32-bit ones otherwise); the
// wait states at the end are those an MFMA reading it next needs.
FP4R_DEV f32x16 zero16() {
  typedef double f64x8 __attribute__((ext_vector_type(8)));
  f64x8 z;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    double d;
    if (k < 7) asm volatile("v_mov_b64 %0, 0" : "=v"(d));
    else asm volatile("v_mov_b64 %0, 0\n\ts_nop 1" : "=v"(d));
    z[k] = d;
  }
  return __builtin_bit_cast(f32x16, z);
}

template <int KB>
using block_t = std::integral_constant<int, KB>;

// LDS of one workgroup in form C.
template <class C>
struct Fp4Lds {
  static constexpr int kOps = C::TM + C::TN;
  // ring of two raw stages per wave (see load_stage)
  static constexpr int kSlot = 512 + 1024 * kOps, kRing = 2 * kSlot;
  // padded row of the FP32 output tile of the epilogue: rows stay 16-byte aligned, and
  // the two half-waves of an MFMA-layout write (rows 4 apart) fall 32 banks apart
  static constexpr int kLdT = C::kTile + 8;
  static constexpr int kMain = C::NW * kRing, kEpi = C::kTile * kLdT * (int)sizeof(float);
  static constexpr int kBytes = kMain > kEpi ? kMain : kEpi;
};
struct Fp4Shared {
  uint64_t flags[kFp4Waves][2][kChainWindows];   // per wave: stages that chain, that continue a group
  uint32_t red[2][kFp4Waves];                    // per-wave amaxes (rows, columns)
};

// Output tile (tm, tn) of matrix `mat` of one product in form C; finp (may be null)
// routes a last update's output to the callers' matrices.  Every kernel entry below
// runs this body.
template <int MODE, class C, bool ACC32>
FP4R_DEV void gemm_fp4_tile(const GemmFp4Args& g, int64_t mat, int tm, int tn, const GemmFin* finp, char* smem,
                            Fp4Shared& sh) {
  constexpr int WN_ = C::WN, TM = C::TM, TN = C::TN, NW = C::NW;
  constexpr int BM = C::kTile, BN = C::kTile, NT = NW * 64;
  constexpr int kOps = Fp4Lds<C>::kOps, kSlot = Fp4Lds<C>::kSlot, kRing = Fp4Lds<C>::kRing, kLdT = Fp4Lds<C>::kLdT;
  constexpr bool kSym = MODE != kModeUpdateX;
  const int64_t row0 = (int64_t)tm * BM, col0 = (int64_t)tn * BN;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int wm = wave / WN_, wn = wave % WN_;
  const int nstages = (int)((g.K + 63) / 64);   // K <= 2^21

  double acc[TM][TN][16];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0;

  // a group chains if rho sigma < 2^48; the limit leaves room for the rounding of
  // the binary32 product rho * sigma
  constexpr float kLim = 281474976710656.0f * (1.0f - 1.0f / 65536.0f);   // 2^48 (1 - 2^-16)
  // the rows a wave covers; diagonal tiles of symmetric products test the tile's rows
  // (see the header)
  const bool diag = kSym && tm == tn;
  const int levels = ACC32 ? 0 : g.a.levels;
  const int ushift = levels > 1 ? 5 : 4;   // rows of a record unit
  const int64_t entries = levels > 1 ? chain_entries(nstages) : nstages;
  const float* const rec_a = g.a.rec + mat * g.a.rec_bstride;
  const float* const rec_b = g.b.rec + mat * g.b.rec_bstride;
  // the largest bound of entry `at` over the units of `rows` rows from `r0` on (units
  // past the matrix hold no rows)
  auto unit_max = [&](const float* rec, int64_t total, int64_t r0, int rows, int64_t at) {
    float mx = 0.0f;
    const int64_t u0 = r0 >> ushift, end = (total + (1 << ushift) - 1) >> ushift;
    for (int k = 0; k < (rows >> ushift); ++k)
      if (u0 + k < end) mx = fmaxf(mx, rec[(u0 + k) * entries + at]);
    return mx;
  };
  // Decides for 64 stages at a time, one per lane: a stage chains if its own bound
  // holds, and continues the group of the stage before it if the bound of an aligned
  // run of two or four stages holds in which it is not the first.
  auto fill_flags = [&]() {
    const int64_t a0 = row0 + (diag ? 0 : wm * TM * 32), b0 = col0 + (diag ? 0 : wn * TN * 32);
    const int ra = diag ? BM : TM * 32, rb = diag ? BN : TN * 32;
    for (int w = 0; w < kChainWindows && 64 * w < nstages; ++w) {
      const int ss = 64 * w + lane;
      bool chain = false, cont = false;
      if (levels > 0 && ss < nstages) {
        chain = unit_max(rec_a, g.M, a0, ra, ss) * unit_max(rec_b, g.N, b0, rb, ss) < kLim;
        if (levels > 1) {
          int64_t at = nstages;
          for (int l = 1; l <= 2; ++l) {
            if (ss & ((1 << l) - 1))
              cont |= unit_max(rec_a, g.M, a0, ra, at + (ss >> l)) * unit_max(rec_b, g.N, b0, rb, at + (ss >> l)) < kLim;
            at += (nstages + (1 << l) - 1) >> l;
          }
        }
      }
      const uint64_t mc = __builtin_amdgcn_ballot_w64(chain), mo = __builtin_amdgcn_ballot_w64(cont);
      if (lane == 0) {
        sh.flags[wave][0][w] = mc;
        sh.flags[wave][1][w] = mo;
      }
    }
  };

  // Operand t = 0 .. TM - 1 are the wave's row tiles of A, the next TN those of B.
  // Rows past the matrix read the last row instead (their outputs are discarded) and
  // stages past the last read the last one (never used), so every load is in range.
  const uint8_t* const codes_a = g.a.codes + mat * g.a.codes_bstride + row0 * 32;
  const uint8_t* const codes_b = g.b.codes + mat * g.b.codes_bstride + col0 * 32;
  const uint8_t* const scales_a = g.a.scales + mat * g.a.scales_bstride + row0 * 4;
  const uint8_t* const scales_b = g.b.scales + mat * g.b.scales_bstride + col0 * 4;
  uint32_t row[kOps];
#pragma unroll
  for (int t = 0; t < kOps; ++t) {
    const int64_t live = t < TM ? g.M - row0 : g.N - col0;
    const int r = (t < TM ? wm * TM + t : wn * TN + t - TM) * 32 + (lane & 31);
    row[t] = (uint32_t)(r < live ? r : (int)live - 1);
  }
  uint32_t co[kOps];
#pragma unroll
  for (int t = 0; t < kOps; ++t) co[t] = row[t] * 32 + (uint32_t)(lane >> 5) * 16 + (4096 - 512 - 1024 * t);
  // scale words of the wave's rows: lane i the word of row i (64 rows with two row
  // tiles; with one, lanes 32 .. 63 repeat its rows), A at slot byte 0
  const int own = TM == 2 ? lane : lane & 31;
  const int64_t live_a = g.M - row0, live_b = g.N - col0;
  const int sr_a = wm * TM * 32 + own, sr_b = wn * TN * 32 + own;
  const uint32_t so_a = (uint32_t)(sr_a < live_a ? sr_a : (int)live_a - 1) * 4;
  const uint32_t so_b = (uint32_t)(sr_b < live_b ? sr_b : (int)live_b - 1) * 4 + (4096 - 256);
  char* const ring = smem + wave * kRing;
  const uint32_t ring_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)ring;
  // the next stage to load; past the last one the pointers stay
  const uint8_t *ca = codes_a - 4096, *cb = codes_b - 4096, *sa = scales_a, *sb = scales_b - 4096;
  const int64_t step_a = g.M * 32, step_b = g.N * 32;
  auto issue = [&](int stage) __attribute__((always_inline)) {
    load_stage<TM, TN>(ring_lds + (stage & 1) * kSlot, co, so_a, so_b, ca, cb, sa, sb);
    const bool more = stage + 1 < nstages;
    const int64_t da = more ? step_a : 0, db = more ? step_b : 0;
    ca += da;
    cb += db;
    sa += da / 8;
    sb += db / 8;
  };
  constexpr int kLoads = kOps + 2;   // vector memory operations of one stage
  uint4 raw[kOps];
  uint32_t rsc[kOps];
  const int lane_sc = (lane & 31) * 4;
  auto read_raw = [&](int stage) __attribute__((always_inline)) {
    const char* slot = ring + (stage & 1) * kSlot;
#pragma unroll
    for (int t = 0; t < kOps; ++t)
      rsc[t] = *reinterpret_cast<const uint32_t*>(slot + (t < TM ? 128 * t : 256 + 128 * (t - TM)) + lane_sc);
#pragma unroll
    for (int t = 0; t < kOps; ++t) raw[t] = *reinterpret_cast<const uint4*>(slot + 512 + 1024 * t + 16 * lane);
  };
  f16x8 op[2][kOps];   // decoded operands of a block, and of the next one
  auto decode = [&](int kb, int t) __attribute__((always_inline)) {
    const f16x2 sc = kb < 2 ? __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(rsc[t], 1.0f, false)
                            : __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(rsc[t], 1.0f, true);
    const uint32_t w = kb == 0 ? raw[t].x : kb == 1 ? raw[t].y : kb == 2 ? raw[t].z : raw[t].w;
    op[kb & 1][t] = fp4_decode(w, sc[kb & 1]);
  };

  const f32x16 zero = {};
  f32x16 p[TM][TN];   // the binary32 chain registers
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) p[i][j] = zero;
  auto fold = [&](int i, int j) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[i][j][e] = acc[i][j][e] + (double)p[i][j][e];
  };

  issue(0);
  issue(1);
  if constexpr (!ACC32) fill_flags();
  wait_loads<kLoads>();
  read_raw(0);
#pragma unroll
  for (int t = 0; t < kOps; ++t) decode(0, t);
  __builtin_amdgcn_sched_barrier(0);
  // Stage s: its raw words are in registers and the operands of its first block are
  // decoded.  Every MFMA is followed by decode work of the next block (the matrix core
  // is busy for 32 cycles, the issue port for 4).  The chain registers hold the open
  // group on entry; the exact products fold it into binary64 before the first block,
  // or before every block where the stage may not chain.
  uint64_t chain_mask = 0, cont_mask = 0;
  for (int s = 0; s < nstages; ++s) {
    if (!ACC32 && (s & 63) == 0) {
      chain_mask = cont_mask = 0;
      if (s < kChainStages) {
        const uint64_t c = sh.flags[wave][0][s >> 6], o = sh.flags[wave][1][s >> 6];
        chain_mask = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(c >> 32)) << 32) |
                     (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)c);
        cont_mask = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(o >> 32)) << 32) |
                    (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)o);
      }
    }
    const bool chains = (chain_mask >> (s & 63)) & 1, continues = (cont_mask >> (s & 63)) & 1;
    // the slot of stage s is free once its words have reached the registers
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    issue(s + 2);
    __builtin_amdgcn_sched_barrier(0);
    // the MFMAs of block kb and the decode of the next block, in a fixed order: one
    // MFMA, then the vector instructions that fit its time on the matrix core
    auto block = [&](auto kb_tag) __attribute__((always_inline)) {
      constexpr int kb = decltype(kb_tag)::value;
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          p[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(op[kb & 1][i], op[kb & 1][TM + j], p[i][j], 0, 0, 0);
#pragma unroll
      for (int t = 0; t < kOps; ++t) {
        decode((kb + 1) & 3, t);
        asm volatile("" : "+v"(op[(kb + 1) & 1][t]));
      }
#pragma unroll
      for (int t = 0; t < TM * TN; ++t) {
        __builtin_amdgcn_sched_group_barrier(kSchedMfma, 1, 0);
        __builtin_amdgcn_sched_group_barrier(kSchedValu, (8 * kOps + TM * TN - 1) / (TM * TN) + 1, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    // a stage that may not chain starts a group at every block
    auto split = [&]() __attribute__((always_inline)) {
      if (!ACC32 && !chains) {
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            fold(i, j);
            p[i][j] = zero16();
          }
      }
    };
    if (!ACC32 && !continues) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          fold(i, j);
          p[i][j] = zero16();
        }
    }
    block(block_t<0>());
    split();
    block(block_t<1>());
    split();
    block(block_t<2>());
    split();
    wait_loads<kLoads>();
    read_raw(s + 1);
    __builtin_amdgcn_sched_barrier(0);
    block(block_t<3>());
  }
  wait_loads<0>();
  if constexpr (!ACC32) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) fold(i, j);
  } else {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][j][e] = (double)p[i][j][e];
  }
  __syncthreads();   // the epilogue reuses the rings

  // epilogue: binary64 formula, one rounding to binary32, staged through LDS, one
  // MFMA tile at a time
  const double sga = (double)g.sc[mat].sg[g.slot_a], sgb = (double)g.sc[mat].sg[g.slot_b];
  const double alpha = sga * sgb;   // exact: product of two binary32 values
  const double fa = (double)g.ca, fb = (double)g.cb, fc = (double)g.cc;
  float* out = g.out + mat * g.out_bstride;
  const float* aux = g.aux ? g.aux + mat * g.out_bstride : nullptr;
  float* tile = reinterpret_cast<float*>(smem);
  // the epilogue operand (A for B, X_k for X_{k+1}) of this lane's outputs of MFMA
  // tile (i, j) (lanes past the edge read 0)
  const int64_t live_rows = g.M - row0 < BM ? g.M - row0 : BM;
  const __amdgpu_buffer_rsrc_t aux_rs = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(aux ? aux + row0 * g.N : out), (short)0, MODE != kModeGramA ? (int)(live_rows * g.N * 4) : 0, kBufWord3);
  float xin[2][16];   // of two tiles in turn: the next one's loads are in flight
  auto load_aux = [&](int i, int j, float (&x)[16]) __attribute__((always_inline)) {
    const int64_t c = col0 + (wn * TN + j) * 32 + (lane & 31);
    const int rl = (wm * TM + i) * 32 + 4 * (lane >> 5);
    const uint32_t off0 = c < g.N ? (uint32_t)((rl * g.N + c) * 4) : kBufOutOfRange;
#pragma unroll
    for (int e = 0; e < 16; ++e)
      x[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                           aux_rs, (int)(off0 + (uint32_t)((8 * (e >> 2) + (e & 3)) * g.N * 4)), 0, 0));
  };
  if (MODE != kModeGramA) load_aux(0, 0, xin[0]);
  // off-diagonal tiles of symmetric products (and a transposed final output): the
  // transposed tile straight from registers (four consecutive rows of a column
  // form a row segment of it)
  const bool mirror = kSym && tm != tn;
  const bool fin = !kSym && finp != nullptr && finp->count > 0;
  float* const fin_out = fin ? finp->out[mat] : nullptr;
  const int64_t fin_ld = fin ? finp->ld[mat] : 0;
  const bool fin_tall = fin && finp->tall[mat] != 0;
  const bool do_rows = g.amax_row_slot >= 0;
  const bool do_cols = g.amax_col_slot >= 0 && (!kSym || mirror);
  float cmax = 0.0f, rmax = 0.0f;
  const int hb = lane >> 5;
  float csg[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) csg[e] = ((g.amax_mask >> ((e & 3) + 4 * hb + 8 * (e >> 2))) & 1u) ? -1.0f : 1.0f;
  const float cs4 = hb ? -1.0f : 1.0f;
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      constexpr int kTiles = TM * TN;
      const int tile_no = i * TN + j;
      if (MODE != kModeGramA && tile_no + 1 < kTiles)
        load_aux((tile_no + 1) / TN, (tile_no + 1) % TN, xin[(tile_no + 1) & 1]);
      const float(&x)[16] = xin[tile_no & 1];
      // this lane's outputs of MFMA tile (i, j) in binary32 (zero outside the matrix)
      float val[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int rl = (wm * TM + i) * 32 + 8 * (e >> 2) + 4 * hb + (e & 3);
        const int cl = (wn * TN + j) * 32 + (lane & 31);
        double v = alpha * acc[i][j][e];
        if (MODE == kModeGramB) v = fb * (double)x[e] + fc * v;
        if (MODE == kModeUpdateX) v = fa * (double)x[e] + v;
        const bool in = row0 + rl < g.M && col0 + cl < g.N;
        val[e] = in ? (float)v : 0.0f;
        tile[rl * kLdT + cl] = val[e];
      }
      const int cl = (wn * TN + j) * 32 + (lane & 31);
      if (fin_tall || mirror) {
#pragma unroll
        for (int e4 = 0; e4 < 4; ++e4) {
          const int rb = (wm * TM + i) * 32 + 8 * e4 + 4 * hb;
          const int64_t tr = col0 + cl, tc = row0 + rb;
          if (tr < g.N && tc < g.M) {
            float* dst = fin_tall ? fin_out + tr * fin_ld + tc : out + tr * g.N + tc;
            *reinterpret_cast<float4*>(dst) = make_float4(val[4 * e4], val[4 * e4 + 1], val[4 * e4 + 2], val[4 * e4 + 3]);
          }
        }
      }
      // rotated amaxes of 16-row blocks of every column (the mirrored tile's rows,
      // or X_{k+1} along m) from registers
      if (do_cols) {
        if (g.amax_rotate) {
          cmax = fmaxf(cmax, rot_cols_max8<0>(val, csg, cs4));
          cmax = fmaxf(cmax, rot_cols_max8<8>(val, csg, cs4));
        } else {
#pragma unroll
          for (int e = 0; e < 16; ++e) cmax = fmaxf(cmax, fabsf(val[e]));
        }
      }
    }
  __syncthreads();
  // rows of the tile: 32 lanes per row, one 16-byte slot each (coalesced stores;
  // a quad of lanes holds one 16-column block), and the rotated amaxes of
  // 16-column blocks of every row
  {
    constexpr int kSlots = BN / 4;
    static_assert(NT % kSlots == 0 && (BM * kSlots) % NT == 0, "the row pass covers the tile");
    const int pq = lane & 3;
    float sg[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) sg[w] = ((g.amax_mask >> (4 * pq + w)) & 1u) ? -1.0f : 1.0f;
    const float s4 = (pq & 1) ? -1.0f : 1.0f;
    constexpr int kIt = BM * kSlots / NT;
#pragma unroll
    for (int it = 0; it < kIt; ++it) {
      const int idx = threadIdx.x + NT * it;
      const float4 u = *reinterpret_cast<const float4*>(tile + (idx / kSlots) * kLdT + 4 * (idx % kSlots));
      const int64_t r = row0 + idx / kSlots, c = col0 + 4 * (idx % kSlots);
      if (r < g.M && c < g.N && !fin_tall)
        *reinterpret_cast<float4*>(fin ? fin_out + r * fin_ld + c : out + r * g.N + c) = u;
      if (do_rows) {
        if (g.amax_rotate) rmax = fmaxf(rmax, rot_rows_max4(u, sg, s4));
        else rmax = fmaxf(rmax, fmaxf(fmaxf(fabsf(u.x), fabsf(u.y)), fmaxf(fabsf(u.z), fabsf(u.w))));
      }
    }
  }
  // one maximum per direction and workgroup, recorded on the workgroup's amax line
  if (do_rows || do_cols) {
    const uint32_t wr = wave_max_bits(rmax), wc = wave_max_bits(cmax);
    if (lane == 0) {
      sh.red[0][wave] = wr;
      sh.red[1][wave] = wc;
    }
    __syncthreads();
    if (threadIdx.x < 2 && (threadIdx.x == 0 ? do_rows : do_cols)) {
      uint32_t m = 0;
#pragma unroll
      for (int w = 0; w < NW; ++w) m = m > sh.red[threadIdx.x][w] ? m : sh.red[threadIdx.x][w];
      const float mf = g.amax_rotate ? 0.25f * __uint_as_float(m) : __uint_as_float(m);
      amax_record(&g.sc[mat], threadIdx.x == 0 ? g.amax_row_slot : g.amax_col_slot, blockIdx.x, mf);
    }
  }
}

// Workgroup `wg` of a launch: in the wide form the first `wide` workgroups take one wide
// tile each and the later ones a quadrant (a narrow tile) of the wide tiles that follow,
// four workgroups per wide tile; in the narrow form every workgroup takes one narrow tile.
// t counts the tiles of the launch in the form's own size.
struct TileSlot {
  int64_t t;
  int quadrant;   // -1: the whole tile
};
FP4R_DEV TileSlot tile_slot(int64_t wg, int64_t wide) {
  if (wg < wide) return TileSlot{wg, -1};
  return TileSlot{wide + (wg - wide) / 4, (int)((wg - wide) & 3)};
}

// The work of a slot whose tile is number t of product g.
template <int MODE, class C, bool ACC32>
FP4R_DEV void run_slot(const GemmFp4Args& g, int64_t t, int quadrant, int tiles_m, int tiles_n, int64_t tiles_per_mat,
                       const GemmFin* fin, char* smem, Fp4Shared& sh) {
  constexpr bool kSym = MODE != kModeUpdateX;
  const int64_t mat = t / tiles_per_mat;
  int tm, tn;
  tile_coords(t % tiles_per_mat, tiles_m, tiles_n, kSym, tm, tn);
  if constexpr (C::kTile == Fp4Wide::kTile) {
    if (quadrant >= 0) {
      const int ntm = 2 * tm + (quadrant >> 1), ntn = 2 * tn + (quadrant & 1);
      if (kSym && ntn < ntm) return;   // the mirror of another quadrant
      if ((int64_t)ntm * Fp4Narrow::kTile >= g.M || (int64_t)ntn * Fp4Narrow::kTile >= g.N) return;
      gemm_fp4_tile<MODE, Fp4Narrow, ACC32>(g, mat, ntm, ntn, fin, smem, sh);
      return;
    }
  }
  gemm_fp4_tile<MODE, C, ACC32>(g, mat, tm, tn, fin, smem, sh);
}

// One product per launch (its arguments at fixed offsets).
template <int MODE, class C, bool ACC32>
__global__ __launch_bounds__(C::NW * 64) __attribute__((amdgpu_waves_per_eu(C::WPE)))
void k_gemm_fp4(GemmFp4Args g, int tiles_m, int tiles_n, int64_t tiles_per_mat, int64_t wide, GemmFin fin) {
  __shared__ __attribute__((aligned(16))) char smem[Fp4Lds<C>::kBytes];
  __shared__ Fp4Shared sh;
  const TileSlot slot = tile_slot(blockIdx.x, wide);
  run_slot<MODE, C, ACC32>(g, slot.t, slot.quadrant, tiles_m, tiles_n, tiles_per_mat, &fin, smem, sh);
}

// Several products of one mode per launch: each workgroup finds its product (uniform
// over the workgroup) from the cumulative tile counts.
template <int MODE, class C, bool ACC32>
__global__ __launch_bounds__(C::NW * 64) __attribute__((amdgpu_waves_per_eu(C::WPE)))
void k_gemm_fp4_multi(GemmFp4Batch gb) {
  __shared__ __attribute__((aligned(16))) char smem[Fp4Lds<C>::kBytes];
  __shared__ Fp4Shared sh;
  const TileSlot slot = tile_slot(blockIdx.x, gb.wide);
  int pi = 0;
  while (pi + 1 < gb.count && slot.t >= gb.tile_end[pi]) ++pi;
  const int64_t t = slot.t - (pi > 0 ? gb.tile_end[pi - 1] : 0);
  run_slot<MODE, C, ACC32>(gb.p[pi], t, slot.quadrant, gb.tiles_m[pi], gb.tiles_n[pi], gb.tiles_per_mat[pi], nullptr,
                           smem, sh);
}

template <int MODE, class C, bool ACC32>
void launch_fp4_form(dim3 grid, hipStream_t st, const GemmFp4Batch& gb, const GemmFin& f) {
  if (gb.count == 1)
    hipLaunchKernelGGL((k_gemm_fp4<MODE, C, ACC32>), grid, dim3(C::NW * 64), 0, st, gb.p[0], (int)gb.tiles_m[0],
                       (int)gb.tiles_n[0], gb.tiles_per_mat[0], gb.wide, f);
  else
    hipLaunchKernelGGL((k_gemm_fp4_multi<MODE, C, ACC32>), grid, dim3(C::NW * 64), 0, st, gb);
}

template <int MODE, bool ACC32>
void launch_fp4_mode(bool wide, dim3 grid, hipStream_t st, const GemmFp4Batch& gb, const GemmFin& f) {
  if (wide) launch_fp4_form<MODE, Fp4Wide, ACC32>(grid, st, gb, f);
  else launch_fp4_form<MODE, Fp4Narrow, ACC32>(grid, st, gb, f);
}

// The kernel of one launch: mode, tile form and accumulation.
template <bool ACC32>
void launch_fp4_kernel(GemmMode mode, bool wide, dim3 grid, hipStream_t st, const GemmFp4Batch& gb,
                       const GemmFin& f) {
  switch (mode) {
    case kModeGramA: launch_fp4_mode<kModeGramA, ACC32>(wide, grid, st, gb, f); break;
    case kModeGramB: launch_fp4_mode<kModeGramB, ACC32>(wide, grid, st, gb, f); break;
    default: launch_fp4_mode<kModeUpdateX, ACC32>(wide, grid, st, gb, f);
  }
}

// Launches of at least one round of resident wide workgroups (two per CU) run wide.
// One NS step, narrow / wide us per launch: Gram of qX 16 / 25 (36 wide tiles), 49 / 50
// (272), 130 / 122 (528), 117 / 99 (600); update 17 / 26 (64), 43 / 48 (396), 85 / 76 (512),
// 153 / 131 (1024).
constexpr int64_t kWideMinTiles = 512;
// A last round of at most this many wide tiles is cut into narrow ones: a wide tile
// alone on its CU has one wave per SIMD and takes most of a full round's time.  Grams of
// 4096 x 4096 (528 tiles) 126 -> 107 and 140 -> 117 us, of 4 x 2048 x 2048 (544) 75 -> 64 and
// 87 -> 72 us, update of 3072 x 3072 (576) 108 -> 92 us; rounds filled by more than a third
// measured the same either way.
constexpr int64_t kFp4Round = 512, kTailMax = 192;

std::atomic<int> g_product_tiling{0};

int swap_product_tiling(int mode) { return g_product_tiling.exchange(mode); }

hipError_t launch_gemm_fp4_batch(GemmMode mode, const GemmFp4Args* list, int count, hipStream_t st,
                                 const GemmFin* fin) {
  if (count < 1 || count > kMaxGemmProblems) return hipErrorInvalidValue;
  if (fin && fin->count > 0 && (count != 1 || mode != kModeUpdateX || fin->count != list[0].batch))
    return hipErrorInvalidValue;
  for (int i = 1; i < count; ++i)
    if (list[i].acc32 != list[0].acc32) return hipErrorInvalidValue;   // one accumulation per launch
  // longest contraction first: its tiles take the longest, the short ones fill the tail
  int order[kMaxGemmProblems];
  for (int i = 0; i < count; ++i) order[i] = i;
  for (int i = 1; i < count; ++i)
    for (int j = i; j > 0 && list[order[j]].K > list[order[j - 1]].K; --j) std::swap(order[j], order[j - 1]);
  const bool sym = mode != kModeUpdateX;
  auto tiles_of = [&](const GemmFp4Args& g, int tile, int& tiles_m, int& tiles_n) {
    tiles_m = (int)((g.M + tile - 1) / tile);
    tiles_n = (int)((g.N + tile - 1) / tile);
    return sym ? (int64_t)tiles_m * (tiles_m + 1) / 2 : (int64_t)tiles_m * tiles_n;
  };
  int64_t wide_tiles = 0;
  for (int i = 0; i < count; ++i) {
    int tm, tn;
    wide_tiles += tiles_of(list[i], Fp4Wide::kTile, tm, tn) * list[i].batch;
  }
  const int forced = g_product_tiling.load(std::memory_order_relaxed);
  const bool wide = forced == 0 ? wide_tiles >= kWideMinTiles : forced == 2;
  GemmFp4Batch gb;
  gb.count = 0;
  int64_t total = 0;
  for (int i = 0; i < count; ++i) {
    const GemmFp4Args& g = list[order[i]];
    int tiles_m, tiles_n;
    const int64_t per = tiles_of(g, wide ? Fp4Wide::kTile : Fp4Narrow::kTile, tiles_m, tiles_n);
    if (per * g.batch == 0) continue;
    const int k = gb.count++;
    gb.p[k] = g;
    gb.tiles_m[k] = tiles_m;
    gb.tiles_n[k] = tiles_n;
    gb.tiles_per_mat[k] = per;
    total += per * g.batch;
    gb.tile_end[k] = total;
  }
  if (gb.count == 0) return hipSuccess;
  const int64_t rest = total % kFp4Round;
  gb.wide = wide && forced == 0 && rest <= kTailMax ? total - rest : total;
  const dim3 grid((uint32_t)(gb.wide + 4 * (total - gb.wide)));
  GemmFin f;
  if (fin) f = *fin;
  if (gb.p[0].acc32) launch_fp4_kernel<true>(mode, wide, grid, st, gb, f);
  else launch_fp4_kernel<false>(mode, wide, grid, st, gb, f);
  return hipGetLastError();
}

}  // namespace fp4r
