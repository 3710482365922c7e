// Bandwidth-bound stages of the NVFP4 Newton-Schulz path on gfx950:
// p99 clipping threshold (exact radix select), Frobenius normalisation,
// canonical copies, and the fused rotate + amax / rotate + encode quantiser.
//
// Paper: Section 2 ("NVFP4 format", "Root optimizer"), Section 3.4 (p99
// clipping, NVFP4 NS iteration, RTN + adaptive 4/6), Table 8 (quantile 0.99).
#include "device.h"
#include "internal.h"

#include <type_traits>

namespace fp4r {

// ---------------------------------------------------------------------------
__global__ void k_fill_u32(uint32_t* p, uint32_t v, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

hipError_t launch_fill_u32(uint32_t* p, uint32_t value, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = (n + 255) / 256;
  hipLaunchKernelGGL(k_fill_u32, dim3((uint32_t)blocks), dim3(256), 0, st, p, value, n);
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_init(uint32_t* status, MatScalars* sc, int64_t n, uint4* hist,
                                              int64_t hist_quads) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i == 0 && status) *status = 0u;
  if (i < n) {
    MatScalars& s = sc[i];
#pragma unroll
    for (int l = 0; l < kAmaxSpread; ++l)
#pragma unroll
      for (int k = 0; k < kNumSlots; ++k) s.amax[l].v[k] = 0u;
#pragma unroll
    for (int k = 0; k < kNumSlots; ++k) s.sg[k] = 0.0f;
    s.tau = __uint_as_float(0x7F800000u);   // +inf: clamping is the identity
    s.inv_norm = 1.0f;
  }
  if (i < hist_quads) hist[i] = make_uint4(0u, 0u, 0u, 0u);
}

hipError_t launch_init(uint32_t* status, MatScalars* sc, int64_t n, uint32_t* hist, int64_t hist_words,
                       hipStream_t st) {
  const int64_t quads = hist ? hist_words / 4 : 0, threads = n > quads ? n : quads;
  if (threads <= 0 && !status) return hipSuccess;
  hipLaunchKernelGGL(k_init, dim3((uint32_t)(threads / 256 + 1)), dim3(256), 0, st, status, sc, n,
                     reinterpret_cast<uint4*>(hist), quads);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Clip threshold: tau = fl32(v[lo] + f (v[lo+1] - v[lo])) over the sorted |M|,
// found with a radix select on the binary32 bit patterns (31-bit keys, digits of 11, 10
// and 10 bits).  Both ranks are tracked in the same passes.
//
// The first pass reads the matrix for the top digit.  The second reads it again for the
// next digit of the elements with the selected top digits (about half a percent of a
// heavy-tailed matrix), and each wave also appends those elements to a segment of its
// own; the last pass reads the segments only (a third full read took as long as each of
// the others, 119 us of 1070 per 3B-set group).  A wave whose segment is too short reads
// its part of the matrix again instead.
//
// The Frobenius norm of clamp(M, tau) comes out of the same passes: tau lies between
// v[lo] and v[lo+1], and no element lies strictly between them, so an element whose
// known prefix is below that of v[lo] is not clipped (its square goes into the binary64
// partial of its part of the matrix) and one above that of v[lo+1] is clipped to tau (it is only
// counted); the elements of the two full prefixes are exactly the last histograms (a key
// is the bit pattern of |x|), which the select step sums in bin order once tau is known.
// Partials are formed and added in a fixed order.

// Walks a range of a matrix's quads from q0 on: thread t takes quads t, t + 256, ..., four
// loads issued before any is used; f(element value) in order.  A range whose length is a
// multiple of 256 may be followed by the next one on the same walk.
struct QuadWalk {
  const float* base;
  int64_t ld;
  uint32_t c4, cc;
  int64_t rr;
  bool flat;
};
FP4R_DEV QuadWalk quad_walk(int64_t rows, int64_t cols, const MatRef& r, int64_t q0) {
  QuadWalk w;
  const int64_t c4 = (r.tall() ? rows : cols) / 4;
  w.ld = r.ld_in();
  w.c4 = (uint32_t)c4;
  w.flat = w.ld == 4 * c4;
  w.base = r.in;
  if (w.flat) {
    w.base += 4 * (q0 + threadIdx.x);
    w.rr = 0;
    w.cc = 0;
  } else {
    const int64_t row = q0 / c4;
    const uint32_t c = (uint32_t)(q0 - row * c4) + threadIdx.x;
    w.rr = row + c / w.c4;
    w.cc = c % w.c4;
  }
  return w;
}
FP4R_DEV float4 walk_load(QuadWalk& w) {   // the next quad of this thread
  if (w.flat) {
    const float4 v = *reinterpret_cast<const float4*>(w.base);
    w.base += 1024;
    return v;
  }
  const float4 v = reinterpret_cast<const float4*>(w.base + w.rr * w.ld)[w.cc];
  w.cc += 256u;
  if (w.cc >= w.c4) {
    const uint32_t d = w.cc / w.c4;
    w.rr += d;
    w.cc -= d * w.c4;
  }
  return v;
}
template <class F>
FP4R_DEV void walk_quads(QuadWalk& w, uint32_t nq, F f) {
  for (uint32_t q0 = threadIdx.x; q0 < nq; q0 += 1024u) {
    float4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      v[u] = q0 + 256u * u < nq ? walk_load(w) : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool live = q0 + 256u * u < nq;
      f(v[u].x, live);
      f(v[u].y, live);
      f(v[u].z, live);
      f(v[u].w, live);
    }
  }
}

// Fixed-order sum over 256 threads (thread 0 gets it).
FP4R_DEV double block_sum_256(double v, double* red) {
  red[threadIdx.x] = v;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) red[threadIdx.x] = red[threadIdx.x] + red[threadIdx.x + off];
    __syncthreads();
  }
  return red[0];
}

// Number of floats of a wave's segment in a part of nq quads, and where it starts.
FP4R_DEV uint32_t seg_cap(const ClipArgs& a, uint32_t nq) { return nq >> a.cand_shift; }
FP4R_DEV float* seg_base(const ClipArgs& a, int mi, uint32_t part, uint32_t nq, uint32_t wave) {
  return a.cand + (int64_t)mi * a.cand_stride + (((int64_t)part * a.part_quads * 4) >> a.cand_shift) +
         (int64_t)wave * seg_cap(a, nq);
}

// WIDE: the global counts have 64 bits (a tile's own, at most 2^31, always fit in 32).
template <int PASS, bool WIDE>
FP4R_DEV void radix_hist_tile(const MatRef& r, int64_t rows, int64_t cols, const MatScalars& sm, uint32_t* status,
                              const ClipArgs& a, int mi, uint32_t tile) {
  constexpr int kBins = PASS == 0 ? 2048 : 1024, kSets = PASS == 0 ? 1 : 2;
  __shared__ uint32_t h[kSets][kBins];
  __shared__ double part_sum[kMaxTileParts][4];   // per part and wave
  __shared__ uint32_t above_all;
  for (int i = threadIdx.x; i < kSets * kBins; i += 256) (&h[0][0])[i] = 0;
  if (threadIdx.x == 0) above_all = 0;
  __syncthreads();
  const bool last = PASS == 2 && a.cand != nullptr;   // reads the segments
  const int64_t quads = rows * cols / 4;
  const uint32_t p0 = PASS > 0 ? sm.sel_prefix[0] : 0u, p1 = PASS > 0 ? sm.sel_prefix[1] : 0u;
  const bool two = PASS > 0 && p0 != p1;
  const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  double acc = 0.0;     // squares of the part's elements below prefix p0, in this thread's order
  uint32_t above = 0;   // elements above prefix p1
  bool bad = false;
  // one element of the digit's candidates and the norm (pre: the prefix known so far)
  auto count_key = [&](uint32_t key, uint32_t pre, uint32_t digit, bool live) {
    if (live && pre == p0) atomicAdd(&h[0][digit], 1u);
    if (kSets > 1 && two && live && pre == p1) atomicAdd(&h[kSets - 1][digit], 1u);
    if (a.psum) {
      if (live && pre < p0) {
        const double x = (double)__uint_as_float(key);
        acc = acc + x * x;
      } else if (live && pre > p1) {
        ++above;
      }
    }
  };
  const uint32_t first = tile * a.tile_parts, end = min(first + a.tile_parts, a.parts);
  QuadWalk walk = quad_walk(rows, cols, r, (int64_t)first * a.part_quads);
  const uint32_t lane = threadIdx.x & 63;
  uint32_t seg_n = 0;   // lane i: the elements in this wave's segment of part first + i
  if (last && lane < end - first) seg_n = a.cnt[((int64_t)mi * a.parts + first + lane) * 4 + wave];
  for (uint32_t part = first; part < end; ++part) {
    const int64_t q0 = (int64_t)part * a.part_quads;
    const uint32_t nq = (uint32_t)(quads - q0 < a.part_quads ? quads - q0 : a.part_quads);
    acc = 0.0;
    if constexpr (PASS == 0) {
      walk_quads(walk, nq, [&](float x, bool live) {
        const uint32_t key = __float_as_uint(x) & 0x7FFFFFFFu;
        if (!live) return;
        if (key >= 0x7F800000u) { bad = true; return; }
        atomicAdd(&h[0][key >> 20], 1u);
      });
    } else if constexpr (PASS == 1) {
      float* const seg = a.cand ? seg_base(a, mi, part, nq, wave) : nullptr;
      const uint32_t cap = seg_cap(a, nq);
      uint32_t n = 0;   // elements collected by this wave (uniform)
      walk_quads(walk, nq, [&](float x, bool live) {
        const uint32_t key = __float_as_uint(x) & 0x7FFFFFFFu;
        live = live && key < 0x7F800000u;
        const uint32_t pre = key >> 20;
        count_key(key, pre, (key >> 10) & 1023u, live);
        if (a.cand) {
          const bool mine = live && (pre == p0 || pre == p1);
          const uint64_t mask = __builtin_amdgcn_ballot_w64(mine);
          if (mask) {
            const uint32_t at = n + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                              __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            if (mine && at < cap) seg[at] = x;
            n += (uint32_t)__builtin_popcountll(mask);
          }
        }
      });
      // lanes leave the walk together or not at all, except past the end of the part: the
      // count of the lane that stayed longest (lane 0) is the wave's
      n = __builtin_amdgcn_readfirstlane(n);
      if (a.cand && lane == 0) a.cnt[((int64_t)mi * a.parts + part) * 4 + wave] = n;
    } else if (last) {
      const uint32_t cap = seg_cap(a, nq);
      const uint32_t n = __builtin_amdgcn_readlane(seg_n, (int)(part - first));
      if (n <= cap) {
        const float* const seg = seg_base(a, mi, part, nq, wave);
        for (uint32_t i = lane; i < n; i += 64) {
          const uint32_t key = __float_as_uint(seg[i]) & 0x7FFFFFFFu;
          count_key(key, key >> 10, key & 1023u, true);
        }
      } else {
        QuadWalk w = quad_walk(rows, cols, r, q0);
        walk_quads(w, nq, [&](float x, bool live) {
          const uint32_t key = __float_as_uint(x) & 0x7FFFFFFFu, top = key >> 20;
          count_key(key, key >> 10, key & 1023u, live && (top == p0 >> 10 || top == p1 >> 10));
        });
      }
    } else {
      walk_quads(walk, nq, [&](float x, bool live) {
        const uint32_t key = __float_as_uint(x) & 0x7FFFFFFFu;
        count_key(key, key >> 10, key & 1023u, live && key < 0x7F800000u);
      });
    }
    if (PASS > 0 && a.psum) {
      const double sum = wave_sum_d(acc);
      if (lane == 0) part_sum[part - first][wave] = sum;
    }
  }
  if (PASS == 0 && bad) atomicOr(status, kStatusNonFinite);
  if (PASS > 0 && a.psum && above) atomicAdd(&above_all, above);
  __syncthreads();
  if (PASS > 0 && a.psum && threadIdx.x < end - first) {
    // partials: one per part from the second pass, then one per part from the last
    const double* const w = part_sum[threadIdx.x];
    const int64_t at = (int64_t)mi * 2 * a.parts + (PASS == 2 ? a.parts : 0u) + first + threadIdx.x;
    a.psum[at] = (w[0] + w[1]) + (w[2] + w[3]);
    a.pcnt[at] = threadIdx.x == 0 ? above_all : 0u;
  }
  using Count = std::conditional_t<WIDE, unsigned long long, uint32_t>;
  Count* const hist = reinterpret_cast<Count*>(a.hist) + mi * 2 * kHistBins;
  for (int b = threadIdx.x; b < kBins; b += 256) {
    if (h[0][b]) atomicAdd(&hist[b], (Count)h[0][b]);
    if (kSets > 1 && two && h[kSets - 1][b]) atomicAdd(&hist[kHistBins + b], (Count)h[kSets - 1][b]);
  }
}

template <int PASS, bool WIDE>
__global__ __launch_bounds__(256) void k_radix_hist(MatChunk ch, const MatScalars* sc, uint32_t* status, ClipArgs a) {
  const int mi = (int)(blockIdx.x / a.tiles);
  radix_hist_tile<PASS, WIDE>(ch.m[mi], ch.rows, ch.cols, sc[mi], status, a, mi, blockIdx.x - (uint32_t)mi * a.tiles);
}

// The same passes over the matrices of several shape groups (see ClipSets).
template <int PASS>
__global__ __launch_bounds__(256) void k_radix_hist_sets(ClipSets cs, uint32_t* status) {
  int i = 0;
  while (i + 1 < cs.count && blockIdx.x >= cs.s[i].tile_end) ++i;
  const ClipSet& g = cs.s[i];
  const uint32_t wg = blockIdx.x - (i ? cs.s[i - 1].tile_end : 0u);
  const int mi = (int)(wg / g.a.tiles);
  radix_hist_tile<PASS, false>(cs.m[g.first + mi], g.rows, g.cols, g.sc[mi], status, g.a, mi,
                               wg - (uint32_t)mi * g.a.tiles);
}

// Selects the digit of both ranks from the histograms (cleared for the next pass): one
// workgroup per matrix, bins in thread order, a shuffle scan over each wave and the wave
// totals through LDS (8.4 us as a 256-entry LDS scan per rank).
template <int PASS, bool WIDE>
FP4R_DEV void radix_select(int64_t rows, int64_t cols, int64_t lo, double frac, MatScalars& s, const ClipArgs& a, float eps,
                           int mi) {
  constexpr int kPer = (PASS == 0 ? 2048 : 1024) / 256;   // bins per thread
  using Count = std::conditional_t<WIDE, unsigned long long, uint32_t>;
  typedef Count Count4 __attribute__((ext_vector_type(4)));
  __shared__ Count wsum[2][4];
  __shared__ uint32_t found_prefix[2];
  __shared__ Count found_rank[2];
  __shared__ double red[256];
  __shared__ unsigned long long above_all;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int64_t n = rows * cols;
  const uint32_t pre0 = PASS > 0 ? s.sel_prefix[0] : 0u, pre1 = PASS > 0 ? s.sel_prefix[1] : 0u;
  const bool two = pre0 != pre1;
  Count* const hist = reinterpret_cast<Count*>(a.hist) + (int64_t)mi * 2 * kHistBins;
  Count c[2][kPer], local[2], incl[2];
#pragma unroll
  for (int rr = 0; rr < 2; ++rr) {
    const Count4* hh = reinterpret_cast<const Count4*>(hist + (two ? rr : 0) * kHistBins + t * kPer);
    local[rr] = 0;
#pragma unroll
    for (int j = 0; j < kPer / 4; ++j) {
      const Count4 v = hh[j];
      c[rr][4 * j] = v.x; c[rr][4 * j + 1] = v.y; c[rr][4 * j + 2] = v.z; c[rr][4 * j + 3] = v.w;
      local[rr] += v.x + v.y + v.z + v.w;
    }
    incl[rr] = local[rr];
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const Count up = __shfl_up(incl[rr], off, 64);
      if (lane >= off) incl[rr] += up;
    }
    if (lane == 63) wsum[rr][wave] = incl[rr];
  }
  if (t < 2) found_prefix[t] = found_rank[t] = 0;   // ranks past the counted (finite) elements
  if (t == 0) above_all = 0;
  __syncthreads();
#pragma unroll
  for (int rr = 0; rr < 2; ++rr) {
    Count before = 0;
#pragma unroll
    for (int w = 0; w < 3; ++w)
      if (w < wave) before += wsum[rr][w];
    Count cum = before + incl[rr] - local[rr];
    const Count target = PASS > 0 ? (Count)s.sel_rank[rr] : (Count)(rr == 0 || lo + 1 >= n ? lo : lo + 1);
    if (target >= cum && target - cum < local[rr]) {   // exactly one thread owns the target rank
#pragma unroll
      for (int j = 0; j < kPer; ++j) {
        if (target >= cum && target - cum < c[rr][j]) {
          const uint32_t bin = (uint32_t)(t * kPer + j);
          found_prefix[rr] = PASS == 0 ? bin : (((rr ? pre1 : pre0) << 10) | bin);
          found_rank[rr] = target - cum;
        }
        cum += c[rr][j];
      }
    }
  }
  __syncthreads();
  const uint32_t f0 = found_prefix[0], f1 = found_prefix[1];
  if (PASS == 2) {
    const double v0 = (double)__uint_as_float(f0), v1 = (double)__uint_as_float(f1);
    const float tau = (float)__dadd_rn(v0, __dmul_rn(frac, __dsub_rn(v1, v0)));
    if (t == 0) s.tau = tau;
    if (a.psum) {
      // ||clamp(M, tau)||^2 in a fixed order: the partials below v[lo]'s prefix, the
      // elements of the two prefixes from the histograms (bin order), the elements above
      // at tau^2 each
      const int64_t np = (int64_t)2 * a.parts;
      double below = 0.0;
      unsigned long long above = 0;
      for (int64_t i = t; i < np; i += 256) {
        below = below + a.psum[mi * np + i];
        above += a.pcnt[mi * np + i];
      }
      double cand = 0.0;
#pragma unroll
      for (int rr = 0; rr < 2; ++rr) {
        if (rr == 1 && !two) break;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
          const uint32_t bin = (uint32_t)(t * kPer + j);
          if (c[rr][j]) {
            const double x = (double)fminf(__uint_as_float(((rr ? pre1 : pre0) << 10) | bin), tau);
            cand = cand + (double)c[rr][j] * (x * x);
          }
        }
      }
      if (above) atomicAdd(&above_all, above);
      const double sum_below = block_sum_256(below, red);
      __syncthreads();
      const double sum_cand = block_sum_256(cand, red);
      if (t == 0) {
        const double tt = (double)tau * (double)tau;
        const double total = __dadd_rn(__dadd_rn(sum_below, sum_cand), __dmul_rn((double)above_all, tt));
        const double nu = __dsqrt_rn(total);
        s.inv_norm = (float)__ddiv_rn(1.0, __dadd_rn(nu, (double)eps));
      }
    }
  }
  for (int b = t; b < 2 * kHistBins * (int)sizeof(Count) / 16; b += 256)
    reinterpret_cast<uint4*>(hist)[b] = make_uint4(0u, 0u, 0u, 0u);
  if (t == 0) {
    s.sel_prefix[0] = f0;
    s.sel_prefix[1] = f1;
    s.sel_rank[0] = found_rank[0];
    s.sel_rank[1] = found_rank[1];
  }
}

template <int PASS, bool WIDE>
__global__ __launch_bounds__(256) void k_radix_select(MatChunk ch, MatScalars* sc, ClipArgs a, float eps) {
  radix_select<PASS, WIDE>(ch.rows, ch.cols, ch.lo, ch.frac, sc[blockIdx.x], a, eps, (int)blockIdx.x);
}
template <int PASS>
__global__ __launch_bounds__(256) void k_radix_select_sets(ClipSets cs, float eps) {
  int i = 0;
  while (i + 1 < cs.count && blockIdx.x >= cs.s[i + 1].first) ++i;
  const ClipSet& g = cs.s[i];
  const int mi = (int)(blockIdx.x - g.first);
  radix_select<PASS, false>(g.rows, g.cols, g.lo, g.frac, g.sc[mi], g.a, eps, mi);
}

ClipArgs clip_args(const ClipScratch& w, int64_t quads, int64_t count) {
  ClipArgs a;
  a.hist = w.hist; a.cand = w.cand; a.cand_stride = w.cand_stride; a.cnt = w.cnt; a.psum = w.psum; a.pcnt = w.pcnt;
  a.part_quads = (uint32_t)hist_part_quads(quads);
  a.parts = (uint32_t)hist_parts(quads);
  a.tile_parts = (uint32_t)hist_tile_parts(quads, count);
  a.tiles = (a.parts + a.tile_parts - 1) / a.tile_parts;
  a.cand_shift = w.cand_shift;
  return a;
}

template <bool WIDE>
void launch_radix(const MatChunk& ch, MatScalars* sc, uint32_t* status, const ClipArgs& a, float eps, hipStream_t st) {
  const dim3 full(a.tiles * (uint32_t)ch.count), sel((uint32_t)ch.count), wg(256);
  hipLaunchKernelGGL((k_radix_hist<0, WIDE>), full, wg, 0, st, ch, sc, status, a);
  hipLaunchKernelGGL((k_radix_select<0, WIDE>), sel, wg, 0, st, ch, sc, a, eps);
  hipLaunchKernelGGL((k_radix_hist<1, WIDE>), full, wg, 0, st, ch, sc, status, a);
  hipLaunchKernelGGL((k_radix_select<1, WIDE>), sel, wg, 0, st, ch, sc, a, eps);
  hipLaunchKernelGGL((k_radix_hist<2, WIDE>), full, wg, 0, st, ch, sc, status, a);
  hipLaunchKernelGGL((k_radix_select<2, WIDE>), sel, wg, 0, st, ch, sc, a, eps);
}

hipError_t launch_clip_threshold(const MatChunk& ch, MatScalars* sc, uint32_t* status, const ClipScratch& w, float eps,
                                 hipStream_t st) {
  if (ch.count < 1) return hipSuccess;
  if (w.psum && !w.cand) return hipErrorInvalidValue;
  const ClipArgs a = clip_args(w, ch.rows * ch.cols / 4, ch.count);
  // 64-bit counts from 2^32 elements on, where a rank or a bin may need them
  if (wide_counts(ch.rows * ch.cols)) launch_radix<true>(ch, sc, status, a, eps, st);
  else launch_radix<false>(ch, sc, status, a, eps, st);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Frobenius norm of the matrices without clipping: per-part binary64 partials in a
// fixed order, then one fixed-order sum per matrix (deterministic).

__global__ __launch_bounds__(256) void k_sumsq(MatChunk ch, double* partial, uint32_t* status, uint32_t part_quads,
                                               uint32_t parts, uint32_t tile_parts, uint32_t tiles) {
  __shared__ double part_sum[kMaxTileParts][4];
  const int mi = (int)(blockIdx.x / tiles);
  const uint32_t first = (blockIdx.x - (uint32_t)mi * tiles) * tile_parts, end = min(first + tile_parts, parts);
  const int64_t quads = ch.rows * ch.cols / 4;
  QuadWalk walk = quad_walk(ch.rows, ch.cols, ch.m[mi], (int64_t)first * part_quads);
  bool bad = false;   // a NaN or infinite entry
  for (uint32_t part = first; part < end; ++part) {
    const int64_t left = quads - (int64_t)part * part_quads;
    double acc = 0.0;
    walk_quads(walk, (uint32_t)(left < part_quads ? left : part_quads), [&](float v, bool live) {   // quads past the end are zero
      bad |= live && !(fabsf(v) <= 3.40282347e38f);
      const double x = (double)fminf(fmaxf(v, -__builtin_inff()), __builtin_inff());
      acc = acc + x * x;
    });
    const double sum = wave_sum_d(acc);
    if ((threadIdx.x & 63) == 0) part_sum[part - first][threadIdx.x >> 6] = sum;
  }
  if (__builtin_amdgcn_ballot_w64(bad) != 0 && (threadIdx.x & 63) == 0) atomicOr(status, kStatusNonFinite);
  __syncthreads();
  if (threadIdx.x < end - first) {
    const double* const w = part_sum[threadIdx.x];
    partial[(int64_t)mi * parts + first + threadIdx.x] = (w[0] + w[1]) + (w[2] + w[3]);
  }
}

__global__ __launch_bounds__(256) void k_norm_final(MatScalars* sc, const double* partial, float eps, uint32_t parts) {
  __shared__ double red[256];
  const int mi = blockIdx.x;
  double acc = 0.0;
  for (uint32_t i = threadIdx.x; i < parts; i += 256) acc = acc + partial[(int64_t)mi * parts + i];
  const double total = block_sum_256(acc, red);
  if (threadIdx.x == 0) {
    const double nu = __dsqrt_rn(total);
    sc[mi].inv_norm = (float)__ddiv_rn(1.0, __dadd_rn(nu, (double)eps));
  }
}

// The status code of a call (0, or FP4ROOT_ERR_NONFINITE = -4 when a NaN or Inf
// was seen) from its device status word, into a caller's device word.
__global__ void k_status_out(const uint32_t* status, int32_t* out) {
  if (threadIdx.x == 0) *out = (*status & kStatusNonFinite) ? -4 : 0;
}

hipError_t launch_status_out(const uint32_t* status, int32_t* out, hipStream_t st) {
  hipLaunchKernelGGL(k_status_out, dim3(1), dim3(64), 0, st, status, out);
  return hipGetLastError();
}

hipError_t launch_inv_norm(const MatChunk& ch, MatScalars* sc, double* partial, float eps,
                           uint32_t* status, hipStream_t st) {
  const ClipArgs a = clip_args(ClipScratch{}, ch.rows * ch.cols / 4, ch.count);
  hipLaunchKernelGGL(k_sumsq, dim3(a.tiles * (uint32_t)ch.count), dim3(256), 0, st, ch, partial, status, a.part_quads,
                     a.parts, a.tile_parts, a.tiles);
  hipLaunchKernelGGL(k_norm_final, dim3(ch.count), dim3(256), 0, st, sc, (const double*)partial, eps, a.parts);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Tiled copies through LDS (64 x 64 tiles, coalesced on both sides).

constexpr int kT = 64;

__host__ __device__ inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Block-wide max of non-negative floats; thread 0 returns the result.
FP4R_DEV float block_max_256(float v, float* red) {
  v = warp_max(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

// Prep: canonical X = fl32(clamp(M) * inv) (transposed when rows > cols), staged
// through a 64 x 64 LDS tile that also yields the amaxes of X rotated along n
// (16-column blocks) and along m (16-row blocks) for the first NS step.
FP4R_DEV void prep_tile(const MatRef& d, int64_t xm, int64_t xn, MatScalars& sm, float* X, uint32_t mask, int rotate,
                        int slot_n, int slot_m, uint32_t tt) {   // canonical X: xm x xn
  __shared__ float tile[kT][kT + 1];
  __shared__ float red[4];
  const uint32_t tcols = (uint32_t)cdiv(xn, kT);
  const bool tall = d.tall();
  const int64_t ld_in = d.ld_in();
  const int64_t xr0 = (int64_t)(tt / tcols) * kT, xc0 = (int64_t)(tt % tcols) * kT;   // canonical tile origin
  const float tau = sm.tau;
  const float inv = sm.inv_norm;
  // tile[i][j] = canonical X[xr0 + i][xc0 + j]; 16-byte accesses of M and X (rows of
  // both are 16-byte aligned and m, n are multiples of 16): thread -> four quads
  // v = threadIdx.x + 256 k, row v / 16 of the tile, columns 4 (v % 16) .. + 3
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int v = (int)threadIdx.x + 256 * k, i = v >> 4, q = v & 15;
    if (!tall) {
      const int64_t r = xr0 + i, c = xc0 + 4 * q;
      if (r < xm && c < xn) {
        float4 a = *reinterpret_cast<const float4*>(d.in + r * ld_in + c);
        a.x = fminf(fmaxf(a.x, -tau), tau) * inv;
        a.y = fminf(fmaxf(a.y, -tau), tau) * inv;
        a.z = fminf(fmaxf(a.z, -tau), tau) * inv;
        a.w = fminf(fmaxf(a.w, -tau), tau) * inv;
        *reinterpret_cast<float4*>(X + r * xn + c) = a;
        tile[i][4 * q] = a.x; tile[i][4 * q + 1] = a.y; tile[i][4 * q + 2] = a.z; tile[i][4 * q + 3] = a.w;
      }
    } else {
      // M row xc0 + i, M columns xr0 + 4q .. + 3  ->  X rows xr0 + 4q .. + 3, column xc0 + i
      const int64_t r = xc0 + i, c = xr0 + 4 * q;
      if (r < xn && c < xm) {
        const float4 a = *reinterpret_cast<const float4*>(d.in + r * ld_in + c);
        tile[4 * q][i] = fminf(fmaxf(a.x, -tau), tau) * inv;
        tile[4 * q + 1][i] = fminf(fmaxf(a.y, -tau), tau) * inv;
        tile[4 * q + 2][i] = fminf(fmaxf(a.z, -tau), tau) * inv;
        tile[4 * q + 3][i] = fminf(fmaxf(a.w, -tau), tau) * inv;
      }
    }
  }
  __syncthreads();
  if (tall) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int v = (int)threadIdx.x + 256 * k, i = v >> 4, q = v & 15;
      const int64_t r = xr0 + i, c = xc0 + 4 * q;
      if (r < xm && c < xn)
        *reinterpret_cast<float4*>(X + r * xn + c) =
            make_float4(tile[i][4 * q], tile[i][4 * q + 1], tile[i][4 * q + 2], tile[i][4 * q + 3]);
    }
  }
  // rotated amaxes: thread -> one 16-column block and one 16-row block of the tile
  float mr = 0.0f, mc = 0.0f;
  {
    const int i = threadIdx.x >> 2, b = threadIdx.x & 3;
    if (xr0 + i < xm && xc0 + 16 * b < xn) {
      float u[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) u[k] = tile[i][16 * b + k];
      if (rotate) {
        mr = 0.25f * rot16_absmax4(u, mask);
      } else {
#pragma unroll
        for (int k = 0; k < 16; ++k) mr = fmaxf(mr, fabsf(u[k]));
      }
    }
  }
  {
    const int j = threadIdx.x & 63, b = threadIdx.x >> 6;
    if (xc0 + j < xn && xr0 + 16 * b < xm) {
      float u[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) u[k] = tile[16 * b + k][j];
      if (rotate) {
        mc = 0.25f * rot16_absmax4(u, mask);
      } else {
#pragma unroll
        for (int k = 0; k < 16; ++k) mc = fmaxf(mc, fabsf(u[k]));
      }
    }
  }
  const float br = block_max_256(mr, red);
  __syncthreads();
  const float bc = block_max_256(mc, red);
  if (threadIdx.x == 0) {
    amax_record(&sm, slot_n, tt, br);
    amax_record(&sm, slot_m, tt, bc);
  }
}

__global__ __launch_bounds__(256) void k_prep_copy(MatChunk ch, MatScalars* sc, float* xbase,
                                                   int64_t x_bstride, uint32_t mask, int rotate,
                                                   int slot_n, int slot_m) {
  const uint32_t per = (uint32_t)(cdiv(ch.rows, kT) * cdiv(ch.cols, kT));
  const int mi = (int)(blockIdx.x / per);
  prep_tile(ch.m[mi], ch.rows, ch.cols, sc[mi], xbase + (int64_t)mi * x_bstride, mask, rotate, slot_n, slot_m,
            blockIdx.x - (uint32_t)mi * per);
}
__global__ __launch_bounds__(256) void k_prep_copy_sets(ClipSets cs, uint32_t mask, int rotate, int slot_n,
                                                        int slot_m) {
  int i = 0;
  while (i + 1 < cs.count && blockIdx.x >= cs.s[i].prep_end) ++i;
  const ClipSet& g = cs.s[i];
  const uint32_t wg = blockIdx.x - (i ? cs.s[i - 1].prep_end : 0u);
  const uint32_t per = (uint32_t)(cdiv(g.rows, kT) * cdiv(g.cols, kT));
  const int mi = (int)(wg / per);
  prep_tile(cs.m[g.first + mi], g.rows, g.cols, g.sc[mi], g.X + (int64_t)mi * g.rows * g.cols, mask, rotate, slot_n,
            slot_m, wg - (uint32_t)mi * per);
}

void clip_set(ClipSets& cs, const MatChunk& ch, MatScalars* sc, float* X, const ClipScratch& w) {
  ClipSet& g = cs.s[cs.count];
  const uint32_t tiles = cs.count ? cs.s[cs.count - 1].tile_end : 0u, prep = cs.count ? cs.s[cs.count - 1].prep_end : 0u;
  g.first = cs.mats;
  for (int i = 0; i < ch.count; ++i) cs.m[cs.mats++] = ch.m[i];
  g.rows = ch.rows; g.cols = ch.cols; g.lo = ch.lo; g.frac = ch.frac;
  g.sc = sc;
  g.X = X;
  g.a = clip_args(w, ch.rows * ch.cols / 4, ch.count);
  g.tile_end = tiles + g.a.tiles * (uint32_t)ch.count;
  g.prep_end = prep + (uint32_t)(cdiv(ch.rows, kT) * cdiv(ch.cols, kT)) * (uint32_t)ch.count;
  ++cs.count;
}

hipError_t launch_clip_prep(const ClipSets& cs, uint32_t* status, float eps, uint32_t mask, bool rotate, int slot_n,
                            int slot_m, hipStream_t st) {
  if (cs.count < 1) return hipSuccess;
  const ClipSet& g = cs.s[cs.count - 1];
  const dim3 full(g.tile_end), sel(cs.mats), wg(256);
  hipLaunchKernelGGL(k_radix_hist_sets<0>, full, wg, 0, st, cs, status);
  hipLaunchKernelGGL(k_radix_select_sets<0>, sel, wg, 0, st, cs, eps);
  hipLaunchKernelGGL(k_radix_hist_sets<1>, full, wg, 0, st, cs, status);
  hipLaunchKernelGGL(k_radix_select_sets<1>, sel, wg, 0, st, cs, eps);
  hipLaunchKernelGGL(k_radix_hist_sets<2>, full, wg, 0, st, cs, status);
  hipLaunchKernelGGL(k_radix_select_sets<2>, sel, wg, 0, st, cs, eps);
  hipLaunchKernelGGL(k_prep_copy_sets, dim3(g.prep_end), wg, 0, st, cs, mask, (int)rotate, slot_n, slot_m);
  return hipGetLastError();
}

// Rotated amaxes of X along n and along m from one read (X as given, no clipping): the
// tile and the block passes of k_prep_copy.  A block with a non-finite element sets the
// status and does not count.  One read instead of one per axis: 167 -> 134 us on
// 4 x 3072 x 8192.
__global__ __launch_bounds__(256) void k_amax_x2(const float* x, int64_t m, int64_t n, int64_t x_bstride,
                                                 uint32_t mask, int rotate, MatScalars* sc, int slot_n,
                                                 int slot_m, uint32_t* status) {
  __shared__ float tile[kT][kT + 1];
  __shared__ float red[4];
  const int64_t b = blockIdx.y;
  const uint32_t tn = (uint32_t)cdiv(n, kT);
  const int64_t r0 = (int64_t)(blockIdx.x / tn) * kT, c0 = (int64_t)(blockIdx.x % tn) * kT;
  const float* X = x + b * x_bstride;
  bool bad = false;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int v = (int)threadIdx.x + 256 * k, i = v >> 4, q = v & 15;
    if (r0 + i < m && c0 + 4 * q < n) {
      const float4 a = *reinterpret_cast<const float4*>(X + (r0 + i) * n + c0 + 4 * q);
      tile[i][4 * q] = a.x; tile[i][4 * q + 1] = a.y; tile[i][4 * q + 2] = a.z; tile[i][4 * q + 3] = a.w;
      bad |= !(fabsf(a.x) <= 3.40282347e38f) | !(fabsf(a.y) <= 3.40282347e38f) |
             !(fabsf(a.z) <= 3.40282347e38f) | !(fabsf(a.w) <= 3.40282347e38f);
    }
  }
  const bool any_bad = __syncthreads_or(bad);
  if (any_bad && threadIdx.x == 0) atomicOr(status, kStatusNonFinite);
  auto block_amax = [&](float (&u)[16]) {
    bool ok = true;
    if (any_bad) {
#pragma unroll
      for (int k = 0; k < 16; ++k) ok = ok && ((__float_as_uint(u[k]) & 0x7F800000u) != 0x7F800000u);
    }
    float v = 0.0f;
    if (rotate) {
      v = 0.25f * rot16_absmax4(u, mask);
    } else {
#pragma unroll
      for (int k = 0; k < 16; ++k) v = fmaxf(v, fabsf(u[k]));
    }
    return ok ? v : 0.0f;
  };
  float mr = 0.0f, mc = 0.0f;
  {
    const int i = threadIdx.x >> 2, q = threadIdx.x & 3;
    if (r0 + i < m && c0 + 16 * q < n) {
      float u[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) u[k] = tile[i][16 * q + k];
      mr = block_amax(u);
    }
  }
  {
    const int j = threadIdx.x & 63, q = threadIdx.x >> 6;
    if (c0 + j < n && r0 + 16 * q < m) {
      float u[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) u[k] = tile[16 * q + k][j];
      mc = block_amax(u);
    }
  }
  const float br = block_max_256(mr, red);
  __syncthreads();
  const float bc = block_max_256(mc, red);
  if (threadIdx.x == 0) {
    amax_record(&sc[b], slot_n, blockIdx.x, br);
    amax_record(&sc[b], slot_m, blockIdx.x, bc);
  }
}

hipError_t launch_amax_x2(const float* x, int64_t batch, int64_t m, int64_t n, int64_t x_bstride, uint32_t sign_mask,
                          bool rotate, MatScalars* sc, int slot_n, int slot_m, uint32_t* status, hipStream_t st) {
  const dim3 grid((uint32_t)(cdiv(m, kT) * cdiv(n, kT)), (uint32_t)batch);
  hipLaunchKernelGGL(k_amax_x2, grid, dim3(256), 0, st, x, m, n, x_bstride, sign_mask, (int)rotate, sc, slot_n,
                     slot_m, status);
  return hipGetLastError();
}

// Copy-out: caller M (rows x cols) from canonical X (transposed back when tall).
__global__ __launch_bounds__(256) void k_copy_out(MatChunk ch, const float* xbase, int64_t x_bstride) {
  __shared__ float tile[kT][kT + 1];
  const int64_t per = cdiv(ch.rows, kT) * cdiv(ch.cols, kT);
  const int mi = (int)(blockIdx.x / per);
  const uint32_t tt = (uint32_t)(blockIdx.x - mi * per);
  const MatRef& d = ch.m[mi];
  const bool tall = d.tall();
  const int64_t rows = tall ? ch.cols : ch.rows, cols = tall ? ch.rows : ch.cols, ld_out = d.ld_out();
  const uint32_t tcols = (uint32_t)cdiv(cols, kT);
  const int64_t br = (int64_t)(tt / tcols) * kT, bc = (int64_t)(tt % tcols) * kT;   // tile origin in M coordinates
  const float* X = xbase + (int64_t)mi * x_bstride;
  const int64_t xld = tall ? rows : cols;
  // 16-byte accesses (see k_prep_copy): thread -> quads v = threadIdx.x + 256 k,
  // row v / 16 of the tile, columns 4 (v % 16) .. + 3
  if (!tall) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int v = (int)threadIdx.x + 256 * k, i = v >> 4, q = v & 15;
      const int64_t r = br + i, c = bc + 4 * q;
      if (r < rows && c < cols)
        *reinterpret_cast<float4*>(d.out + r * ld_out + c) = *reinterpret_cast<const float4*>(X + r * xld + c);
    }
    return;
  }
  // X row bc + i, X columns br + 4q .. + 3  ->  M rows br + 4q .. + 3, column bc + i
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int v = (int)threadIdx.x + 256 * k, i = v >> 4, q = v & 15;
    const int64_t c = bc + i, r = br + 4 * q;
    if (r < rows && c < cols) {
      const float4 a = *reinterpret_cast<const float4*>(X + c * xld + r);
      tile[4 * q][i] = a.x; tile[4 * q + 1][i] = a.y; tile[4 * q + 2][i] = a.z; tile[4 * q + 3][i] = a.w;
    }
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int v = (int)threadIdx.x + 256 * k, i = v >> 4, q = v & 15;
    const int64_t r = br + i, c = bc + 4 * q;
    if (r < rows && c < cols)
      *reinterpret_cast<float4*>(d.out + r * ld_out + c) =
          make_float4(tile[i][4 * q], tile[i][4 * q + 1], tile[i][4 * q + 2], tile[i][4 * q + 3]);
  }
}

hipError_t launch_prep_copy(const MatChunk& ch, MatScalars* sc, float* x, int64_t x_bstride,
                            uint32_t mask, bool rotate, int slot_n, int slot_m, hipStream_t st) {
  hipLaunchKernelGGL(k_prep_copy, dim3((uint32_t)(cdiv(ch.rows, kT) * cdiv(ch.cols, kT) * ch.count)), dim3(256), 0, st, ch, sc, x,
                     x_bstride, mask, (int)rotate, slot_n, slot_m);
  return hipGetLastError();
}

hipError_t launch_copy_out(const MatChunk& ch, const float* x, int64_t x_bstride, hipStream_t st) {
  hipLaunchKernelGGL(k_copy_out, dim3((uint32_t)(cdiv(ch.rows, kT) * cdiv(ch.cols, kT) * ch.count)), dim3(256), 0, st, ch, x, x_bstride);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The rotation ahead of the quantiser: with a tensor scale of at least 2^-40 the
// factor 1/4 is left to the quantiser's scales (returns kf = 4, see quant_block);
// otherwise the block is rotated in full (kf = 1).
FP4R_DEV float rotate_for_quant(float (&u)[16], uint32_t mask, int rotate, float sg) {
  if (!rotate) return 1.0f;
  hadamard16(u, mask);
  if (sg >= 0x1p-40f) return 4.0f;
  quarter16(u);
  return 1.0f;
}

// Quantiser: one thread per 16-element block.  Axis 1: blocks along a row,
// consecutive threads take consecutive blocks of a row (contiguous 64-byte
// reads).  Axis 0: blocks down a column, consecutive threads take consecutive
// columns (each of the 16 loads is a contiguous 256-byte wave access).

template <int AXIS>
FP4R_DEV void block_pos(const Batch& in, int64_t g, int64_t& r, int64_t& c) {
  if (AXIS == 1) {
    const int64_t nbr = in.cols / 16;
    r = g / nbr;
    c = (g % nbr) * 16;
  } else {
    c = g % in.cols;
    r = (g / in.cols) * 16;
  }
}

template <int AXIS>
FP4R_DEV bool load_block_at(const Batch& in, int64_t b, int64_t r, int64_t c, float (&u)[16]) {
  const float* x = in.x + b * in.bstride;
  if (AXIS == 1) {
    const float4* p = reinterpret_cast<const float4*>(x + r * in.ld + c);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 v = p[q];
      u[4 * q] = v.x; u[4 * q + 1] = v.y; u[4 * q + 2] = v.z; u[4 * q + 3] = v.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < 16; ++i) u[i] = x[(r + i) * in.ld + c];
  }
  return finite16(u);
}

template <int AXIS>
__global__ __launch_bounds__(256) void k_amax(Batch in, uint32_t mask, int rotate, int clip,
                                              MatScalars* sc, int slot, uint32_t* status) {
  __shared__ float red[4];
  const int64_t b = blockIdx.y;
  const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t nblk = in.rows * in.cols / 16;
  float m = 0.0f;
  if (g < nblk) {
    float u[16];
    int64_t r, c;
    block_pos<AXIS>(in, g, r, c);
    const bool ok = load_block_at<AXIS>(in, b, r, c, u);
    if (!ok) atomicOr(status, kStatusNonFinite);
    if (clip) {
      const float tau = sc[b].tau;
#pragma unroll
      for (int i = 0; i < 16; ++i) u[i] = fminf(fmaxf(u[i], -tau), tau);
    }
    if (rotate) {
      m = 0.25f * rot16_absmax4(u, mask);
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) m = fmaxf(m, fabsf(u[i]));
    }
    if (!ok) m = 0.0f;
  }
  m = warp_max(m);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    const float mm = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    amax_record(&sc[b], slot, blockIdx.x, mm);
  }
}

// E2M1 magnitude of index 0..7 (the hardware decode of the code, exact).
FP4R_DEV double e2m1_grid(uint32_t idx) {
  return (double)__builtin_bit_cast(float2, __builtin_amdgcn_cvt_scalef32_pk_f32_fp4(idx, 1.0f, 0)).x;
}

// Stochastic rounding of one block's magnitudes (the first-moment state; see
// fp4root_momentum_update): u holds kf times the rotated block, `scale` is the
// chosen E4M3 code and `rtn` the round-to-nearest codes with that scale; element
// e0 + i takes 24 bits of SplitMix64 output (e0 + i) / 2 + 1 of `key` (two elements
// per output, see below).  With x = |u| / r exact
// (r = fl32(s s_g)), the floor grid point of x is the nearest one or the one
// below it (the round-to-nearest quotient is within one ulp of x), and
// rho (hi - lo) r < (|u| - lo r) 2^24 is exact in binary64 (every term has at
// most 48 significant bits; |u| - lo r is a difference of numbers within a factor 2).
FP4R_DEV uint64_t sr_block_codes_exact(const float (&u)[16], float kf, float r, uint64_t rtn, uint64_t key,
                                       uint64_t e0) {
  const double rd = (double)r;
  // element e0 + i takes 24 bits of SplitMix64 output (e0 + i) / 2 + 1 (e0 is even):
  // bits 40..63 for even i, bits 16..39 for odd i
  const uint64_t z0 = key + 0x9E3779B97F4A7C15ull * (e0 / 2 + 1);
  uint64_t zk = 0;
  uint64_t out = 0;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    if ((i & 1) == 0) zk = splitmix64_mix(z0 + 0x9E3779B97F4A7C15ull * (uint64_t)(i / 2));
    const float ui = kf == 1.0f ? u[i] : u[i] * 0.25f;
    const double a = (double)fabsf(ui);
    const uint32_t c = (uint32_t)(rtn >> (4 * i)) & 15u;
    uint32_t idx = c & 7u;
    double lo = e2m1_grid(idx);
    if (idx > 0 && lo * rd > a) {
      --idx;
      lo = e2m1_grid(idx);
    }
    if (idx < 7) {
      const double hi = e2m1_grid(idx + 1);
      const uint32_t rho = (uint32_t)(zk >> ((i & 1) ? 16 : 40)) & 0xFFFFFFu;
      if ((double)rho * (hi - lo) * rd < (a - lo * rd) * 16777216.0) ++idx;
    }
    out |= (uint64_t)((c & 8u) | idx) << (4 * i);
  }
  return out;
}

// The same codes decided in binary32 wherever that is certain.  The index, with the
// grid's points as its whole numbers, is the concave p(x) = min(2 x, x + 2, x / 2 + 4, 7),
// and the rule above is floor(p(x) + 1 - rho 2^-24) away from whole values of that sum.
// It is computed with x = |u| rcp(r): rcp within 2^-23, a slope times x of at most 4, and
// two roundings of at most 2^-22, so within 2^-20 in all; a block with an element within
// 2^-19 of a whole number (one in 2^14) takes the binary64 comparisons.  Both passes that
// encode this way were bound by issue: four 8192 x 3072 moments 176 -> 134 us, the AdamW step's
// second pass over 25 M elements 55 -> 44 us.
FP4R_DEV uint64_t sr_block_codes(const float (&u)[16], float kf, uint32_t scale, float sg, uint64_t rtn,
                                 uint64_t key, uint64_t e0) {
  const float r = e4m3_value(scale) * sg;
  if (!(r > 0.0f)) return rtn & 0x8888888888888888ull;   // magnitudes 0, signs kept
  bool sure = r > 0x1p-100f && r < 0x1p+100f;
  const float i1 = __builtin_amdgcn_rcpf(r) * (kf == 1.0f ? 1.0f : 0.25f), i2 = i1 + i1, ih = 0.5f * i1;
  const uint64_t z0 = key + 0x9E3779B97F4A7C15ull * (e0 / 2 + 1);
  uint64_t zk = 0;
  uint32_t w[2] = {0u, 0u};
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    if ((i & 1) == 0) zk = splitmix64_mix(z0 + 0x9E3779B97F4A7C15ull * (uint64_t)(i / 2));
    const uint32_t rho = (uint32_t)(zk >> ((i & 1) ? 16 : 40)) & 0xFFFFFFu;
    const float a = fabsf(u[i]);
    const float p = fminf(fminf(fminf(fmaf(a, i2, 1.0f), fmaf(a, i1, 3.0f)), fmaf(a, ih, 5.0f)), 8.0f);
    const float t = fmaf((float)rho, -0x1p-24f, p);
    sure = sure & (fabsf(__builtin_amdgcn_fractf(t) - 0.5f) < 0.5f - 0x1p-19f);   // false for NaN
    w[i >> 3] |= (uint32_t)t << (4 * (i & 7));
  }
  if (!sure) return sr_block_codes_exact(u, kf, r, rtn, key, e0);
  return (rtn & 0x8888888888888888ull) | (uint64_t)w[0] | ((uint64_t)w[1] << 32);
}

template <int AXIS, bool SR = false>
__global__ __launch_bounds__(256) void k_encode(Batch in, uint32_t mask, int rotate, int clip,
                                                int adaptive, MatScalars* sc, int slot, QOut out,
                                                float* tensor_scale, float* tau_out, uint64_t sr_key) {
  const int64_t b = blockIdx.y;
  const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t nblk = in.rows * in.cols / 16;
  const float sg = tensor_scale_from_amax(amax_read(sc[b], slot));
  if (g == 0) {
    sc[b].sg[slot] = sg;
    if (tensor_scale) tensor_scale[b] = sg;
    if (tau_out) tau_out[b] = sc[b].tau;
  }
  if (g >= nblk) return;
  int64_t r = 0, c = 0;
  block_pos<AXIS>(in, g, r, c);
  {
    float u[16];
    load_block_at<AXIS>(in, b, r, c, u);
    if (clip) {
      const float tau = sc[b].tau;
#pragma unroll
      for (int i = 0; i < 16; ++i) u[i] = fminf(fmaxf(u[i], -tau), tau);
    }
    const float kf = rotate_for_quant(u, mask, rotate, sg);
    uint32_t scale;
    uint64_t codes;
    uint32_t n2;
    quant_block(u, sg, adaptive != 0, scale, codes, n2, false, kf);
    if constexpr (SR)
      codes = sr_block_codes(u, kf, scale, sg, codes, sr_key, (uint64_t)((b * in.rows + r) * in.cols + c));
    int64_t code_off, scale_off;
    if (AXIS == 1) {   // [rows][cols/2], [rows][cols/16]
      code_off = r * (in.cols / 2) + c / 2;
      scale_off = r * (in.cols / 16) + c / 16;
    } else {           // transposed: [cols][rows/2], [cols][rows/16]
      code_off = c * (in.rows / 2) + r / 2;
      scale_off = c * (in.rows / 16) + r / 16;
    }
    *reinterpret_cast<uint2*>(out.codes + b * out.codes_bstride + code_off) =
        make_uint2((uint32_t)codes, (uint32_t)(codes >> 32));
    out.scales[b * out.scales_bstride + scale_off] = (uint8_t)scale;
  }
}

// The words that lane q of a quad stores (8 bytes at 8 q of the row's 32 bytes of a
// stage-major stage): first halves of blocks 0 .. 3, then their second halves.  Lane q
// holds block q's codes; all lanes of the wave must be active.
FP4R_DEV uint2 quad_stage_words(uint64_t codes, int q) {
  const uint32_t lo = (uint32_t)codes, hi = (uint32_t)(codes >> 32);
  const uint32_t l0 = dpp_u<0x88>(lo), l1 = dpp_u<0xDD>(lo);   // lanes 0, 2, 0, 2 and 1, 3, 1, 3
  const uint32_t h0 = dpp_u<0x88>(hi), h1 = dpp_u<0xDD>(hi);
  return q < 2 ? make_uint2(l0, l1) : make_uint2(h0, h1);
}

// The operand encoders take several problems per launch (one per shape group of a step:
// ten launches of 5 us instead of five for two groups of small matrices, and no gap between
// them), each workgroup finding its own; one problem alone needs no search, and its matrices
// are the grid's second dimension.
struct EncodeSlot {
  int problem;
  int64_t mat;
  uint32_t wg;   // within the matrix
};
template <bool MULTI>
FP4R_DEV EncodeSlot encode_slot(const EncodeBatch& eb) {
  if (!MULTI) return EncodeSlot{0, (int64_t)blockIdx.y, blockIdx.x};
  int i = 0;
  while (i + 1 < eb.count && blockIdx.x >= eb.end[i]) ++i;
  const uint32_t local = blockIdx.x - (i ? eb.end[i - 1] : 0u), mat = local / eb.per[i];
  return EncodeSlot{i, (int64_t)mat, local - mat * eb.per[i]};
}

// The table of a launch over list[0 .. count) with per(i) workgroups per matrix; false when
// the problems must go one by one.
template <class F>
bool encode_table(const EncodeArgs* list, int count, F per, EncodeBatch& eb) {
  eb.count = count;
  int64_t end = 0;
  for (int i = 0; i < count; ++i) {
    eb.p[i] = list[i];
    const int64_t n = per(list[i]);
    end += n * list[i].batch;
    if (count > 1 && end > kMaxSharedBlocks) return false;
    eb.per[i] = (uint32_t)n;
    eb.end[i] = (uint32_t)end;
  }
  return true;
}

// A products' operand from row blocks: each wave takes 16 rows x one 64-element stage,
// lane 4i + k block k of row i (consecutive waves take consecutive stages of a row
// group, so a workgroup reads whole 256-byte row segments).
template <bool MULTI>
__global__ __launch_bounds__(256) void k_encode_operand(EncodeBatch eb, uint32_t mask, int rotate, int adaptive,
                                                        int slot) {
  const EncodeSlot es = encode_slot<MULTI>(eb);
  const EncodeArgs& ea = eb.p[es.problem];
  const float* const x = ea.x;
  const int64_t rows = ea.rows, K = ea.K, bstride = ea.bstride, b = es.mat;
  MatScalars* const sc = ea.sc;
  const OperandOut& out = ea.q;
  const uint32_t nst = (uint32_t)((K + 63) / 64);
  // uniform over the wave, so the division by the stage count is scalar work
  const uint32_t wv = es.wg * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const float sg = tensor_scale_from_amax(amax_read(sc[b], slot));
  if (es.wg == 0 && threadIdx.x == 0) sc[b].sg[slot] = sg;
  const uint32_t rg = wv / nst, st = wv - rg * nst;
  if ((int64_t)rg * 16 >= rows) return;   // rows is a multiple of 16: whole waves leave
  const int lane = (int)(threadIdx.x & 63), q = lane & 3;
  const int64_t r = (int64_t)rg * 16 + (lane >> 2), c = ((int64_t)st * 4 + q) * 16;
  uint32_t scale = 0, n2 = 0;
  uint64_t codes = 0;
  const bool want = out.words != nullptr || out.rec != nullptr;
  if (c < K) {
    float u[16];
    const float4* p = reinterpret_cast<const float4*>(x + b * bstride + r * K + c);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const float4 v = p[k];
      u[4 * k] = v.x; u[4 * k + 1] = v.y; u[4 * k + 2] = v.z; u[4 * k + 3] = v.w;
    }
    const float kf = rotate_for_quant(u, mask, rotate, sg);
    quant_block(u, sg, adaptive != 0, scale, codes, n2, want, kf);
  }
  const int64_t row = (int64_t)st * rows + r;
  *reinterpret_cast<uint2*>(out.codes + b * out.codes_bstride + row * 32 + 8 * q) = quad_stage_words(codes, q);
  out.scales[b * out.scales_bstride + row * 4 + q] = (uint8_t)scale;
  if (want) {
    const uint32_t w = quad_row_word(n2, scale);
    if (out.words) {
      if (q == 0) out.words[b * out.words_bstride + row] = w;
    } else {
      const float rho = wave_max_pos(word_rho(w));
      if (lane == 0) out.rec[b * out.rec_bstride + (int64_t)rg * nst + st] = rho;
    }
  }
}

hipError_t launch_encode_operand(const EncodeArgs* list, int count, uint32_t sign_mask, bool rotate, bool adaptive46,
                                 int slot, hipStream_t st) {
  if (count < 1 || count > kMaxEncode) return hipErrorInvalidValue;
  for (int i = 0; i < count; ++i)
    if (list[i].rows % 16 != 0 || list[i].K % 16 != 0) return hipErrorInvalidValue;
  EncodeBatch eb;
  auto per = [](const EncodeArgs& e) { return (e.rows / 16 * ((e.K + 63) / 64) + 3) / 4; };
  if (!encode_table(list, count, per, eb)) {
    for (int i = 0; i < count; ++i) {
      const hipError_t e = launch_encode_operand(list + i, 1, sign_mask, rotate, adaptive46, slot, st);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  if (count == 1)
    hipLaunchKernelGGL(k_encode_operand<false>, dim3(eb.per[0], (uint32_t)list[0].batch), dim3(256), 0, st, eb,
                       sign_mask, (int)rotate, (int)adaptive46, slot);
  else
    hipLaunchKernelGGL(k_encode_operand<true>, dim3(eb.end[count - 1]), dim3(256), 0, st, eb, sign_mask, (int)rotate,
                       (int)adaptive46, slot);
  return hipGetLastError();
}

// Both quantisations of X from one read: a 64 x 64 tile is staged in LDS; each
// thread encodes one 16-column block (qX, along n) and one 16-row block (qXt,
// along m, written transposed).
// Eight waves per SIMD (64 VGPRs and 24 bytes of scratch per lane) rather than the
// six its 73 registers would allow: the extra waves cover part of its LDS and
// memory waits (about 2.5 % less time per launch).
template <bool MULTI>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8))) void k_encode_x2(EncodeBatch eb, uint32_t mask, int rotate, int adaptive,
                                                   int slot_n, int slot_m, uint32_t reset_mask) {
  const EncodeSlot es = encode_slot<MULTI>(eb);
  const EncodeArgs& ea = eb.p[es.problem];
  const int64_t m = ea.rows, n = ea.K, b = es.mat;
  MatScalars* const sc = ea.sc;
  const OperandOut &qx = ea.q, &qxt = ea.qt;
  // rows padded to 68 floats: 16-byte row slices for the row blocks.  gfx950 serves
  // a 128-bit LDS read 16 lanes per cycle over 64 banks and a 128-bit write 8 lanes
  // per cycle over 32 banks: the 16 lanes of one read (4 rows x 4 slices) and 64
  // consecutive columns of one row fall in distinct banks, and so do the 8 lanes of
  // one write (2 rows x 4 slices) because lanes with bit 1 of q set store their
  // four slices in the order k ^ 2
  __shared__ __align__(16) float tile[kT][kT + 4];
  const uint32_t tn = (uint32_t)cdiv(n, kT);   // tiles per row of tiles (grid.x < 2^32)
  const int64_t r0 = (int64_t)(es.wg / tn) * kT, c0 = (int64_t)(es.wg % tn) * kT;
  const float* X = ea.x + b * ea.bstride;
  const float sgn = tensor_scale_from_amax(amax_read(sc[b], slot_n));
  const float sgm = tensor_scale_from_amax(amax_read(sc[b], slot_m));
  if (es.wg == 0) {
    if (threadIdx.x == 0) {
      sc[b].sg[slot_n] = sgn;
      sc[b].sg[slot_m] = sgm;
    }
    // amax slots the next kernels record into (this kernel reads only slot_n, slot_m)
    if (threadIdx.x < kAmaxSpread * kNumSlots) {
      const int line = (int)threadIdx.x / kNumSlots, slot = (int)threadIdx.x % kNumSlots;
      if ((reset_mask >> slot) & 1u) sc[b].amax[line].v[slot] = 0u;
    }
  }
  {
    const int i = threadIdx.x >> 2, q = threadIdx.x & 3;   // row i, 16 columns at 16 q
    if (r0 + i < m && c0 + 16 * q < n) {
      const float4* p = reinterpret_cast<const float4*>(X + (r0 + i) * n + c0 + 16 * q);
      float4* t = reinterpret_cast<float4*>(&tile[i][16 * q]);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int kk = k ^ (q & 2);
        t[kk] = p[kk];
      }
    }
  }
  __syncthreads();
  const bool want = qx.words != nullptr || qx.rec != nullptr;
  {
    const int i = threadIdx.x >> 2, q = threadIdx.x & 3;
    const int64_t r = r0 + i, c = c0 + 16 * q;
    uint32_t n2 = 0, scale = 0;
    uint64_t codes = 0;
    if (r < m && c < n) {
      float u[16];
      const float4* t = reinterpret_cast<const float4*>(&tile[i][16 * q]);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const float4 v = t[k];
        u[4 * k] = v.x; u[4 * k + 1] = v.y; u[4 * k + 2] = v.z; u[4 * k + 3] = v.w;
      }
      const float kf = rotate_for_quant(u, mask, rotate, sgn);
      quant_block(u, sgn, adaptive != 0, scale, codes, n2, want, kf);
    }
    const int64_t row = (c0 / 64) * m + r;
    const uint2 w = quad_stage_words(codes, q);
    if (r < m) {
      *reinterpret_cast<uint2*>(qx.codes + b * qx.codes_bstride + row * 32 + 8 * q) = w;
      qx.scales[b * qx.scales_bstride + row * 4 + q] = (uint8_t)scale;
    }
    // chain bound of row i's stage (lanes 4i .. 4i + 3 hold its four blocks; blocks past
    // the edge count as zero), or the largest over this wave's 16 rows
    if (want) {
      const uint32_t rw = quad_row_word(n2, scale);
      if (qx.words) {
        if (q == 0 && r < m) qx.words[b * qx.words_bstride + row] = rw;
      } else {
        const float rho = wave_max_pos(word_rho(rw));
        if ((threadIdx.x & 63) == 0 && r0 + 16 * (threadIdx.x >> 6) < m)
          qx.rec[b * qx.rec_bstride + ((r0 / 16) + (threadIdx.x >> 6)) * cdiv(n, 64) + c0 / 64] = rho;
      }
    }
  }
  {
    const int j = threadIdx.x & 63, q = threadIdx.x >> 6;   // column j, 16 rows at 16 q
    const int64_t c = c0 + j, r = r0 + 16 * q;
    uint32_t n2 = 0, scale = 0;
    uint64_t codes = 0;
    if (r < m && c < n) {
      float u[16];
#pragma unroll
      for (int k = 0; k < 16; ++k) u[k] = tile[16 * q + k][j];
      const float kf = rotate_for_quant(u, mask, rotate, sgm);
      quant_block(u, sgm, adaptive != 0, scale, codes, n2, want, kf);
    }
    // the four blocks of column j (one row of qXt's stage) sit in the four waves:
    // exchange in LDS (the tile is no longer read once every thread has passed the
    // barrier); thread 4 j' + q' then stores 8 bytes of row j'
    __syncthreads();
    uint32_t* const xc = reinterpret_cast<uint32_t*>(&tile[0][0]);   // [8][64] code words (half, block), rows
    float* const xt = reinterpret_cast<float*>(xc + 512);            // [4][64] n2 4^E
    uint32_t* const xs = xc + 768;                                   // [4][64] scale | e << 8
    xc[q * 64 + j] = (uint32_t)codes;
    xc[(4 + q) * 64 + j] = (uint32_t)(codes >> 32);
    xs[q * 64 + j] = scale | (block_unit(scale) << 8);
    if (want) xt[q * 64 + j] = block_square(n2, scale);
    __syncthreads();
    const int j2 = threadIdx.x >> 2, q2 = threadIdx.x & 3;
    const int64_t row = (r0 / 64) * n + c0 + j2;
    uint32_t sw[4];
    float t = 0.0f;
    if (q2 == 0) {
#pragma unroll
      for (int k = 0; k < 4; ++k) sw[k] = xs[k * 64 + j2];
    }
    if (c0 + j2 < n) {
      *reinterpret_cast<uint2*>(qxt.codes + b * qxt.codes_bstride + row * 32 + 8 * q2) =
          make_uint2(xc[(2 * q2) * 64 + j2], xc[(2 * q2 + 1) * 64 + j2]);
      if (q2 == 0)
        *reinterpret_cast<uint32_t*>(qxt.scales + b * qxt.scales_bstride + row * 4) =
            (sw[0] & 0xFFu) | ((sw[1] & 0xFFu) << 8) | ((sw[2] & 0xFFu) << 16) | ((sw[3] & 0xFFu) << 24);
    }
    if (want) {
      uint32_t rw = 0;
      if (q2 == 0) {
        t = (xt[j2] + xt[64 + j2]) + (xt[128 + j2] + xt[192 + j2]);
        rw = row_word(t, min(min(sw[0] >> 8, sw[1] >> 8), min(sw[2] >> 8, sw[3] >> 8)));
      }
      if (qxt.words) {
        if (q2 == 0 && c0 + j2 < n) qxt.words[b * qxt.words_bstride + row] = rw;
      } else {
        const float rho = wave_max_pos(word_rho(rw));   // the wave's 16 rows (0 in the other lanes)
        if ((threadIdx.x & 63) == 0 && c0 + j2 < n)
          qxt.rec[b * qxt.rec_bstride + ((c0 + j2) / 16) * cdiv(m, 64) + r0 / 64] = rho;
      }
    }
  }
}

// Chain levels (see chain_entries): each wave takes two units of 32 rows (one per half
// wave, a row per lane) x four stages.
__global__ __launch_bounds__(256) void k_chain_levels(ChainList list) {
  int oi = 0;
  while (oi + 1 < list.count && (int64_t)blockIdx.x >= list.wg_end[oi]) ++oi;
  const ChainOp& op = list.op[oi];
  const int64_t wg = (int64_t)blockIdx.x - (oi > 0 ? list.wg_end[oi - 1] : 0);
  const int quads = (op.nst + 3) / 4;
  const int64_t per = ((op.rows + 63) / 64) * quads;   // waves of one matrix
  const int64_t wv = wg * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t b = wv / per;
  if (b >= op.batch) return;
  const int64_t left = wv - b * per;
  const int quad = (int)(left % quads);
  const int lane = (int)(threadIdx.x & 63);
  const int64_t row = (left / quads) * 64 + lane;
  const uint32_t* words = op.words + b * op.words_bstride;
  uint32_t w[4];
#pragma unroll
  for (int k = 0; k < 4; ++k)
    w[k] = row < op.rows && 4 * quad + k < op.nst ? words[(int64_t)(4 * quad + k) * op.rows + row] : 15u;
  float v[7];   // runs of one stage (4), two (2) and four (1)
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = word_rho(w[k]);
#pragma unroll
  for (int k = 0; k < 2; ++k)
    v[4 + k] = ldexpf(word_square(w[2 * k]) + word_square(w[2 * k + 1]),
                      -2 * (int)min(w[2 * k] & 15u, w[2 * k + 1] & 15u));
  v[6] = ldexpf((word_square(w[0]) + word_square(w[1])) + (word_square(w[2]) + word_square(w[3])),
                -2 * (int)min(min(w[0] & 15u, w[1] & 15u), min(w[2] & 15u, w[3] & 15u)));
#pragma unroll
  for (int k = 0; k < 7; ++k) {
    const uint32_t h = row16_max_bits(__float_as_uint(v[k]));
    v[k] = __uint_as_float(max(h, (uint32_t)__shfl_xor((int)h, 16, 64))) * (1.0f + 0x1p-20f);   // past the sums' roundings
  }
  const int64_t unit = row / 32;
  if ((lane & 31) != 0 || unit * 32 >= op.rows) return;
  const int n1 = op.nst, n2 = (op.nst + 1) / 2;
  float* rec = op.rec + b * op.rec_bstride + unit * chain_entries(op.nst);
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (4 * quad + k < n1) rec[4 * quad + k] = v[k];
#pragma unroll
  for (int k = 0; k < 2; ++k)
    if (2 * quad + k < n2) rec[n1 + 2 * quad + k] = v[4 + k];
  rec[n1 + n2 + quad] = v[6];
}

hipError_t launch_chain_levels(const ChainOp* ops, int count, hipStream_t st) {
  if (count < 1 || count > kMaxChainOps) return hipErrorInvalidValue;
  ChainList list;
  list.count = count;
  int64_t total = 0;
  for (int i = 0; i < count; ++i) {
    list.op[i] = ops[i];
    total += (ops[i].batch * ((ops[i].rows + 63) / 64) * ((ops[i].nst + 3) / 4) + 3) / 4;
    list.wg_end[i] = total;
  }
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(k_chain_levels, dim3((uint32_t)total), dim3(256), 0, st, list);
  return hipGetLastError();
}

// One thread per (row, stage) of a matrix: 32 code bytes and 4 scale bytes from the
// stage-major layout to the row-major one (a last partial stage copies its blocks only).
__global__ __launch_bounds__(256) void k_untile_nvfp4(const uint8_t* codes, const uint8_t* scales, int64_t rows,
                                                       int64_t K, uint8_t* out_codes, uint8_t* out_scales) {
  const int64_t b = blockIdx.y;
  const int64_t nst = (K + 63) / 64;
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= rows * nst) return;
  const int64_t st = t / rows, r = t % rows;
  const int nb = (int)(K / 16 - 4 * st < 4 ? K / 16 - 4 * st : 4);   // blocks in this stage
  const uint8_t* sc = codes + b * tiled_code_bytes(rows, K) + (st * rows + r) * 32;
  const uint8_t* ss = scales + b * tiled_scale_bytes(rows, K) + (st * rows + r) * 4;
  uint8_t* dc = out_codes ? out_codes + b * rows * (K / 2) + r * (K / 2) + st * 32 : nullptr;
  uint8_t* ds = out_scales ? out_scales + b * rows * (K / 16) + r * (K / 16) + st * 4 : nullptr;
  for (int k = 0; k < nb; ++k) {
    if (out_codes)
      *reinterpret_cast<uint2*>(dc + 8 * k) =
          make_uint2(reinterpret_cast<const uint32_t*>(sc)[k], reinterpret_cast<const uint32_t*>(sc)[4 + k]);
    if (out_scales) ds[k] = ss[k];
  }
}

hipError_t launch_untile_nvfp4(const uint8_t* codes, const uint8_t* scales, int64_t batch, int64_t rows,
                               int64_t K, uint8_t* out_codes, uint8_t* out_scales, hipStream_t st) {
  const int64_t n = rows * ((K + 63) / 64);
  if (n == 0 || batch == 0) return hipSuccess;
  if (K % 16 != 0) return hipErrorInvalidValue;
  const dim3 grid((uint32_t)((n + 255) / 256), (uint32_t)batch);
  hipLaunchKernelGGL(k_untile_nvfp4, grid, dim3(256), 0, st, codes, scales, rows, K, out_codes, out_scales);
  return hipGetLastError();
}

hipError_t launch_encode_x2(const EncodeArgs* list, int count, uint32_t sign_mask, bool rotate, bool adaptive46,
                            int slot_n, int slot_m, hipStream_t st, uint32_t reset_mask) {
  if (count < 1 || count > kMaxEncode) return hipErrorInvalidValue;
  if (reset_mask & ((1u << slot_n) | (1u << slot_m))) return hipErrorInvalidValue;
  EncodeBatch eb;
  auto per = [](const EncodeArgs& e) { return cdiv(e.rows, kT) * cdiv(e.K, kT); };
  if (!encode_table(list, count, per, eb)) {
    for (int i = 0; i < count; ++i) {
      const hipError_t e =
          launch_encode_x2(list + i, 1, sign_mask, rotate, adaptive46, slot_n, slot_m, st, reset_mask);
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  if (count == 1)
    hipLaunchKernelGGL(k_encode_x2<false>, dim3(eb.per[0], (uint32_t)list[0].batch), dim3(256), 0, st, eb, sign_mask,
                       (int)rotate, (int)adaptive46, slot_n, slot_m, reset_mask);
  else
    hipLaunchKernelGGL(k_encode_x2<true>, dim3(eb.end[count - 1]), dim3(256), 0, st, eb, sign_mask, (int)rotate,
                       (int)adaptive46, slot_n, slot_m, reset_mask);
  return hipGetLastError();
}

hipError_t launch_amax(const Batch& in, int axis, uint32_t sign_mask, bool rotate, bool clip,
                       MatScalars* sc, int slot, uint32_t* status, hipStream_t st) {
  const int64_t nblk = in.rows * in.cols / 16;
  const dim3 grid((uint32_t)((nblk + 255) / 256), (uint32_t)in.batch);
  if (axis == 1)
    hipLaunchKernelGGL(k_amax<1>, grid, dim3(256), 0, st, in, sign_mask, (int)rotate, (int)clip, sc,
                       slot, status);
  else
    hipLaunchKernelGGL(k_amax<0>, grid, dim3(256), 0, st, in, sign_mask, (int)rotate, (int)clip, sc,
                       slot, status);
  return hipGetLastError();
}

hipError_t launch_encode(const Batch& in, int axis, uint32_t sign_mask, bool rotate, bool clip,
                         bool adaptive46, MatScalars* sc, int slot, const QOut& out,
                         float* tensor_scale, hipStream_t st, float* tau_out) {
  const int64_t nblk = in.rows * in.cols / 16;
  const dim3 grid((uint32_t)((nblk + 255) / 256), (uint32_t)in.batch);
  if (axis == 1)
    hipLaunchKernelGGL((k_encode<1, false>), grid, dim3(256), 0, st, in, sign_mask, (int)rotate, (int)clip,
                       (int)adaptive46, sc, slot, out, tensor_scale, tau_out, (uint64_t)0);
  else
    hipLaunchKernelGGL((k_encode<0, false>), grid, dim3(256), 0, st, in, sign_mask, (int)rotate, (int)clip,
                       (int)adaptive46, sc, slot, out, tensor_scale, tau_out, (uint64_t)0);
  return hipGetLastError();
}

hipError_t launch_encode_sr(const Batch& in, uint32_t sign_mask, bool rotate, bool adaptive46,
                            MatScalars* sc, int slot, const QOut& out, float* tensor_scale,
                            uint64_t sr_key, hipStream_t st) {
  const int64_t nblk = in.rows * in.cols / 16;
  const dim3 grid((uint32_t)((nblk + 255) / 256), (uint32_t)in.batch);
  hipLaunchKernelGGL((k_encode<1, true>), grid, dim3(256), 0, st, in, sign_mask, (int)rotate, 0,
                     (int)adaptive46, sc, slot, out, tensor_scale, (float*)nullptr, sr_key);
  return hipGetLastError();
}


// ---------------------------------------------------------------------------
// First-moment update: one thread per 16-element row block of a contiguous
// matrix.  Decodes the previous NVFP4 state (one rounding of q s s_g, then the
// inverse rotation), forms m = fl32(b1 m_hat + b2 g) (exact products, one binary64
// rounding, then binary32), writes m and records the amax of m rotated with
// `mask` (the tensor scale of the next state) in amax slot 0.
FP4R_DEV void mom_update_block(const float* g, float* m, int64_t e0, bool in, const uint8_t* codes,
                               const uint8_t* scales, float prev_sg, int has_prev, uint32_t prev_mask,
                               uint32_t mask, int rotate, float b1, float b2, MatScalars* sc, uint32_t wg,
                               uint32_t* status) {
  __shared__ float red[4];
  float amax = 0.0f;
  if (in) {
    float x[16];
    const float4* gp = reinterpret_cast<const float4*>(g + e0);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const float4 v = gp[q];
      x[4 * q] = v.x; x[4 * q + 1] = v.y; x[4 * q + 2] = v.z; x[4 * q + 3] = v.w;
    }
    const bool ok = finite16(x);
    if (!ok) atomicOr(status, kStatusNonFinite);
    float mv[16];
    mom_block(x, codes, scales, e0, prev_sg, has_prev, prev_mask, rotate, b1, b2, mv);
    float4* mp = reinterpret_cast<float4*>(m + e0);
#pragma unroll
    for (int q = 0; q < 4; ++q) mp[q] = make_float4(mv[4 * q], mv[4 * q + 1], mv[4 * q + 2], mv[4 * q + 3]);
    if (rotate) {
      amax = 0.25f * rot16_absmax4(mv, mask);
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) amax = fmaxf(amax, fabsf(mv[i]));
    }
    if (!ok) amax = 0.0f;
  }
  amax = warp_max(amax);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = amax;
  __syncthreads();
  if (threadIdx.x == 0) {
    const float mm = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    amax_record(sc, 0, wg, mm);
  }
}

__global__ __launch_bounds__(256) void k_mom_update(const float* g, float* m, int64_t rows, int64_t cols,
                                                    const uint8_t* codes, const uint8_t* scales,
                                                    const float* prev_sg, int has_prev, uint32_t prev_mask,
                                                    uint32_t mask, int rotate, float b1, float b2,
                                                    MatScalars* sc, uint32_t* status) {
  const int64_t b = blockIdx.y;
  const int64_t blk = (int64_t)blockIdx.x * 256 + threadIdx.x;
  mom_update_block(g, m, b * rows * cols + blk * 16, blk < rows * cols / 16, codes, scales,
                   has_prev ? prev_sg[b] : 0.0f, has_prev, prev_mask, mask, rotate, b1, b2, &sc[b], blockIdx.x,
                   status);
}

// The two passes over the parameters of an optimizer step.  One launch of each kind for up
// to kMaxRootChunk of them: small parameters are bound by the launches (12 parameters of 64
// to 256 K elements: 188 us in 49 launches of their own, 25 in 4).
__global__ __launch_bounds__(256) void k_root_mom_update(RootChunk ch, int has_prev, int rotate, float b1, float b2,
                                                         MatScalars* sc, uint32_t* status) {
  uint32_t wg;
  const int i = root_param(ch, blockIdx.x, wg);
  const RootRef& p = ch.p[i];
  const int64_t blk = (int64_t)wg * 256 + threadIdx.x;
  mom_update_block(p.g, p.m, blk * 16, blk < p.nblk, p.codes, p.scales, has_prev ? p.tensor_scale[0] : 0.0f, has_prev,
                   p.prev_mask, p.mask, rotate, b1, b2, &sc[i], wg, status);
}

template <bool SR>
__global__ __launch_bounds__(256) void k_root_mom_encode(RootChunk ch, int rotate, int adaptive, MatScalars* sc) {
  uint32_t wg;
  const int i = root_param(ch, blockIdx.x, wg);
  const RootRef& p = ch.p[i];
  const int64_t blk = (int64_t)wg * 256 + threadIdx.x;
  const float sg = tensor_scale_from_amax(amax_read(sc[i], 0));
  if (blk == 0) p.tensor_scale[0] = sg;
  if (blk >= p.nblk) return;
  float u[16];
  const float4* mp = reinterpret_cast<const float4*>(p.m + blk * 16);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float4 v = mp[q];
    u[4 * q] = v.x; u[4 * q + 1] = v.y; u[4 * q + 2] = v.z; u[4 * q + 3] = v.w;
  }
  const float kf = rotate_for_quant(u, p.mask, rotate, sg);
  uint32_t scale, n2;
  uint64_t c;
  quant_block(u, sg, adaptive != 0, scale, c, n2, false, kf);
  if constexpr (SR) c = sr_block_codes(u, kf, scale, sg, c, p.sr_key, (uint64_t)(blk * 16));
  *reinterpret_cast<uint2*>(p.codes + blk * 8) = make_uint2((uint32_t)c, (uint32_t)(c >> 32));
  p.scales[blk] = (uint8_t)scale;
}

hipError_t launch_root_momentum(const RootChunk& ch, bool has_prev, bool rotate, bool adaptive, bool sr, float b1,
                                float b2, MatScalars* sc, uint32_t* status, hipStream_t st) {
  const dim3 grid(ch.end[ch.count - 1]);
  hipLaunchKernelGGL(k_root_mom_update, grid, dim3(256), 0, st, ch, (int)has_prev, (int)rotate, b1, b2, sc, status);
  if (sr)
    hipLaunchKernelGGL(k_root_mom_encode<true>, grid, dim3(256), 0, st, ch, (int)rotate, (int)adaptive, sc);
  else
    hipLaunchKernelGGL(k_root_mom_encode<false>, grid, dim3(256), 0, st, ch, (int)rotate, (int)adaptive, sc);
  return hipGetLastError();
}

// Re-encode the first moment of a flat parameter (batch 1, n elements) in place,
// recomputing m_t = fl32(b1 decode(old state) + b2 g) exactly as mom_block does:
// the quantized-state AdamW step's second pass (its first pass recorded the rotated
// amax of m_t in slot 0 and saved the previous tensor scale in sg[kSlotPrevState]).
// Each thread reads and writes only its own block of the state.
template <bool SR>
__global__ __launch_bounds__(256) void k_mom_encode(const float* g, uint8_t* codes, uint8_t* scales,
                                                    int64_t nblk, int has_prev, uint32_t prev_mask,
                                                    uint32_t mask, int rotate, int adaptive, float b1, float b2,
                                                    MatScalars* sc, float* tensor_scale, uint64_t sr_key) {
  const int64_t blk = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const float sg = tensor_scale_from_amax(amax_read(sc[0], 0));
  if (blk == 0) {
    sc[0].sg[0] = sg;
    tensor_scale[0] = sg;
  }
  if (blk >= nblk) return;
  const int64_t e0 = blk * 16;
  float x[16];
  const float4* gp = reinterpret_cast<const float4*>(g + e0);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float4 v = gp[q];
    x[4 * q] = v.x; x[4 * q + 1] = v.y; x[4 * q + 2] = v.z; x[4 * q + 3] = v.w;
  }
  float u[16];
  mom_block(x, codes, scales, e0, sc[0].sg[kSlotPrevState], has_prev != 0, prev_mask, rotate != 0, b1, b2, u);
  const float kf = rotate_for_quant(u, mask, rotate, sg);
  uint32_t scale, n2;
  uint64_t c;
  quant_block(u, sg, adaptive != 0, scale, c, n2, false, kf);
  if constexpr (SR) c = sr_block_codes(u, kf, scale, sg, c, sr_key, (uint64_t)e0);
  *reinterpret_cast<uint2*>(codes + e0 / 2) = make_uint2((uint32_t)c, (uint32_t)(c >> 32));
  scales[blk] = (uint8_t)scale;
}

hipError_t launch_mom_encode(const float* g, uint8_t* codes, uint8_t* scales, int64_t n, bool has_prev,
                             uint32_t prev_mask, uint32_t mask, bool rotate, bool adaptive, bool sr, float b1,
                             float b2, MatScalars* sc, float* tensor_scale, uint64_t sr_key, hipStream_t st) {
  const int64_t nblk = n / 16;
  const dim3 grid((uint32_t)((nblk + 255) / 256));
  if (sr)
    hipLaunchKernelGGL(k_mom_encode<true>, grid, dim3(256), 0, st, g, codes, scales, nblk, (int)has_prev, prev_mask,
                       mask, (int)rotate, (int)adaptive, b1, b2, sc, tensor_scale, sr_key);
  else
    hipLaunchKernelGGL(k_mom_encode<false>, grid, dim3(256), 0, st, g, codes, scales, nblk, (int)has_prev, prev_mask,
                       mask, (int)rotate, (int)adaptive, b1, b2, sc, tensor_scale, sr_key);
  return hipGetLastError();
}

hipError_t launch_mom_update(const float* g, float* m, int64_t batch, int64_t rows, int64_t cols,
                             const uint8_t* codes, const uint8_t* scales, const float* prev_sg,
                             bool has_prev, uint32_t prev_mask, uint32_t mask, bool rotate, float b1,
                             float b2, MatScalars* sc, uint32_t* status, hipStream_t st) {
  const int64_t nblk = rows * cols / 16;
  const dim3 grid((uint32_t)((nblk + 255) / 256), (uint32_t)batch);
  hipLaunchKernelGGL(k_mom_update, grid, dim3(256), 0, st, g, m, rows, cols, codes, scales, prev_sg,
                     (int)has_prev, prev_mask, mask, (int)rotate, b1, b2, sc, status);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// BF16 comparison path.

// Xb = bf16(X): four elements per thread, 16-byte reads and 8-byte writes.
__global__ __launch_bounds__(256) void k_cast_bf16(const float* x, int64_t mn, int64_t x_bstride, uint16_t* xb) {
  const int64_t b = blockIdx.y;
  const int64_t i = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= mn) return;
  const float4 v = *reinterpret_cast<const float4*>(x + b * x_bstride + i);
  uint2 o;
  o.x = (uint32_t)bf16_rne(v.x) | ((uint32_t)bf16_rne(v.y) << 16);
  o.y = (uint32_t)bf16_rne(v.z) | ((uint32_t)bf16_rne(v.w) << 16);
  *reinterpret_cast<uint2*>(xb + b * mn + i) = o;
}

hipError_t launch_cast_bf16(const float* x, int64_t batch, int64_t m, int64_t n, int64_t x_bstride,
                            uint16_t* xb, hipStream_t st) {
  // rows are contiguous with row stride n, so each matrix is m*n consecutive floats
  // (m*n and x_bstride are multiples of 4)
  const int64_t mn = m * n;
  if (batch == 0 || mn == 0) return hipSuccess;
  const dim3 grid((uint32_t)((mn / 4 + 255) / 256), (uint32_t)batch);
  hipLaunchKernelGGL(k_cast_bf16, grid, dim3(256), 0, st, x, mn, x_bstride, xb);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Small per-matrix scalar kernels.

__global__ void k_export_scalar(const MatScalars* sc, int64_t n, int which, int slot, float* out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  out[i] = which == 0 ? sc[i].tau : sc[i].sg[slot];
}

hipError_t launch_export_scalar(const MatScalars* sc, int64_t n, int which, int slot, float* out,
                                hipStream_t st) {
  if (n <= 0 || !out) return hipSuccess;
  hipLaunchKernelGGL(k_export_scalar, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, st, sc, n,
                     which, slot, out);
  return hipGetLastError();
}

}  // namespace fp4r
