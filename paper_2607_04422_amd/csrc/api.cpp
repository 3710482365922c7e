// C ABI of libfp4root: argument validation, workspace planning, grouping by
// canonical shape, and the stream-ordered launch sequence of each operation.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <map>
#include <mutex>
#include <utility>
#include <vector>

#include "../../include/fp4root.h"
#include "internal.h"

using namespace fp4r;

namespace {

constexpr int kVersion = 200;   // 0.2.0
constexpr size_t kAlign = 256;

#define FP4R_TRY(expr)                                   \
  do {                                                   \
    if ((expr) != hipSuccess) return FP4ROOT_ERR_HIP;    \
  } while (0)

// SplitMix64 (Steele, Lea, Flood 2014): output number `index` of the stream
// started at `state`.  Bit i of output k+1 selects the sign of Hadamard row i
// in NS step k.
uint64_t splitmix64(uint64_t state, uint64_t index) {
  uint64_t z = state + 0x9E3779B97F4A7C15ull * index;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

uint32_t sign_mask(uint64_t seed, int32_t step) {
  return (uint32_t)(splitmix64(seed, (uint64_t)step + 1) & 0xFFFFu);
}

// Bump allocator over the caller's workspace; with base == nullptr it only sizes.
#define FP4R_TRY_RC(expr)             \
  do {                                \
    const int rc_ = (expr);           \
    if (rc_ != FP4ROOT_OK) return rc_; \
  } while (0)

struct Carver {
  char* base;
  size_t off = 0;
  explicit Carver(void* b) : base((char*)b) {}
  template <class T>
  T* take(size_t count) {
    off = (off + kAlign - 1) / kAlign * kAlign;
    T* p = base ? reinterpret_cast<T*>(base + off) : nullptr;
    off += count * sizeof(T);
    return p;
  }
};

bool aligned(const void* p, size_t a) { return ((uintptr_t)p % a) == 0; }

// Each side at most 2^21: the products address one 128-row tile of an operand or
// of the output with 32-bit byte offsets (128 * 2^21 * 4 bytes = 2^30).  At most
// 2^36 elements: 256 GiB of FP32, about what the device holds.
constexpr int64_t kMaxDim = int64_t(1) << 21;
constexpr int64_t kMaxElems = int64_t(1) << 36;
// Row strides of the matrix lists (MatRef keeps them in 31 bits of 16-byte units): 16 rows of
// 2^33 - 4 floats are 512 GiB, more than the device holds.
constexpr int64_t kMaxLd = (int64_t(1) << 33) - 4;
bool dims_ok(int64_t r, int64_t c) {
  return r > 0 && c > 0 && r % 16 == 0 && c % 16 == 0 && r <= kMaxDim && c <= kMaxDim && r * c <= kMaxElems;
}

// ---------------------------------------------------------------------------
// Default coefficients: per aspect bucket r = round-half-up(long/short) clamped
// to [1, 4], five per-step (a, b, c) rows.  Generated by coeff_fit.py (this
// library's own fit; the paper does not print Root's values).
#include "coeffs_table.inc"

void default_coeffs_impl(int64_t rows, int64_t cols, int32_t steps, float* out3) {
  const int64_t lo = std::min(rows, cols), hi = std::max(rows, cols);
  int r = (int)((2 * hi + lo) / (2 * lo));   // round half up of hi/lo
  r = std::min(std::max(r, 1), kCoeffBuckets);
  const float(*t)[3] = kCoeffTable[r - 1];
  for (int32_t k = 0; k < steps; ++k) {
    const int row = std::min<int32_t>(k, kCoeffSteps - 1);
    out3[3 * k + 0] = t[row][0];
    out3[3 * k + 1] = t[row][1];
    out3[3 * k + 2] = t[row][2];
  }
}

// ---------------------------------------------------------------------------
// Kernel timer for measurement harnesses: while enabled, every product launch
// is bracketed by HIP events recorded on its own stream.

struct TimerRec {
  int kernel;
  double flop;
  hipEvent_t start, stop;
};

std::mutex g_timer_mu;
bool g_timer_on = false;
std::vector<TimerRec> g_timer_recs;
std::vector<hipEvent_t> g_event_pool;

hipEvent_t pooled_event() {
  if (!g_event_pool.empty()) {
    hipEvent_t e = g_event_pool.back();
    g_event_pool.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

template <class Launch>
hipError_t timed(int kernel, double flop, hipStream_t st, Launch launch) {
  if (!g_timer_on) return launch();
  std::lock_guard<std::mutex> lk(g_timer_mu);
  TimerRec r{kernel, flop, pooled_event(), pooled_event()};
  if (!r.start || !r.stop) return hipErrorOutOfMemory;
  hipError_t e = hipEventRecord(r.start, st);
  if (e == hipSuccess) e = launch();
  if (e == hipSuccess) e = hipEventRecord(r.stop, st);
  g_timer_recs.push_back(r);
  return e;
}

double gram_flop(int64_t batch, int64_t m, int64_t k) { return (double)batch * m * (m + 1) * k; }
double gemm_flop(int64_t batch, int64_t m, int64_t n, int64_t k) { return 2.0 * batch * m * n * k; }

// ---------------------------------------------------------------------------
// Workspace of one batched NS step over `batch` m x n matrices.
// Scratch of the library GEMM of the BF16 path: the needs it reports reach 72 MiB (1500 sizes
// from 16 x 16 to 8192 x 32768 and batches up to 300).
constexpr size_t kBlasltWsBytes = size_t(128) << 20;

struct StepWs {
  MatScalars* sc = nullptr;
  // NVFP4 path
  uint8_t *qx_c = nullptr, *qx_s = nullptr, *qxt_c = nullptr, *qxt_s = nullptr;
  float* A = nullptr;
  uint8_t *qa_c = nullptr, *qa_s = nullptr;
  // chain bounds of qX, qXt and qA / qB: row words and levels (ChainOp), or the
  // encoders' own records alone (see use_levels)
  uint32_t *words_x = nullptr, *words_xt = nullptr, *words_a = nullptr;
  float *rec_x = nullptr, *rec_xt = nullptr, *rec_a = nullptr;
  // BF16 path
  uint16_t *xb = nullptr, *a16 = nullptr, *b16 = nullptr;
  char* blaslt_ws = nullptr;   // scratch of the library GEMM (update product)
};

// Chain bounds over runs of up to four stages take one more launch per encoder (about 5 us);
// with few stages the encoders' own one-stage records do.  Bounds from 512 elements on
// instead of 1024: 256 matrices of 512 x 512 3759 -> 3831 us per call, one of 256 x 512 244 -> 258.
// From 2048 on: 12 parameters of 256 x 256 and 256 x 1024 384 -> 370, three ragged groups of 1040
// to 4112 773 -> 764, one 4096 x 4096 and a step of a 3B-shaped block the same within 0.1 %.
constexpr int64_t kLevelsMinK = 1024;
bool use_levels(int64_t K) { return K >= kLevelsMinK; }
int64_t words_stride(int64_t rows, int64_t K) { return (K + 63) / 64 * rows; }
int64_t rec_stride(int64_t rows, int64_t K) {
  return use_levels(K) ? chain_level_count(rows, K) : rows / 16 * ((K + 63) / 64);
}

void carve_step(Carver& cv, int64_t batch, int64_t m, int64_t n, bool bf16, StepWs& w) {
  w.sc = cv.take<MatScalars>((size_t)batch);
  if (!bf16) {
    // the products' operands, stage-major (see OperandOut)
    w.qx_c = cv.take<uint8_t>((size_t)(batch * tiled_code_bytes(m, n)));
    w.qx_s = cv.take<uint8_t>((size_t)(batch * tiled_scale_bytes(m, n)));
    w.qxt_c = cv.take<uint8_t>((size_t)(batch * tiled_code_bytes(n, m)));
    w.qxt_s = cv.take<uint8_t>((size_t)(batch * tiled_scale_bytes(n, m)));
    w.A = cv.take<float>((size_t)(batch * m * m));
    w.qa_c = cv.take<uint8_t>((size_t)(batch * tiled_code_bytes(m, m)));
    w.qa_s = cv.take<uint8_t>((size_t)(batch * tiled_scale_bytes(m, m)));
    w.rec_x = cv.take<float>((size_t)(batch * rec_stride(m, n)));
    w.rec_xt = cv.take<float>((size_t)(batch * rec_stride(n, m)));
    w.rec_a = cv.take<float>((size_t)(batch * rec_stride(m, m)));
    if (use_levels(n)) w.words_x = cv.take<uint32_t>((size_t)(batch * words_stride(m, n)));
    if (use_levels(m)) {
      w.words_xt = cv.take<uint32_t>((size_t)(batch * words_stride(n, m)));
      w.words_a = cv.take<uint32_t>((size_t)(batch * words_stride(m, m)));
    }
  } else {
    w.xb = cv.take<uint16_t>((size_t)(batch * m * n));
    w.a16 = cv.take<uint16_t>((size_t)(batch * m * m));
    w.b16 = cv.take<uint16_t>((size_t)(batch * m * m));
    w.blaslt_ws = cv.take<char>(kBlasltWsBytes);
  }
}

template <class T>
hipError_t copy_trace(T* dst, const T* src, size_t count, hipStream_t st) {
  if (!dst) return hipSuccess;
  return hipMemcpyAsync(dst, src, count * sizeof(T), hipMemcpyDeviceToDevice, st);
}

// A stage-major operand exported in the row-major layout of fp4root_quantize (either
// output may be null).
hipError_t export_operand(uint8_t* codes, uint8_t* scales, const uint8_t* tc, const uint8_t* ts, int64_t batch,
                          int64_t rows, int64_t K, hipStream_t st) {
  if (!codes && !scales) return hipSuccess;
  return launch_untile_nvfp4(tc, ts, batch, rows, K, codes, scales, st);
}

// Operand views of the stage-major buffers of one step.
OperandOut operand_out(uint8_t* c, uint8_t* s, int64_t rows, int64_t K, uint32_t* words, float* rec) {
  OperandOut q{c, s, tiled_code_bytes(rows, K), tiled_scale_bytes(rows, K)};
  if (!rec) return q;   // binary32 accumulation: no chain bounds
  if (words) {
    q.words = words;
    q.words_bstride = words_stride(rows, K);
  } else {
    q.rec = rec;
    q.rec_bstride = rec_stride(rows, K);
  }
  return q;
}
Fp4Operand tiled_operand(const uint8_t* c, const uint8_t* s, int64_t rows, int64_t K, const float* rec) {
  Fp4Operand o{c, s, tiled_code_bytes(rows, K), tiled_scale_bytes(rows, K)};
  if (!rec) return o;
  o.rec = rec;
  o.rec_bstride = rec_stride(rows, K);
  o.levels = use_levels(K) ? 3 : 1;
  return o;
}
// The operand of the matrices from `first` on.
void advance(Fp4Operand& o, int64_t first) {
  o.codes += first * o.codes_bstride;
  o.scales += first * o.scales_bstride;
  if (o.rec) o.rec += first * o.rec_bstride;
}
// The chain levels of an operand's row words.
ChainOp chain_op(const uint32_t* words, float* rec, int64_t batch, int64_t rows, int64_t K) {
  return ChainOp{words, rec, words_stride(rows, K), rec_stride(rows, K), rows, (int32_t)((K + 63) / 64),
                 (int32_t)batch};
}
// Collects operands whose words await reduction; launches when full or flushed.
struct ChainQueue {
  ChainOp op[kMaxChainOps];
  int count = 0;
  hipStream_t st;
  explicit ChainQueue(hipStream_t s) : st(s) {}
  hipError_t add(const OperandOut& q, float* rec, int64_t batch, int64_t rows, int64_t K) {
    if (!q.words) return hipSuccess;
    op[count++] = chain_op(q.words, rec, batch, rows, K);
    return count == kMaxChainOps ? flush() : hipSuccess;
  }
  hipError_t flush() {
    if (count == 0) return hipSuccess;
    const hipError_t e = launch_chain_levels(op, count, st);
    count = 0;
    return e;
  }
};

// Encoders of several shape groups, kMaxEncode per launch.
struct EncodeQueue {
  EncodeArgs e[kMaxEncode];
  int count = 0;
  template <class F>
  hipError_t add(const EncodeArgs& a, F launch) {
    e[count++] = a;
    return count == kMaxEncode ? flush(launch) : hipSuccess;
  }
  template <class F>
  hipError_t flush(F launch) {
    const int n = count;
    count = 0;
    return n ? launch(e, n) : hipSuccess;
  }
};

// One shape group in one NVFP4 NS step: a batch of m x n matrices at x (matrix
// stride bstride), its step workspace, its coefficients, and (last step of a
// call) the callers' matrices the update writes straight into.
struct StepGroup {
  float* x;
  int64_t batch, m, n, bstride;
  const StepWs* w;
  float a, b, c;
  const std::vector<MatChunk>* fin = nullptr;
};

// The product args of one group's step, common parts.
GemmFp4Args product_args(const StepGroup& sg, uint32_t mask, bool rot, bool acc32) {
  GemmFp4Args g{};
  g.acc32 = acc32 ? 1 : 0;
  g.batch = sg.batch;
  g.sc = sg.w->sc;
  g.amax_mask = mask;
  g.amax_rotate = rot ? 1 : 0;
  return g;
}

// Products of one mode over several groups, kMaxGemmProblems per launch (one timer
// record per launch, its FLOP the sum over the launch's products).
template <class F>
int launch_products(GemmMode mode, int timer_kernel, const StepGroup* gs, int count, F make_args, hipStream_t st,
                    const GemmFin* fin = nullptr) {
  for (int i0 = 0; i0 < count; i0 += kMaxGemmProblems) {
    const int cnt = std::min(count - i0, kMaxGemmProblems);
    GemmFp4Args list[kMaxGemmProblems];
    double flop = 0.0;
    for (int i = 0; i < cnt; ++i) {
      list[i] = make_args(gs[i0 + i]);
      flop += mode == kModeUpdateX ? gemm_flop(list[i].batch, list[i].M, list[i].N, list[i].K)
                                   : gram_flop(list[i].batch, list[i].M, list[i].K);
    }
    FP4R_TRY(timed(timer_kernel, flop, st, [&] { return launch_gemm_fp4_batch(mode, list, cnt, st, fin); }));
  }
  return FP4ROOT_OK;
}

// A round of wide tiles.  Shared update products run narrow below it; exactly that many, and
// launches forced to the wide form, run wide.
constexpr int64_t kShareTiles = 512;

// One NVFP4 NS step on `count` shape groups at once: each kernel of the step runs
// for every group before the next kernel, and the two Gram products of all groups
// share launches (the short groups' tiles fill the long ones' last round).
// xs selects the amax / tensor-scale slot pair of X_k (0 or 2); its amaxes are
// already recorded (by the copy-in stage or the previous update product) unless
// x_amax_needed is set.  The update product records the amaxes of X_{k+1}
// (rotated with the next step's signs) in the other pair.  A trace needs count 1.
int run_step_fp4(const StepGroup* gs, int count, uint32_t flags, uint64_t seed, int32_t step, int xs,
                 bool x_amax_needed, uint32_t* status, const fp4root_ns_trace* tr, hipStream_t st) {
  if (tr && count != 1) return FP4ROOT_ERR_UNSUPPORTED;
  const bool rot = flags & FP4ROOT_F_HADAMARD, ad = flags & FP4ROOT_F_ADAPTIVE46;
  // binary32 accumulation: one MFMA chain per product, so no chain records
  const bool acc32 = flags & FP4ROOT_F_FP32_ACCUM;
  auto rec = [acc32](float* r) { return acc32 ? nullptr : r; };
  const uint32_t mask = sign_mask(seed, step), next_mask = sign_mask(seed, step + 1);
  const int xn = xs, xm = xs + 1, nxn = xs ^ 2, nxm = (xs ^ 2) + 1;
  ChainQueue chains(st);
  // qX and qXt; the amax slots recorded later in the step are cleared by the encoder
  // of X (a single step starts with every slot clear)
  EncodeQueue enc;
  const uint32_t reset = x_amax_needed ? 0u : (1u << kSlotA) | (1u << kSlotB) | (1u << nxn) | (1u << nxm);
  auto encode_x2 = [&](const EncodeArgs* e, int n) {
    return launch_encode_x2(e, n, mask, rot, ad, xn, xm, st, reset);
  };
  for (int i = 0; i < count; ++i) {
    const StepGroup& sg = gs[i];
    const StepWs& w = *sg.w;
    if (x_amax_needed)
      FP4R_TRY(launch_amax_x2(sg.x, sg.batch, sg.m, sg.n, sg.bstride, mask, rot, w.sc, xn, xm, status, st));
    FP4R_TRY(enc.add(EncodeArgs{sg.x, sg.batch, sg.m, sg.n, sg.bstride, w.sc,
                                operand_out(w.qx_c, w.qx_s, sg.m, sg.n, w.words_x, rec(w.rec_x)),
                                operand_out(w.qxt_c, w.qxt_s, sg.n, sg.m, w.words_xt, rec(w.rec_xt))},
                     encode_x2));
  }
  FP4R_TRY(enc.flush(encode_x2));
  for (int i = 0; i < count; ++i) {
    const StepGroup& sg = gs[i];
    const StepWs& w = *sg.w;
    FP4R_TRY(chains.add(operand_out(w.qx_c, w.qx_s, sg.m, sg.n, w.words_x, rec(w.rec_x)), w.rec_x, sg.batch, sg.m, sg.n));
    FP4R_TRY(chains.add(operand_out(w.qxt_c, w.qxt_s, sg.n, sg.m, w.words_xt, rec(w.rec_xt)), w.rec_xt, sg.batch, sg.n, sg.m));
  }
  FP4R_TRY(chains.flush());
  // A = qX qX^T, recording amax(A H)
  FP4R_TRY(launch_products(kModeGramA, 0, gs, count, [&](const StepGroup& sg) {
    GemmFp4Args g = product_args(sg, mask, rot, acc32);
    g.a = tiled_operand(sg.w->qx_c, sg.w->qx_s, sg.m, sg.n, rec(sg.w->rec_x));
    g.b = g.a;
    g.M = sg.m; g.N = sg.m; g.K = sg.n;
    g.slot_a = g.slot_b = xn;
    g.out = sg.w->A; g.out_bstride = sg.m * sg.m; g.aux = nullptr;
    g.amax_row_slot = g.amax_col_slot = kSlotA;
    return g;
  }, st));
  if (tr) FP4R_TRY(copy_trace(tr->A, gs[0].w->A, (size_t)(gs[0].batch * gs[0].m * gs[0].m), st));
  // Q of the symmetric matrices of groups [first, last), in the qA buffers
  auto encode_sym = [&](int first, int last, int slot) -> hipError_t {
    auto run = [&](const EncodeArgs* e, int n) { return launch_encode_operand(e, n, mask, rot, ad, slot, st); };
    auto out = [&](const StepGroup& sg) {
      return operand_out(sg.w->qa_c, sg.w->qa_s, sg.m, sg.m, sg.w->words_a, rec(sg.w->rec_a));
    };
    for (int i = first; i < last; ++i) {
      const StepGroup& sg = gs[i];
      const hipError_t e =
          enc.add(EncodeArgs{sg.w->A, sg.batch, sg.m, sg.m, sg.m * sg.m, sg.w->sc, out(sg), OperandOut{}}, run);
      if (e != hipSuccess) return e;
    }
    hipError_t e = enc.flush(run);
    for (int i = first; i < last && e == hipSuccess; ++i)
      e = chains.add(out(gs[i]), gs[i].w->rec_a, gs[i].batch, gs[i].m, gs[i].m);
    return e == hipSuccess ? chains.flush() : e;
  };
  // qA
  FP4R_TRY(encode_sym(0, count, kSlotA));
  if (tr) {
    const StepGroup& sg = gs[0];
    FP4R_TRY(export_operand(tr->qa_codes, tr->qa_scales, sg.w->qa_c, sg.w->qa_s, sg.batch, sg.m, sg.m, st));
    FP4R_TRY(launch_export_scalar(sg.w->sc, sg.batch, 1, kSlotA, tr->qa_sg, st));
  }
  // B = b A + c qA qA^T, written over A, recording amax(B H)
  FP4R_TRY(launch_products(kModeGramB, 1, gs, count, [&](const StepGroup& sg) {
    GemmFp4Args g = product_args(sg, mask, rot, acc32);
    g.a = tiled_operand(sg.w->qa_c, sg.w->qa_s, sg.m, sg.m, rec(sg.w->rec_a));
    g.b = g.a;
    g.M = sg.m; g.N = sg.m; g.K = sg.m;
    g.slot_a = g.slot_b = kSlotA;
    g.out = sg.w->A; g.out_bstride = sg.m * sg.m; g.aux = sg.w->A;
    g.cb = sg.b; g.cc = sg.c;
    g.amax_row_slot = g.amax_col_slot = kSlotB;
    return g;
  }, st));
  if (tr) FP4R_TRY(copy_trace(tr->B, gs[0].w->A, (size_t)(gs[0].batch * gs[0].m * gs[0].m), st));
  // qB (reusing the qA buffers), then the update product while qB is fresh in the caches:
  // X <- a X + qB qXt^T, recording the amaxes of X_{k+1} for the next step.  Consecutive
  // groups share launches while together they leave room in one round of workgroups (12
  // parameters of 256 x 256 and 256 x 1024, with shared encoders: 524 -> 417 us per step); larger
  // ones fill rounds of their own.
  // Last step: X_{k+1} goes straight to the callers' matrices, a chunk per launch.
  for (int i = 0, last; i < count; i = last) {
    int64_t tiles = 0;
    for (last = i; last < count; ++last) {
      tiles += ((gs[last].m + 127) / 128) * ((gs[last].n + 127) / 128) * gs[last].batch;
      if (last > i && (tiles > kShareTiles || last - i == kMaxGemmProblems)) break;
    }
    FP4R_TRY(encode_sym(i, last, kSlotB));
    if (tr) {
      const StepGroup& sg = gs[i];
      const StepWs& w = *sg.w;
      FP4R_TRY(export_operand(tr->qx_codes, tr->qx_scales, w.qx_c, w.qx_s, sg.batch, sg.m, sg.n, st));
      FP4R_TRY(launch_export_scalar(w.sc, sg.batch, 1, xn, tr->qx_sg, st));
      FP4R_TRY(export_operand(tr->qxt_codes, tr->qxt_scales, w.qxt_c, w.qxt_s, sg.batch, sg.n, sg.m, st));
      FP4R_TRY(launch_export_scalar(w.sc, sg.batch, 1, xm, tr->qxt_sg, st));
      FP4R_TRY(export_operand(tr->qb_codes, tr->qb_scales, w.qa_c, w.qa_s, sg.batch, sg.m, sg.m, st));
      FP4R_TRY(launch_export_scalar(w.sc, sg.batch, 1, kSlotB, tr->qb_sg, st));
    }
    auto update = [&](const StepGroup& u) {
      GemmFp4Args g = product_args(u, next_mask, rot, acc32);
      g.a = tiled_operand(u.w->qa_c, u.w->qa_s, u.m, u.m, rec(u.w->rec_a));
      g.b = tiled_operand(u.w->qxt_c, u.w->qxt_s, u.n, u.m, rec(u.w->rec_xt));
      g.M = u.m; g.N = u.n; g.K = u.m;
      g.slot_a = kSlotB; g.slot_b = xm;
      g.out = u.x; g.out_bstride = u.bstride; g.aux = u.x;
      g.ca = u.a;
      g.amax_row_slot = nxn; g.amax_col_slot = nxm;
      return g;
    };
    if (!gs[i].fin) {   // all groups of a call are at the same step
      FP4R_TRY_RC(launch_products(kModeUpdateX, 2, gs + i, last - i, update, st));
      continue;
    }
    for (int k = i; k < last; ++k)
      for (size_t c = 0; c < gs[k].fin->size(); ++c) {
        const int64_t first = (int64_t)c * kMaxChunk;
        const MatChunk& ch = (*gs[k].fin)[c];
        GemmFin fin;
        fin.count = ch.count;
        for (int f = 0; f < ch.count; ++f) {
          fin.out[f] = ch.m[f].out;
          fin.ld[f] = ch.m[f].ld_out();
          fin.tall[f] = ch.m[f].tall() ? 1 : 0;
        }
        FP4R_TRY_RC(launch_products(kModeUpdateX, 2, gs + k, 1, [&](const StepGroup& u) {
          GemmFp4Args g = update(u);
          g.amax_row_slot = g.amax_col_slot = -1;   // no amaxes needed
          g.batch = fin.count;
          g.sc += first;
          advance(g.a, first);
          advance(g.b, first);
          g.out += first * g.out_bstride;
          g.aux += first * g.out_bstride;
          return g;
        }, st, &fin));
      }
  }
  return FP4ROOT_OK;
}

// One BF16 NS step; Xb must hold bf16(X) on entry and holds bf16(X_{k+1}) on exit.
int run_step_bf16(float* x, int64_t batch, int64_t m, int64_t n, int64_t bstride, float a, float b,
                  float c, const StepWs& w, hipStream_t st) {
  GemmBf16Args g{};
  g.batch = batch;
  // A16 = Xb Xb^T
  g.a = w.xb; g.b = w.xb; g.a_bstride = g.b_bstride = m * n;
  g.M = m; g.N = m; g.K = n;
  g.out16 = w.a16; g.out16_bstride = m * m;
  FP4R_TRY(timed(0, gram_flop(batch, m, n), st, [&] { return launch_gemm_bf16(kModeGramA, g, st); }));
  // B16 = b A16 + c A16 A16^T
  g.a = w.a16; g.b = w.a16; g.a_bstride = g.b_bstride = m * m;
  g.K = m;
  g.out16 = w.b16; g.aux16 = w.a16;
  g.cb = b; g.cc = c;
  FP4R_TRY(timed(1, gram_flop(batch, m, m), st, [&] { return launch_gemm_bf16(kModeGramB, g, st); }));
  // X <- a X + B16 Xb (library GEMM), then Xb = bf16(X)
  FP4R_TRY(timed(2, gemm_flop(batch, m, n, m), st, [&] {
    return launch_bf16_update_blaslt(w.b16, w.xb, x, batch, m, n, bstride, a, w.blaslt_ws, kBlasltWsBytes, st);
  }));
  FP4R_TRY(launch_cast_bf16(x, batch, m, n, bstride, w.xb, st));
  return FP4ROOT_OK;
}

// ---------------------------------------------------------------------------
// Orthogonalisation groups.

struct Group {
  int64_t m, n;
  std::vector<int64_t> members;
};

std::vector<Group> make_groups(const fp4root_matrix* mats, int64_t count) {
  std::map<std::pair<int64_t, int64_t>, size_t> idx;
  std::vector<Group> groups;
  for (int64_t i = 0; i < count; ++i) {
    const int64_t m = std::min(mats[i].rows, mats[i].cols), n = std::max(mats[i].rows, mats[i].cols);
    auto key = std::make_pair(m, n);
    auto it = idx.find(key);
    if (it == idx.end()) {
      idx[key] = groups.size();
      groups.push_back(Group{m, n, {}});
      it = idx.find(key);
    }
    groups[it->second].members.push_back(i);
  }
  return groups;
}

// The chunk of `count` matrices of a list from `first` on (canonical shape m x n, quantile
// index and fraction as given).
MatChunk make_chunk(const std::vector<MatRef>& all, size_t first, size_t count, int64_t m, int64_t n, int64_t lo,
                    double frac) {
  MatChunk ch;
  std::memset(&ch, 0, sizeof(ch));
  ch.count = (int)count;
  ch.rows = m;
  ch.cols = n;
  ch.lo = lo;
  ch.frac = frac;
  for (size_t i = 0; i < count; ++i) ch.m[i] = all[first + i];
  return ch;
}
size_t chunk_hist_words(int64_t batch, int64_t elems) {
  return (size_t)(std::min<int64_t>(batch, kMaxChunk) * hist_words(elems));
}

void quantile_index(int64_t n, float q, int64_t& lo, double& frac) {
  const double h = (double)q * (double)(n - 1);
  const double f = std::floor(h);
  lo = (int64_t)f;
  frac = h - f;
}

struct GroupWs {
  StepWs step;
  float* X = nullptr;
  uint32_t* hist = nullptr;
  double* partial = nullptr;
  uint32_t* partial_cnt = nullptr;
  uint32_t* cand_cnt = nullptr;
};

void carve_group(Carver& cv, const Group& gr, bool bf16, GroupWs& w) {
  const int64_t B = (int64_t)gr.members.size();
  carve_step(cv, B, gr.m, gr.n, bf16, w.step);
  w.X = cv.take<float>((size_t)(B * gr.m * gr.n));
  w.hist = cv.take<uint32_t>(chunk_hist_words(B, gr.m * gr.n));
  const size_t parts = (size_t)(std::min<int64_t>(B, kMaxChunk) * hist_parts(gr.m * gr.n / 4));
  w.partial = cv.take<double>(parts * 2);
  w.partial_cnt = cv.take<uint32_t>(parts * 2);
  w.cand_cnt = cv.take<uint32_t>(parts * 4);
}

int validate_matrices(const fp4root_matrix* mats, int64_t count) {
  if (count < 0 || (count > 0 && !mats)) return FP4ROOT_ERR_INVALID_ARG;
  for (int64_t i = 0; i < count; ++i) {
    const fp4root_matrix& a = mats[i];
    if (!a.in || !a.out) return FP4ROOT_ERR_INVALID_ARG;
    if (!dims_ok(a.rows, a.cols)) return FP4ROOT_ERR_SHAPE;
    if (a.ld_in < a.cols || a.ld_out < a.cols || a.ld_in % 4 || a.ld_out % 4) return FP4ROOT_ERR_SHAPE;
    if (a.ld_in > kMaxLd || a.ld_out > kMaxLd) return FP4ROOT_ERR_SHAPE;
    if (!aligned(a.in, 16) || !aligned(a.out, 16)) return FP4ROOT_ERR_INVALID_ARG;
    if ((const void*)a.in == (const void*)a.out && a.ld_in != a.ld_out) return FP4ROOT_ERR_INVALID_ARG;
  }
  return FP4ROOT_OK;
}

int validate_config(const fp4root_ns_config* cfg) {
  if (!cfg || cfg->steps < 0) return FP4ROOT_ERR_INVALID_ARG;
  if (cfg->flags & ~(uint32_t)(FP4ROOT_F_CLIP | FP4ROOT_F_HADAMARD | FP4ROOT_F_ADAPTIVE46 |
                               FP4ROOT_F_BF16_PATH | FP4ROOT_F_FP32_ACCUM))
    return FP4ROOT_ERR_INVALID_ARG;
  if ((cfg->flags & FP4ROOT_F_BF16_PATH) && (cfg->flags & FP4ROOT_F_FP32_ACCUM)) return FP4ROOT_ERR_INVALID_ARG;
  if ((cfg->flags & FP4ROOT_F_CLIP) && !(cfg->clip_quantile >= 0.0f && cfg->clip_quantile <= 1.0f))
    return FP4ROOT_ERR_INVALID_ARG;
  if (!(cfg->eps >= 0.0f) || !std::isfinite(cfg->eps)) return FP4ROOT_ERR_INVALID_ARG;
  if (cfg->coeffs)
    for (int32_t k = 0; k < 3 * cfg->steps; ++k)
      if (!std::isfinite(cfg->coeffs[k])) return FP4ROOT_ERR_INVALID_ARG;
  return FP4ROOT_OK;
}

// The NVFP4 path keeps every group's workspace at once (its steps run over all groups
// together); the BF16 path runs the groups one after another in one reused workspace.
size_t orthogonalize_ws_size(const fp4root_matrix* mats, int64_t count, const fp4root_ns_config* cfg) {
  const bool bf16 = cfg->flags & FP4ROOT_F_BF16_PATH;
  size_t need = kAlign;   // status word
  Carver all(nullptr);
  all.off = kAlign;
  for (const Group& gr : make_groups(mats, count)) {
    GroupWs w;
    if (bf16) {
      Carver cv(nullptr);
      cv.off = kAlign;
      carve_group(cv, gr, bf16, w);
      need = std::max(need, cv.off);
    } else {
      carve_group(all, gr, bf16, w);
      need = std::max(need, all.off);
    }
  }
  return need;
}
}  // namespace

// ===========================================================================
// ---------------------------------------------------------------------------
// Fixed scratch of fp4root_quantize_noalloc: a file-scope device array, one copy
// per GPU, shared by every call on that GPU (overlapping calls on one GPU race).
// It holds kNoAllocMaxBatch matrices with clipping (the status word, the per-matrix scalars
// and the radix histograms of one chunk of matrices), and without clipping as many scalars as
// fit in the same bytes.
constexpr int64_t kNoAllocMaxBatch = 256;
constexpr int kNoAllocChunk = 32;
constexpr size_t kNoAllocScratchBytes =
    kAlign + (kNoAllocMaxBatch * sizeof(MatScalars) + kAlign - 1) / kAlign * kAlign +
    (size_t)kNoAllocChunk * 2 * kHistBins * sizeof(uint32_t);
constexpr int64_t kNoAllocMaxPlain = (kNoAllocScratchBytes - kAlign) / sizeof(MatScalars);
static_assert(kNoAllocMaxPlain == 1166, "stated in fp4root.h");
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace {
// The device address of `scratch` on the current device, looked up once per
// device (in host code the array's name is only a host-side stand-in).
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_dev[kMaxDevices] = {};

int scratch_address(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return FP4ROOT_ERR_HIP;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_dev[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return FP4ROOT_ERR_HIP;
    g_scratch_dev[dev] = p;
  }
  *out = g_scratch_dev[dev];
  return FP4ROOT_OK;
}
}  // namespace

extern "C" {

int fp4root_version(void) { return kVersion; }

int fp4root_set_product_tiling(int mode) {
  if (mode < 0 || mode > 2) return FP4ROOT_ERR_INVALID_ARG;
  return swap_product_tiling(mode);
}

int fp4root_timer_enable(int on) {
  std::lock_guard<std::mutex> lk(g_timer_mu);
  g_timer_on = on != 0;
  return FP4ROOT_OK;
}

int fp4root_timer_read(int kernel, double* ms, int64_t* launches, double* flop) {
  if (!ms || !launches || !flop) return FP4ROOT_ERR_INVALID_ARG;
  std::lock_guard<std::mutex> lk(g_timer_mu);
  double t = 0.0, f = 0.0;
  int64_t n = 0;
  for (const TimerRec& r : g_timer_recs) {
    if (kernel >= 0 && r.kernel != kernel) continue;
    if (hipEventSynchronize(r.stop) != hipSuccess) return FP4ROOT_ERR_HIP;
    float e = 0.0f;
    if (hipEventElapsedTime(&e, r.start, r.stop) != hipSuccess) return FP4ROOT_ERR_HIP;
    t += e;
    f += r.flop;
    ++n;
  }
  *ms = t;
  *launches = n;
  *flop = f;
  return FP4ROOT_OK;
}

int fp4root_timer_reset(void) {
  std::lock_guard<std::mutex> lk(g_timer_mu);
  for (const TimerRec& r : g_timer_recs) {
    if (hipEventSynchronize(r.stop) != hipSuccess) return FP4ROOT_ERR_HIP;
    g_event_pool.push_back(r.start);
    g_event_pool.push_back(r.stop);
  }
  g_timer_recs.clear();
  return FP4ROOT_OK;
}

const char* fp4root_status_string(int s) {
  switch (s) {
    case FP4ROOT_OK: return "ok";
    case FP4ROOT_ERR_INVALID_ARG: return "invalid argument";
    case FP4ROOT_ERR_SHAPE: return "invalid shape (dimensions must be positive multiples of 16, at most 2^21, at most 2^36 elements)";
    case FP4ROOT_ERR_WORKSPACE: return "workspace missing or too small";
    case FP4ROOT_ERR_NONFINITE: return "non-finite value in the input";
    case FP4ROOT_ERR_HIP: return "HIP runtime error";
    case FP4ROOT_ERR_UNSUPPORTED: return "unsupported combination";
    default: return "unknown status";
  }
}

int fp4root_default_coeffs(int64_t rows, int64_t cols, int32_t steps, float* out3) {
  if (!out3 || steps < 0) return FP4ROOT_ERR_INVALID_ARG;
  if (!dims_ok(rows, cols)) return FP4ROOT_ERR_SHAPE;
  default_coeffs_impl(rows, cols, steps, out3);
  return FP4ROOT_OK;
}

int fp4root_device_status(const void* ws, void* stream) {
  if (!ws) return FP4ROOT_ERR_INVALID_ARG;
  hipStream_t st = (hipStream_t)stream;
  uint32_t word = 0;
  if (hipStreamSynchronize(st) != hipSuccess) return FP4ROOT_ERR_HIP;
  if (hipMemcpy(&word, ws, sizeof(word), hipMemcpyDeviceToHost) != hipSuccess) return FP4ROOT_ERR_HIP;
  if (word & kStatusNonFinite) return FP4ROOT_ERR_NONFINITE;
  return FP4ROOT_OK;
}

namespace {
// Count words of the clip passes' segments (4 per part of a chunk's matrices); none for a
// shape that the call refuses.
int64_t quantize_cand_counts(int64_t batch, int64_t rows, int64_t cols) {
  if (batch <= 0 || !dims_ok(rows, cols)) return 0;
  return 4 * std::min<int64_t>(batch, kMaxChunk) * hist_parts(rows * cols / 4);
}
}  // namespace

size_t fp4root_quantize_workspace(int64_t batch, int64_t rows, int64_t cols, uint32_t flags) {
  if (batch < 0) return 0;
  Carver cv(nullptr);
  cv.off = kAlign;
  cv.take<MatScalars>((size_t)batch);
  if (flags & FP4ROOT_F_CLIP) {
    cv.take<uint32_t>(chunk_hist_words(batch, dims_ok(rows, cols) ? rows * cols : 0));
    cv.take<uint32_t>((size_t)quantize_cand_counts(batch, rows, cols));
  }
  return cv.off;
}

namespace {
// Synchronous argument checks of fp4root_quantize (everything but the workspace).
int check_quantize(const float* x, int64_t batch, int64_t rows, int64_t cols, int64_t ld, int64_t batch_stride,
                   int axis, uint32_t flags, float clip_quantile, const uint8_t* codes, const uint8_t* scales,
                   const float* tensor_scale) {
  if (batch < 0 || !x || !codes || !scales || !tensor_scale || (axis != 0 && axis != 1))
    return FP4ROOT_ERR_INVALID_ARG;
  if (flags & ~(uint32_t)(FP4ROOT_F_CLIP | FP4ROOT_F_HADAMARD | FP4ROOT_F_ADAPTIVE46))
    return FP4ROOT_ERR_INVALID_ARG;
  if (!dims_ok(rows, cols)) return FP4ROOT_ERR_SHAPE;
  if (ld < cols || ld % 4 || (batch > 1 && batch_stride < rows * ld) || batch_stride % 4)
    return FP4ROOT_ERR_SHAPE;
  if ((flags & FP4ROOT_F_CLIP) && ld > kMaxLd) return FP4ROOT_ERR_SHAPE;
  if (!aligned(x, 16) || !aligned(codes, 8)) return FP4ROOT_ERR_INVALID_ARG;
  if ((flags & FP4ROOT_F_CLIP) && !(clip_quantile >= 0.0f && clip_quantile <= 1.0f)) return FP4ROOT_ERR_INVALID_ARG;
  return FP4ROOT_OK;
}

// The launches of fp4root_quantize (arguments checked, batch > 0) on the scratch
// memory at ws: with `collect` fp4root_quantize_workspace bytes, otherwise
// kNoAllocScratchBytes (the clip passes then read the matrix three times, in chunks of
// kNoAllocChunk).  Every part that must start at zero is cleared by a kernel first.
int quantize_launch(const float* x, int64_t batch, int64_t rows, int64_t cols, int64_t ld, int64_t batch_stride,
                    int axis, uint32_t flags, float clip_quantile, uint64_t seed, int32_t step, uint8_t* codes,
                    uint8_t* scales, float* tensor_scale, float* clip_threshold, void* ws, bool collect,
                    hipStream_t st) {
  const bool clip = flags & FP4ROOT_F_CLIP;
  // half as many matrices of 64-bit counts fit in the fixed scratch
  const size_t chunk = collect ? kMaxChunk : wide_counts(rows * cols) ? kNoAllocChunk / 2 : kNoAllocChunk;
  const size_t hist_n = std::min((size_t)batch, chunk) * (size_t)hist_words(rows * cols);
  Carver cv(ws);
  uint32_t* status = cv.take<uint32_t>(1);
  MatScalars* sc = cv.take<MatScalars>((size_t)batch);
  uint32_t* hist = clip ? cv.take<uint32_t>(hist_n) : nullptr;
  uint32_t* cnt = clip && collect ? cv.take<uint32_t>((size_t)quantize_cand_counts(batch, rows, cols)) : nullptr;
  FP4R_TRY(launch_init(status, sc, batch, hist, clip ? (int64_t)hist_n : 0, st));
  if (clip) {
    int64_t lo;
    double frac;
    quantile_index(rows * cols, clip_quantile, lo, frac);
    std::vector<MatRef> all((size_t)batch);
    for (int64_t b = 0; b < batch; ++b) all[(size_t)b] = MatRef{x + b * batch_stride, nullptr, (uint32_t)(ld / 4), 0u};
    for (size_t c0 = 0; c0 < all.size(); c0 += chunk) {
      const size_t cnt_mats = std::min(all.size() - c0, chunk);
      const MatChunk ch = make_chunk(all, c0, cnt_mats, rows, cols, lo, frac);
      ClipScratch cs;
      cs.hist = hist;
      if (collect) {
        // segments in the code output, written by the encoder later: half a byte per element
        cs.cand = reinterpret_cast<float*>(codes + (int64_t)c0 * (rows * cols / 2));
        cs.cand_stride = rows * cols / 8;
        cs.cand_shift = 3;
        cs.cnt = cnt;
      }
      FP4R_TRY(launch_clip_threshold(ch, sc + c0, status, cs, 0.0f, st));
    }
  }
  const Batch in{x, batch, rows, cols, ld, batch_stride};
  const QOut q{codes, scales, rows * cols / 2, rows * cols / 16};
  const bool rot = flags & FP4ROOT_F_HADAMARD, ad = flags & FP4ROOT_F_ADAPTIVE46;
  const uint32_t mask = sign_mask(seed, step);
  FP4R_TRY(launch_amax(in, axis, mask, rot, clip, sc, 0, status, st));
  FP4R_TRY(launch_encode(in, axis, mask, rot, clip, ad, sc, 0, q, tensor_scale, st, clip_threshold));
  return FP4ROOT_OK;
}
}  // namespace

int fp4root_quantize(const float* x, int64_t batch, int64_t rows, int64_t cols, int64_t ld,
                     int64_t batch_stride, int axis, uint32_t flags, float clip_quantile,
                     uint64_t seed, int32_t step, uint8_t* codes, uint8_t* scales,
                     float* tensor_scale, float* clip_threshold, void* ws, size_t ws_bytes,
                     void* stream) {
  const int rc = check_quantize(x, batch, rows, cols, ld, batch_stride, axis, flags, clip_quantile, codes, scales,
                                tensor_scale);
  if (rc != FP4ROOT_OK) return rc;
  if (!ws || ws_bytes < fp4root_quantize_workspace(batch, rows, cols, flags)) return FP4ROOT_ERR_WORKSPACE;
  if (batch == 0) return FP4ROOT_OK;
  return quantize_launch(x, batch, rows, cols, ld, batch_stride, axis, flags, clip_quantile, seed, step, codes,
                         scales, tensor_scale, clip_threshold, ws, true, (hipStream_t)stream);
}

size_t fp4root_momentum_workspace(int64_t batch, int64_t rows, int64_t cols) {
  if (batch < 0 || !dims_ok(rows, cols)) return 0;
  Carver cv(nullptr);
  cv.off = kAlign;
  cv.take<MatScalars>((size_t)batch);
  return std::max<size_t>(cv.off, kAlign);
}

namespace {
// Synchronous argument checks of fp4root_momentum_update (everything but the workspace).
int check_momentum(const float* g, const float* m, int64_t batch, int64_t rows, int64_t cols,
                   const uint8_t* codes, const uint8_t* scales, const float* tensor_scale, float beta,
                   uint32_t flags, int32_t step) {
  if (batch < 0 || step < 0 || !g || !m || !codes || !scales || !tensor_scale) return FP4ROOT_ERR_INVALID_ARG;
  if (flags & ~(uint32_t)(FP4ROOT_F_HADAMARD | FP4ROOT_F_ADAPTIVE46 | FP4ROOT_F_STOCHASTIC))
    return FP4ROOT_ERR_INVALID_ARG;
  if (!(beta >= 0.0f && beta <= 1.0f)) return FP4ROOT_ERR_INVALID_ARG;
  if (!dims_ok(rows, cols)) return FP4ROOT_ERR_SHAPE;
  if (!aligned(g, 16) || !aligned(m, 16) || !aligned(codes, 8)) return FP4ROOT_ERR_INVALID_ARG;
  return FP4ROOT_OK;
}

// The launches of fp4root_momentum_update (arguments already checked).
int momentum_update_launch(const float* g, float* m, int64_t batch, int64_t rows, int64_t cols, uint8_t* codes,
                           uint8_t* scales, float* tensor_scale, float beta, uint32_t flags, uint64_t seed,
                           int32_t step, void* ws, hipStream_t st) {
  if (batch == 0) return FP4ROOT_OK;
  Carver cv(ws);
  uint32_t* status = cv.take<uint32_t>(1);
  MatScalars* sc = cv.take<MatScalars>((size_t)batch);
  const bool rot = flags & FP4ROOT_F_HADAMARD, ad = flags & FP4ROOT_F_ADAPTIVE46;
  const float b1 = beta, b2 = 1.0f - beta;   // b2 = fl32(1 - beta)
  const uint32_t mask = sign_mask(seed, step), prev_mask = step > 0 ? sign_mask(seed, step - 1) : 0u;
  FP4R_TRY(launch_init(status, sc, batch, nullptr, 0, st));
  FP4R_TRY(launch_mom_update(g, m, batch, rows, cols, codes, scales, tensor_scale, step > 0, prev_mask,
                             mask, rot, b1, b2, sc, status, st));
  const Batch in{m, batch, rows, cols, cols, rows * cols};
  const QOut q{codes, scales, rows * cols / 2, rows * cols / 16};
  if (flags & FP4ROOT_F_STOCHASTIC) {
    const uint64_t key = splitmix64(seed ^ 0x5352ull, (uint64_t)step + 1);
    FP4R_TRY(launch_encode_sr(in, mask, rot, ad, sc, 0, q, tensor_scale, key, st));
  } else {
    FP4R_TRY(launch_encode(in, 1, mask, rot, false, ad, sc, 0, q, tensor_scale, st));
  }
  return FP4ROOT_OK;
}
}  // namespace

int fp4root_momentum_update(const float* g, float* m, int64_t batch, int64_t rows, int64_t cols,
                            uint8_t* codes, uint8_t* scales, float* tensor_scale, float beta,
                            uint32_t flags, uint64_t seed, int32_t step, void* ws, size_t ws_bytes,
                            void* stream) {
  const int rc = check_momentum(g, m, batch, rows, cols, codes, scales, tensor_scale, beta, flags, step);
  if (rc != FP4ROOT_OK) return rc;
  if (!ws || ws_bytes < fp4root_momentum_workspace(batch, rows, cols)) return FP4ROOT_ERR_WORKSPACE;
  return momentum_update_launch(g, m, batch, rows, cols, codes, scales, tensor_scale, beta, flags, seed, step, ws,
                                (hipStream_t)stream);
}

namespace {
// A rows x cols view of a flat parameter for the first-moment kernels (blocks of
// 16, draws and codes are indexed by the flat position, so every view with
// cols % 16 == 0 gives the same state): 16 x n/16 up to 2^25 elements, else
// n/256 x 256.  Returns false when neither fits the kernels' limits.
bool flat_view(int64_t n, int64_t& rows, int64_t& cols) {
  if (n <= 0 || n % 256) return false;
  if (n / 16 <= (int64_t(1) << 21)) {
    rows = 16;
    cols = n / 16;
  } else {
    rows = n / 256;
    cols = 256;
  }
  return dims_ok(rows, cols);
}
}  // namespace

size_t fp4root_qadamw_workspace(int64_t n) {
  int64_t r, c;
  if (!flat_view(n, r, c)) return 0;
  return fp4root_momentum_workspace(1, r, c);
}

int fp4root_qadamw_update(uint16_t* w, const float* g, float* m, int64_t n, uint8_t* m_codes,
                          uint8_t* m_scales, float* m_tensor_scale, uint8_t* v_codes, uint16_t* v_scales,
                          uint16_t* v_means, float lr, float wd, float beta1, float beta2, float eps,
                          uint32_t flags, uint64_t seed, int32_t step, void* ws, size_t ws_bytes,
                          void* stream) {
  int64_t vr = 0, vc = 0;
  if (!flat_view(n, vr, vc)) return FP4ROOT_ERR_SHAPE;
  if (step < 0 || !w || !g || !m_codes || !m_scales || !m_tensor_scale || !v_codes || !v_scales || !v_means)
    return FP4ROOT_ERR_INVALID_ARG;
  if (!aligned(w, 16) || !aligned(g, 16) || (m && !aligned(m, 16)) || !aligned(m_codes, 8) || !aligned(v_codes, 8))
    return FP4ROOT_ERR_INVALID_ARG;
  // the second pass reads g again: the first-moment output may not overlap it
  if (m && (const char*)m < (const char*)(g + n) && (const char*)g < (const char*)(m + n))
    return FP4ROOT_ERR_INVALID_ARG;
  if (flags & ~(uint32_t)(FP4ROOT_F_HADAMARD | FP4ROOT_F_ADAPTIVE46 | FP4ROOT_F_STOCHASTIC))
    return FP4ROOT_ERR_INVALID_ARG;
  if (!std::isfinite(lr) || !std::isfinite(wd) || !std::isfinite(eps) || !(beta1 >= 0.0f && beta1 <= 1.0f) ||
      !(beta2 >= 0.0f && beta2 <= 1.0f))
    return FP4ROOT_ERR_INVALID_ARG;
  if (!ws || ws_bytes < fp4root_qadamw_workspace(n)) return FP4ROOT_ERR_WORKSPACE;
  hipStream_t st = (hipStream_t)stream;
  Carver cv(ws);
  uint32_t* status = cv.take<uint32_t>(1);
  MatScalars* sc = cv.take<MatScalars>(1);
  auto bias_correction = [](float beta, int32_t t) {
    double p = 1.0;
    for (int32_t k = 0; k <= t; ++k) p *= (double)beta;
    return (float)(1.0 - p);
  };
  const bool rot = flags & FP4ROOT_F_HADAMARD, ad = flags & FP4ROOT_F_ADAPTIVE46;
  const uint32_t mask = sign_mask(seed, step), prev_mask = step > 0 ? sign_mask(seed, step - 1) : 0u;
  FP4R_TRY(launch_init(status, sc, 1, nullptr, 0, st));
  // pass 1: first moment (read only), its rotated amax, second moment and weights
  QAdamWLaunch q;
  q.w = w; q.g = g; q.m_out = m; q.mcodes = m_codes; q.mscales = m_scales; q.m_prev_sg = m_tensor_scale;
  q.b1 = beta1;
  q.c1m = 1.0f - beta1;
  q.sc = sc;
  q.vcodes = v_codes; q.vscales = v_scales; q.vmeans = v_means; q.n = n;
  q.has_prev = step > 0;
  q.rotate = rot;
  q.adaptive = ad;
  q.prev_mask = prev_mask;
  q.mask = mask;
  q.b2 = beta2;
  q.c2 = 1.0f - beta2;
  q.bc1 = bias_correction(beta1, step);
  q.bc2 = bias_correction(beta2, step);
  q.eps = eps;
  q.lr = lr;
  const float lw = lr * wd;
  q.c1w = 1.0f - lw;
  q.status = status;
  FP4R_TRY(launch_qadamw(q, st));
  // pass 2: the first moment re-derived and encoded in place
  const uint64_t key = splitmix64(seed ^ 0x5352ull, (uint64_t)step + 1);
  FP4R_TRY(launch_mom_encode(g, m_codes, m_scales, n, step > 0, prev_mask, mask, rot, ad,
                             flags & FP4ROOT_F_STOCHASTIC, beta1, 1.0f - beta1, sc, m_tensor_scale, key, st));
  return FP4ROOT_OK;
}

int fp4root_apply_update(uint16_t* w, const float* o, int64_t count, float lr, float wd, float scale,
                         void* stream) {
  if (count < 0 || count % 8) return FP4ROOT_ERR_SHAPE;
  if (count > 0 && (!w || !o || !aligned(w, 16) || !aligned(o, 16))) return FP4ROOT_ERR_INVALID_ARG;
  if (!std::isfinite(lr) || !std::isfinite(wd) || !std::isfinite(scale)) return FP4ROOT_ERR_INVALID_ARG;
  const float lw = lr * wd, c1 = 1.0f - lw, c2 = lr * scale;   // one binary32 rounding each
  FP4R_TRY(launch_apply_update(w, o, count, c1, c2, (hipStream_t)stream));
  return FP4ROOT_OK;
}

namespace {
std::vector<fp4root_matrix> root_matrices(const fp4root_param* p, int64_t count) {
  std::vector<fp4root_matrix> mats((size_t)count);
  for (int64_t i = 0; i < count; ++i)
    mats[(size_t)i] = fp4root_matrix{p[i].m, p[i].m, p[i].rows, p[i].cols, p[i].cols, p[i].cols};
  return mats;
}
}  // namespace

size_t fp4root_root_step_workspace(const fp4root_param* params, int64_t count, const fp4root_ns_config* ns) {
  if (count < 0 || (count > 0 && !params) || !ns) return 0;
  size_t need = kAlign;
  for (int64_t i = 0; i < count; ++i) {
    if (!dims_ok(params[i].rows, params[i].cols)) return 0;
  }
  need = std::max(need, fp4root_momentum_workspace(std::min<int64_t>(count, kMaxRootChunk), 16, 16));
  if (count > 0) {
    const std::vector<fp4root_matrix> mats = root_matrices(params, count);
    const size_t ow = fp4root_orthogonalize_workspace(mats.data(), count, ns);
    if (ow == 0) return 0;
    need = std::max(need, ow);
  }
  return need;
}

namespace {
int orthogonalize_launch(const fp4root_matrix* mats, int64_t count, const fp4root_ns_config* cfg, void* ws,
                         bool reset_status, hipStream_t st);
}  // namespace

namespace {
bool overlap(const void* a, int64_t na, const void* b, int64_t nb) {
  const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
  return x < y + (uintptr_t)nb && y < x + (uintptr_t)na;
}

// Two parameters that must not share a launch: one writes what the other reads or writes
// (one weight listed twice, for instance), so their order counts.
bool depend(const fp4root_param& a, const fp4root_param& b) {
  const int64_t na = a.rows * a.cols, nb = b.rows * b.cols;
  return overlap(a.w, 2 * na, b.w, 2 * nb) || overlap(a.m, 4 * na, b.m, 4 * nb) || overlap(a.g, 4 * na, b.m, 4 * nb) ||
         overlap(a.m, 4 * na, b.g, 4 * nb) || overlap(a.m_codes, na / 2, b.m_codes, nb / 2) ||
         overlap(a.m_scales, na / 16, b.m_scales, nb / 16) || a.m_tensor_scale == b.m_tensor_scale;
}

// The longest run of parameters from `first` on that one launch of each kind can take.
void root_chunk(const fp4root_param* params, int64_t count, int64_t first, const fp4root_root_config& rc,
                RootChunk& ch) {
  ch.count = 0;
  int64_t end = 0;
  for (int64_t i = first; i < count && ch.count < kMaxRootChunk; ++i) {
    const fp4root_param& p = params[i];
    const int64_t nblk = p.rows * p.cols / 16, wgs = (nblk + 255) / 256;
    bool fits = end + wgs <= kMaxSharedBlocks;
    for (int64_t k = first; k < i && fits; ++k) fits = !depend(params[k], p);
    if (ch.count > 0 && !fits) break;
    const uint64_t seed = rc.momentum_seed + (uint64_t)i;
    // scale 0: the default update scale sqrt(max(1, rows / cols)), rounded once
    const float s = p.scale > 0.0f ? p.scale
                                   : (float)std::sqrt(std::max(1.0, (double)p.rows / (double)p.cols));
    end += wgs;
    ch.p[ch.count] = RootRef{p.g, p.m, p.m_codes, p.m_scales, p.m_tensor_scale, p.w, nblk,
                             splitmix64(seed ^ 0x5352ull, (uint64_t)rc.step + 1), sign_mask(seed, rc.step),
                             rc.step > 0 ? sign_mask(seed, rc.step - 1) : 0u, rc.lr * s};
    ch.end[ch.count++] = (uint32_t)end;
  }
}
}  // namespace

int fp4root_root_step(const fp4root_param* params, int64_t count, const fp4root_root_config* rc,
                      const fp4root_ns_config* ns, void* ws, size_t ws_bytes, void* stream) {
  if (count < 0 || (count > 0 && !params) || !rc || !ns) return FP4ROOT_ERR_INVALID_ARG;
  // every argument is checked before the first launch, so an error leaves every
  // parameter's state unchanged
  for (int64_t i = 0; i < count; ++i) {
    const fp4root_param& p = params[i];
    if (!p.w || !aligned(p.w, 16) || !std::isfinite(p.scale) || p.scale < 0.0f) return FP4ROOT_ERR_INVALID_ARG;
    const int c = check_momentum(p.g, p.m, 1, p.rows, p.cols, p.m_codes, p.m_scales, p.m_tensor_scale, rc->beta,
                                 rc->momentum_flags, rc->step);
    if (c != FP4ROOT_OK) return c;
  }
  if (!std::isfinite(rc->lr) || !std::isfinite(rc->wd)) return FP4ROOT_ERR_INVALID_ARG;
  int c = validate_config(ns);
  if (c != FP4ROOT_OK) return c;
  const std::vector<fp4root_matrix> mats = root_matrices(params, count);
  c = validate_matrices(mats.data(), count);
  if (c != FP4ROOT_OK) return c;
  const size_t need = fp4root_root_step_workspace(params, count, ns);
  if (need == 0) return FP4ROOT_ERR_INVALID_ARG;
  if (!ws || ws_bytes < need) return FP4ROOT_ERR_WORKSPACE;
  hipStream_t st = (hipStream_t)stream;
  // one status word for the whole step (the first word of the workspace, shared by
  // the stages, which run in stream order and reuse the rest of the workspace)
  uint32_t* status = reinterpret_cast<uint32_t*>(ws);
  if (count == 0) FP4R_TRY(launch_fill_u32(status, 0u, 1, st));
  Carver cv(ws);
  cv.take<uint32_t>(1);
  MatScalars* sc = cv.take<MatScalars>((size_t)std::min<int64_t>(count, kMaxRootChunk));
  const float b1 = rc->beta, b2 = 1.0f - b1;   // b2 = fl32(1 - beta)
  const uint32_t mf = rc->momentum_flags;
  const float lw = rc->lr * rc->wd, c1 = 1.0f - lw;
  RootChunk ch;
  for (int64_t i = 0; i < count; i += ch.count) {
    root_chunk(params, count, i, *rc, ch);
    FP4R_TRY(launch_init(i == 0 ? status : nullptr, sc, ch.count, nullptr, 0, st));
    FP4R_TRY(launch_root_momentum(ch, rc->step > 0, mf & FP4ROOT_F_HADAMARD, mf & FP4ROOT_F_ADAPTIVE46,
                                  mf & FP4ROOT_F_STOCHASTIC, b1, b2, sc, status, st));
  }
  const int rc2 = orthogonalize_launch(mats.data(), count, ns, ws, false, st);
  if (rc2 != FP4ROOT_OK) return rc2;
  for (int64_t i = 0; i < count; i += ch.count) {
    root_chunk(params, count, i, *rc, ch);
    FP4R_TRY(launch_root_apply(ch, c1, st));
  }
  return FP4ROOT_OK;
}

size_t fp4root_ns_step_workspace(int64_t batch, int64_t m, int64_t n, uint32_t flags) {
  if (batch < 0 || !dims_ok(m, n)) return 0;
  Carver cv(nullptr);
  cv.off = kAlign;
  StepWs w;
  carve_step(cv, batch, m, n, flags & FP4ROOT_F_BF16_PATH, w);
  return cv.off;
}

int fp4root_ns_step(float* x, int64_t batch, int64_t m, int64_t n, int64_t batch_stride, float a,
                    float b, float c, uint32_t flags, uint64_t seed, int32_t step,
                    const fp4root_ns_trace* trace, void* ws, size_t ws_bytes, void* stream) {
  if (batch < 0 || !x) return FP4ROOT_ERR_INVALID_ARG;
  if (flags & ~(uint32_t)(FP4ROOT_F_HADAMARD | FP4ROOT_F_ADAPTIVE46 | FP4ROOT_F_BF16_PATH | FP4ROOT_F_CLIP |
                          FP4ROOT_F_FP32_ACCUM))
    return FP4ROOT_ERR_INVALID_ARG;
  if ((flags & FP4ROOT_F_BF16_PATH) && (flags & FP4ROOT_F_FP32_ACCUM)) return FP4ROOT_ERR_INVALID_ARG;
  if (!std::isfinite(a) || !std::isfinite(b) || !std::isfinite(c)) return FP4ROOT_ERR_INVALID_ARG;
  if (!dims_ok(m, n)) return FP4ROOT_ERR_SHAPE;
  if ((batch > 1 && batch_stride < m * n) || batch_stride % 4) return FP4ROOT_ERR_SHAPE;
  if (!aligned(x, 16)) return FP4ROOT_ERR_INVALID_ARG;
  const bool bf16 = flags & FP4ROOT_F_BF16_PATH;
  if (bf16 && trace) return FP4ROOT_ERR_UNSUPPORTED;
  if (!ws || ws_bytes < fp4root_ns_step_workspace(batch, m, n, flags)) return FP4ROOT_ERR_WORKSPACE;
  if (batch == 0) return FP4ROOT_OK;
  hipStream_t st = (hipStream_t)stream;
  Carver cv(ws);
  uint32_t* status = cv.take<uint32_t>(1);
  StepWs w;
  carve_step(cv, batch, m, n, bf16, w);
  FP4R_TRY(launch_init(status, w.sc, batch, nullptr, 0, st));
  if (bf16) {
    if (batch_stride != m * n && batch > 1) return FP4ROOT_ERR_UNSUPPORTED;
    FP4R_TRY(launch_cast_bf16(x, batch, m, n, batch_stride, w.xb, st));
    return run_step_bf16(x, batch, m, n, batch_stride, a, b, c, w, st);
  }
  const StepGroup sg{x, batch, m, n, batch_stride, &w, a, b, c};
  return run_step_fp4(&sg, 1, flags, seed, step, 0, true, status, trace, st);
}

int fp4root_quantize_noalloc(const float* x, int64_t batch, int64_t rows, int64_t cols, int64_t ld,
                             int64_t batch_stride, int axis, uint32_t flags, float clip_quantile, uint64_t seed,
                             int32_t step, uint8_t* codes, uint8_t* scales, float* tensor_scale,
                             float* clip_threshold, int32_t* status, void* stream) {
  const int rc = check_quantize(x, batch, rows, cols, ld, batch_stride, axis, flags, clip_quantile, codes, scales,
                                tensor_scale);
  if (rc != FP4ROOT_OK) return rc;
  if (batch > ((flags & FP4ROOT_F_CLIP) ? kNoAllocMaxBatch : kNoAllocMaxPlain)) return FP4ROOT_ERR_WORKSPACE;
  hipStream_t st = (hipStream_t)stream;
  void* ws = nullptr;
  const int rs = scratch_address(&ws);
  if (rs != FP4ROOT_OK) return rs;
  if (batch > 0)
    FP4R_TRY_RC(quantize_launch(x, batch, rows, cols, ld, batch_stride, axis, flags, clip_quantile, seed, step,
                                codes, scales, tensor_scale, clip_threshold, ws, false, st));
  else
    FP4R_TRY(launch_fill_u32(reinterpret_cast<uint32_t*>(ws), 0u, 1, st));
  // the status word is the scratch's first word (see quantize_launch)
  if (status) FP4R_TRY(launch_status_out(reinterpret_cast<const uint32_t*>(ws), status, st));
  return FP4ROOT_OK;
}

size_t fp4root_orthogonalize_workspace(const fp4root_matrix* mats, int64_t count,
                                       const fp4root_ns_config* cfg) {
  if (validate_config(cfg) != FP4ROOT_OK || count < 0 || (count > 0 && !mats)) return 0;
  for (int64_t i = 0; i < count; ++i)
    if (!dims_ok(mats[i].rows, mats[i].cols)) return 0;
  return orthogonalize_ws_size(mats, count, cfg);
}

namespace {
// The launches of fp4root_orthogonalize (arguments and workspace already checked);
// the status word is cleared first only when reset_status is set.
int orthogonalize_launch(const fp4root_matrix* mats, int64_t count, const fp4root_ns_config* cfg, void* ws,
                         bool reset_status, hipStream_t st) {
  const bool bf16 = cfg->flags & FP4ROOT_F_BF16_PATH;
  const bool clip = cfg->flags & FP4ROOT_F_CLIP;
  uint32_t* status = reinterpret_cast<uint32_t*>(ws);
  if (count == 0) return reset_status && launch_fill_u32(status, 0u, 1, st) != hipSuccess ? FP4ROOT_ERR_HIP : FP4ROOT_OK;
  const std::vector<Group> groups = make_groups(mats, count);
  const size_t ng = groups.size();

  // per group: descriptors, workspace, coefficients, output route
  std::vector<GroupWs> gw(ng);
  std::vector<std::vector<MatRef>> gall(ng);
  std::vector<std::vector<float>> gco(ng);
  std::vector<std::vector<MatChunk>> gout(ng);   // chunks of the last update's outputs
  Carver shared(ws);   // NVFP4: every group's workspace side by side
  shared.off = kAlign;
  auto prepare = [&](size_t gi) -> int {
    const Group& gr = groups[gi];
    const int64_t B = (int64_t)gr.members.size(), m = gr.m, n = gr.n;
    GroupWs& w = gw[gi];
    std::vector<MatRef>& all = gall[gi];
    all.resize((size_t)B);
    for (int64_t i = 0; i < B; ++i) {
      const fp4root_matrix& a = mats[gr.members[(size_t)i]];
      all[(size_t)i] = MatRef{a.in, a.out, (uint32_t)(a.ld_in / 4),
                              (uint32_t)(a.ld_out / 4) | (a.rows > a.cols ? 0x80000000u : 0u)};
    }
    int64_t lo = 0;
    double frac = 0.0;
    if (clip) quantile_index(m * n, cfg->clip_quantile, lo, frac);
    FP4R_TRY(launch_init(reset_status && gi == 0 ? status : nullptr, w.step.sc, B, w.hist,
                         clip ? (int64_t)chunk_hist_words(B, m * n) : 0, st));
    // the last update is written straight to the callers' matrices
    if (!bf16 && cfg->steps > 0)
      for (size_t c0 = 0; c0 < all.size(); c0 += kMaxChunk)
        gout[gi].push_back(make_chunk(all, c0, std::min(all.size() - c0, (size_t)kMaxChunk), m, n, lo, frac));
    std::vector<float>& co = gco[gi];
    co.assign((size_t)std::max(cfg->steps, 1) * 3, 0.0f);
    if (cfg->coeffs)
      std::memcpy(co.data(), cfg->coeffs, sizeof(float) * 3 * (size_t)cfg->steps);
    else
      default_coeffs_impl(m, n, cfg->steps, co.data());
    return FP4ROOT_OK;
  };
  // clip, normalise, orient: with clipping, the passes also yield the norm of the clipped
  // matrix; they collect elements in X, which the copy overwrites.  Small groups share launches.
  ClipSets sets;
  int64_t set_elems = 0;
  const uint32_t mask0 = sign_mask(cfg->seed, 0);
  const bool rot = cfg->flags & FP4ROOT_F_HADAMARD;
  auto flush_sets = [&]() -> int {
    const hipError_t e = sets.count ? launch_clip_prep(sets, status, cfg->eps, mask0, rot, kSlotXn, kSlotXm, st) : hipSuccess;
    sets.count = 0;
    sets.mats = 0;
    set_elems = 0;
    return e == hipSuccess ? FP4ROOT_OK : FP4ROOT_ERR_HIP;
  };
  auto copy_in = [&](size_t gi) -> int {
    const int64_t m = groups[gi].m, n = groups[gi].n;
    const GroupWs& w = gw[gi];
    const std::vector<MatRef>& all = gall[gi];
    int64_t lo = 0;
    double frac = 0.0;
    if (clip) quantile_index(m * n, cfg->clip_quantile, lo, frac);
    for (size_t c0 = 0; c0 < all.size(); c0 += kMaxChunk) {
      const size_t cnt = std::min(all.size() - c0, (size_t)kMaxChunk);
      const MatChunk ch = make_chunk(all, c0, cnt, m, n, lo, frac);
      float* const X = w.X + (int64_t)c0 * m * n;
      if (clip) {
        ClipScratch cs;
        cs.hist = w.hist;
        cs.cand = X;
        cs.cand_stride = m * n;
        cs.cnt = w.cand_cnt;
        cs.psum = w.partial;
        cs.pcnt = w.partial_cnt;
        const int64_t elems = (int64_t)all.size() * m * n;
        if (!bf16 && ng > 1 && all.size() <= (size_t)kMaxClipSetMats && elems <= kClipSetElems) {
          if (sets.count == kMaxClipSets || sets.mats + cnt > (size_t)kMaxClipSetMats ||
              set_elems + elems > kClipSetElems)
            FP4R_TRY_RC(flush_sets());
          clip_set(sets, ch, w.step.sc, X, cs);
          set_elems += elems;
          continue;
        }
        FP4R_TRY(launch_clip_threshold(ch, w.step.sc + c0, status, cs, cfg->eps, st));
      } else {
        FP4R_TRY(launch_inv_norm(ch, w.step.sc + c0, w.partial, cfg->eps, status, st));
      }
      FP4R_TRY(launch_prep_copy(ch, w.step.sc + c0, X, m * n, mask0, rot, kSlotXn, kSlotXm, st));
    }
    return FP4ROOT_OK;
  };
  // without an update product that writes the outputs (no steps, or the BF16 path)
  auto write_back = [&](size_t gi) -> int {
    const Group& gr = groups[gi];
    if (!gout[gi].empty()) return FP4ROOT_OK;
    for (size_t c0 = 0; c0 < gall[gi].size(); c0 += kMaxChunk) {
      const size_t cnt = std::min(gall[gi].size() - c0, (size_t)kMaxChunk);
      const MatChunk ch = make_chunk(gall[gi], c0, cnt, gr.m, gr.n, 0, 0.0);
      FP4R_TRY(launch_copy_out(ch, gw[gi].X + (int64_t)c0 * gr.m * gr.n, gr.m * gr.n, st));
    }
    return FP4ROOT_OK;
  };

  if (bf16) {
    // one group after another in the same workspace
    for (size_t gi = 0; gi < ng; ++gi) {
      const Group& gr = groups[gi];
      const int64_t B = (int64_t)gr.members.size(), m = gr.m, n = gr.n;
      Carver cv(ws);
      cv.off = kAlign;
      carve_group(cv, gr, bf16, gw[gi]);
      int rc = prepare(gi);
      if (rc == FP4ROOT_OK) rc = copy_in(gi);
      if (rc != FP4ROOT_OK) return rc;
      if (cfg->steps > 0) FP4R_TRY(launch_cast_bf16(gw[gi].X, B, m, n, m * n, gw[gi].step.xb, st));
      for (int32_t k = 0; k < cfg->steps; ++k) {
        const float* c3 = &gco[gi][3 * (size_t)k];
        rc = run_step_bf16(gw[gi].X, B, m, n, m * n, c3[0], c3[1], c3[2], gw[gi].step, st);
        if (rc != FP4ROOT_OK) return rc;
      }
      rc = write_back(gi);
      if (rc != FP4ROOT_OK) return rc;
    }
    return FP4ROOT_OK;
  }

  // NVFP4: every group prepared, then each NS step over all groups at once
  for (size_t gi = 0; gi < ng; ++gi) {
    carve_group(shared, groups[gi], false, gw[gi]);
    int rc = prepare(gi);
    if (rc == FP4ROOT_OK) rc = copy_in(gi);
    if (rc != FP4ROOT_OK) return rc;
  }
  FP4R_TRY_RC(flush_sets());
  std::vector<StepGroup> sgs(ng);
  for (int32_t k = 0; k < cfg->steps; ++k) {
    for (size_t gi = 0; gi < ng; ++gi) {
      const Group& gr = groups[gi];
      const float* c3 = &gco[gi][3 * (size_t)k];
      sgs[gi] = StepGroup{gw[gi].X, (int64_t)gr.members.size(), gr.m, gr.n, gr.m * gr.n, &gw[gi].step,
                          c3[0], c3[1], c3[2], k == cfg->steps - 1 ? &gout[gi] : nullptr};
    }
    const int rc = run_step_fp4(sgs.data(), (int)ng, cfg->flags, cfg->seed, k, 2 * (k & 1), false, status,
                                nullptr, st);
    if (rc != FP4ROOT_OK) return rc;
  }
  for (size_t gi = 0; gi < ng; ++gi) {
    const int rc = write_back(gi);
    if (rc != FP4ROOT_OK) return rc;
  }
  return FP4ROOT_OK;
}
}  // namespace

int fp4root_orthogonalize(const fp4root_matrix* mats, int64_t count, const fp4root_ns_config* cfg,
                          void* ws, size_t ws_bytes, void* stream) {
  int rc = validate_config(cfg);
  if (rc != FP4ROOT_OK) return rc;
  rc = validate_matrices(mats, count);
  if (rc != FP4ROOT_OK) return rc;
  if (!ws || ws_bytes < orthogonalize_ws_size(mats, count, cfg)) return FP4ROOT_ERR_WORKSPACE;
  return orthogonalize_launch(mats, count, cfg, ws, true, (hipStream_t)stream);
}

}  // extern "C"
