// C ABI of libstreambp and the host-side chunk loops (paper Sec. 3.2.1, 3.2.2).
// Host code only validates, carves the caller's workspace and enqueues kernels
// on the caller's stream; it never allocates or synchronises.
#include "../../include/streambp.h"
#include "launch.h"

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#ifdef __SANITIZE_ADDRESS__
#include <sanitizer/asan_interface.h>
#endif

using namespace sbp;

namespace {

thread_local char g_err[512] = "";

int32_t fail(int32_t code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

#define HIPCHK(expr)                                                                       \
  do {                                                                                     \
    hipError_t e__ = (expr);                                                               \
    if (e__ != hipSuccess)                                                                 \
      return fail(SBP_ERR_HIP, "%s failed: %s (%s:%d)", #expr, hipGetErrorString(e__), __FILE__, __LINE__); \
  } while (0)

// Bump allocator over the caller's workspace (256-byte granularity).  In a host build under the address sanitizer the bytes between two
// carved buffers, and a gap added for that, are out of bounds.
struct Carver {
  char* base; size_t off = 0;
  explicit Carver(void* p) : base((char*)p) {}
  template <typename T> T* take(size_t n_elems) { return (T*)take_bytes(n_elems * sizeof(T)); }
  void* take_bytes(size_t bytes) {
    void* p = base ? base + off : nullptr;
    off += align_up(bytes, 256);
#ifdef __SANITIZE_ADDRESS__
    off += 256;
    if (base) {
      ASAN_UNPOISON_MEMORY_REGION(p, bytes);
      ASAN_POISON_MEMORY_REGION((char*)p + bytes, (size_t)(base + off - (char*)p) - bytes);
    }
#endif
    return p;
  }
};

// fp32 buffers that one fill clears: a region of its own, so that nothing else can come to lie between them.
struct Cleared { void* p = nullptr; size_t bytes = 0; };
struct ClearedCarver {
  Carver& cv; Cleared r;
  explicit ClearedCarver(Carver& c) : cv(c) { r.p = c.base ? c.base + c.off : nullptr; }
  float* take(size_t n) {
    float* p = (float*)(r.p ? (char*)r.p + r.bytes : nullptr);
    r.bytes += align_up(n * sizeof(float), 256);
    return p;
  }
  Cleared close() {
    cv.take_bytes(r.bytes);
    return r;
  }
};

bool valid_dtype(int32_t dt) { return dt == SBP_F32 || dt == SBP_BF16; }
// weight gradients: fp32, or bf16 next to bf16 weights
int32_t check_grad_dtype(int32_t dt, int32_t grad_dt) {
  if (!valid_dtype(grad_dt)) return fail(SBP_ERR_UNSUPPORTED, "grad_dtype %d not supported", grad_dt);
  if (grad_dt == SBP_BF16 && dt != SBP_BF16) return fail(SBP_ERR_UNSUPPORTED, "bf16 gradients need dtype == SBP_BF16");
  return SBP_OK;
}

// Weight gradients are added once per group (one read-modify-write pass over every dW per group instead of one per chunk), at most MAX_DW_GROUP chunks
// or passes (the GEMM kernels take up to eight reduction segments per output), the operands of which stay alive until the launch.  Head: as many chunks
// as it takes to reach dw_group_rows rows.  Layer: that group sets the bytes, and how often bf16 gradients may be rounded; how many passes share a launch
// is plan_layer's.
constexpr int MAX_DW_GROUP = 8;
// Defaults (dw_group_rows == 0).  Measured at 7B widths, chunk 2048: the head's dW pass (2.2 GB read-modify-written) still
// gains from eight chunks per pass over four; the layer's seven dW (0.93 GB) do not, so the layer has room for four.
constexpr int DW_GROUP_ROWS_LAYER = 8192;
constexpr int DW_GROUP_ROWS_HEAD = 16384;
int dw_group_for(size_t chunk_rows, int32_t cfg_rows, int default_rows) {   // cfg_rows: the config's dw_group_rows (0 = default)
  const size_t rows = cfg_rows > 0 ? (size_t)cfg_rows : (size_t)default_rows;
  return (int)std::max<size_t>(1, std::min<size_t>(MAX_DW_GROUP, rows / std::max<size_t>(chunk_rows, 1)));
}

// ------------------------------------------------------------- layer ------
// A pass of the chunk loop works on `rows` rows of a sequence, or on `seqs` whole sequences (then rows = seq_len), the rows of which are one
// behind the other; `sets` passes share a weight-gradient launch.
struct LayerPlan { int seqs, rows, sets; };
struct LayerWs {
  void *K, *V;                 // [seqs, T, Hkv*dh] dt   cached for the whole sequence(s)
  float *dK, *dV;              // [seqs, T, Hkv*dh] fp32 prefix accumulators
  Cleared kv_grads;            // both
  float2* rope;                // [T, dh/2] cos/sin
  // Rows of a pass, dt.  a, o, m, gate, up, act, dh1_t, dq, dkc and dvc are the operands of its weight-gradient GEMMs; act holds dact before
  // the SwiGLU adjoint replaces it.
  void *q, *d_o;
  void *a, *o, *m, *gate, *up, *act, *dh1_t, *dq, *dkc, *dvc;
  // fp32 [rows, d].  f0: output projection, then h1 (the sum of the attention side, in place), at the end da; f1: dm, then dh1 (in place); the
  // plain forward's down projection
  float *f0, *f1;
  float *rstd1, *rstd2, *lse, *delta;
  float* partial[MAX_DW_GROUP][2];      // rows that the norm gains' gradients are the column sums of, per pass of a weight-gradient group: g1, g2
  float* gemm_scratch; size_t gemm_scratch_bytes;
  // Further copies of the operands of the weight-gradient GEMMs: a pass's operands stay alive while the next passes of its group run.
  LayerPlan plan;
  void* alt[MAX_DW_GROUP - 1][10];
  size_t bytes;
};
// The workspace view a pass uses: set 0 = the primary operand buffers, sets 1.. the further copies.
LayerWs pass_view(const LayerWs& s, int set) {
  LayerWs v = s;
  if (set > 0) {
    void** ptrs[10] = {&v.a, &v.o, &v.m, &v.gate, &v.up, &v.act, &v.dh1_t, &v.dq, &v.dkc, &v.dvc};
    for (int i = 0; i < 10; ++i) *ptrs[i] = s.alt[set - 1][i];
  }
  return v;
}

int32_t check_layer_cfg(const sbp_layer_cfg* c) {
  if (!c) return fail(SBP_ERR_NULL, "cfg is NULL");
  if (!valid_dtype(c->dtype)) return fail(SBP_ERR_UNSUPPORTED, "dtype %d not supported", c->dtype);
  if (int32_t rc = check_grad_dtype(c->dtype, c->grad_dtype)) return rc;
  if (c->dw_group_rows < 0) return fail(SBP_ERR_SHAPE, "dw_group_rows must be >= 0");
  if (c->batch < 1 || c->seq_len < 1 || c->chunk < 1) return fail(SBP_ERR_SHAPE, "batch, seq_len and chunk must be >= 1");
  if (c->hidden < 1 || c->mlp_width < 1) return fail(SBP_ERR_SHAPE, "hidden and mlp_width must be >= 1");
  if (c->n_q_heads < 1 || c->n_kv_heads < 1 || c->n_q_heads % c->n_kv_heads != 0)
    return fail(SBP_ERR_SHAPE, "n_q_heads (%d) must be a positive multiple of n_kv_heads (%d)", c->n_q_heads, c->n_kv_heads);
  if (c->head_dim < 2 || (c->head_dim & 1) || c->head_dim > 256)
    return fail(SBP_ERR_SHAPE, "head_dim must be even and in [2, 256]");
  if (!(c->rms_eps >= 0.f) || !(c->rope_theta > 0.f)) return fail(SBP_ERR_SHAPE, "rms_eps must be >= 0 and rope_theta > 0");
  if (c->window < 0) return fail(SBP_ERR_SHAPE, "window must be >= 0");
  if (c->seq_first)
    for (int b = 0; b < c->batch; ++b)
      if (c->seq_first[b] < 0 || c->seq_first[b] > c->seq_len)
        return fail(SBP_ERR_SHAPE, "seq_first[%d] = %d is outside [0, seq_len]", b, c->seq_first[b]);
  return SBP_OK;
}

// The workspace a layer call asks for: K, V and their gradients, and what a chunk of `chunk` rows at a time needs with every intermediate in a buffer
// of its own and a copy of the ten operand buffers per chunk of a weight-gradient group.  The passes are planned inside these bytes (plan_layer).
size_t layer_budget(const sbp_layer_cfg* c) {
  const size_t es = dtype_size(c->dtype);
  const size_t T = c->seq_len, cm = (size_t)std::min(c->chunk, c->seq_len);
  const size_t d = c->hidden, F = c->mlp_width, qd = (size_t)c->n_q_heads * c->head_dim, kd = (size_t)c->n_kv_heads * c->head_dim;
  Carver cv(nullptr);
  for (int i = 0; i < 2; ++i) cv.take_bytes(T * kd * es);
  cv.take_bytes(2 * align_up(T * kd * sizeof(float), 256));
  cv.take<float2>(T * (c->head_dim / 2));
  const size_t operands[10] = {cm * d * es, cm * qd * es, cm * d * es, cm * F * es, cm * F * es, cm * F * es, cm * d * es, cm * qd * es, cm * kd * es, cm * kd * es};
  const int sets = dw_group_for(cm, c->dw_group_rows, DW_GROUP_ROWS_LAYER);
  for (int g = 0; g < sets; ++g) {
    for (int i = 0; i < 2; ++i) cv.take<float>(rmsnorm_bwd_partial_floats((int)cm, (int)d));
    for (size_t bytes : operands) cv.take_bytes(bytes);
  }
  for (size_t bytes : {cm * qd * es, cm * F * es, cm * qd * es}) cv.take_bytes(bytes);      // q, dact, do
  for (int i = 0; i < 5; ++i) cv.take<float>(cm * d);                                        // h1, dm, dh1, da, the output projection
  for (int i = 0; i < 2; ++i) cv.take<float>(cm);
  cv.take<float>(cm * c->n_q_heads);
  cv.take<float>(2 * cm * c->n_q_heads);
  cv.take_bytes(c->dtype == SBP_BF16 ? gemm_scratch_bytes((int)cm, (int)std::max(d, qd)) : 0);
  return cv.off;
}

// backward = false: the plain forward, which keeps no operands and no gradients
LayerWs carve_layer(const sbp_layer_cfg* c, void* ws, const LayerPlan& plan, bool backward) {
  const size_t es = dtype_size(c->dtype);
  const size_t T = (size_t)c->seq_len * plan.seqs, n = (size_t)plan.rows * plan.seqs;
  const size_t d = c->hidden, F = c->mlp_width, qd = (size_t)c->n_q_heads * c->head_dim, kd = (size_t)c->n_kv_heads * c->head_dim;
  Carver cv(ws);
  LayerWs w{};
  w.plan = plan;
  w.K = cv.take_bytes(T * kd * es);
  w.V = cv.take_bytes(T * kd * es);
  w.rope = cv.take<float2>((size_t)c->seq_len * (c->head_dim / 2));
  w.q = cv.take_bytes(n * qd * es);
  w.a = cv.take_bytes(n * d * es);
  w.o = cv.take_bytes(n * qd * es);
  w.m = cv.take_bytes(n * d * es);
  w.gate = cv.take_bytes(n * F * es);
  w.up = cv.take_bytes(n * F * es);
  w.act = cv.take_bytes(n * F * es);
  w.f0 = cv.take<float>(n * d);
  w.f1 = cv.take<float>(n * d);
  w.rstd1 = cv.take<float>(n);
  w.rstd2 = cv.take<float>(n);
  w.lse = cv.take<float>(n * c->n_q_heads);
  // (a chunk's worth, as the call's bytes have it: a partial tile per CU from chunks of 256 rows at widths of 2560 on.  Smaller ones leave room for fewer - 64
  // for 64 rows at 7B widths, 27 for 256 rows at 256 - so that the products of their passes split less, and share no last round)
  w.gemm_scratch_bytes = c->dtype == SBP_BF16 ? gemm_scratch_bytes((int)std::min(n, (size_t)std::min(c->chunk, c->seq_len)), (int)std::max(d, qd)) : 0;
  w.gemm_scratch = (float*)cv.take_bytes(w.gemm_scratch_bytes);
  if (backward) {
    ClearedCarver grads(cv);
    w.dK = grads.take(T * kd);
    w.dV = grads.take(T * kd);
    w.kv_grads = grads.close();
    w.d_o = cv.take_bytes(n * qd * es);
    w.dh1_t = cv.take_bytes(n * d * es);
    w.dq = cv.take_bytes(n * qd * es);
    w.dkc = cv.take_bytes(n * kd * es);
    w.dvc = cv.take_bytes(n * kd * es);
    w.delta = cv.take<float>(2 * n * c->n_q_heads);
    const size_t sizes[10] = {n * d * es, n * qd * es, n * d * es, n * F * es, n * F * es, n * F * es,
                              n * d * es, n * qd * es, n * kd * es, n * kd * es};   // a, o, m, gate, up, act, dh1_t, dq, dkc, dvc
    for (int g = 0; g < plan.sets; ++g)
      for (float*& p : w.partial[g]) p = cv.take<float>(rmsnorm_bwd_partial_floats((int)n, (int)d));
    for (int g = 1; g < plan.sets; ++g)
      for (int i = 0; i < 10; ++i) w.alt[g - 1][i] = cv.take_bytes(sizes[i]);
  }
  w.bytes = cv.off;
  return w;
}

// How the rows of a call are dealt to passes.  The paper's partition bounds the memory; inside those bytes fewer and larger passes are faster: every
// pass streams all weights and is some twenty dependent launches.  fits(plan): the plan's buffers are within the call's workspace.
//
// Candidates: for every number of sets, whole sequences, as many as fit, or, where not even one does, the longest stretch of a sequence; both evened
// out, and with up to two passes more, which may waste less of the last row of tiles.  Taken is the one with the least estimated time: a pass costs
// its launches, two readings of the weights and the products of its rows, rounded up to tiles; a weight-gradient launch a reading and a
// writing of the gradients.  `products`: multiples of 2 flops per weight and row.
//
// bf16 gradients are rounded once per weight-gradient launch (per pass where a launch cannot take several), so no plan makes more launches than groups of
// dw_group_rows rows, chunk by chunk, would, nor more passes than there are chunks.  Error of dW_gate against fp64 and time, chunk by chunk / with more launches where
// that is faster / with this bound: 8192 tokens at 4096 / 14336, chunk 1024, 4.529e-3 12.2 ms / 4.679e-3 10.9 / 4.529e-3 11.6; 32768 at 2048 / 5632, chunk 1024,
// 4.688e-3 39.3 / 5.240e-3 27.8 / 4.689e-3 29.1; 4 x 500 at 2048 / 5632, chunk 128, 4.450e-3 / 4.748e-3 / 4.450e-3.
//
// Measured, chunk by chunk as the config says / in planned passes of the same bytes: four sequences of 640 tokens at 7B widths, chunk 512, eight passes / one
// 5.47 -> 3.63 ms; 8192 tokens at 4096 / 14336, chunk 1024, bf16 gradients, eight / four 12.2 -> 11.6; 32768 at 7B widths, chunk 2048, sixteen / eight 70.9 -> 69.9; a
// 1024-wide stack of two layers, 2 x 1023 tokens, chunk 512, 3.27 -> 2.65.  SPAN_ROWS: 8192 rows a pass are slower again (8192 tokens at
// 4096 / 14336 11.85 ms, 32768 at 7B widths 71.7): the MLP's tensors, 230 to 310 MB each, no longer stay in the 256 MB cache from one product to the next.
constexpr int SPAN_ROWS = 4096;
constexpr int SPAN_SEQS = ATTN_MAX_SEQS;
template <typename Fits>
LayerPlan plan_layer(const sbp_layer_cfg* c, int max_sets, double products, bool dw, Fits fits) {
  const int T = c->seq_len, cm = std::min(c->chunk, T), rows_max = std::max(cm, SPAN_ROWS), grain = c->dtype == SBP_BF16 ? 256 : 32;
  const double d = c->hidden, qd = (double)c->n_q_heads * c->head_dim, kd = (double)c->n_kv_heads * c->head_dim;
  const double weights = 2.0 * d * qd + 2.0 * d * kd + 3.0 * d * c->mlp_width;
  const double row_us = 2.0 * products * weights / (c->dtype == SBP_BF16 ? 1.3e9 : 7e7);
  const double pass_us = 60.0 + weights * 2.0 * dtype_size(c->dtype) / 5e6, dw_us = dw ? weights * 2.0 * dtype_size(c->grad_dtype) / 5e6 : 0.0;
  auto largest = [&](int hi, auto ok) {      // largest n <= hi with ok(n), or 0
    int lo = 0;
    while (lo < hi) {
      const int mid = lo + (hi - lo + 1) / 2;
      if (ok(mid)) lo = mid; else hi = mid - 1;
    }
    return lo;
  };
  const bool rounds = dw && c->grad_dtype == SBP_BF16;
  const int group = dw ? dw_group_for((size_t)cm, c->dw_group_rows, DW_GROUP_ROWS_LAYER) : 1;
  const int64_t most_passes = c->batch * cdiv(T, cm), most_launches = cdiv(most_passes, group);      // of a plan that `rounds`
  LayerPlan best{1, cm, group};      // (chunk by chunk: what the bytes are made for)
  double best_us = -1.0;
  for (int sets = 1; sets <= max_sets; ++sets) {
    const int seqs = T > rows_max ? 0 : largest(std::min(std::min(c->batch, SPAN_SEQS), rows_max / T), [&](int n) { return fits(LayerPlan{n, T, sets}); });
    const int rows = seqs > 0 ? T : largest(std::min(T, rows_max), [&](int n) { return fits(LayerPlan{1, n, sets}); });
    if (rows < 1) break;                                 // (more sets need more)
    const int64_t least = seqs > 0 ? cdiv(c->batch, seqs) : cdiv(T, rows);
    for (int64_t parts = least; parts <= least + 2; ++parts) {
      LayerPlan p{1, rows, sets};
      int64_t passes, tiles;                             // tiles: rows of all passes, in units of `grain`
      if (seqs > 0) {
        p.seqs = (int)cdiv(c->batch, parts);
        passes = cdiv(c->batch, p.seqs);
        tiles = (passes - 1) * cdiv((int64_t)p.seqs * T, grain) + cdiv((c->batch - (passes - 1) * p.seqs) * T, grain);
      } else {
        const int even = (int)cdiv(T, parts), up = (int)align_up((size_t)even, (size_t)grain);
        p.rows = up <= rows ? up : even;
        passes = cdiv(T, p.rows);
        tiles = ((passes - 1) * cdiv(p.rows, grain) + cdiv(T - (passes - 1) * p.rows, grain)) * c->batch;
        passes *= c->batch;
      }
      if (sets > 1 && sets > passes) continue;
      if (rounds && (passes > most_passes || cdiv(passes, sets) > most_launches)) continue;
      const double us = (double)passes * pass_us + (double)(tiles * grain) * row_us + (double)cdiv(passes, sets) * dw_us;
      if (best_us < 0.0 || us < best_us) { best = p; best_us = us; }
    }
  }
  return best;
}
LayerPlan plan_backward(const sbp_layer_cfg* c) {
  const size_t budget = layer_budget(c);
  return plan_layer(c, MAX_DW_GROUP, 3.0, true, [&](const LayerPlan& p) { return carve_layer(c, nullptr, p, true).bytes <= budget; });
}
LayerPlan plan_forward(const sbp_layer_cfg* c) {
  const size_t budget = layer_budget(c);
  return plan_layer(c, 1, 1.0, false, [&](const LayerPlan& p) { return carve_layer(c, nullptr, p, false).bytes <= budget; });
}

// split-K scratch of the entry point currently running on this host thread
thread_local float* t_gemm_scratch = nullptr;
thread_local size_t t_gemm_scratch_bytes = 0;

GemmArgs mk(const void* A, const void* B, void* C, int M, int N, int K, int64_t lda, int64_t ldb, int64_t ldc,
            bool ta, bool tb, int in_dt, int out_dt, bool acc) {
  GemmArgs g{A, B, C, M, N, K, lda, ldb, ldc, ta, tb, in_dt, out_dt, acc};
  g.scratch = t_gemm_scratch;
  g.scratch_bytes = t_gemm_scratch_bytes;
  g.few_ok = true;
  return g;
}
// Y[M,N] = X[M,K] W[N,K]^T
GemmArgs fwd_gemm(const void* X, const void* W, void* Y, int M, int N, int K, int dt, int out_dt) {
  return mk(X, W, Y, M, N, K, K, K, N, false, true, dt, out_dt, false);
}
// RoPE of K in the store of its product: fp32 products, heads that divide the kernel's tiles.  False: a pass over K is left to do.
bool rope_in_store(GemmArgs& g, const float2* table, int period, int dh) {
  if (g.in_dt != DT_F32 || dh % 2 != 0 || GEMM_ROPE_COLS % dh != 0) return false;
  g.rope = table; g.rope_dim = dh; g.rope_period = period;
  return true;
}
// dX[M,K] (=|+=) dY[M,N] W[N,K]
GemmArgs dx_gemm(const void* dY, const void* W, void* dX, int M, int N, int K, int dt, int out_dt, bool acc) {
  return mk(dY, W, dX, M, K, N, N, K, K, false, false, dt, out_dt, acc);
}
// dW[N,K] += dY[M,N]^T X[M,K]
GemmArgs dw_gemm(const void* dY, const void* X, void* dW, int M, int N, int K, int dt, int grad_dt) {
  return mk(dY, X, dW, N, K, M, N, K, K, true, false, dt, grad_dt, true);
}

const char* at(const void* p, size_t row, size_t width, size_t es) { return (const char*)p + row * width * es; }
char* at(void* p, size_t row, size_t width, size_t es) { return (char*)p + row * width * es; }

int32_t check_layer_ptrs(const sbp_layer_weights* w) {
  if (!w) return fail(SBP_ERR_NULL, "weights table is NULL");
  const void* ps[] = {w->wq, w->wk, w->wv, w->wo, w->wgate, w->wup, w->wdown, w->g1, w->g2};
  for (const void* p : ps) if (!p) return fail(SBP_ERR_NULL, "a weight pointer is NULL");
  return SBP_OK;
}

// The rows of one pass: n rows from r0 on of sequence b0, or (r0 = 0, n = T) the sequences b0 .. b0 + seqs - 1
struct Pass { int b0, seqs, r0, n; bool whole; };      // whole: all rows of its sequences
int64_t pass_rows(const Pass& p) { return (int64_t)p.seqs * p.n; }

// K and V of the pass's sequences, once (cached for all passes over them).  Where a pass takes whole sequences it does so itself, from
// the rows normalised for q (chunk_reforward).  Else row blocks as large as the operand buffers that the coming pass will fill allow (gate, up,
// act are contiguous: 3 n F elements hold the normalised rows of 3 n F / d positions), so that the two projections are GEMMs with enough output
// tiles to fill the chip on their own; nothing proportional to T is added to the workspace.
int32_t kv_prepass(const sbp_layer_cfg* c, const sbp_layer_weights* w, const LayerWs& s, const char* xb, hipStream_t st) {
  const int dt = c->dtype;
  const size_t es = dtype_size(dt);
  const int T = c->seq_len, d = c->hidden;
  const int kd = c->n_kv_heads * c->head_dim;
  void* a_rows = s.a;
  int block = s.plan.rows;
  const size_t idle_rows = (size_t)((const char*)s.act + (size_t)s.plan.rows * c->mlp_width * es - (const char*)s.gate) / ((size_t)d * es);
  if (idle_rows > (size_t)block) {
    a_rows = s.gate;
    block = (int)std::min<size_t>((size_t)T, idle_rows);
  }
  for (int r0 = 0; r0 < T; r0 += block) {
    const int n = std::min(block, T - r0);
    HIPCHK(rmsnorm_fwd(dt, at(xb, r0, d, es), nullptr, w->g1, a_rows, nullptr, nullptr, n, d, c->rms_eps, st));
    GemmArgs kv[2] = {fwd_gemm(a_rows, w->wk, at(s.K, r0, kd, es), n, kd, d, dt, dt),
                      fwd_gemm(a_rows, w->wv, at(s.V, r0, kd, es), n, kd, d, dt, dt)};
    const bool rotated = rope_in_store(kv[0], s.rope + (size_t)r0 * (c->head_dim / 2), n, c->head_dim);
    HIPCHK(gemm_batch(kv, 2, st));
    if (!rotated) HIPCHK(rope_apply(dt, at(s.K, r0, kd, es), s.rope + (size_t)r0 * (c->head_dim / 2), n, n, c->n_kv_heads, c->head_dim, false, st));
  }
  return SBP_OK;
}

// The attention call of a pass; backward adds its own tensors
AttnArgs pass_attn(const sbp_layer_cfg* c, const LayerWs& s, const Pass& p) {
  AttnArgs aa{};
  aa.dt = c->dtype; aa.Hq = c->n_q_heads; aa.Hkv = c->n_kv_heads; aa.dh = c->head_dim;
  aa.batch = p.seqs; aa.q_start = p.r0; aa.q_len = p.n; aa.scale = 1.0f / std::sqrt((float)c->head_dim);
  aa.window = c->window; aa.kv_first = c->seq_first ? *std::min_element(c->seq_first + p.b0, c->seq_first + p.b0 + p.seqs) : 0;      // rows before it are padding in front of the sequence
  aa.kv_firsts = c->seq_first && p.seqs > 1 ? c->seq_first + p.b0 : nullptr;
  aa.q = s.q; aa.k = s.K; aa.v = s.V; aa.o = s.o; aa.lse = s.lse;
  if (fusion_mask() & FUSE_ROPE_Q) aa.rope_q = s.rope + (size_t)p.r0 * (c->head_dim / 2);
  return aa;
}

// Partitioned reforward of a pass's rows: fills a, q, o, lse, f0 = h1, m, gate, up (with_act = false: the backward, which gets act from swiglu_bwd), and
// K and V where the pass takes whole sequences.
// with_act = true (the plain forward): fills act, and gate and up only where the gated store does not take the products.
int32_t chunk_reforward(const sbp_layer_cfg* c, const sbp_layer_weights* w, const LayerWs& s, const char* xc, const Pass& p, bool with_act, hipStream_t st) {
  const int dt = c->dtype;
  const int d = c->hidden, F = c->mlp_width, qd = c->n_q_heads * c->head_dim, kd = c->n_kv_heads * c->head_dim;
  const int n = (int)pass_rows(p);
  HIPCHK(rmsnorm_fwd(dt, xc, nullptr, w->g1, s.a, nullptr, s.rstd1, n, d, c->rms_eps, st));
  GemmArgs qkv[3] = {fwd_gemm(s.a, w->wq, s.q, n, qd, d, dt, dt), fwd_gemm(s.a, w->wk, s.K, n, kd, d, dt, dt), fwd_gemm(s.a, w->wv, s.V, n, kd, d, dt, dt)};
  // q with K and V in one launch, as a grouped one or on the kernels for few tiles.  Whole layer, q apart / in one: 64 rows at 7B widths 923 -> 895 us
  // (forward 213 -> 192), 300 rows 1181 -> 1167 (320 -> 303), 640 at 4096 / 14336 1448 -> 1428 (412 -> 385), 1023 at 2048 / 5632 581 -> 574
  // (175 -> 167), 1023 at 1024 / 2816 283 -> 278 (104 -> 100), 2560 at 7B widths 3330 -> 3279; 900 rows at 4096 / 14336 and 7B widths the same.
  const bool rotated = p.whole && rope_in_store(qkv[1], s.rope, p.n, c->head_dim);
  HIPCHK(gemm_batch(qkv, p.whole ? 3 : 1, st));
  if (p.whole && !rotated) {
    HIPCHK(rope_apply(dt, s.K, s.rope, n, p.n, c->n_kv_heads, c->head_dim, false, st));
  }
  const AttnArgs aa = pass_attn(c, s, p);      // with RoPE(q) inside the kernel, which leaves s.q rotated
  if (!aa.rope_q) HIPCHK(rope_apply(dt, s.q, s.rope + (size_t)p.r0 * (c->head_dim / 2), n, p.n, c->n_q_heads, c->head_dim, false, st));
  HIPCHK(attn_forward(aa, st));
  HIPCHK(gemm(fwd_gemm(s.o, w->wo, s.f0, n, d, qd, dt, DT_F32), st));
  HIPCHK(rmsnorm_fwd(dt, xc, s.f0, w->g2, s.m, s.f0, s.rstd2, n, d, c->rms_eps, st));
  if (with_act) {      // the forward needs neither gate nor up: one product of both whose store applies the gate
    GemmArgs ga = fwd_gemm(s.m, w->wgate, s.act, n, F, d, dt, dt);
    ga.glu_up = w->wup;
    if (gemm_glu_supported(ga)) {
      HIPCHK(gemm(ga, st));
      return SBP_OK;
    }
  }
  {
    const GemmArgs gu[2] = {fwd_gemm(s.m, w->wgate, s.gate, n, F, d, dt, dt), fwd_gemm(s.m, w->wup, s.up, n, F, d, dt, dt)};
    HIPCHK(gemm_batch(gu, 2, st));
  }
  if (with_act) HIPCHK(swiglu_fwd(dt, s.gate, s.up, s.act, (int64_t)n * F, st));
  return SBP_OK;
}

}  // namespace

extern "C" {

const char* streambp_version(void) { return "streambp-mi355x 0.1 (gfx950)"; }
const char* streambp_last_error(void) { return g_err; }

size_t streambp_layer_workspace_bytes(const sbp_layer_cfg* cfg) {
  if (check_layer_cfg(cfg) != SBP_OK) return 0;
  return layer_budget(cfg);
}

// Low-rank adapter mode of the layer backward (App. D, experiment setup: rank-32 adapters, adapter gradients only).
// The chunk loop runs on the effective matrices W + s B A (built once per call); instead of the seven weight gradients
// of a chunk it forms, per adapted matrix, P = X A^T, Q = dY B (chunk x rank, the rank rounded up to a multiple of 8) and
// accumulates dB += dY^T P, dA += Q^T X - the chain rule through B A without ever forming dW.
constexpr int LORA_MAX_RANK = 256;
struct LoraCtx {
  int n;                           // adapted matrices
  int pad;                         // adapter rank rounded up to a multiple of 8 (the GEMMs' 16-byte granule); the
                                   // MFMA GEMMs take such widths with a masked ragged tile
  int which[7];                    // index into the order wq, wk, wv, wo, wgate, wup, wdown
  int out_dim[7], in_dim[7];
  void *a_pad[7], *b_pad[7];       // [pad, in], [out, pad] in the storage type, zero beyond the rank
  float *da_pad[7], *db_pad[7];    // fp32 accumulators of the same shapes
  Cleared grads;                   // all of them
  void *P[7], *Q[7];               // [chunk, pad] per adapted matrix
};
} // extern "C"

namespace {
int32_t layer_backward_impl(const sbp_layer_cfg* c, const sbp_layer_weights* w, const void* x, const void* dy, void* dx,
                            const sbp_layer_grads* g, const LoraCtx* lora, const LayerWs& s_all, hipStream_t st) {
  int32_t rc;
  t_gemm_scratch = s_all.gemm_scratch; t_gemm_scratch_bytes = s_all.gemm_scratch_bytes;
  const int dt = c->dtype, gdt = c->grad_dtype;
  const size_t es = dtype_size(dt);
  const int T = c->seq_len, d = c->hidden, F = c->mlp_width;
  const int qd = c->n_q_heads * c->head_dim, kd = c->n_kv_heads * c->head_dim, half = c->head_dim / 2;
  const LayerPlan plan = s_all.plan;
  HIPCHK(rope_table(s_all.rope, T, c->head_dim, c->rope_theta, c->pos_offset, s_all.kv_grads.p, s_all.kv_grads.bytes, st));
  // Weight-gradient GEMMs waiting for their launch (a group of passes' worth).  A group may span sequences: short samples would
  // otherwise read and write every dW once each (four samples of 640 tokens at 7B widths: 2.3 of 8.8 ms).
  GemmArgs dws[7 * MAX_DW_GROUP];
  int n_dws = 0;
  ColumnSums gains{};          // of the same passes (adapter mode: the gains are frozen)
  if (!lora) { gains.dg[0] = g->g1; gains.dg[1] = g->g2; }
  for (int b0 = 0; b0 < c->batch; b0 += plan.seqs) {
    const int n_chunks = (int)cdiv(T, plan.rows), seqs = std::min(plan.seqs, c->batch - b0);
    if (n_chunks > 1 && (rc = kv_prepass(c, w, pass_view(s_all, n_dws / 7), at(x, (size_t)b0 * T, d, es), st))) return rc;
    if (b0 > 0) HIPCHK(fill_zero(s_all.kv_grads.p, s_all.kv_grads.bytes, st));      // (of the first: with the table)
    // Chunks run last to first: rows of dK/dV belonging to chunk i are final once
    // chunks >= i are done (later queries are the only other readers of those
    // keys), so the K/V-side gradient and dx of the chunk can be finished at once.
    for (int ci = n_chunks - 1; ci >= 0; --ci) {
      const Pass p{b0, seqs, ci * plan.rows, std::min(plan.rows, T - ci * plan.rows), n_chunks == 1};
      const int n = (int)pass_rows(p), set = n_dws / 7;
      const LayerWs s = pass_view(s_all, set);
      const size_t row0 = (size_t)b0 * T + p.r0;
      const char *xc = at(x, row0, d, es), *dyc = at(dy, row0, d, es);
      float *partial1 = lora ? nullptr : s_all.partial[set][0], *partial2 = lora ? nullptr : s_all.partial[set][1];
      if ((rc = chunk_reforward(c, w, s, xc, p, false, st))) return rc;
      // ---- MLP backward (the weight-gradient GEMMs of the chunk are deferred to one grouped launch below)
      {   // dact = dy W_d (in act), then the SwiGLU adjoint: gate <- dgate, up <- dup, act <- silu(gate) up.  The adjoint can run as
          // the GEMM's epilogue (dact is then never stored); measured slower than the elementwise pass, so off by default.
        GemmArgs gd = dx_gemm(dyc, w->wdown, s.act, n, d, F, dt, dt, false);
        if ((fusion_mask() & FUSE_SWIGLU) || !gemm_uses_mfma(gd)) {      // (the shape-agnostic kernel's launches are what it costs)
          gd.swiglu_gate = s.gate; gd.swiglu_up = s.up; gd.swiglu_act = s.act;
          HIPCHK(gemm(gd, st));
        } else {
          HIPCHK(gemm(gd, st));
          HIPCHK(swiglu_bwd(dt, s.gate, s.up, s.act, s.act, (int64_t)n * F, st));
        }
      }
      {   // dm = dgate W_g + dup W_u: two operand pairs, one launch
        GemmArgs gm = dx_gemm(s.gate, w->wgate, s.f1, n, F, d, dt, DT_F32, false);
        gm.A2 = s.up; gm.B2 = w->wup;
        HIPCHK(gemm(gm, st));
      }
      HIPCHK(rmsnorm_bwd(dt, s.f1, s.f0, true, w->g2, s.rstd2, dyc, false, s.f1, s.dh1_t, partial2, n, d, st));      // f1: dm -> dh1
      // ---- attention-side backward
      HIPCHK(gemm(dx_gemm(s.dh1_t, w->wo, s.d_o, n, d, qd, dt, dt, false), st));
      AttnArgs aa = pass_attn(c, s, p);            // (with rope_q dq leaves the kernel rotated back, RoPE's adjoint)
      aa.d_o = s.d_o; aa.dq = s.dq; aa.dk = s.dK; aa.dv = s.dV; aa.delta = s.delta;
      if (dt == DT_BF16) aa.dkv_slices = attn_dkv_slices(aa, s.gemm_scratch_bytes);
      if (aa.dkv_slices > 1) aa.dkv_scratch = s.gemm_scratch;                                   // (idle between GEMMs)
      // K/V side of the pass's rows: final now
      aa.dkc = s.dkc; aa.dvc = s.dvc; aa.rope_k = s.rope + (size_t)p.r0 * half;
      HIPCHK(attn_backward(aa, st));
      if (!aa.rope_q) HIPCHK(rope_apply(dt, s.dq, s.rope + (size_t)p.r0 * half, n, p.n, c->n_q_heads, c->head_dim, true, st));
      // the last pass of a weight-gradient group
      const bool group_done = !lora && (n_dws + 7 == 7 * plan.sets || (ci == 0 && b0 + seqs == c->batch));
      // da = dq W_q + dkc W_k + dvc W_v; fp32: with the weight gradients in one launch, where they are launched and it has room
      const GemmArgs qkv[3] = {dx_gemm(s.dq, w->wq, s.f0, n, qd, d, dt, DT_F32, false), dx_gemm(s.dkc, w->wk, s.f0, n, kd, d, dt, DT_F32, true),
                               dx_gemm(s.dvc, w->wv, s.f0, n, kd, d, dt, DT_F32, true)};
      const bool da_with_dw = group_done && dt == DT_F32 && n_dws + 10 <= 7 * MAX_DW_GROUP;
      if (!da_with_dw) HIPCHK(gemm_sum(qkv, 3, st));
      if (!lora) {
        // ---- the seven weight gradients of the chunk, dW += dY^T X (Eq. 1 summand): queued, and launched together
        //      with those of the other chunks of the group (one pass over every dW for the group's rows)
        const GemmArgs mine[7] = {dw_gemm(dyc, s.act, g->wdown, n, d, F, dt, gdt),  dw_gemm(s.gate, s.m, g->wgate, n, F, d, dt, gdt),
                                  dw_gemm(s.up, s.m, g->wup, n, F, d, dt, gdt),    dw_gemm(s.dh1_t, s.o, g->wo, n, d, qd, dt, gdt),
                                  dw_gemm(s.dq, s.a, g->wq, n, qd, d, dt, gdt),    dw_gemm(s.dkc, s.a, g->wk, n, kd, d, dt, gdt),
                                  dw_gemm(s.dvc, s.a, g->wv, n, kd, d, dt, gdt)};
        for (int i = 0; i < 7; ++i) dws[n_dws++] = mine[i];
        if (group_done) {
          if (da_with_dw) n_dws = (int)(std::copy_n(qkv, 3, dws + n_dws) - dws);
          HIPCHK(gemm_batch(dws, n_dws, st));
          n_dws = 0;
        }
      } else {
        // ---- adapter gradients of the chunk (Eq. 1 summands of dA and dB): four grouped launches of skinny GEMMs
        const void* dYs[7] = {s.dq, s.dkc, s.dvc, s.dh1_t, s.gate, s.up, dyc};     // order wq, wk, wv, wo, wgate, wup, wdown
        const void* Xs[7] = {s.a, s.a, s.a, s.o, s.m, s.m, s.act};
        GemmArgs gp[7], gq[7], gb[7], ga[7];
        const int rp = lora->pad;
        for (int j = 0; j < lora->n; ++j) {
          const int i = lora->which[j], out = lora->out_dim[j], in = lora->in_dim[j];
          gp[j] = fwd_gemm(Xs[i], lora->a_pad[j], lora->P[j], n, rp, in, dt, dt);                                   // P = X A^T
          gq[j] = mk(dYs[i], lora->b_pad[j], lora->Q[j], n, rp, out, out, rp, rp, false, false, dt, dt, false);    // Q = dY B
          gb[j] = dw_gemm(dYs[i], lora->P[j], lora->db_pad[j], n, out, rp, dt, DT_F32);                             // dB += dY^T P
          ga[j] = dw_gemm(lora->Q[j], Xs[i], lora->da_pad[j], n, rp, in, dt, DT_F32);                               // dA += Q^T X
        }
        // P and Q are chunk x rank: a handful of output tiles each.  Those with a long reduction (the MLP width) go out
        // alone, where the dispatcher splits the reduction over the chip; the short ones share one grouped launch.
        auto launch_skinny = [&](const GemmArgs* gs, int cnt) -> int32_t {
          GemmArgs shortk[7];
          int n_short = 0;
          for (int j = 0; j < cnt; ++j) {
            if (gs[j].K >= 8192) HIPCHK(gemm(gs[j], st));
            else shortk[n_short++] = gs[j];
          }
          if (n_short == 1) HIPCHK(gemm(shortk[0], st));
          else if (n_short > 1) HIPCHK(gemm_batch(shortk, n_short, st, true));
          return SBP_OK;
        };
        if ((rc = launch_skinny(gp, lora->n))) return rc;
        if ((rc = launch_skinny(gq, lora->n))) return rc;
        if (lora->n == 1) {
          HIPCHK(gemm(gb[0], st)); HIPCHK(gemm(ga[0], st));
        } else {
          HIPCHK(gemm_batch(gb, lora->n, st, true));
          HIPCHK(gemm_batch(ga, lora->n, st, true));
        }
      }
      HIPCHK(rmsnorm_bwd(dt, s.f0, xc, false, w->g1, s.rstd1, s.f1, true, nullptr, at(dx, row0, d, es), partial1, n, d, st));
      if (!lora) {
        gains.partial[0][set] = partial1; gains.partial[1][set] = partial2;
        gains.blocks[set] = rmsnorm_bwd_partial_rows(n);
        gains.n = set + 1;
        if (n_dws == 0) {      // the group's weight gradients are launched
          HIPCHK(column_sums(gains, 2, d, st));
          gains.n = 0;
        }
      }
    }
  }
  return SBP_OK;
}
}  // namespace

extern "C" {

int32_t streambp_layer_backward(const sbp_layer_cfg* c, const sbp_layer_weights* w, const void* x, const void* dy,
                                void* dx, const sbp_layer_grads* g, void* workspace, size_t workspace_bytes,
                                void* hip_stream) {
  int32_t rc = check_layer_cfg(c);
  if (rc) return rc;
  if ((rc = check_layer_ptrs(w))) return rc;
  if (!x || !dy || !dx || !g || !workspace) return fail(SBP_ERR_NULL, "x, dy, dx, dw and workspace must be non-NULL");
  {
    const void* ps[] = {g->wq, g->wk, g->wv, g->wo, g->wgate, g->wup, g->wdown, g->g1, g->g2};
    for (const void* p : ps) if (!p) return fail(SBP_ERR_NULL, "a gradient pointer is NULL");
  }
  if (dx == x || dx == dy) return fail(SBP_ERR_SHAPE, "dx may not alias x or dy");
  if ((uintptr_t)workspace & 255) return fail(SBP_ERR_WORKSPACE, "workspace must be 256-byte aligned");
  const size_t need = layer_budget(c);
  if (workspace_bytes < need) return fail(SBP_ERR_WORKSPACE, "workspace too small: %zu < %zu", workspace_bytes, need);
  const LayerWs s_all = carve_layer(c, workspace, plan_backward(c), true);
  return layer_backward_impl(c, w, x, dy, dx, g, nullptr, s_all, (hipStream_t)hip_stream);
}

// ---- adapter mode ---------------------------------------------------------------------------------------------
namespace {
int32_t check_lora(const sbp_layer_cfg* c, const sbp_lora_adapters* ad) {
  if (!ad) return fail(SBP_ERR_NULL, "adapters table is NULL");
  if (ad->rank < 1 || ad->rank > LORA_MAX_RANK) return fail(SBP_ERR_SHAPE, "adapter rank must be in [1, %d]", LORA_MAX_RANK);
  if (!std::isfinite(ad->scale)) return fail(SBP_ERR_SHAPE, "adapter scale must be finite");
  if (c->grad_dtype != SBP_F32) return fail(SBP_ERR_UNSUPPORTED, "adapter gradients are fp32");
  int n = 0;
  for (int i = 0; i < 7; ++i) {
    if ((ad->a[i] == nullptr) != (ad->b[i] == nullptr)) return fail(SBP_ERR_NULL, "adapter %d: A and B must be given together", i);
    n += ad->a[i] != nullptr;
  }
  if (n == 0) return fail(SBP_ERR_NULL, "no matrix is adapted");
  return SBP_OK;
}
struct LoraWs { LoraCtx ctx; sbp_layer_weights w_eff; void* bt[7]; sbp_layer_cfg layer_cfg; void* layer_ws; size_t bytes; };      // bytes: up to layer_ws
LoraWs carve_lora(const sbp_layer_cfg* c, const sbp_layer_weights* w, const sbp_lora_adapters* ad, void* ws, size_t rows) {
  const size_t es = dtype_size(c->dtype);
  const int d = c->hidden, F = c->mlp_width, qd = c->n_q_heads * c->head_dim, kd = c->n_kv_heads * c->head_dim;
  const int outs[7] = {qd, kd, kd, d, F, F, d}, ins[7] = {d, d, d, qd, d, d, F};
  Carver cv(ws);
  LoraWs L{};
  if (w) L.w_eff = *w;
  const void** eff[7] = {&L.w_eff.wq, &L.w_eff.wk, &L.w_eff.wv, &L.w_eff.wo, &L.w_eff.wgate, &L.w_eff.wup, &L.w_eff.wdown};
  LoraCtx& x = L.ctx;
  x.n = 0;
  x.pad = (ad->rank + 7) & ~7;
  const size_t rp = (size_t)x.pad;
  for (int i = 0; i < 7; ++i) {
    if (!ad->a[i]) continue;
    const int j = x.n++;
    x.which[j] = i; x.out_dim[j] = outs[i]; x.in_dim[j] = ins[i];
    *eff[i] = cv.take_bytes((size_t)outs[i] * ins[i] * es);                      // W + s B A
    x.a_pad[j] = cv.take_bytes(rp * ins[i] * es);
    x.b_pad[j] = cv.take_bytes((size_t)outs[i] * rp * es);
    L.bt[j] = cv.take_bytes((size_t)ad->rank * outs[i] * es);                    // s B^T, the merge GEMM's operand
    x.P[j] = cv.take_bytes(rows * rp * es);
    x.Q[j] = cv.take_bytes(rows * rp * es);
  }
  ClearedCarver grads(cv);
  for (int j = 0; j < x.n; ++j) {
    x.da_pad[j] = grads.take(rp * x.in_dim[j]);
    x.db_pad[j] = grads.take((size_t)x.out_dim[j] * rp);
  }
  x.grads = grads.close();
  L.layer_cfg = *c;
  L.layer_cfg.dw_group_rows = 1;          // no weight-gradient passes to group: one set of chunk buffers
  L.layer_ws = cv.take_bytes(0);
  L.bytes = cv.off;
  return L;
}
size_t lora_budget(const sbp_layer_cfg* c, const sbp_lora_adapters* ad) {
  const LoraWs L = carve_lora(c, nullptr, ad, nullptr, (size_t)std::min(c->chunk, c->seq_len));
  return L.bytes + layer_budget(&L.layer_cfg);
}
LayerPlan plan_lora(const sbp_layer_cfg* c, const sbp_lora_adapters* ad) {
  const size_t budget = lora_budget(c, ad);
  return plan_layer(c, 1, 2.0, false, [&](const LayerPlan& p) {
    return carve_lora(c, nullptr, ad, nullptr, (size_t)p.seqs * p.rows).bytes + carve_layer(c, nullptr, p, true).bytes <= budget;
  });
}
}  // namespace

size_t streambp_layer_lora_workspace_bytes(const sbp_layer_cfg* cfg, const sbp_lora_adapters* ad) {
  if (check_layer_cfg(cfg) != SBP_OK || check_lora(cfg, ad) != SBP_OK) return 0;
  return lora_budget(cfg, ad);
}

int32_t streambp_layer_lora_backward(const sbp_layer_cfg* c, const sbp_layer_weights* w, const sbp_lora_adapters* ad,
                                     const void* x, const void* dy, void* dx, const sbp_lora_grads* g, void* workspace,
                                     size_t workspace_bytes, void* hip_stream) {
  int32_t rc = check_layer_cfg(c);
  if (rc) return rc;
  if ((rc = check_layer_ptrs(w))) return rc;
  if ((rc = check_lora(c, ad))) return rc;
  if (!x || !dy || !dx || !g || !workspace) return fail(SBP_ERR_NULL, "x, dy, dx, the gradient table and workspace must be non-NULL");
  for (int i = 0; i < 7; ++i)
    if (ad->a[i] && (!g->da[i] || !g->db[i])) return fail(SBP_ERR_NULL, "adapter %d: da and db must be non-NULL", i);
  if (dx == x || dx == dy) return fail(SBP_ERR_SHAPE, "dx may not alias x or dy");
  if ((uintptr_t)workspace & 255) return fail(SBP_ERR_WORKSPACE, "workspace must be 256-byte aligned");
  const size_t need = lora_budget(c, ad);
  if (workspace_bytes < need) return fail(SBP_ERR_WORKSPACE, "workspace too small: %zu < %zu", workspace_bytes, need);
  const LayerPlan plan = plan_lora(c, ad);
  const LoraWs L = carve_lora(c, w, ad, workspace, (size_t)plan.seqs * plan.rows);
  hipStream_t st = (hipStream_t)hip_stream;
  const int dt = c->dtype;
  const size_t es = dtype_size(dt);
  const void* base[7] = {w->wq, w->wk, w->wv, w->wo, w->wgate, w->wup, w->wdown};
  const void* eff[7] = {L.w_eff.wq, L.w_eff.wk, L.w_eff.wv, L.w_eff.wo, L.w_eff.wgate, L.w_eff.wup, L.w_eff.wdown};
  const LoraCtx& X = L.ctx;
  t_gemm_scratch = nullptr; t_gemm_scratch_bytes = 0;
  // Operands with the rank rounded up to a multiple of 8, and the effective matrices W + s B A: one pass that reads W, adds the rank-r product
  // in fp32 and rounds once
  PadJobs pads{};
  GemmArgs merge[7];
  for (int j = 0; j < X.n; ++j) {
    const int i = X.which[j], out = X.out_dim[j], in = X.in_dim[j], r = ad->rank;
    pads.job[pads.n++] = PadJob{ad->a[i], X.a_pad[j], r, in, 0, X.pad, in, 1.0f, 0};
    pads.job[pads.n++] = PadJob{ad->b[i], X.b_pad[j], out, r, 0, out, X.pad, 1.0f, 0};
    pads.job[pads.n++] = PadJob{ad->b[i], L.bt[j], r, out, 1, r, out, ad->scale, 0};
    merge[j] = mk(L.bt[j], X.a_pad[j], (void*)eff[i], out, in, r, out, in, in, true, false, dt, dt, true);
    merge[j].C0 = base[i];
  }
  HIPCHK(pad_matrices(dt, pads, st));
  HIPCHK(gemm_batch(merge, X.n, st));
  if (X.n > 0) HIPCHK(fill_zero(X.grads.p, X.grads.bytes, st));
  const LayerWs s_all = carve_layer(&L.layer_cfg, L.layer_ws, plan, true);
  if ((rc = layer_backward_impl(&L.layer_cfg, &L.w_eff, x, dy, dx, nullptr, &X, s_all, st))) return rc;
  AddJobs adds{};
  for (int j = 0; j < X.n; ++j) {
    const int i = X.which[j];
    adds.job[adds.n++] = AddJob{X.da_pad[j], X.in_dim[j], g->da[i], ad->rank, X.in_dim[j], 0};
    adds.job[adds.n++] = AddJob{X.db_pad[j], X.pad, g->db[i], X.out_dim[j], ad->rank, 0};
  }
  HIPCHK(add_scaled_blocks(adds, ad->scale, st));
  return SBP_OK;
}

int32_t streambp_layer_forward(const sbp_layer_cfg* c, const sbp_layer_weights* w, const void* x, void* y,
                               void* workspace, size_t workspace_bytes, void* hip_stream) {
  int32_t rc = check_layer_cfg(c);
  if (rc) return rc;
  if ((rc = check_layer_ptrs(w))) return rc;
  if (!x || !y || !workspace) return fail(SBP_ERR_NULL, "x, y and workspace must be non-NULL");
  if ((uintptr_t)workspace & 255) return fail(SBP_ERR_WORKSPACE, "workspace must be 256-byte aligned");
  const size_t need = layer_budget(c);
  if (workspace_bytes < need) return fail(SBP_ERR_WORKSPACE, "workspace too small: %zu < %zu", workspace_bytes, need);
  const LayerWs s = carve_layer(c, workspace, plan_forward(c), false);
  hipStream_t st = (hipStream_t)hip_stream;
  t_gemm_scratch = s.gemm_scratch; t_gemm_scratch_bytes = s.gemm_scratch_bytes;
  const int dt = c->dtype;
  const size_t es = dtype_size(dt);
  const int T = c->seq_len, d = c->hidden, F = c->mlp_width;
  HIPCHK(rope_table(s.rope, T, c->head_dim, c->rope_theta, c->pos_offset, nullptr, 0, st));
  for (int b0 = 0; b0 < c->batch; b0 += s.plan.seqs) {
    const int seqs = std::min(s.plan.seqs, c->batch - b0);
    const bool whole = s.plan.rows >= T;
    if (!whole && (rc = kv_prepass(c, w, s, at(x, (size_t)b0 * T, d, es), st))) return rc;
    for (int r0 = 0; r0 < T; r0 += s.plan.rows) {
      const Pass p{b0, seqs, r0, std::min(s.plan.rows, T - r0), whole};
      const int n = (int)pass_rows(p);
      const size_t row0 = (size_t)b0 * T + r0;
      if ((rc = chunk_reforward(c, w, s, at(x, row0, d, es), p, true, st))) return rc;
      HIPCHK(gemm(fwd_gemm(s.act, w->wdown, s.f1, n, d, F, dt, DT_F32), st));
      HIPCHK(add_store(dt, s.f0, s.f1, at(y, row0, d, es), (int64_t)n * d, st));
    }
  }
  return SBP_OK;
}

// --------------------------------------------------------------- LM head --
static int32_t check_head_cfg(const sbp_head_cfg* c) {
  if (!c) return fail(SBP_ERR_NULL, "cfg is NULL");
  if (!valid_dtype(c->dtype)) return fail(SBP_ERR_UNSUPPORTED, "dtype %d not supported", c->dtype);
  if (int32_t rc = check_grad_dtype(c->dtype, c->grad_dtype)) return rc;
  if (c->dw_group_rows < 0) return fail(SBP_ERR_SHAPE, "dw_group_rows must be >= 0");
  if (c->batch < 1 || c->seq_len < 1 || c->chunk < 1 || c->hidden < 1 || c->vocab < 1)
    return fail(SBP_ERR_SHAPE, "batch, seq_len, chunk, hidden and vocab must be >= 1");
  if (c->objective < SBP_OBJ_SFT || c->objective > SBP_OBJ_DPO) return fail(SBP_ERR_UNSUPPORTED, "objective %d not supported", c->objective);
  if (c->objective == SBP_OBJ_DPO && c->batch != 2) return fail(SBP_ERR_SHAPE, "DPO needs batch == 2 (chosen, rejected)");
  return SBP_OK;
}

// The weight gradient of the head is accumulated once per group of chunks (dw_group_for): dz and the gathered h rows of that
// many chunks stay alive and one GEMM adds them into dW, so the 8 bytes per element of
// read-modify-write traffic on dW (the largest tensor of the path) are paid once per group instead of once per
// chunk.  The fp32 logits - the dominant term - still exist for one chunk only.
struct HeadWs {
  int dw_group;
  float* z; void* dz; float *row_loss, *target_logit, *seq_weight, *ell;      // dz, row_loss: the group's rows
  float2* stats; int n_stat;          // per row and 256-column block of the chunk's logits: (max, sum of exp), written by the logits GEMM
  int64_t ldz;                        // row stride of z and dz: bf16 rows are padded to the GEMMs' reduction step (zeros), so that any vocabulary fits
  int32_t *index, *chunk_rows; void *hc, *dhc;   // active-row compaction: row list, rows per chunk; gathered rows of h (the group's; ht: a chunk's), rows of dh
  bool ht;                            // the weight gradient's h rows are kept transposed, hT [hidden, ldt] per chunk of the group
  int64_t ldt; void* hT;
  float* gemm_scratch; size_t gemm_scratch_bytes; size_t bytes;
};
// Chunks whose rows the products of a small chunk run on at once (see streambp_lmhead_ce_backward): whole spans per weight-gradient group
constexpr int HEAD_SPAN_ROWS = 2048;
static int head_span_chunks(int dw_group, int cm) {
  int chunks = std::max(1, std::min(dw_group, HEAD_SPAN_ROWS / cm));
  while (dw_group % chunks != 0) --chunks;
  return chunks;
}
static HeadWs carve_head(const sbp_head_cfg* c, void* ws) {
  const int64_t rows = (int64_t)c->batch * c->seq_len;
  const size_t cm = (size_t)std::min<int64_t>(c->chunk, rows);
  Carver cv(ws);
  HeadWs h;
  h.ldz = c->dtype == SBP_BF16 ? (int64_t)align_up((size_t)c->vocab, 64) : c->vocab;
  h.z = cv.take<float>(cm * (size_t)h.ldz);
  h.dw_group = dw_group_for(cm, c->dw_group_rows, DW_GROUP_ROWS_HEAD);
  const size_t group = (size_t)std::min<int64_t>((int64_t)cm * h.dw_group, rows);      // rows of a weight-gradient group
  h.dz = cv.take_bytes(group * (size_t)h.ldz * dtype_size(c->dtype));
  h.row_loss = cv.take<float>(group);
  h.target_logit = cv.take<float>(cm);
  h.n_stat = (int)cdiv(c->vocab, GEMM_STAT_COLS);
  h.stats = cv.take<float2>(cm * (size_t)h.n_stat);
  h.seq_weight = cv.take<float>(c->batch);
  h.ell = cv.take<float>(1);
  h.index = cv.take<int32_t>((size_t)rows);
  h.chunk_rows = cv.take<int32_t>(2 * (size_t)cdiv(rows, (int64_t)cm) + 1);
  // With h^T the weight gradient's GEMM reads one operand instead of two through transposing LDS loads: 152064 x 3584, 8192 rows: 7.50 -> 7.20 ms;
  // the copy takes 6 us per 2048-row chunk.  Whole call, 3584 x 152064: 32768 rows 86.2 -> 85.4 ms, 6000 13.10 -> 12.88, 1500 4.58 -> 4.53, 300 the
  // same.  With / without it, 8192 rows and 1500: 51 million outputs 0.985-0.989 and 1.00, 66 0.99 and 0.995, 84 0.98-0.99 and 0.995, 102 0.977 and 0.99, 263
  // 0.99, 545 0.99: the line lies where the gain passes the spread of the runs (1.5 %) and pays for the copies' room.
  h.ht = c->dtype == SBP_BF16 && c->hidden % 8 == 0 && (int64_t)c->vocab * c->hidden >= 100000000;
  h.ldt = (int64_t)align_up(cm, 64);
  h.hc = cv.take_bytes((h.ht ? cm : group) * c->hidden * dtype_size(c->dtype));
  // (or, a multiple of ldt wide, per unit of several chunks: as many copies as the chunks of the call, whole units)
  const int64_t chunks = align_up((size_t)cdiv(rows, (int64_t)cm), (size_t)head_span_chunks(h.dw_group, (int)cm));
  h.hT = h.ht ? cv.take_bytes((size_t)std::min<int64_t>(h.dw_group, chunks) * c->hidden * h.ldt * 2) : nullptr;
  h.dhc = cv.take_bytes(cm * c->hidden * dtype_size(c->dtype));
  h.gemm_scratch_bytes = c->dtype == SBP_BF16 ? gemm_scratch_bytes((int)cm, c->hidden) : 0;
  h.gemm_scratch = (float*)cv.take_bytes(h.gemm_scratch_bytes);
  h.bytes = cv.off;
  return h;
}

size_t streambp_lmhead_workspace_bytes(const sbp_head_cfg* cfg) {
  if (check_head_cfg(cfg) != SBP_OK) return 0;
  return carve_head(cfg, nullptr).bytes;
}

int32_t streambp_lmhead_ce_backward(const sbp_head_cfg* c, const void* w, const void* h, const int32_t* targets,
                                    const float* old_logp, const float* ref_logp, const float* advantages, void* dh,
                                    void* dw, float* loss, int64_t* n_active, void* workspace, size_t workspace_bytes,
                                    void* hip_stream) {
  int32_t rc = check_head_cfg(c);
  if (rc) return rc;
  if (!w || !h || !targets || !dh || !dw || !loss || !n_active || !workspace)
    return fail(SBP_ERR_NULL, "w, h, targets, dh, dw, loss, n_active and workspace must be non-NULL");
  if (c->objective == SBP_OBJ_GRPO && (!ref_logp || !advantages)) return fail(SBP_ERR_NULL, "GRPO needs ref_logp and advantages");
  if (c->objective == SBP_OBJ_DPO && !ref_logp) return fail(SBP_ERR_NULL, "DPO needs ref_logp");
  if ((uintptr_t)workspace & 255) return fail(SBP_ERR_WORKSPACE, "workspace must be 256-byte aligned");
  const HeadWs s = carve_head(c, workspace);
  if (workspace_bytes < s.bytes) return fail(SBP_ERR_WORKSPACE, "workspace too small: %zu < %zu", workspace_bytes, s.bytes);

  hipStream_t st = (hipStream_t)hip_stream;
  const int dt = c->dtype;
  const size_t es = dtype_size(dt);
  t_gemm_scratch = s.gemm_scratch; t_gemm_scratch_bytes = s.gemm_scratch_bytes;
  const int64_t rows = (int64_t)c->batch * c->seq_len;
  const int cm = (int)std::min<int64_t>(c->chunk, rows);
  const int d = c->hidden, V = c->vocab;

  // Rows with an ignored target contribute nothing (dz = 0): only the active rows are pushed through the
  // GEMMs.  Positions are independent (Sec. 3.2.1), so the active rows of all sequences are chunked as one
  // flat list; the list and the per-chunk row counts live on the device (no host synchronisation), and the
  // kernels of a chunk read their row count at run time.
  // How many rows the products run on at once: one chunk, or as many chunks as make HEAD_SPAN_ROWS.  dz is kept for them anyway, and the buffer of the
  // fp32 logits has room for what else they need: the numerator form never holds logits (there it takes the statistics and the rows of h and dh of
  // the whole span, and every product runs on the span), the logits of fp32 heads are formed where their dz will be (the same, without statistics),
  // else they are dead when the span's last chunk is done (it takes dh, and that product alone runs on the span).  Small chunks are what this is for: the logits of 1024 rows at 7B widths are 2376 output tiles, a tenth round
  // of the CUs for 72 of them.  GRPO group of 8 x 1111 rows, chunk 1024, 18.8 -> 18.0 ms; fp32 layer and head of 256 rows, chunk 64 (five launches a
  // chunk) 371 -> 335 us with dh alone, later 138 -> 108 with all products and fewer launches around them; two-layer stack of 1024 wide layers, vocabulary 50257, chunk 512, 3.36 -> 3.30 ms.
  // More rows than HEAD_SPAN_ROWS gain no more: all 16384 of a group at once, dh takes 26.0 instead of 26.9 ms per 32768 rows, the row
  // kernel, which finds less of dz in the caches, 4.2 instead of 3.65, and the whole call the same.
  const bool padded = dt == DT_BF16;      // bf16 rows of z and dz are padded to a multiple of 64, dz with zeros: the products with dz need no particular vocabulary
  auto numerators = [&](const void* hc, void* dz, int n, const int* n_dev, const int32_t* idx, float2* stats, float* target_logit) {
    GemmArgs g = fwd_gemm(hc, w, dz, n, V, d, dt, DT_BF16);
    g.ldc = s.ldz;
    g.rows_dev = n_dev; g.row_stats = stats;
    g.numer_targets = targets; g.numer_row_index = idx; g.numer_target_value = target_logit;
    return g;
  };
  const bool numer = (fusion_mask() & FUSE_NUMERATORS) && dt == DT_BF16 && s.n_stat > 0 &&
                     gemm_numerators_supported(numerators(s.hc, s.dz, cm, s.chunk_rows, s.index, s.stats, s.target_logit));
  const bool in_place = dt == SBP_F32, wide = numer || in_place;      // fp32 dz takes the place of the logits; wide: a unit may be a span
  void *hc = s.hc, *dhc = s.dhc;
  float2* stats = s.stats;
  float* target_logit = s.target_logit;
  int chunks = head_span_chunks(s.dw_group, cm);
  const int span = (int)std::min<int64_t>(rows, (int64_t)cm * chunks);
  size_t z_used = 0;      // bytes of the fp32-logits buffer that other things take
  if (span > cm) {
    auto carve = [&](void* base) {
      if (!numer) { dhc = base; return (size_t)span * d * es; }
      Carver cv(base);
      dhc = cv.take_bytes((size_t)span * d * es);
      stats = cv.take<float2>((size_t)span * s.n_stat);
      target_logit = cv.take<float>(span);
      if (s.ht) hc = cv.take_bytes((size_t)span * d * es);
      return cv.off;
    };
    if (carve(nullptr) <= (size_t)cm * s.ldz * sizeof(float)) z_used = carve(s.z);
    else { dhc = s.dhc; stats = s.stats; target_logit = s.target_logit; hc = s.hc; chunks = 1; }
  } else chunks = 1;
  const int cu = chunks > 1 && wide ? span : cm;          // rows of a unit: what the logits are formed of at once
  const int dh_units = chunks > 1 && !wide ? chunks : 1, per_group = wide ? s.dw_group / chunks : s.dw_group;      // units of a span of dh, of a weight-gradient group
  const bool gather_span = dh_units > 1 && !s.ht;         // all rows of a span fetched at once
  const int n_units = (int)cdiv(rows, (int64_t)cu);
  int32_t* unit_rows = s.chunk_rows;                      // [n_units], then all active rows, then the rows per span
  int32_t* span_rows = unit_rows + n_units + 1;
  const int n_spans = dh_units > 1 ? (int)cdiv(rows, (int64_t)span) : 0, n_groups = (int)cdiv(n_units, per_group), group_units = std::min(per_group, n_units);
  int32_t* group_rows = span_rows + n_spans;
  // All units of the list but the last active one are full, so that the rows of dz and h (the columns of h^T) of a group's units are one matrix of as many rows:
  // one reduction without a break, whose last round may be split, in place of a segment per unit (about 3 us each and tile, the pipeline emptied and filled
  // again).  50257 x 1024, 1842 rows in four units 294 -> 240 + 10 us; 152064 x 3584, 16384 rows in eight 13.95 -> 13.85 ms, 151936 x 3584, 8888 in five, the call
  // 18.02 -> 17.94.  Where h^T is kept a unit has to end with 64 columns, and its rows start 64 columns further apart than they are long where there is room for it:
  // the fp32-logits buffer, which the numerator form leaves idle (rows 32 KB apart: 13.98 ms).  The list of the groups' rows has to fit behind the others.
  const bool joined = n_units > 1 && (!s.ht || cu % 64 == 0) && n_units + 1 + n_spans + n_groups <= 2 * (int)cdiv(rows, (int64_t)cm) + 1;
  int64_t ldt = s.ht && joined ? (int64_t)group_units * cu : (int64_t)align_up((size_t)cu, 64);
  char* hT_all = (char*)s.hT;
  if (s.ht && joined && numer && align_up(z_used, 256) + (size_t)d * (ldt + 64) * 2 <= (size_t)cm * s.ldz * sizeof(float)) {
    hT_all = (char*)s.z + align_up(z_used, 256);
    ldt += 64;
  }
  {
    HeadBegin b{};
    b.targets = targets; b.B = c->batch; b.T = c->seq_len; b.V = V;
    b.seq_weight = s.seq_weight; b.n_active = n_active; b.ell = c->objective == SBP_OBJ_DPO ? s.ell : nullptr;
    b.index = s.index; b.unit_rows = unit_rows; b.unit = cu; b.n_units = n_units;
    b.span_rows = span_rows; b.span = span; b.n_spans = n_spans;
    b.group_rows = group_rows; b.group = group_units * cu; b.n_groups = joined ? n_groups : 0;
    b.dh = dh; b.dh_bytes = (size_t)rows * d * es;           // ignored rows of dh: exact zeros
    HIPCHK(head_begin(b, st));
  }
  GemmArgs pending[MAX_DW_GROUP + 1];
  int n_pending = 0;
  // rows [first, first + n) of the list of active rows: at most n, the rest of them on the device
  auto moved = [&](bool scatter, int64_t first, int64_t n, const int32_t* n_dev, void* buf) {
    const int m = (int)std::max<int64_t>(0, std::min<int64_t>(n, rows - first));
    return m == 0 ? RowMove{} : scatter ? RowMove{buf, s.index + first, n_dev, dh, m} : RowMove{h, s.index + first, n_dev, buf, m};
  };
  for (int ci = 0; ci < n_units; ++ci) {
    const int64_t first = (int64_t)ci * cu, group_first = (int64_t)(ci - n_pending) * cu, span_first = first - (int64_t)(ci % dh_units) * cu;
    const int32_t* idx = s.index + first;
    const int* n_dev = unit_rows + ci;
    const int n = (int)std::min<int64_t>(cu, rows - first);      // upper bound of the unit's rows
    void* hcu = s.ht ? hc : at(hc, (size_t)n_pending * cu, d, es);
    void* dz = at(s.dz, (size_t)n_pending * cu, s.ldz, es);
    void* hT = s.ht ? hT_all + (size_t)n_pending * (joined ? (size_t)cu : (size_t)d * ldt) * 2 : nullptr;
    if (ci == 0) HIPCHK(move_rows(dt, RowMove{}, gather_span ? moved(false, 0, span, span_rows, hc) : moved(false, 0, cu, n_dev, hcu), d, st));
    if (s.ht) HIPCHK(transpose_rows(hcu, n_dev, n, d, hT, ldt, st));
    // The logits: fp32 with (max, sum of exp) per row and 256-column block out of the GEMM's epilogue where the MFMA kernel
    // takes the problem - or, better, never as logits at all: the numerator form leaves exp(z - block max) in bf16 directly in
    // the chunk's dz buffer plus the target logits, and the row kernel finishes dz in place.
    GemmArgs gz = numerators(hcu, dz, n, n_dev, idx, stats, target_logit);
    if (!numer) {
      gz = fwd_gemm(hcu, w, in_place ? dz : s.z, n, V, d, dt, DT_F32);
      gz.ldc = s.ldz; gz.c_padded = padded;
      gz.rows_dev = n_dev;
      gz.row_stats = s.stats;
    }
    const bool has_stats = numer || (s.n_stat > 0 && gemm_row_stats_supported(gz));   // the LSE statistics come out of the GEMM's epilogue
    if (!has_stats) gz.row_stats = nullptr;
    HIPCHK(gemm(gz, st));
    HeadRowArgs a{};
    a.stats = has_stats ? stats : nullptr; a.n_stat = s.n_stat;
    a.target_logit = numer ? target_logit : nullptr;
    a.dt = dt; a.objective = c->objective; a.z = in_place ? (const float*)dz : s.z; a.dz = dz; a.ldz = s.ldz; a.targets = targets;
    a.old_logp = old_logp; a.ref_logp = ref_logp;
    a.advantages = advantages; a.seq_weight = s.seq_weight; a.row0 = 0; a.row_index = idx; a.rows_dev = n_dev;
    a.rows = n; a.V = V; a.T = c->seq_len;
    a.loss_scale = c->loss_scale; a.clip_eps = c->clip_eps; a.kl_beta = c->kl_beta; a.kl_mode = c->kl_mode;
    a.row_loss = s.row_loss + (size_t)n_pending * cu;
    HIPCHK(head_rows(a, st));
    pending[n_pending] = dw_gemm(dz, hcu, dw, n, V, d, dt, c->grad_dtype);
    if (s.ht) {
      pending[n_pending].B = hT; pending[n_pending].tb = true;
      pending[n_pending].ldb = ldt; pending[n_pending].b_padded = true;
    }
    pending[n_pending].lda = s.ldz; pending[n_pending].a_padded = padded;
    pending[n_pending].rows_dev = n_dev;
    const bool span_done = (ci + 1) % dh_units == 0 || ci + 1 == n_units;
    const int* span_dev = dh_units > 1 ? span_rows + ci / dh_units : n_dev;
    const bool group_done = n_pending + 1 == per_group || ci + 1 == n_units, dh_with_dw = span_done && group_done && dt == DT_F32;      // dh and dW in one launch
    if (span_done) {
      GemmArgs gh = dx_gemm((char*)dz - (size_t)(first - span_first) * s.ldz * es, w, dhc, (int)(first + n - span_first), V, d, dt, dt, false);
      gh.lda = s.ldz; gh.a_padded = padded;
      gh.rows_dev = span_dev;
      if (!dh_with_dw) HIPCHK(gemm(gh, st));
      else {      // (the longer reduction first)
        std::copy_backward(pending, pending + n_pending + 1, pending + n_pending + 2);
        pending[0] = gh;
      }
    }
    LossSum sum{};
    ++n_pending;
    if (group_done) {
      int n_products = n_pending;
      if (joined) {
        GemmArgs& g = pending[dh_with_dw];      // the group's first unit, and all rows behind it
        g.K = (int)(first + n - group_first);
        g.rows_dev = group_rows + group_first / ((int64_t)group_units * cu);
        n_products = 1;
      }
      HIPCHK(gemm_batch(pending, n_products + dh_with_dw, st));
      // the active rows of the group's chunks are one list: its loss terms are summed together
      sum = LossSum{s.row_loss, (int)(first + n - group_first), c->objective == SBP_OBJ_DPO ? s.ell : loss, unit_rows + n_units,
                    (int)std::min<int64_t>(group_first, INT32_MAX)};
      n_pending = 0;
    }
    // rows of dh out, the next rows of h in: independent of each other
    const RowMove out = span_done ? moved(true, span_first, first + n - span_first, span_dev, dhc) : RowMove{};
    void* next = s.ht ? hc : at(hc, (size_t)n_pending * cu, d, es);
    RowMove in{};
    if (!gather_span) in = moved(false, first + cu, cu, n_dev + 1, next);
    else if (span_done) in = moved(false, first + cu, span, span_dev + 1, next);
    HIPCHK(move_rows(dt, out, in, d, st, sum));
  }
  if (c->objective == SBP_OBJ_DPO)
    HIPCHK(dpo_finish(dt, s.ell, c->kl_beta, dh, rows * d, dw, c->grad_dtype, (int64_t)V * d, loss, st));
  return SBP_OK;
}

// -------------------------------------------------------- chunk attention --
static int32_t check_attn_cfg(const sbp_attn_cfg* c) {
  if (!c) return fail(SBP_ERR_NULL, "cfg is NULL");
  if (!valid_dtype(c->dtype)) return fail(SBP_ERR_UNSUPPORTED, "dtype %d not supported", c->dtype);
  if (c->n_q_heads < 1 || c->n_kv_heads < 1 || c->n_q_heads % c->n_kv_heads != 0)
    return fail(SBP_ERR_SHAPE, "n_q_heads must be a positive multiple of n_kv_heads");
  if (c->head_dim < 1 || c->head_dim > 256) return fail(SBP_ERR_SHAPE, "head_dim must be in [1, 256]");
  if (c->q_start < 0 || c->q_len < 0) return fail(SBP_ERR_SHAPE, "q_start and q_len must be >= 0");
  if ((int64_t)c->q_start + c->q_len > INT32_MAX) return fail(SBP_ERR_SHAPE, "q_start + q_len overflows");
  // the kernels take row maxima of the raw scores before scaling them, which is only right for a positive finite scale
  if (!(c->scale > 0.f) || !std::isfinite(c->scale)) return fail(SBP_ERR_SHAPE, "scale must be positive and finite");
  if (c->window < 0 || c->kv_first < 0) return fail(SBP_ERR_SHAPE, "window and kv_first must be >= 0");
  return SBP_OK;
}

// delta and log-sum-exp of the chunk's (query, head) pairs: what the backward cannot do without
static size_t attn_stats_bytes(const sbp_attn_cfg* c) { return align_up((size_t)2 * std::max(c->q_len, 1) * c->n_q_heads * sizeof(float), 256); }
static AttnArgs attn_args(const sbp_attn_cfg* c) {
  AttnArgs a{};
  a.dt = c->dtype; a.Hq = c->n_q_heads; a.Hkv = c->n_kv_heads; a.dh = c->head_dim;
  a.q_start = c->q_start; a.q_len = c->q_len; a.scale = c->scale; a.window = c->window; a.kv_first = c->kv_first;
  if (c->dtype == SBP_BF16 && (c->head_dim == 128 || c->head_dim == 64)) a.dkv_slices = attn_dkv_slices(a, SIZE_MAX);
  return a;
}

size_t streambp_attn_workspace_bytes(const sbp_attn_cfg* cfg) {
  if (check_attn_cfg(cfg) != SBP_OK) return 0;
  const AttnArgs a = attn_args(cfg);
  return attn_stats_bytes(cfg) + align_up(attn_dkv_scratch_bytes(a, a.dkv_slices), 256);
}

int32_t streambp_attn_chunk_forward(const sbp_attn_cfg* c, const void* q, const void* k, const void* v, void* o,
                                    float* lse, void* hip_stream) {
  int32_t rc = check_attn_cfg(c);
  if (rc) return rc;
  if (c->q_len == 0) return SBP_OK;   // empty chunk: nothing to do
  if (!q || !k || !v || !o || !lse) return fail(SBP_ERR_NULL, "q, k, v, o and lse must be non-NULL");
  AttnArgs a = attn_args(c);
  a.q = q; a.k = k; a.v = v; a.o = o; a.lse = lse;
  HIPCHK(attn_forward(a, (hipStream_t)hip_stream));
  return SBP_OK;
}

int32_t streambp_attn_chunk_backward(const sbp_attn_cfg* c, const void* q, const void* k, const void* v, const void* o,
                                     const float* lse, const void* d_o, void* dq, float* dk, float* dv,
                                     void* workspace, size_t workspace_bytes, void* hip_stream) {
  int32_t rc = check_attn_cfg(c);
  if (rc) return rc;
  if (c->q_len == 0) return SBP_OK;
  if (!q || !k || !v || !o || !lse || !d_o || !dq || !dk || !dv || !workspace)
    return fail(SBP_ERR_NULL, "all tensor pointers and workspace must be non-NULL");
  if ((uintptr_t)workspace & 255) return fail(SBP_ERR_WORKSPACE, "workspace must be 256-byte aligned");
  if (workspace_bytes < attn_stats_bytes(c)) return fail(SBP_ERR_WORKSPACE, "workspace too small");
  AttnArgs a = attn_args(c);
  // with less than the query's bytes the same slices run one after the other: the same results
  if (a.dkv_slices > 1 && workspace_bytes >= streambp_attn_workspace_bytes(c)) a.dkv_scratch = (float*)((char*)workspace + attn_stats_bytes(c));
  a.q = q; a.k = k; a.v = v; a.o = (void*)o; a.lse = (float*)lse;
  a.d_o = d_o; a.dq = dq; a.dk = dk; a.dv = dv; a.delta = (float*)workspace;
  HIPCHK(attn_backward(a, (hipStream_t)hip_stream));
  return SBP_OK;
}

// Which kernels a configuration gets.  The bf16 MFMA GEMMs need every matrix dimension of the layer (hidden, the q and
// k/v widths, mlp_width - resp. the head's hidden) to be a multiple of 64 (the reduction step; output tiles are 256 wide with
// a masked ragged last tile), the MFMA attention head_dim 128.  The head's rows of logits are padded to 64 columns, so that its
// products take any vocabulary; the softmax-numerator store needs a multiple of 8.  64-wide heads and other vocabularies run on MFMA
// kernels too, below the full rate; anything else runs on the shape-agnostic fp32 kernels, which are much slower.
int32_t streambp_layer_fast_path(const sbp_layer_cfg* c) {
  if (int32_t rc = check_layer_cfg(c)) return rc;
  if (c->dtype != SBP_BF16) return fail(0, "fp32 storage: the shape-agnostic kernels are the only path"), 0;
  const int qd = c->n_q_heads * c->head_dim, kd = c->n_kv_heads * c->head_dim;
  if (c->head_dim != 128) return fail(0, "head_dim %d: the full-rate MFMA attention kernels take 128 only", c->head_dim), 0;
  const int dims[4] = {c->hidden, qd, kd, c->mlp_width};
  const char* names[4] = {"hidden", "n_q_heads*head_dim", "n_kv_heads*head_dim", "mlp_width"};
  for (int i = 0; i < 4; ++i)   // every width is the reduction length of some GEMM of the layer
    if (dims[i] % 64) return fail(0, "%s = %d is not a multiple of 64: its GEMMs leave the MFMA kernels", names[i], dims[i]), 0;
  return 1;
}
int32_t streambp_lmhead_fast_path(const sbp_head_cfg* c) {
  if (int32_t rc = check_head_cfg(c)) return rc;
  if (c->dtype != SBP_BF16) return fail(0, "fp32 storage: the shape-agnostic kernels are the only path"), 0;
  if (c->hidden % 64) return fail(0, "hidden = %d is not a multiple of 64: the head's GEMMs leave the MFMA kernels", c->hidden), 0;
  if (c->vocab % 8) return fail(0, "vocab = %d is not a multiple of 8: the head keeps fp32 logits instead of softmax numerators", c->vocab), 0;
  return 1;
}
int64_t streambp_generic_launches(void) { return (int64_t)generic_bf16_launches(); }

// ---- the same backward for callers that cannot allocate ------------------------------------------------------
// The per-call scratch of the attention backward (delta and the log2-domain log-sum-exp, 2 floats per (query, head)
// pair) lives in device memory that belongs to the library's code object instead of a caller workspace.  Every GPU
// the library runs on holds its own copy of the array at its own address; the address is looked up once per device
// (a symbol query, not an allocation) and only that pointer - never the array's name, which on the host is a stand-in
// and not a device address - is handed to kernels.
constexpr int64_t STATIC_SCRATCH_PAIRS = 1 << 18;            // q_len * n_q_heads <= 262144 (2 MiB of scratch)
static __device__ __align__(256) float g_static_scratch[2 * STATIC_SCRATCH_PAIRS];
constexpr int STATIC_MAX_DEVICES = 64;
static float* g_static_scratch_ptr[STATIC_MAX_DEVICES];      // per device, filled on the first call on that device
static std::mutex g_static_scratch_mu;

int32_t streambp_attn_chunk_backward_noalloc(const sbp_attn_cfg* c, const void* q, const void* k, const void* v, const void* o,
                                             const float* lse, const void* d_o, void* dq, float* dk, float* dv,
                                             void* hip_stream) {
  int32_t rc = check_attn_cfg(c);
  if (rc) return rc;
  if (c->q_len == 0) return SBP_OK;
  if (!q || !k || !v || !o || !lse || !d_o || !dq || !dk || !dv) return fail(SBP_ERR_NULL, "all tensor pointers must be non-NULL");
  const int64_t pairs = (int64_t)c->q_len * c->n_q_heads;
  if (pairs > STATIC_SCRATCH_PAIRS)
    return fail(SBP_ERR_WORKSPACE, "q_len * n_q_heads = %lld exceeds the %lld pairs the built-in scratch holds; use "
                "streambp_attn_chunk_backward with a caller workspace", (long long)pairs, (long long)STATIC_SCRATCH_PAIRS);
  int dev = -1;
  HIPCHK(hipGetDevice(&dev));
  if (dev < 0 || dev >= STATIC_MAX_DEVICES) return fail(SBP_ERR_UNSUPPORTED, "device index %d out of range", dev);
  float* scratch;
  {
    std::lock_guard<std::mutex> lock(g_static_scratch_mu);
    if (!g_static_scratch_ptr[dev]) {
      void* p = nullptr;
      HIPCHK(hipGetSymbolAddress(&p, HIP_SYMBOL(g_static_scratch)));
      if (!p) return fail(SBP_ERR_HIP, "hipGetSymbolAddress returned a null address for the built-in scratch");
      g_static_scratch_ptr[dev] = (float*)p;
    }
    scratch = g_static_scratch_ptr[dev];
  }
  AttnArgs a = attn_args(c);
  a.q = q; a.k = k; a.v = v; a.o = (void*)o; a.lse = (float*)lse;
  a.d_o = d_o; a.dq = dq; a.dk = dk; a.dv = dv; a.delta = scratch;
  HIPCHK(attn_backward(a, (hipStream_t)hip_stream));
  return SBP_OK;
}

int64_t streambp_attn_tile_pairs(int32_t q_start, int32_t q_len, int32_t* tile_q, int32_t* tile_k) {
  // Work is skipped per wave: a wave owns ATTN_WAVE_Q query rows and walks key tiles of ATTN_TILE_K.
  if (tile_q) *tile_q = ATTN_WAVE_Q;
  if (tile_k) *tile_k = ATTN_TILE_K;
  if (q_start < 0 || q_len <= 0) return 0;
  int64_t pairs = 0;
  for (int64_t t0 = 0; t0 < q_len; t0 += ATTN_WAVE_Q) {
    const int64_t last_q = q_start + std::min<int64_t>(t0 + ATTN_WAVE_Q, q_len) - 1;   // last query position of the wave
    pairs += last_q / ATTN_TILE_K + 1;                                                 // key tiles that start at or before it
  }
  return pairs;
}

// ------------------------------------------------------------ stack loop --
namespace {
struct StackWs { void *h, *dh, *ga, *gb; void* sub; size_t sub_bytes; size_t bytes; };
sbp_head_cfg stack_head_cfg(const sbp_stack_cfg* c) {
  sbp_head_cfg h{};
  h.dtype = c->layer.dtype; h.batch = c->layer.batch; h.seq_len = c->layer.seq_len; h.chunk = c->head_chunk;
  h.hidden = c->layer.hidden; h.vocab = c->vocab; h.objective = c->objective; h.loss_scale = c->loss_scale;
  h.clip_eps = c->clip_eps; h.kl_beta = c->kl_beta; h.kl_mode = c->kl_mode; h.grad_dtype = c->layer.grad_dtype; h.dw_group_rows = c->layer.dw_group_rows;
  return h;
}
int32_t check_stack_cfg(const sbp_stack_cfg* c) {
  if (!c) return fail(SBP_ERR_NULL, "cfg is NULL");
  int32_t rc = check_layer_cfg(&c->layer);
  if (rc) return rc;
  if (c->n_layers < 1) return fail(SBP_ERR_SHAPE, "n_layers must be >= 1");
  if (!(c->final_eps >= 0.f)) return fail(SBP_ERR_SHAPE, "final_eps must be >= 0");
  const sbp_head_cfg h = stack_head_cfg(c);
  return check_head_cfg(&h);
}
StackWs carve_stack(const sbp_stack_cfg* c, void* ws) {
  const size_t rows = (size_t)c->layer.batch * c->layer.seq_len, d = c->layer.hidden, es = dtype_size(c->layer.dtype);
  const sbp_head_cfg h = stack_head_cfg(c);
  Carver cv(ws);
  StackWs s;
  s.h = cv.take_bytes(rows * d * es);      // RMSNorm(ckpt[L])
  s.dh = cv.take_bytes(rows * d * es);     // gradient wrt h
  s.ga = cv.take_bytes(rows * d * es);     // running dL/dx, ping
  s.gb = cv.take_bytes(rows * d * es);     // pong
  s.sub_bytes = std::max(std::max(streambp_layer_workspace_bytes(&c->layer), streambp_lmhead_workspace_bytes(&h)),
                         streambp_rmsnorm_workspace_bytes((int64_t)rows, (int32_t)d));
  s.sub = cv.take_bytes(s.sub_bytes);
  s.bytes = cv.off;
  return s;
}
}  // namespace

extern "C" size_t streambp_stack_workspace_bytes(const sbp_stack_cfg* cfg) {
  if (check_stack_cfg(cfg) != SBP_OK) return 0;
  return carve_stack(cfg, nullptr).bytes;
}

extern "C" int32_t streambp_stack_forward(const sbp_stack_cfg* c, const sbp_layer_weights* layers, const void* emb,
                                          const int32_t* ids, void* const* ckpt, void* workspace, size_t workspace_bytes,
                                          void* hip_stream) {
  int32_t rc = check_stack_cfg(c);
  if (rc) return rc;
  if (!layers || !ckpt || !workspace) return fail(SBP_ERR_NULL, "layers, ckpt and workspace must be non-NULL");
  if ((emb == nullptr) != (ids == nullptr)) return fail(SBP_ERR_NULL, "emb and ids must be given together");
  for (int l = 0; l <= c->n_layers; ++l) if (!ckpt[l]) return fail(SBP_ERR_NULL, "ckpt[%d] is NULL", l);
  if ((uintptr_t)workspace & 255) return fail(SBP_ERR_WORKSPACE, "workspace must be 256-byte aligned");
  const StackWs s = carve_stack(c, workspace);
  if (workspace_bytes < s.bytes) return fail(SBP_ERR_WORKSPACE, "workspace too small: %zu < %zu", workspace_bytes, s.bytes);
  const int64_t rows = (int64_t)c->layer.batch * c->layer.seq_len;
  if (emb && (rc = streambp_embedding_forward(c->layer.dtype, rows, c->layer.hidden, c->vocab, ids, emb, ckpt[0], hip_stream))) return rc;
  for (int l = 0; l < c->n_layers; ++l)
    if ((rc = streambp_layer_forward(&c->layer, &layers[l], ckpt[l], ckpt[l + 1], s.sub, s.sub_bytes, hip_stream))) return rc;
  return SBP_OK;
}

extern "C" int32_t streambp_stack_backward(const sbp_stack_cfg* c, const sbp_layer_weights* layers, const void* g_final,
                                           const void* w_head, void* const* ckpt, const int32_t* ids, const int32_t* targets,
                                           const float* old_logp, const float* ref_logp, const float* advantages,
                                           const sbp_layer_grads* dlayers, float* dg_final, void* dw_head, float* demb,
                                           void* dx0, float* loss, int64_t* n_active, void* workspace,
                                           size_t workspace_bytes, void* hip_stream) {
  int32_t rc = check_stack_cfg(c);
  if (rc) return rc;
  if (!layers || !g_final || !w_head || !ckpt || !targets || !dlayers || !dg_final || !dw_head || !loss || !n_active || !workspace)
    return fail(SBP_ERR_NULL, "a required pointer is NULL");
  if ((demb == nullptr) != (ids == nullptr)) return fail(SBP_ERR_NULL, "demb and ids must be given together");
  for (int l = 0; l <= c->n_layers; ++l) if (!ckpt[l]) return fail(SBP_ERR_NULL, "ckpt[%d] is NULL", l);
  if ((uintptr_t)workspace & 255) return fail(SBP_ERR_WORKSPACE, "workspace must be 256-byte aligned");
  const StackWs s = carve_stack(c, workspace);
  if (workspace_bytes < s.bytes) return fail(SBP_ERR_WORKSPACE, "workspace too small: %zu < %zu", workspace_bytes, s.bytes);
  const int64_t rows = (int64_t)c->layer.batch * c->layer.seq_len;
  const int d = c->layer.hidden, dt = c->layer.dtype;
  const sbp_head_cfg hc = stack_head_cfg(c);
  const int L = c->n_layers;
  // head on h = RMSNorm(x_L), then the final norm's adjoint
  if ((rc = streambp_rmsnorm_forward(dt, rows, d, c->final_eps, ckpt[L], g_final, s.h, hip_stream))) return rc;
  if ((rc = streambp_lmhead_ce_backward(&hc, w_head, s.h, targets, old_logp, ref_logp, advantages, s.dh, dw_head, loss, n_active,
                                        s.sub, s.sub_bytes, hip_stream))) return rc;
  if ((rc = streambp_rmsnorm_backward(dt, rows, d, c->final_eps, ckpt[L], g_final, s.dh, s.ga, dg_final, s.sub, s.sub_bytes, hip_stream))) return rc;
  // layers L-1 .. 0: dL/dx of layer l is dL/dy of layer l-1 (Sec. 3.1)
  void* gin = s.ga;
  void* gout = s.gb;
  for (int l = L - 1; l >= 0; --l) {
    void* dst = (l == 0 && dx0) ? dx0 : gout;
    if ((rc = streambp_layer_backward(&c->layer, &layers[l], ckpt[l], gin, dst, &dlayers[l], s.sub, s.sub_bytes, hip_stream))) return rc;
    gout = gin;
    gin = dst;
  }
  if (demb && (rc = streambp_embedding_backward(dt, rows, d, c->vocab, ids, gin, demb, hip_stream))) return rc;
  return SBP_OK;
}

// ------------------------------------------------------------ stack glue --
struct RmsnormWs { float *rstd, *partial; size_t bytes; };
static RmsnormWs carve_rmsnorm(int n_rows, int hidden, void* ws) {
  Carver cv(ws);
  RmsnormWs w;
  w.rstd = cv.take<float>((size_t)std::max(n_rows, 1));
  w.partial = cv.take<float>(rmsnorm_bwd_partial_floats(n_rows, hidden) + 64);
  w.bytes = cv.off;
  return w;
}
size_t streambp_rmsnorm_workspace_bytes(int64_t n_rows, int32_t hidden) {
  if (n_rows < 0 || n_rows > INT32_MAX || hidden < 1) return 0;
  return carve_rmsnorm((int)n_rows, hidden, nullptr).bytes;
}
int32_t streambp_rmsnorm_forward(int32_t dtype, int64_t n_rows, int32_t hidden, float eps, const void* x, const void* g,
                                 void* y, void* hip_stream) {
  if (!valid_dtype(dtype)) return fail(SBP_ERR_UNSUPPORTED, "dtype %d not supported", dtype);
  if (n_rows < 0 || n_rows > INT32_MAX || hidden < 1 || !(eps >= 0.f)) return fail(SBP_ERR_SHAPE, "bad shape");
  if (!x || !g || !y) return fail(SBP_ERR_NULL, "x, g and y must be non-NULL");
  HIPCHK(rmsnorm_fwd(dtype, x, nullptr, g, y, nullptr, nullptr, (int)n_rows, hidden, eps, (hipStream_t)hip_stream));
  return SBP_OK;
}
int32_t streambp_rmsnorm_backward(int32_t dtype, int64_t n_rows, int32_t hidden, float eps, const void* x, const void* g,
                                  const void* dy, void* dx, float* dg, void* workspace, size_t workspace_bytes,
                                  void* hip_stream) {
  if (!valid_dtype(dtype)) return fail(SBP_ERR_UNSUPPORTED, "dtype %d not supported", dtype);
  if (n_rows < 0 || n_rows > INT32_MAX || hidden < 1 || !(eps >= 0.f)) return fail(SBP_ERR_SHAPE, "bad shape");
  if (!x || !g || !dy || !dx || !dg || !workspace) return fail(SBP_ERR_NULL, "x, g, dy, dx, dg and workspace must be non-NULL");
  if ((uintptr_t)workspace & 255) return fail(SBP_ERR_WORKSPACE, "workspace must be 256-byte aligned");
  if (workspace_bytes < streambp_rmsnorm_workspace_bytes(n_rows, hidden)) return fail(SBP_ERR_WORKSPACE, "workspace too small");
  const RmsnormWs s = carve_rmsnorm((int)n_rows, hidden, workspace);
  hipStream_t st = (hipStream_t)hip_stream;
  HIPCHK(rmsnorm_fwd(dtype, x, nullptr, g, nullptr, nullptr, s.rstd, (int)n_rows, hidden, eps, st));
  HIPCHK(rmsnorm_bwd_plain(dtype, dy, x, g, s.rstd, dx, dg, s.partial, (int)n_rows, hidden, st));
  return SBP_OK;
}
int32_t streambp_embedding_forward(int32_t dtype, int64_t n_rows, int32_t hidden, int32_t vocab, const int32_t* ids,
                                   const void* emb, void* x, void* hip_stream) {
  if (!valid_dtype(dtype)) return fail(SBP_ERR_UNSUPPORTED, "dtype");
  if (n_rows < 0 || hidden < 1 || vocab < 1 || n_rows > INT32_MAX) return fail(SBP_ERR_SHAPE, "bad shape");
  if (!ids || !emb || !x) return fail(SBP_ERR_NULL, "NULL pointer");
  HIPCHK(embedding_fwd(dtype, ids, emb, x, n_rows, hidden, vocab, (hipStream_t)hip_stream));
  return SBP_OK;
}
int32_t streambp_embedding_backward(int32_t dtype, int64_t n_rows, int32_t hidden, int32_t vocab, const int32_t* ids,
                                    const void* dx, float* demb, void* hip_stream) {
  if (!valid_dtype(dtype)) return fail(SBP_ERR_UNSUPPORTED, "dtype");
  if (n_rows < 0 || hidden < 1 || vocab < 1 || n_rows > INT32_MAX) return fail(SBP_ERR_SHAPE, "bad shape");
  if (!ids || !dx || !demb) return fail(SBP_ERR_NULL, "NULL pointer");
  HIPCHK(embedding_bwd(dtype, ids, dx, demb, n_rows, hidden, vocab, (hipStream_t)hip_stream));
  return SBP_OK;
}

}  // extern "C"
