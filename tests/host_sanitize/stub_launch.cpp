// Host stand-ins for every kernel launcher declared in csrc/launch.h.  Nothing is computed: each launcher touches the
// first and the last byte of every operand extent its kernels would read or write, so that the address sanitizer
// sees exactly the memory ranges the C-ABI layer (workspace carving, chunk offsets, leading dimensions, ragged last
// chunks) hands to the kernels.  An extent that leaves its allocation is a heap-buffer-overflow report, one that leaves its buffer
// inside the workspace a use-after-poison report (the carver poisons what lies between two buffers).
#include "launch.h"

#include <algorithm>
#include <atomic>
#include <cstdio>
#include <functional>

namespace sbp {

// what a driver wants to see of the calls (plans.cpp): attention calls (backward or not), and the problems of a launch
std::function<void(const AttnArgs&, bool)> stub_on_attn;
std::function<void(const GemmArgs*, int)> stub_on_gemm_batch;

static std::atomic<long long> g_touches{0};
long long stub_touches() { return g_touches.load(); }
// a planted mistake: the head's row kernel writes one element past the last padded row of dz
bool stub_overrun = false;

static void rd(const void* p, size_t bytes) {
  if (!p || bytes == 0) return;
  volatile const unsigned char* c = (volatile const unsigned char*)p;
  (void)c[0];
  (void)c[bytes - 1];
  ++g_touches;
}
static void wr(void* p, size_t bytes) {
  if (!p || bytes == 0) return;
  volatile unsigned char* c = (volatile unsigned char*)p;
  c[0] = c[0];
  c[bytes - 1] = c[bytes - 1];
  ++g_touches;
}
static size_t es(int dt) { return dtype_size(dt); }

static void touch_gemm(const GemmArgs& g) {
  if (g.M <= 0 || g.N <= 0 || g.K <= 0) return;
  // padded operands: A is read to the next multiple of 64 reduction columns (NN) resp. of 8 output rows (TN), C written to the next
  // multiple of 4 columns
  const size_t a_m = g.ta && g.a_padded ? align_up(g.M, 8) : g.M, a_k = !g.ta && g.a_padded ? align_up(g.K, 64) : g.K;
  const size_t a_el = g.ta ? (size_t)(g.K - 1) * g.lda + a_m : (size_t)(g.M - 1) * g.lda + a_k;
  const size_t b_el = g.tb ? (size_t)(g.N - 1) * g.ldb + (g.b_padded ? align_up(g.K, 64) : g.K) : (size_t)(g.K - 1) * g.ldb + g.N;
  const size_t c_el = (size_t)(g.M - 1) * g.ldc + (g.c_padded ? align_up(g.N, 4) : g.N);
  rd(g.A, a_el * es(g.in_dt)); rd(g.B, b_el * es(g.in_dt));
  if (g.glu_up) rd(g.glu_up, b_el * es(g.in_dt));
  if (g.C0) rd(g.C0, c_el * es(g.out_dt));
  if (g.A2) { rd(g.A2, a_el * es(g.in_dt)); rd(g.B2, b_el * es(g.in_dt)); }
  if (g.swiglu_gate) {
    wr(g.swiglu_gate, c_el * es(g.out_dt)); wr(g.swiglu_up, c_el * es(g.out_dt)); wr(g.swiglu_act, c_el * es(g.out_dt));
  } else {
    wr(g.C, c_el * es(g.out_dt));
  }
  if (g.row_stats) wr(g.row_stats, (size_t)g.M * cdiv(g.N, GEMM_STAT_COLS) * sizeof(float2));
  if (g.numer_targets) { wr(g.numer_target_value, (size_t)g.M * 4); if (g.numer_row_index) rd(g.numer_row_index, (size_t)g.M * 4); }
  if (g.rows_dev) rd(g.rows_dev, sizeof(int));
  if (g.scratch) wr(g.scratch, g.scratch_bytes);     // split reductions may fill all that they are given
}
static bool nt_mfma(const GemmArgs& g) {              // the MFMA kernels' rule for C = A B^T
  return g.in_dt == DT_BF16 && !g.ta && g.tb && !g.acc && g.K % 64 == 0 && (g.N % 8 == 0 || (g.c_padded && g.ldc % 8 == 0 && g.ldc >= g.N));
}
bool gemm_row_stats_supported(const GemmArgs& g) { return nt_mfma(g) && g.out_dt == DT_F32; }
bool gemm_numerators_supported(const GemmArgs& g) {
  return nt_mfma(g) && g.out_dt == DT_BF16 && g.row_stats && g.numer_targets && g.numer_target_value;
}
bool gemm_glu_supported(const GemmArgs& g) { return g.glu_up && nt_mfma(g) && cdiv(g.M, 256) * cdiv(g.N, 128) >= 200; }
size_t gemm_scratch_bytes(int max_m, int max_n) {     // at most one partial tile per CU, 27 per output tile, of the rows that exist
  return (size_t)std::min<int64_t>(256, cdiv(max_m, 256) * cdiv(max_n, 256) * 27) * std::min(max_m, 256) * 256 * sizeof(float);
}
hipError_t gemm(const GemmArgs& g, hipStream_t) { touch_gemm(g); return hipSuccess; }
hipError_t gemm_batch(const GemmArgs* gs, int n, hipStream_t, bool) {
  if (stub_on_gemm_batch) stub_on_gemm_batch(gs, n);
  for (int i = 0; i < n; ++i) touch_gemm(gs[i]);
  return hipSuccess;
}
hipError_t gemm_sum(const GemmArgs* gs, int n, hipStream_t) { for (int i = 0; i < n; ++i) touch_gemm(gs[i]); return hipSuccess; }
bool gemm_uses_mfma(const GemmArgs& g) { return g.in_dt == DT_BF16; }
void gemm_set_force_generic(bool) {}
static int g_mask = FUSE_ROPE_Q | FUSE_NUMERATORS;
int fusion_mask() { return g_mask; }
void set_fusion_mask(int m) { g_mask = m; }
long long generic_bf16_launches() { return 0; }
void note_generic_bf16_launch() {}
namespace prof { Scope::Scope(int, double, bool, hipStream_t s) : st(s) {} Scope::~Scope() {} }

hipError_t rope_table(float2* tab, int n_pos, int dh, float, int, void* zeros, size_t zero_bytes, hipStream_t) {
  wr(tab, (size_t)n_pos * (dh / 2) * sizeof(float2)); wr(zeros, zero_bytes); return hipSuccess;
}
hipError_t rope_apply(int dt, void* x, const float2* tab, int rows, int period, int H, int dh, bool, hipStream_t) {
  wr(x, (size_t)rows * H * dh * es(dt)); rd(tab, (size_t)std::min(rows, period) * (dh / 2) * sizeof(float2)); return hipSuccess;
}
size_t rmsnorm_bwd_partial_floats(int rows, int d) { return (size_t)cdiv(rows, 4) * (size_t)d; }
hipError_t rmsnorm_fwd(int dt, const void* x, const float* add, const void* g, void* out, float* sum_out, float* rstd, int rows, int d, float, hipStream_t) {
  const size_t n = (size_t)rows * d;
  rd(x, n * es(dt)); rd(add, n * 4); rd(g, (size_t)d * es(dt)); wr(out, n * es(dt)); wr(sum_out, n * 4); wr(rstd, (size_t)rows * 4);
  return hipSuccess;
}
int rmsnorm_bwd_partial_rows(int rows) { return (int)cdiv(rows, 4); }
hipError_t rmsnorm_bwd(int dt, const float* dnorm, const void* xin, bool x_is_f32, const void* g, const float* rstd, const void* res,
                       bool res_is_f32, float* out_f32, void* out_t, float* partial, int rows, int d, hipStream_t) {
  const size_t n = (size_t)rows * d;
  rd(dnorm, n * 4); rd(xin, n * (x_is_f32 ? 4 : es(dt))); rd(g, (size_t)d * es(dt)); rd(rstd, (size_t)rows * 4);
  rd(res, n * (res_is_f32 ? 4 : es(dt))); wr(out_f32, n * 4); wr(out_t, n * es(dt));
  wr(partial, rmsnorm_bwd_partial_floats(rows, d) * 4);
  return hipSuccess;
}
hipError_t column_sums(const ColumnSums& cs, int n_dg, int d, hipStream_t) {
  for (int w = 0; w < n_dg; ++w) {
    for (int i = 0; i < cs.n; ++i) rd(cs.partial[w][i], (size_t)cs.blocks[i] * d * 4);
    wr(cs.dg[w], (size_t)d * 4);
  }
  return hipSuccess;
}
hipError_t rmsnorm_bwd_plain(int dt, const void* dy, const void* x, const void* g, const float* rstd, void* dx, float* dg, float* partial,
                             int rows, int d, hipStream_t) {
  const size_t n = (size_t)rows * d;
  rd(dy, n * es(dt)); rd(x, n * es(dt)); rd(g, (size_t)d * es(dt)); rd(rstd, (size_t)rows * 4); wr(dx, n * es(dt)); wr(dg, (size_t)d * 4);
  wr(partial, rmsnorm_bwd_partial_floats(rows, d) * 4);
  return hipSuccess;
}
hipError_t swiglu_fwd(int dt, const void* gate, const void* up, void* act, int64_t n, hipStream_t) {
  rd(gate, n * es(dt)); rd(up, n * es(dt)); wr(act, n * es(dt)); return hipSuccess;
}
hipError_t swiglu_bwd(int dt, void* gate, void* up, const void* dact, void* act, int64_t n, hipStream_t) {
  wr(gate, n * es(dt)); wr(up, n * es(dt)); rd(dact, n * es(dt)); wr(act, n * es(dt)); return hipSuccess;
}
hipError_t add_store(int dt, const float* a, const float* b, void* y, int64_t n, hipStream_t) { rd(a, n * 4); rd(b, n * 4); wr(y, n * es(dt)); return hipSuccess; }
hipError_t kv_grad_finish(int dt, const float* dK, const float* dV, const float2* tab, void* dkc, void* dvc, int rows, int H, int dh, hipStream_t) {
  const size_t n = (size_t)rows * H * dh;
  rd(dK, n * 4); rd(dV, n * 4); rd(tab, (size_t)rows * (dh / 2) * sizeof(float2)); wr(dkc, n * es(dt)); wr(dvc, n * es(dt)); return hipSuccess;
}
hipError_t fill_zero(void* p, size_t bytes, hipStream_t) { wr(p, bytes); return hipSuccess; }
hipError_t transpose_rows(const void* src, const int32_t* rows_dev, int R, int C, void* dst, int64_t ld, hipStream_t) {
  if (rows_dev) rd(rows_dev, 4);
  rd(src, (size_t)R * C * 2); wr(dst, ((size_t)(C - 1) * ld + align_up(R, 64)) * 2);
  return hipSuccess;
}
hipError_t pad_matrices(int dt, PadJobs jobs, hipStream_t) {
  for (int k = 0; k < jobs.n; ++k) {
    const PadJob& p = jobs.job[k];
    rd(p.src, (size_t)p.R * p.C * es(dt)); wr(p.dst, (size_t)p.R2 * p.C2 * es(dt));
  }
  return hipSuccess;
}
hipError_t add_scaled_blocks(AddJobs jobs, float, hipStream_t) {
  for (int k = 0; k < jobs.n; ++k) {
    const AddJob& p = jobs.job[k];
    if (p.R > 0 && p.C > 0) { rd(p.src, ((size_t)(p.R - 1) * p.ld + p.C) * 4); wr(p.dst, (size_t)p.R * p.C * 4); }
  }
  return hipSuccess;
}
hipError_t embedding_fwd(int dt, const int32_t* ids, const void* emb, void* x, int64_t rows, int d, int vocab, hipStream_t) {
  rd(ids, rows * 4); rd(emb, (size_t)vocab * d * es(dt)); wr(x, (size_t)rows * d * es(dt)); return hipSuccess;
}
hipError_t embedding_bwd(int dt, const int32_t* ids, const void* dx, float* demb, int64_t rows, int d, int vocab, hipStream_t) {
  rd(ids, rows * 4); rd(dx, (size_t)rows * d * es(dt)); wr(demb, (size_t)vocab * d * 4); return hipSuccess;
}

static void touch_attn(const AttnArgs& a, bool bwd) {
  if (stub_on_attn) stub_on_attn(a, bwd);
  const size_t nb = a.batch, qn = nb * a.q_len * a.Hq * a.dh, kn = nb * (a.q_start + a.q_len) * a.Hkv * a.dh;
  if (a.rope_q && !bwd) wr((void*)a.q, qn * es(a.dt)); else rd(a.q, qn * es(a.dt));
  rd(a.k, kn * es(a.dt)); rd(a.v, kn * es(a.dt));
  if (a.rope_q) rd(a.rope_q, (size_t)a.q_len * (a.dh / 2) * sizeof(float2));
  if (!bwd) { wr(a.o, qn * es(a.dt)); wr(a.lse, nb * a.Hq * a.q_len * 4); return; }
  rd(a.o, qn * es(a.dt)); rd(a.lse, nb * a.Hq * a.q_len * 4); rd(a.d_o, qn * es(a.dt)); wr(a.dq, qn * es(a.dt));
  wr(a.dk, kn * 4); wr(a.dv, kn * 4); wr(a.delta, nb * 2 * a.Hq * a.q_len * 4);
  if (a.dkc) {
    const size_t cn = nb * a.q_len * a.Hkv * a.dh * es(a.dt);
    wr(a.dkc, cn); wr(a.dvc, cn); rd(a.rope_k, (size_t)a.q_len * (a.dh / 2) * sizeof(float2));
  }
  if (a.dkv_scratch) wr(a.dkv_scratch, attn_dkv_scratch_bytes(a, a.dkv_slices));     // the parts of split key blocks
}
hipError_t attn_forward(const AttnArgs& a, hipStream_t) { if (a.q_len > 0) touch_attn(a, false); return hipSuccess; }
hipError_t attn_backward(const AttnArgs& a, hipStream_t) { if (a.q_len > 0) touch_attn(a, true); return hipSuccess; }
bool attn_uses_mfma(int dt, int dh, int Hq, int Hkv) { return dt == DT_BF16 && (dh == 128 || dh == 64) && Hq % Hkv == 0; }
void attn_set_force_generic(bool) {}

hipError_t head_rows(const HeadRowArgs& a, hipStream_t) {
  const size_t n = (size_t)a.rows * a.ldz;            // rows are padded; dz is written to their end
  if (a.target_logit) { rd(a.target_logit, (size_t)a.rows * 4); rd(a.dz, n * es(a.dt)); }
  else rd(a.z, ((size_t)(a.rows - 1) * a.ldz + (a.ldz % 4 == 0 ? align_up(a.V, 4) : a.V)) * 4);
  wr(a.dz, n * es(a.dt) + (stub_overrun ? 1 : 0)); wr(a.row_loss, (size_t)a.rows * 4);
  if (a.stats) rd(a.stats, (size_t)a.rows * a.n_stat * sizeof(float2));
  if (a.row_index) rd(a.row_index, (size_t)a.rows * 4);
  if (a.rows_dev) rd(a.rows_dev, 4);
  return hipSuccess;
}
hipError_t head_begin(const HeadBegin& a, hipStream_t) {
  const size_t rows = (size_t)a.B * a.T;
  rd(a.targets, rows * 4); wr(a.seq_weight, (size_t)a.B * 4); wr(a.n_active, 8); wr(a.ell, 4); wr(a.index, rows * 4); wr(a.unit_rows, (size_t)(a.n_units + 1) * 4);
  if (a.n_spans) wr(a.span_rows, (size_t)a.n_spans * 4);
  wr(a.dh, a.dh_bytes); return hipSuccess;
}
hipError_t move_rows(int dt, const RowMove& scatter, const RowMove& gather, int d, hipStream_t, const LossSum& sum) {
  if (sum.n > 0) { rd(sum.v, (size_t)sum.n * 4); wr(sum.out, 4); rd(sum.n_dev, 4); }
  if (scatter.max_rows > 0) { rd(scatter.src, (size_t)scatter.max_rows * d * es(dt)); rd(scatter.index, (size_t)scatter.max_rows * 4); rd(scatter.rows_dev, 4); }
  if (gather.max_rows > 0) { rd(gather.index, (size_t)gather.max_rows * 4); rd(gather.rows_dev, 4); wr(gather.dst, (size_t)gather.max_rows * d * es(dt)); }
  return hipSuccess;
}
hipError_t dpo_finish(int dt, const float* ell, float, void* dh, int64_t n_dh, void* dw, int dw_dt, int64_t n_dw, float* loss, hipStream_t) {
  rd(ell, 4); wr(dh, n_dh * es(dt)); wr(dw, n_dw * es(dw_dt)); wr(loss, 4); return hipSuccess;
}

}  // namespace sbp
