// Host-side launchers of the HIP kernels.  Every function only enqueues work on
// `st`; none allocates or synchronises.  Shapes are validated by the callers in
// api.hip before anything is launched.
#pragma once
#include "common.h"

namespace sbp {

// C[M,N] (=|+=) sum_k A(m,k) * B(k,n), fp32 accumulation.
//   A(m,k) = ta ? A[k*lda + m] : A[m*lda + k]
//   B(k,n) = tb ? B[n*ldb + k] : B[k*ldb + n]
// in_dt: element type of A and B; out_dt: element type of C; acc: C += (fp32 C only).
struct GemmArgs {
  const void* A; const void* B; void* C;
  int M, N, K;
  int64_t lda, ldb, ldc;
  bool ta, tb;
  int in_dt, out_dt;
  bool acc;
  float* scratch = nullptr;      // optional fp32 scratch for split-K partial tiles
  size_t scratch_bytes = 0;
  // Optional device-side count of valid "rows" (the M dimension of NT / NN problems, the K dimension of the
  // dW form): the kernels read it at run time and skip the work beyond it; the host-side M (resp. K) is the
  // upper bound the launch is sized for.
  const int* rows_dev = nullptr;
  // Optional second operand pair of the same shapes and leading dimensions: C (=|+=) A B + A2 B2 in one launch, as one reduction of
  // twice the length (split over workgroups or not), also in the shape-agnostic kernel; two launches where the MFMA kernel takes one pair alone.
  const void* A2 = nullptr;
  const void* B2 = nullptr;
  // Optional row statistics of the output (store form C = A B^T with fp32 C, MFMA kernel only: ask
  // gemm_row_stats_supported first): row_stats[m * ceil(N / GEMM_STAT_COLS) + t] = (max, sum of exp(c - max)) of row m
  // over the columns [t * GEMM_STAT_COLS, (t + 1) * GEMM_STAT_COLS), taken from the fp32 accumulators.
  float2* row_stats = nullptr;
  // Optional "softmax numerators" form of the row-statistics store (C bf16, MFMA kernel only: ask
  // gemm_numerators_supported first).  C does not receive the product c but exp(c - max), max being the row's maximum
  // over the element's block of GEMM_STAT_COLS columns - the same (max, sum of exp) pairs go to row_stats, the sums
  // taken from the unrounded fp32 values - and the product's value in column numer_targets[r] of row m goes to
  // numer_target_value[m] (fp32), r = numer_row_index ? numer_row_index[m] : m; a target outside [0, N) matches no
  // column and leaves the entry untouched.  What a softmax over the row needs is then all there in half the bytes:
  // softmax(c)[n] = C[m, n] * exp(max_block(n) - lse(m)).
  const int32_t* numer_targets = nullptr;
  const int32_t* numer_row_index = nullptr;
  float* numer_target_value = nullptr;
  // Optional fused SwiGLU adjoint (store form C = A B with the same row-major [M, N] layout and leading dimension for
  // C, gate, up and act; bf16): the product is the gradient wrt act = silu(gate) * up and is never stored; instead the
  // epilogue reads the tile's gate and up values and writes act (what the forward would have produced; optional),
  // gate <- d gate and up <- d up in place.  The shape-agnostic kernel has the same epilogue.  Where the MFMA kernel cannot take
  // it the dispatcher runs the plain product into C and the elementwise kernel - same results up to the rounding of the product to bf16.
  void* swiglu_gate = nullptr;
  void* swiglu_up = nullptr;
  void* swiglu_act = nullptr;
  // A is padded: its rows (NN: columns K .. next multiple of 64, which hold zeros; TN: columns M .. next multiple of 8, any finite
  // values) reach further than the operand, so K (NN) and M (TN) need not be multiples of anything.
  bool a_padded = false;
  // B of C += A^T B^T (stored [N, K]) is padded: its rows reach to the next multiple of 64 with finite values
  bool b_padded = false;
  // C = A B^T is padded: its rows reach to ldc, a multiple of 8, so N need not be a multiple of anything (columns N .. next multiple of 4
  // receive finite values of no meaning).
  bool c_padded = false;
  // Optional second B of the store form C = A B^T (bf16): C receives silu(A B^T) * (A glu_up^T), neither product is stored (MFMA kernel only: ask
  // gemm_glu_supported first)
  const void* glu_up = nullptr;
  // Accumulated bf16 C: C = C0 + A B instead (C0 laid out like C)
  const void* C0 = nullptr;
  // Optional rotary embedding of a stored C = A B^T (fp32, one of a launch's problems): heads of rope_dim columns, a divisor of GEMM_ROPE_COLS, row r by row
  // r % rope_period of the table
  const float2* rope = nullptr;
  int rope_dim = 0, rope_period = 0;
  // Outputs of few tiles may go to the kernels of gemm_few.hip (which split no reduction over workgroups and leave `scratch` alone)
  bool few_ok = false;
};
constexpr int GEMM_STAT_COLS = 256;
constexpr int GEMM_ROPE_COLS = 32;      // (of a tile of the shape-agnostic kernel, which all fp32 products run on)
bool gemm_row_stats_supported(const GemmArgs& g);
bool gemm_numerators_supported(const GemmArgs& g);
bool gemm_glu_supported(const GemmArgs& g);
// upper bound of the scratch a GEMM with M <= max_m rows and N <= max_n columns may use
size_t gemm_scratch_bytes(int max_m, int max_n);
hipError_t gemm(const GemmArgs& g, hipStream_t st);
// n independent GEMMs (distinct outputs); one grouped launch when the MFMA kernel can take them all, or the shape-agnostic one (of that also several that add to
// one output, after one that stores it)
// group_small: take the grouped launch also when the problems together have few output tiles (skinny problems)
hipError_t gemm_batch(const GemmArgs* gs, int n, hipStream_t st, bool group_small = false);
struct FewChoice { int tm, tn; double us; };      // output tile of gemm_few_k (0: not for it) and estimated time
// C = sum of n products (gs[0] stores, the others, with acc set, add to the same C): one launch where the kernels for few output tiles are the
// faster ones, otherwise gemm(gs[0]) and gemm_batch of the rest
hipError_t gemm_sum(const GemmArgs* gs, int n, hipStream_t st);
// true when the bf16 MFMA kernel can take this problem (used by tests / tile accounting)
bool gemm_uses_mfma(const GemmArgs& g);
// force the generic kernel (debug / A-B tests)
void gemm_set_force_generic(bool on);
// which of the optional fusions the entry points use (A/B measurements): bit 0 = SwiGLU adjoint in the epilogue of the
// dact GEMM, bit 1 = rotary embedding of q / its adjoint on dq inside the attention kernels, bit 2 = the LM head's logits
// GEMM stores bf16 softmax numerators (and the target logits) instead of fp32 logits
enum { FUSE_SWIGLU = 1, FUSE_ROPE_Q = 2, FUSE_NUMERATORS = 4 };
int fusion_mask();
void set_fusion_mask(int mask);
// bf16 problems that have run on the shape-agnostic kernels since the library was loaded
long long generic_bf16_launches();
void note_generic_bf16_launch();

// ---- optional per-launch timing (off unless streambp_debug_profile_begin was called) ----
namespace prof {
// kinds 0..11: gemm_mfma_k<layout, mode> with layout NT=0, NN=1, TN=2 and mode 0, 1, 2 (slot 3 unused); 12..23: the grouped kernel;
// then the shape-agnostic GEMM, the attention forward / backward launch sequences, the segmented weight-gradient GEMM and the
// store form with row statistics (gemm_mfma_k<NT, 5>), the input-gradient form with the fused SwiGLU adjoint (gemm_mfma_k<NN, 6>)
// and the softmax-numerator store (gemm_mfma_k<NT, 7>), the kernels for outputs of few tiles (gemm_few_k), the gated
// store (gemm_mfma_k<NT, 8>)
enum { GEMM_SINGLE = 0, GEMM_GROUP = 12, GEMM_GENERIC = 24, ATTN_FWD = 25, ATTN_BWD = 26, GEMM_SEG = 27, GEMM_STATS = 28, GEMM_SWIGLU = 29,
       GEMM_NUMER = 30, GEMM_FEW = 31, GEMM_GLU = 32, N_KIND = 33 };
struct Scope {
  hipStream_t st; bool active = false; int kind = 0; double work = 0; bool bounded = false; hipEvent_t e0{}, e1{};
  // bounded: `work` was computed from a host-side upper bound of a run-time row count
  Scope(int kind, double work, bool bounded, hipStream_t st);
  ~Scope();
};
}  // namespace prof

// ---- elementwise / row kernels (dt = storage type of the T-typed tensors) ----
// cos/sin table [n_pos, dh/2] (float2), angles evaluated in fp64; in the same launch zeros (16-byte aligned, zero_bytes % 16 == 0) become zero.
hipError_t rope_table(float2* tab, int n_pos, int dh, float theta, int pos_offset, void* zeros, size_t zero_bytes, hipStream_t st);
// in-place rotation of x [rows, H, dh]; tab points at the row of position 0 of these rows, which starts again after `period` of them.
hipError_t rope_apply(int dt, void* x, const float2* tab, int rows, int period, int H, int dh, bool inverse, hipStream_t st);
// out = g * (x + add) * rstd ; sum_out = x + add (fp32, optional, may be add itself) ; rstd per row
hipError_t rmsnorm_fwd(int dt, const void* x, const float* add, const void* g, void* out, float* sum_out,
                       float* rstd, int rows, int d, float eps, hipStream_t st);
// adjoint: dnorm [rows,d] fp32 is the gradient wrt the normalised output.
//   xin: the tensor that was normalised (x_is_f32 ? fp32 : dt);  res: gradient flowing around the norm
//   (res_is_f32 ? fp32 : dt);  out_f32 / out_t (either may be NULL) = res + dx_norm; out_f32 may be dnorm itself;
//   partial (may be NULL; rmsnorm_bwd_partial_floats floats) = rows whose column sums are those of dnorm * xin * rstd: what dg grows by, through
//   column_sums (two-stage, deterministic)
hipError_t rmsnorm_bwd(int dt, const float* dnorm, const void* xin, bool x_is_f32, const void* g,
                       const float* rstd, const void* res, bool res_is_f32, float* out_f32, void* out_t,
                       float* partial, int rows, int d, hipStream_t st);
size_t rmsnorm_bwd_partial_floats(int rows, int d);
int rmsnorm_bwd_partial_rows(int rows);
// dg[w] += column sums of n buffers partial[w][i] of blocks[i] rows, w < n_dg
struct ColumnSums { int n; int blocks[8]; const float* partial[2][8]; float* dg[2]; };
hipError_t column_sums(const ColumnSums& cs, int n_dg, int d, hipStream_t st);
// dy, x, dx in dt; no residual branch
hipError_t rmsnorm_bwd_plain(int dt, const void* dy, const void* x, const void* g, const float* rstd, void* dx,
                             float* dg, float* partial, int rows, int d, hipStream_t st);
// recompute rstd only (used when the statistic was not kept): not needed by the layer path
hipError_t swiglu_fwd(int dt, const void* gate, const void* up, void* act, int64_t n, hipStream_t st);
// in place: gate <- dgate, up <- dup, given dact; act (optional, may be dact itself) <- silu(gate) * up of the incoming values, the same
// numbers swiglu_fwd writes (for callers that need act only in the backward)
hipError_t swiglu_bwd(int dt, void* gate, void* up, const void* dact, void* act, int64_t n, hipStream_t st);
// y = T(a + b) with a, b fp32
hipError_t add_store(int dt, const float* a, const float* b, void* y, int64_t n, hipStream_t st);
// dkc = T(RoPE^T(dK rows)), dvc = T(dV rows);  dK, dV fp32 [rows, H, dh]
hipError_t kv_grad_finish(int dt, const float* dK, const float* dV, const float2* tab, void* dkc, void* dvc,
                          int rows, int H, int dh, hipStream_t st);
hipError_t fill_zero(void* p, size_t bytes, hipStream_t st);
// MFMA rate probe: operands = 32768 bf16 values on the device, sink = workgroups * 512 floats; lds_reads = 0, 6 or 8 of the
// eight A fragments of a round re-read from LDS
hipError_t mfma_rate_probe(const void* operands, float* sink, int workgroups, int iters, int lds_reads, hipStream_t st);
hipError_t copy_bytes(void* dst, const void* src, size_t bytes, hipStream_t st);     // 16-byte aligned, bytes % 16 == 0 fast path
// Small matrices, up to 21 in one launch: dst [R2, C2] (dt, dense) = zero-padded scale * src, src [R, C] (dt, dense) or its transpose (src [C, R])
struct PadJob { const void* src; void* dst; int R, C, transposed, R2, C2; float scale; int64_t begin; };      // begin: set by pad_matrices
struct PadJobs { int n; PadJob job[21]; };
hipError_t pad_matrices(int dt, PadJobs jobs, hipStream_t st);
// ... up to 14: dst [R, C] fp32 (dense) += scale * src[i * ld + j]
struct AddJob { const float* src; int64_t ld; float* dst; int R, C; int64_t begin; };
struct AddJobs { int n; AddJob job[14]; };
hipError_t add_scaled_blocks(AddJobs jobs, float scale, hipStream_t st);
// ids outside [0, vocab) are never used as an index: their x row is zero, their dx row is dropped
hipError_t embedding_fwd(int dt, const int32_t* ids, const void* emb, void* x, int64_t rows, int d, int vocab, hipStream_t st);
hipError_t embedding_bwd(int dt, const int32_t* ids, const void* dx, float* demb, int64_t rows, int d, int vocab, hipStream_t st);

// ---- chunk attention ----
constexpr int ATTN_MAX_SEQS = 32;
struct AttnSeqs { int n; int first[ATTN_MAX_SEQS]; };      // sequences of a launch, the first visible key of each
struct AttnArgs {
  int dt;
  int Hq, Hkv, dh;
  int q_start, q_len;
  float scale;
  int window = 0;          // > 0: a query at position t sees only keys t - window < u <= t
  int kv_first = 0;        // key positions before this one are padding: never visible
  // Several sequences in one call, up to ATTN_MAX_SEQS: `batch` of q_len queries and keys each, one behind the other (q_start = 0; lse [batch, Hq, c],
  // delta [batch, 2, Hq, c]), kv_firsts their kv_first on the host (or NULL: kv_first for all; else kv_first is the least of them).
  int batch = 1;
  const int32_t* kv_firsts = nullptr;
  const void *q, *k, *v;   // q [c,Hq,dh]; k,v [>=s+c,Hkv,dh]
  void* o; float* lse;     // o [c,Hq,dh]; lse [Hq,c]
  const void* d_o; void* dq; float *dk, *dv;
  float* delta;            // [2,Hq,c] scratch (backward): delta, then the log2-domain log-sum-exp
  // dK/dV: slices that the queries of a key block are cut into (attn_dkv_slices), and the optional fp32 scratch (16-byte aligned,
  // attn_dkv_scratch_bytes) that lets a workgroup take each
  int dkv_slices = 1;
  float* dkv_scratch = nullptr;
  // Optional rotary embedding of the chunk's queries folded into the attention kernels: cos/sin rows [c, dh/2] of the
  // chunk's positions.  Forward: q arrives un-rotated, is rotated on load and written back rotated (q must then be
  // writable); backward: q is the rotated tensor the forward left, and dq leaves the kernel already rotated back
  // (the adjoint rotation), i.e. as the gradient wrt the un-rotated projection.
  const float2* rope_q = nullptr;
  // Optional (backward): the chunk's own rows of dK and dV are final after this call; dkc = T(RoPE^T(dK rows)), dvc = T(dV rows), with the
  // cos/sin rows [c, dh/2] of the chunk's positions
  void *dkc = nullptr, *dvc = nullptr;
  const float2* rope_k = nullptr;
};
hipError_t attn_forward(const AttnArgs& a, hipStream_t st);
hipError_t attn_backward(const AttnArgs& a, hipStream_t st);
bool attn_uses_mfma(int dt, int dh, int Hq, int Hkv);
void attn_set_force_generic(bool on);
constexpr int ATTN_TILE_Q = 256;   // rows of queries per workgroup in the MFMA kernels (8 waves x 32 rows)
constexpr int ATTN_WAVE_Q = 32;    // rows of queries per wave: the granularity at which key tiles are skipped
constexpr int ATTN_TILE_K = 64;    // keys per inner step
constexpr int ATTN_KV_TILE = 128;  // dK/dV: keys per workgroup
constexpr int ATTN_KV_QUERIES = 64;   // dK/dV: queries per step

// dK/dV of the MFMA kernels: one workgroup per 128 keys and K/V head walks the query tiles of the group's heads.  Where these are not whole
// rounds of the 256 CUs the walk is cut into slices, a workgroup each: their sums meet in scratch, in a fixed order.  The number of
// slices is a property of the sizes - without the scratch one workgroup walks them in turn - so the results of the attention entry
// points do not depend on the scratch.  Cost of s slices in steps (one step, 64 queries, takes about 1.9 us): the rounds, each with the share's steps and about
// three more for a workgroup's start and the 128 KB that it leaves, and the pass that adds the parts (2 us, 4 TB/s).
// max_bytes bounds the scratch that the slices need.
inline int attn_first_key_block(const AttnArgs& a) {
  const int first_visible = a.window > 0 && a.q_start - a.window + 1 > a.kv_first ? a.q_start - a.window + 1 : a.kv_first;
  return (first_visible > 0 ? first_visible : 0) / ATTN_KV_TILE;
}
constexpr int ATTN_MAX_SLICES = 32;
inline size_t attn_dkv_scratch_bytes(const AttnArgs& a, int slices) {      // [sequence][slice][dk | dv][key][kv head][dh] fp32, keys from the first visible block on
  const int64_t keys = (int64_t)a.q_start + a.q_len - (int64_t)attn_first_key_block(a) * ATTN_KV_TILE;
  return slices < 2 || keys <= 0 ? 0 : (size_t)(a.batch * slices * 2 * keys * a.Hkv * a.dh) * sizeof(float);
}
inline int attn_dkv_slices(const AttnArgs& a, size_t max_bytes) {
  const int64_t blocks = (cdiv((int64_t)a.q_start + a.q_len, ATTN_KV_TILE) - attn_first_key_block(a)) * a.Hkv * a.batch;
  if (blocks <= 0) return 1;
  int64_t tiles = cdiv(a.q_len, ATTN_KV_QUERIES);
  if (a.window > 0 && tiles > cdiv((int64_t)a.window + ATTN_KV_TILE, ATTN_KV_QUERIES) + 1) tiles = cdiv((int64_t)a.window + ATTN_KV_TILE, ATTN_KV_QUERIES) + 1;
  const int64_t steps = tiles * (a.Hq / a.Hkv);
  int best = 1;
  double best_cost = 0.0;
  for (int s = 1; s == 1 || (s <= ATTN_MAX_SLICES && blocks * s <= 512 && steps / s >= 2 && attn_dkv_scratch_bytes(a, s) <= max_bytes); ++s) {
    const double cost = (double)cdiv(blocks * s, 256) * (double)(cdiv(steps, s) + 3) + (s > 1 ? 1.0 + 0.02 * (double)(blocks * s) : 0.0);
    if (s == 1 || cost < best_cost) { best = s; best_cost = cost; }
  }
  return best;
}

// ---- LM head rows ----
struct HeadRowArgs {
  int dt;                   // type of dz
  int objective;            // 0 SFT, 1 GRPO, 2 DPO
  const float* z;           // [rows, ldz] fp32 logits (unused in the numerator form); fp32 dz may be the same buffer
  void* dz;                 // [rows, ldz] dt, columns V .. ldz become zeros; numerator form (target_logit != NULL): holds exp(z - block max) on entry
  int64_t ldz;
  const int32_t* targets;   // [rows] (already offset to the chunk)
  const float* old_logp;    // [rows] or NULL
  const float* ref_logp;    // [rows] or NULL
  const float* advantages;  // [B] or NULL
  const float* seq_weight;  // [B] GRPO: 1/(B*T_o,j); NULL otherwise
  int64_t row0;             // global row index of the chunk's first row (row / T = sequence)
  const int32_t* row_index; // optional: original row of each chunk row (compacted chunks); then targets / old_logp /
                            // ref_logp are indexed by it and row0 is ignored
  const int* rows_dev;      // optional device-side count of valid chunk rows (<= rows)
  const float2* stats;      // optional [rows, n_stat]: per row and column block (max, sum of exp(z - max)) from the logits
  int n_stat;               // GEMM; the kernel then reads z once instead of twice
  const float* target_logit; // optional [rows]: z[row, target] from the logits GEMM's numerator form (needs stats, bf16 dz)
  int rows, V, T;
  float loss_scale, clip_eps, kl_beta; int kl_mode;
  float* row_loss;          // [rows] scratch: per-row loss term (DPO: per-row signed log-ratio)
};
hipError_t head_rows(const HeadRowArgs& a, hipStream_t st);
// What a head call starts with.  Active rows: 0 <= target < V; seq_weight[j] = 1/(B*T_o,j) of the active rows T_o,j of sequence j (0 if there are none);
// n_active: their total - or minus the number of targets >= V if there is any; index[0..n_active): the active rows in increasing order;
// unit_rows[i] = clamp(n_active - i*unit, 0, unit) for i < n_units, unit_rows[n_units] = n_active; span_rows, group_rows: the same for n_spans spans of `span` rows and
// n_groups groups of `group`;
// ell (or NULL) and dh_bytes of dh become zeros
struct HeadBegin {
  const int32_t* targets; int B, T, V;
  float* seq_weight; int64_t* n_active; float* ell;
  int32_t* index; int32_t* unit_rows; int unit, n_units; int32_t* span_rows; int span, n_spans; int32_t* group_rows; int group, n_groups;
  void* dh; size_t dh_bytes;
};
hipError_t head_begin(const HeadBegin& a, hipStream_t st);
// A gather, dst[r,:] = src[index[r],:] for r < *rows_dev, zero rows after, and a scatter, dst[index[r],:] = src[r,:] for r < *rows_dev, independent of
// each other, in one launch; max_rows 0: none.  With them out += sum(v[0..n)), n > 0, in a fixed order; n_dev: device-side count of the list that v[0]
// is entry `first` of
struct RowMove { const void* src; const int32_t* index; const int* rows_dev; void* dst; int max_rows; };
struct LossSum { const float* v; int n; float* out; const int* n_dev; int first; };
hipError_t move_rows(int dt, const RowMove& scatter, const RowMove& gather, int d, hipStream_t st, const LossSum& sum = LossSum{});
// dst [C, ld] = src [R, C]^T (bf16, C % 8 == 0, 16-byte aligned); rows_dev: only the first *rows_dev rows count.  Columns from there to the next
// multiple of 64 become zeros (ld reaches to R's next multiple of 64, % 8 == 0); those after it are not written.
hipError_t transpose_rows(const void* src, const int32_t* rows_dev, int R, int C, void* dst, int64_t ld, hipStream_t st);
// DPO fix-up: factor = sigmoid(beta*ell)-1 ; scales dh (dt) and dw (fp32) in place, loss += -log sigmoid(beta*ell)
hipError_t dpo_finish(int dt, const float* ell, float beta, void* dh, int64_t n_dh, void* dw, int dw_dt, int64_t n_dw,
                      float* loss, hipStream_t st);

}  // namespace sbp
