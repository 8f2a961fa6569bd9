// Shape-agnostic chunk attention (any head_dim <= 256, fp32 or bf16 storage, fp32 products and sums): the path of the fp32
// configuration and of head sizes the bf16 MFMA kernels do not take.  Query row t of the chunk sits at global position
// q_start + t and sees keys 0 .. q_start + t; the causal mask is an integer
// comparison of positions, never a stored tensor, and so are the two optional
// rules: a sliding window (keys t - window < u <= t) and padding in front of the
// sequence (keys before kv_first hidden).  A query that sees no key gets o = 0,
// lse = -inf and sends no gradient.  No atomics: every output element has
// exactly one owner, so results are reproducible.
//
// fp32 MFMAs (v_mfma_f32_16x16x4_f32) straight from registers, 16 queries (forward, dQ) or 16 keys (dK/dV) of a head per workgroup, the
// other dimension dealt to its eight waves in blocks of 16, which meet in LDS at the end.  What bounds the calls of the small configuration
// is the chain of dependent loads, not arithmetic: one query (key) per workgroup, with its second product on as many threads as the
// head is wide, walked 256 keys one after the other (64 queries, 4 heads of 16, up to 256 keys, with the rotary embedding: forward 14.8 -> 5.8 us, dQ
// with delta 13.5 -> 5.3, dK/dV 11.8 -> 4.8).
//
// Layout: a score block has 16 rows (keys; dK/dV: queries) in registers, rows 4 (l / 16) + r, and its 16 columns across lanes, l % 16.  MFMA j
// of the first product takes element j of both operands' four at head_dim 16 d + 4 (l / 16) .. + 3; MFMA r of the second product takes
// accumulator register r as its B operand, i.e. row 4 (l / 16) + r of the block as its reduction index.
#include "launch.h"
#include "device.h"

namespace sbp {

constexpr int AG_WAVES = 8, AG_THREADS = AG_WAVES * 64;
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef bf16_t bf16x4 __attribute__((ext_vector_type(4)));

// four elements of a head from element e on; past the head: zeros
template <typename T>
__device__ __forceinline__ f32x4 head4(const T* __restrict__ p, int e, int dh, bool vec) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (vec && e < dh) {           // (heads of a multiple of four elements)
    if constexpr (sizeof(T) == 4) v = *(const f32x4*)(p + e);
    else {
      const bf16x4 w = *(const bf16x4*)(p + e);
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = (float)w[j];
    }
  } else if (!vec) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (e + j < dh) v[j] = ldf(p + e + j);
  }
  return v;
}
template <typename T> __device__ __forceinline__ float stored(float x) { T t; stf(&t, x); return ldf(&t); }      // as T holds it
// Heads of up to 64 elements load a block's operands before its products; wider ones, whose registers they would not fit, one 16-wide piece at a time.
template <int DB> constexpr bool AHEAD = DB <= 4;
template <int DB, typename F>
struct Pieces {
  f32x4 held[AHEAD<DB> ? DB : 1];
  F load;
  __device__ __forceinline__ explicit Pieces(F f) : load(f) {
    if constexpr (AHEAD<DB>) {
#pragma unroll
      for (int d = 0; d < DB; ++d) held[d] = load(d);
    }
  }
  __device__ __forceinline__ f32x4 operator()(int d) const {
    if constexpr (AHEAD<DB>) return held[d];
    else return load(d);
  }
};
template <int DB, typename F> __device__ __forceinline__ Pieces<DB, F> pieces(F f) { return Pieces<DB, F>(f); }
#define AG_PIECE_DONE(d) do { if (!AHEAD<DB> && ((d) & 1)) __builtin_amdgcn_sched_barrier(0); } while (0)
#define AG_MFMA(a, b, c) __builtin_amdgcn_mfma_f32_16x16x4f32((a), (b), (c), 0, 0, 0)
__device__ __forceinline__ float over_groups(float x) { x += __shfl_xor(x, 16, WAVE); return x + __shfl_xor(x, 32, WAVE); }

// acc^T [element][column] += X^T [element][row] P [row][column], X's 16 rows as frag(d)[r] = X[4 (l / 16) + r][16 d + l % 16].  `edge`: some (row, column)
// pairs of the block are hidden, seen[r] says which are not: a row that holds infinities or NaN must not reach the columns it is hidden
// from (0 * NaN), so such blocks go pair by pair, with x(row, element).
template <int DB, typename F, typename X>
__device__ __forceinline__ void second_product(f32x4 (&acc)[DB], const F& frag, const f32x4& p, bool edge, const bool (&seen)[4], int dh, X x) {
  if (edge) {
    bool odd = false;
#pragma unroll
    for (int d = 0; d < DB; ++d) {
      const f32x4 v = frag(d);
#pragma unroll
      for (int r = 0; r < 4; ++r) odd = odd || !(fabsf(v[r]) < INFINITY);
      AG_PIECE_DONE(d);
    }
    if (__builtin_amdgcn_ballot_w64(odd) != 0) {
      const int li = threadIdx.x & 15, lg = (threadIdx.x & 63) >> 4;
#pragma unroll 1
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float pr = __shfl(p[r], g * 16 + li, WAVE);
          const bool vis = __shfl(seen[r] ? 1 : 0, g * 16 + li, WAVE) != 0;
#pragma unroll
          for (int d = 0; d < DB; ++d)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (vis && d * 16 + 4 * lg + e < dh) acc[d][e] = fmaf(x(4 * g + r, d * 16 + 4 * lg + e), pr, acc[d][e]);
        }
      return;
    }
  }
#pragma unroll
  for (int d = 0; d < DB; ++d) {
    const f32x4 v = frag(d);
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[d] = AG_MFMA(v[r], p[r], acc[d]);
    AG_PIECE_DONE(d);
  }
}

struct AgShape { int Hq, Hkv, dh, q_start, c; float scale; int window, kv_first, vec; };
__device__ __forceinline__ int first_key(const AgShape& a, int pos) { return max(a.kv_first, a.window > 0 ? pos - a.window + 1 : 0); }

// ---- forward.  rope: q arrives un-rotated, is rotated on load and written back rotated.
template <typename T, int DB>
__global__ __launch_bounds__(AG_THREADS) void attn_fwd_generic_k(T* q, const T* __restrict__ k, const T* __restrict__ v, T* __restrict__ o,
                                                                 float* __restrict__ lse, AgShape a, const float2* __restrict__ rope) {
  __shared__ float sO[AG_WAVES][DB * 16][17];
  __shared__ float sM[AG_WAVES][16], sL[AG_WAVES][16];
  const int h = blockIdx.y, t0 = blockIdx.x * 16, kvh = h / (a.Hq / a.Hkv);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), li = threadIdx.x & 15, lg = (threadIdx.x & 63) >> 4;
  const bool vec = a.vec != 0;
  const int64_t kv_stride = (int64_t)a.Hkv * a.dh;
  const T *kb = k + (int64_t)kvh * a.dh, *vb = v + (int64_t)kvh * a.dh;
  const int t = min(t0 + li, a.c - 1), pos = a.q_start + t;                    // my query
  const int lo = first_key(a, pos), n_keys = a.q_start + min(t0 + 16, a.c);
  f32x4 qf[DB];
  if (rope) {
    const int half = a.dh / 2;
    float* rot = &sO[0][0][0];                                                 // [16][DB * 16]
    for (int i = threadIdx.x; i < 16 * a.dh; i += AG_THREADS) {
      const int row = i / a.dh, e = i % a.dh, tr = min(t0 + row, a.c - 1);
      const T* p = q + ((int64_t)tr * a.Hq + h) * a.dh;
      const bool up = e >= half;
      const float2 cs = rope[(int64_t)tr * half + (up ? e - half : e)];
      const float other = ldf(p + (up ? e - half : e + half));
      rot[row * (DB * 16) + e] = stored<T>(ldf(p + e) * cs.x + (up ? other : -other) * cs.y);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 16 * a.dh; i += AG_THREADS) {
      const int row = i / a.dh, e = i % a.dh;
      if (t0 + row < a.c) stf(q + ((int64_t)(t0 + row) * a.Hq + h) * a.dh + e, rot[row * (DB * 16) + e]);
    }
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int j = 0; j < 4; ++j) qf[d][j] = d * 16 + 4 * lg + j < a.dh ? rot[li * (DB * 16) + d * 16 + 4 * lg + j] : 0.f;
    __syncthreads();
  } else {
#pragma unroll
    for (int d = 0; d < DB; ++d) qf[d] = head4(q + ((int64_t)t * a.Hq + h) * a.dh, d * 16 + 4 * lg, a.dh, vec);
  }
#pragma unroll
  for (int d = 0; d < DB; ++d) qf[d] *= a.scale;
  float m = -INFINITY, l = 0.f;
  f32x4 acc[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d) acc[d] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int b0 = first_key(a, a.q_start + t0) / 16, b1 = (n_keys + 15) / 16;
  const int lo_last = first_key(a, a.q_start + min(t0 + 15, a.c - 1));
  for (int b = b0 + wave; b < b1; b += AG_WAVES) {
    const int u0 = b * 16;
    const bool edge = u0 + 15 > a.q_start + t0 || u0 < lo_last;
    bool seen[4];
    const T* kr = kb + (int64_t)min(u0 + li, n_keys - 1) * kv_stride;
    const auto kf = pieces<DB>([&](int d) { return head4(kr, d * 16 + 4 * lg, a.dh, vec); });
    const auto vf = pieces<DB>([&](int d) {
      f32x4 x;
#pragma unroll
      for (int r = 0; r < 4; ++r) x[r] = d * 16 + li < a.dh ? ldf(vb + (int64_t)min(u0 + 4 * lg + r, n_keys - 1) * kv_stride + d * 16 + li) : 0.f;
      return x;
    });
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int d = 0; d < DB; ++d) {
      const f32x4 kd = kf(d);
#pragma unroll
      for (int j = 0; j < 4; ++j) s = AG_MFMA(kd[j], qf[d][j], s);
      AG_PIECE_DONE(d);
    }
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int u = u0 + 4 * lg + r;
      seen[r] = u <= pos && u >= lo;
      s[r] = seen[r] ? s[r] : -INFINITY;
      mx = fmaxf(mx, s[r]);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, WAVE));
    mx = fmaxf(mx, __shfl_xor(mx, 32, WAVE));
    const float m_new = fmaxf(m, mx);
    const float corr = m == -INFINITY ? 0.f : expf(m - m_new);
    m = m_new;
    float sum = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      s[r] = s[r] == -INFINITY ? 0.f : expf(s[r] - m_new);
      sum += s[r];
    }
    l = l * corr + sum;                                                        // (my group's keys)
#pragma unroll
    for (int d = 0; d < DB; ++d) acc[d] *= corr;
    second_product<DB>(acc, vf, s, edge, seen, a.dh, [&](int row, int e) { return ldf(vb + (int64_t)min(u0 + row, n_keys - 1) * kv_stride + e); });
  }
  // acc[d][r]: element d * 16 + 4 lg + r of O of query li
  l = over_groups(l);
  if (lg == 0) { sM[wave][li] = m; sL[wave][li] = l; }
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int r = 0; r < 4; ++r) sO[wave][d * 16 + 4 * lg + r][li] = acc[d][r];
  __syncthreads();
  for (int i = threadIdx.x; i < 16 * a.dh; i += AG_THREADS) {
    const int row = i / a.dh, e = i % a.dh;
    if (t0 + row >= a.c) continue;
    float mt = sM[0][row];
#pragma unroll
    for (int w = 1; w < AG_WAVES; ++w) mt = fmaxf(mt, sM[w][row]);
    float lt = 0.f, ot = 0.f;
#pragma unroll
    for (int w = 0; w < AG_WAVES; ++w) {
      const float f = sM[w][row] == -INFINITY ? 0.f : expf(sM[w][row] - mt);
      lt += sL[w][row] * f;
      ot += sO[w][e][row] * f;
    }
    stf(o + ((int64_t)(t0 + row) * a.Hq + h) * a.dh + e, lt > 0.f ? ot / lt : 0.f);
    if (e == 0) lse[(int64_t)h * a.c + t0 + row] = lt > 0.f ? mt + logf(lt) : -INFINITY;
  }
}

// ---- dQ; also delta[h, t] = sum_j d_o[t,h,j] * o[t,h,j], which dK/dV reads.  rope: dq leaves rotated back.
template <typename T, int DB>
__global__ __launch_bounds__(AG_THREADS) void attn_dq_generic_k(const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                                                                const T* __restrict__ o, const T* __restrict__ d_o, const float* __restrict__ lse,
                                                                float* __restrict__ delta, T* __restrict__ dq, AgShape a,
                                                                const float2* __restrict__ rope) {
  __shared__ float sQ[AG_WAVES][DB * 16][17];
  const int h = blockIdx.y, t0 = blockIdx.x * 16, kvh = h / (a.Hq / a.Hkv);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), li = threadIdx.x & 15, lg = (threadIdx.x & 63) >> 4;
  const bool vec = a.vec != 0;
  const int64_t kv_stride = (int64_t)a.Hkv * a.dh;
  const T *kb = k + (int64_t)kvh * a.dh, *vb = v + (int64_t)kvh * a.dh;
  const int t = min(t0 + li, a.c - 1), pos = a.q_start + t;
  const int lo = first_key(a, pos), n_keys = a.q_start + min(t0 + 16, a.c);
  const int64_t qoff = ((int64_t)t * a.Hq + h) * a.dh;
  f32x4 qf[DB], df[DB];
  float D = 0.f;
#pragma unroll
  for (int d = 0; d < DB; ++d) {
    qf[d] = head4(q + qoff, d * 16 + 4 * lg, a.dh, vec);
    df[d] = head4(d_o + qoff, d * 16 + 4 * lg, a.dh, vec);
    const f32x4 of = head4(o + qoff, d * 16 + 4 * lg, a.dh, vec);
#pragma unroll
    for (int j = 0; j < 4; ++j) D += df[d][j] * of[j];
  }
  D = over_groups(D);
  if (wave == 0 && lg == 0 && t0 + li < a.c) delta[(int64_t)h * a.c + t] = D;
  const float L = lse[(int64_t)h * a.c + t];
  f32x4 acc[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d) acc[d] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int b0 = first_key(a, a.q_start + t0) / 16, b1 = (n_keys + 15) / 16;
  const int lo_last = first_key(a, a.q_start + min(t0 + 15, a.c - 1));
  for (int b = b0 + wave; b < b1; b += AG_WAVES) {
    const int u0 = b * 16;
    const bool edge = u0 + 15 > a.q_start + t0 || u0 < lo_last;
    bool seen[4];
    const int64_t row = (int64_t)min(u0 + li, n_keys - 1) * kv_stride;
    const auto kf = pieces<DB>([&](int d) { return head4(kb + row, d * 16 + 4 * lg, a.dh, vec); });
    const auto vf = pieces<DB>([&](int d) { return head4(vb + row, d * 16 + 4 * lg, a.dh, vec); });
    const auto kt = pieces<DB>([&](int d) {
      f32x4 x;
#pragma unroll
      for (int r = 0; r < 4; ++r) x[r] = d * 16 + li < a.dh ? ldf(kb + (int64_t)min(u0 + 4 * lg + r, n_keys - 1) * kv_stride + d * 16 + li) : 0.f;
      return x;
    });
    f32x4 s = {0.f, 0.f, 0.f, 0.f}, dp = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int d = 0; d < DB; ++d) {
      const f32x4 kd = kf(d), vd = vf(d);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        s = AG_MFMA(kd[j], qf[d][j], s);
        dp = AG_MFMA(vd[j], df[d][j], dp);
      }
      AG_PIECE_DONE(d);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int u = u0 + 4 * lg + r;
      seen[r] = u <= pos && u >= lo;
      s[r] = seen[r] ? expf(s[r] * a.scale - L) * (dp[r] - D) * a.scale : 0.f;
    }
    second_product<DB>(acc, kt, s, edge, seen, a.dh, [&](int row, int e) { return ldf(kb + (int64_t)min(u0 + row, n_keys - 1) * kv_stride + e); });
  }
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int r = 0; r < 4; ++r) sQ[wave][d * 16 + 4 * lg + r][li] = acc[d][r];
  __syncthreads();
  auto total = [&](int row, int e) {
    float x = 0.f;
#pragma unroll
    for (int w = 0; w < AG_WAVES; ++w) x += sQ[w][e][row];
    return x;
  };
  for (int i = threadIdx.x; i < 16 * a.dh; i += AG_THREADS) {
    const int row = i / a.dh, e = i % a.dh;
    if (t0 + row >= a.c) continue;
    float x = total(row, e);
    if (rope) {                                                                // adjoint: rotation by the negative angle
      const int half = a.dh / 2;
      const bool up = e >= half;
      const float2 cs = rope[(int64_t)(t0 + row) * half + (up ? e - half : e)];
      const float other = total(row, up ? e - half : e + half);
      x = x * cs.x + (up ? -other : other) * cs.y;
    }
    stf(dq + ((int64_t)(t0 + row) * a.Hq + h) * a.dh + e, x);
  }
}

// ---- dK/dV (and dkc, dvc of the chunk's own rows, final with this call): 16 keys of one KV head; the waves walk blocks of 16 queries that see some of them, for every query head of the group
template <typename T, int DB>
__global__ __launch_bounds__(AG_THREADS) void attn_dkv_generic_k(const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                                                                 const T* __restrict__ d_o, const float* __restrict__ lse,
                                                                 const float* __restrict__ delta, float* __restrict__ dk, float* __restrict__ dv,
                                                                 AgShape a, T* __restrict__ dkc, T* __restrict__ dvc, const float2* __restrict__ rope) {
  __shared__ float sD[AG_WAVES][DB * 16][17];
  const int kvh = blockIdx.y, u0 = blockIdx.x * 16, G = a.Hq / a.Hkv;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), li = threadIdx.x & 15, lg = (threadIdx.x & 63) >> 4;
  const bool vec = a.vec != 0;
  const int n_total = a.q_start + a.c, u = min(u0 + li, n_total - 1);          // my key
  const int64_t koff = ((int64_t)u * a.Hkv + kvh) * a.dh, q_stride = (int64_t)a.Hq * a.dh;
  const auto kf = pieces<DB>([&](int d) { return head4(k + koff, d * 16 + 4 * lg, a.dh, vec); });
  const auto vf = pieces<DB>([&](int d) { return head4(v + koff, d * 16 + 4 * lg, a.dh, vec); });
  f32x4 ak[DB], av[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d) ak[d] = av[d] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int t_first = max(0, u0 - a.q_start);                                  // rows before it see none of the keys, nor do rows from t_end on
  int t_end = a.c;
  if (a.window > 0) t_end = (int)min((int64_t)a.c, max((int64_t)0, (int64_t)u0 + 15 + a.window - a.q_start));
  if (u0 + 15 < a.kv_first) t_end = 0;
  const int b0 = t_first / 16, n_blocks = max(0, (t_end + 15) / 16 - b0);
  for (int it = wave; it < n_blocks * G; it += AG_WAVES) {
    const int t0 = (b0 + it / G) * 16, h = kvh * G + it % G;
    const T *qb = q + (int64_t)h * a.dh, *db = d_o + (int64_t)h * a.dh;
    const int64_t row = (int64_t)min(t0 + li, a.c - 1) * q_stride;
    const auto qf = pieces<DB>([&](int d) { return head4(qb + row, d * 16 + 4 * lg, a.dh, vec); });
    const auto df = pieces<DB>([&](int d) { return head4(db + row, d * 16 + 4 * lg, a.dh, vec); });
    auto across = [&](const T* __restrict__ p) {
      return [=](int d) {
        f32x4 x;
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = d * 16 + li < a.dh ? ldf(p + (int64_t)min(t0 + 4 * lg + r, a.c - 1) * q_stride + d * 16 + li) : 0.f;
        return x;
      };
    };
    const auto qt = pieces<DB>(across(qb)), dt = pieces<DB>(across(db));
    const bool edge = u0 + 15 > a.q_start + t0 || u0 < first_key(a, a.q_start + t0 + 15) || t0 + 15 >= a.c || u0 + 15 >= n_total;
    bool seen[4];
    float L[4], D[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int t = min(t0 + 4 * lg + r, a.c - 1);
      L[r] = lse[(int64_t)h * a.c + t];
      D[r] = delta[(int64_t)h * a.c + t];
    }
    f32x4 s = {0.f, 0.f, 0.f, 0.f}, dp = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int d = 0; d < DB; ++d) {
      const f32x4 qd = qf(d), dd = df(d), kd = kf(d), vd = vf(d);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        s = AG_MFMA(qd[j], kd[j], s);
        dp = AG_MFMA(dd[j], vd[j], dp);
      }
      AG_PIECE_DONE(d);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int t = t0 + 4 * lg + r, pos = a.q_start + t;
      seen[r] = t < a.c && u0 + li < n_total && u <= pos && u >= first_key(a, pos);
      const float p = seen[r] ? expf(s[r] * a.scale - L[r]) : 0.f;
      s[r] = p;
      dp[r] = seen[r] ? p * (dp[r] - D[r]) * a.scale : 0.f;
    }
    auto at_row = [&](const T* __restrict__ p) { return [=](int row, int e) { return ldf(p + (int64_t)min(t0 + row, a.c - 1) * q_stride + e); }; };
    second_product<DB>(av, dt, s, edge, seen, a.dh, at_row(db));
    second_product<DB>(ak, qt, dp, edge, seen, a.dh, at_row(qb));
  }
  auto leave = [&](const f32x4 (&acc)[DB], float* __restrict__ out, T* __restrict__ fin, bool rotate) {
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int r = 0; r < 4; ++r) sD[wave][d * 16 + 4 * lg + r][li] = acc[d][r];
    __syncthreads();
    auto total = [&](int row, int e) {
      float x = 0.f;
#pragma unroll
      for (int w = 0; w < AG_WAVES; ++w) x += sD[w][e][row];
      float* p = out + ((int64_t)(u0 + row) * a.Hkv + kvh) * a.dh + e;
      return *p += x;
    };
    if (!fin) {
      for (int i = threadIdx.x; i < 16 * a.dh; i += AG_THREADS)
        if (u0 + i / a.dh < n_total) total(i / a.dh, i % a.dh);
    } else {                             // (an even head size: what the rotary embedding pairs)
      const int half = a.dh / 2;
      for (int i = threadIdx.x; i < 16 * half; i += AG_THREADS) {
        const int row = i / half, e = i % half, t = u0 + row - a.q_start;
        if (u0 + row >= n_total) continue;
        const float x = total(row, e), y = total(row, e + half);
        if (t < 0) continue;
        const float2 cs = rotate ? rope[(int64_t)t * half + e] : make_float2(1.f, 0.f);
        T* f = fin + ((int64_t)t * a.Hkv + kvh) * a.dh + e;
        stf(f, rotate ? x * cs.x + y * cs.y : x);               // rotation by the negative angle
        stf(f + half, rotate ? y * cs.x - x * cs.y : y);
      }
    }
    __syncthreads();
  };
  leave(ak, dk, dkc, true);
  leave(av, dv, dvc, false);
}

static AgShape shape_of(const AttnArgs& a, std::initializer_list<const void*> tensors) {
  bool vec = a.dh % 4 == 0;
  for (const void* p : tensors) vec = vec && !((uintptr_t)p & (4 * dtype_size(a.dt) - 1));
  return AgShape{a.Hq, a.Hkv, a.dh, a.q_start, a.q_len, a.scale, a.window, a.kv_first, vec ? 1 : 0};
}
// One instance per power of two of 16-wide blocks of the head
template <typename F>
static void per_blocks(int dh, F f) {
  if (dh <= 16) f(std::integral_constant<int, 1>{});
  else if (dh <= 32) f(std::integral_constant<int, 2>{});
  else if (dh <= 64) f(std::integral_constant<int, 4>{});
  else if (dh <= 128) f(std::integral_constant<int, 8>{});
  else f(std::integral_constant<int, 16>{});
}

template <typename T>
static hipError_t forward_t(const AttnArgs& a, hipStream_t st) {
  const AgShape s = shape_of(a, {a.q, a.k, a.v});
  const dim3 grid((unsigned)cdiv(a.q_len, 16), (unsigned)a.Hq);
  per_blocks(a.dh, [&](auto db) {
    attn_fwd_generic_k<T, decltype(db)::value><<<grid, AG_THREADS, 0, st>>>((T*)a.q, (const T*)a.k, (const T*)a.v, (T*)a.o, a.lse, s, a.rope_q);
  });
  return hipGetLastError();
}
template <typename T>
static hipError_t backward_t(const AttnArgs& a, hipStream_t st) {
  const AgShape s = shape_of(a, {a.q, a.k, a.v, a.o, a.d_o});
  const dim3 gq((unsigned)cdiv(a.q_len, 16), (unsigned)a.Hq), gk((unsigned)cdiv((int64_t)a.q_start + a.q_len, 16), (unsigned)a.Hkv);
  per_blocks(a.dh, [&](auto db) {
    constexpr int DB = decltype(db)::value;
    attn_dq_generic_k<T, DB><<<gq, AG_THREADS, 0, st>>>((const T*)a.q, (const T*)a.k, (const T*)a.v, (const T*)a.o, (const T*)a.d_o, a.lse, a.delta,
                                                        (T*)a.dq, s, a.rope_q);
    attn_dkv_generic_k<T, DB><<<gk, AG_THREADS, 0, st>>>((const T*)a.q, (const T*)a.k, (const T*)a.v, (const T*)a.d_o, a.lse, a.delta, a.dk, a.dv, s,
                                                         (T*)a.dkc, (T*)a.dvc, a.rope_k);
  });
  return hipGetLastError();
}
hipError_t attn_forward_generic(const AttnArgs& a, hipStream_t st) {
  if (a.q_len == 0) return hipSuccess;
  return a.dt == DT_BF16 ? forward_t<bf16_t>(a, st) : forward_t<float>(a, st);
}
hipError_t attn_backward_generic(const AttnArgs& a, hipStream_t st) {
  if (a.q_len == 0) return hipSuccess;
  return a.dt == DT_BF16 ? backward_t<bf16_t>(a, st) : backward_t<float>(a, st);
}

}  // namespace sbp
