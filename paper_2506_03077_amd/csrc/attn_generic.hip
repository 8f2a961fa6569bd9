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
// other dimension dealt to its waves in blocks of 16, which meet in LDS at the end (heads of more than 64 elements: to groups of waves, each with a share of
// the head).  What bounds the calls of the small configuration
// is the chain of dependent loads, not arithmetic: one query (key) per workgroup, with its second product on as many threads as the
// head is wide, walked 256 keys one after the other (64 queries, 4 heads of 16, up to 256 keys, with the rotary embedding: forward 14.8 -> 5.8 us, dQ
// with delta 13.5 -> 5.3, dK/dV 11.8 -> 4.8).
//
// Layout: a score block has 16 rows (keys; dK/dV: queries) in registers, rows 4 (l / 16) + r, and its 16 columns across lanes, l % 16.  MFMA j
// of the first product takes element j of both operands' four at head_dim 16 d + 4 (l / 16) .. + 3; MFMA r of the second product takes
// accumulator register r as its B operand, i.e. row 4 (l / 16) + r of the block as its reduction index.
#include "launch.h"
#include "attn_plan.h"
#include "device.h"

namespace sbp {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef bf16_t bf16x4 __attribute__((ext_vector_type(4)));

template <typename T> __device__ __forceinline__ float stored(float x) { T t; stf(&t, x); return ldf(&t); }      // as T holds it

// Operands stay as they were loaded until the product that uses them, and no load hangs on a lane condition (elements past the head come from its last
// ones): all loads of a block are under way at once, and a block costs one or two round trips to memory however wide the head is.
// Loading 16-wide pieces in front of their products (heads of more than 64 elements, the earlier form) took one for every two pieces.  fp32, 64 queries from 0, 4
// heads: of 80 forward 12.6 -> 7.4 us, backward 36 -> 17.5; of 256 30 -> 9.2, 81 -> 30 (one query per workgroup: 9.4, 30); 512 from 960, 8 / 2 heads of 128 75 -> 50, 333 ->
// 254 (425, 2337).  Where it is still behind one query per workgroup: few queries and heads of more than 128 over 100 to 1000 keys (bf16, one head of 256, 64
// queries from 192: 49 -> 22 us against 16), as a workgroup's sixteen queries then have one CU.
template <typename T> struct Raw;
template <> struct Raw<float> {
  typedef f32x4 four; typedef float one;
  static __device__ __forceinline__ f32x4 value(f32x4 v) { return v; }
  static __device__ __forceinline__ float value(float v) { return v; }
};
template <> struct Raw<bf16_t> {
  typedef bf16x4 four; typedef uint16_t one;
  static __device__ __forceinline__ f32x4 value(bf16x4 v) { return f32x4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]}; }
  static __device__ __forceinline__ float value(uint16_t v) { return (float)__builtin_bit_cast(bf16_t, v); }
};
// Addresses: a uniform base and a 32-bit byte offset (sixteen rows of at most 65535 heads of 256).  Rows and their four-element pieces start anywhere: the
// vector types are aligned like their elements, which the loads of this chip take.
template <typename T> struct AnyFour { typedef typename Raw<T>::four type __attribute__((aligned(sizeof(T)))); };
// DB pieces d0 .. of row `row` (of rows `stride` apart): piece d = elements 16 d + e4 .. + 3, from the head's end on its last four (which element a place
// holds does not matter, as both operands of a product have the same there).  first: the instance of DB blocks that takes the whole head, whose
// pieces below DB / 2 are always whole.
template <typename T, int DB>
__device__ __forceinline__ void load_row(typename Raw<T>::four (&v)[DB], const T* __restrict__ base, int row, int stride, bool first, int d0, int e4, int dh) {
  const char* p = (const char*)base;
  if (dh >= 4) {
#pragma unroll
    for (int i = 0; i < DB; ++i) {
      const int e = (d0 + i) * 16 + e4;
      v[i] = *(const typename AnyFour<T>::type*)(p + (uint32_t)((row * stride + (first && i < DB / 2 ? e : min(e, dh - 4))) * (int)sizeof(T)));
    }
  } else {
#pragma unroll
    for (int i = 0; i < DB; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) v[i][j] = *(const T*)(p + (uint32_t)((row * stride + max(0, dh - 4 + j)) * (int)sizeof(T)));
  }
}
// ... and the values of its piece i: zeros past the head and where an element has had its place before
template <typename T, int DB>
__device__ __forceinline__ f32x4 row_piece(f32x4 v, bool first, int d0, int i, int e4, int dh) {
  if (!first || i >= DB / 2) {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = (d0 + i) * 16 + e4 - (dh - 4) <= j ? v[j] : 0.f;
  }
  return v;
}
// DB pieces d0 .. across rows row0 .. row0 + 3, at most `last`: element 16 d + li of each (past the head: its last one again, for sums that nothing stores)
template <typename T, int DB>
__device__ __forceinline__ void load_across(typename Raw<T>::one (&v)[DB][4], const T* __restrict__ base, int row0, int last, int stride, bool first, int d0, int li, int dh) {
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = min(row0 + r, last) * stride;
#pragma unroll
    for (int i = 0; i < DB; ++i) {
      const int e = (d0 + i) * 16 + li;
      v[i][r] = *(const typename Raw<T>::one*)((const char*)base + (uint32_t)((row + (first && i < DB / 2 ? e : min(e, dh - 1))) * (int)sizeof(T)));
    }
  }
}
#define AG_MFMA(a, b, c) __builtin_amdgcn_mfma_f32_16x16x4f32((a), (b), (c), 0, 0, 0)
__device__ __forceinline__ float over_groups(float x) { x += __shfl_xor(x, 16, WAVE); return x + __shfl_xor(x, 32, WAVE); }

// acc^T [element][column] += X^T [element][row] P [row][column] for pieces d0 .., X's 16 rows as v[i][r] = X[4 (l / 16) + r][16 (d0 + i) + l % 16].
// `edge`: some (row, column) pairs of the block are hidden, seen[r] says which are not: a row that holds infinities or NaN must not
// reach the columns it is hidden from (0 * NaN), so such blocks go pair by pair, with x(row, element).
template <typename T, int DB, typename X>
__device__ __forceinline__ void second_product(f32x4 (&acc)[DB], int d0, const typename Raw<T>::one (&v)[DB][4], const f32x4& p, bool edge, const bool (&seen)[4],
                                               int dh, X x) {
  if (edge) {
    bool odd = false;
#pragma unroll
    for (int i = 0; i < DB; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) odd = odd || !(fabsf(Raw<T>::value(v[i][r])) < INFINITY);
    if (__builtin_amdgcn_ballot_w64(odd) != 0) {
      const int li = threadIdx.x & 15, lg = (threadIdx.x & 63) >> 4;
#pragma unroll 1
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float pr = __shfl(p[r], g * 16 + li, WAVE);
          const bool vis = __shfl(seen[r] ? 1 : 0, g * 16 + li, WAVE) != 0;
#pragma unroll
          for (int i = 0; i < DB; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const int el = (d0 + i) * 16 + 4 * lg + e;
              if (vis && el < dh) acc[i][e] = fmaf(x(4 * g + r, el), pr, acc[i][e]);
            }
        }
      return;
    }
  }
#pragma unroll
  for (int i = 0; i < DB; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[i] = AG_MFMA(Raw<T>::value(v[i][r]), p[r], acc[i]);
}

// The sums of the slots meet in LDS: part[slot][row][element], rows ROW apart
template <int DB, int P, int W> struct Parts {
  static constexpr int HEAD = DB * P, ROW = HEAD * 16 + 4, THREADS = W * 64, SLOTS = W / P, SLOT = 16 * ROW, FLOATS = SLOTS * SLOT;
  static constexpr int PAIRS = (16 * HEAD * 8 + THREADS - 1) / THREADS;     // of elements that a thread finishes: e and e + half of a row (what the rotary embedding
  struct Pair { int row, e; bool in; };                      // pairs; an odd head's last pair is one element)
  static __device__ __forceinline__ Pair pair(int n, int half) {
    const int i = n * THREADS + (int)threadIdx.x, row = i / (HEAD * 8), e = i % (HEAD * 8);
    return Pair{min(row, 15), e, row < 16 && e < half};
  }
  static __device__ __forceinline__ void leave(float* part, int slot, int d0, const f32x4 (&acc)[DB], int li, int lg4) {
#pragma unroll
    for (int d = 0; d < DB; ++d) *(f32x4*)(part + slot * SLOT + li * ROW + (d0 + d) * 16 + lg4) = acc[d];
  }
  template <typename F>
  static __device__ __forceinline__ void sums(const float* part, int half, float (&x)[PAIRS], float (&y)[PAIRS], F weight) {
#pragma unroll
    for (int n = 0; n < PAIRS; ++n) x[n] = y[n] = 0.f;
#pragma unroll
    for (int w = 0; w < SLOTS; ++w)
#pragma unroll
      for (int n = 0; n < PAIRS; ++n) {
        const Pair p = pair(n, half);
        const float* s = part + w * SLOT + p.row * ROW + p.e;
        const float f = weight(w, p.row);
        x[n] += s[0] * f;
        y[n] += s[half] * f;
      }
  }
};
// Heads of more than 64 elements: P waves share a block, each with DB pieces of the head, and exchange their N sums of the first product; every one
// gets the same totals.  x: [2][slot][N][P][64], the halves used in turn, so that one barrier per round is enough.
template <int P, int N, int W> constexpr int EXCHANGE = P == 1 ? 1 : 2 * W * N * 64;
template <int P, int N, int W>
__device__ __forceinline__ void exchange(f32x4* x, int turn, int slot, int share, bool on, f32x4 (&s)[N]) {
  if constexpr (P > 1) {
    f32x4* b = x + ((turn & 1) * (W / P) + slot) * (N * P * 64) + (threadIdx.x & 63);
    if (on) {
#pragma unroll
      for (int n = 0; n < N; ++n) b[(n * P + share) * 64] = s[n];
    }
    __syncthreads();
    if (on) {
#pragma unroll
      for (int n = 0; n < N; ++n) {
        s[n] = b[n * P * 64];
#pragma unroll
        for (int i = 1; i < P; ++i) s[n] += b[(n * P + i) * 64];
      }
    }
  }
}

struct AgShape { int Hq, Hkv, dh, q_start, c; float scale; int window, kv_first; };
__device__ __forceinline__ int first_key(const AgShape& a, int pos) { return max(a.kv_first, a.window > 0 ? pos - a.window + 1 : 0); }

// What a wave is: a slot takes every SLOTS-th block, its waves a share of the head each
#define AG_WAVE_SETUP                                                                                             \
  using Pt = Parts<DB, P, W>;                                                                                    \
  constexpr int SLOTS = Pt::SLOTS;                                                                               \
  constexpr bool FIRST = P == 1;                                                                                 \
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), slot = wave / P, share = wave % P, d0 = share * DB; \
  const int li = threadIdx.x & 15, lg4 = (threadIdx.x & 63) >> 4 << 2
// (P == 1: a wave's own number of rounds; else all waves run the same, for the barrier in each)
#define AG_ROUNDS(n) (P == 1 ? ((n) - slot + SLOTS - 1) / SLOTS : ((n) + SLOTS - 1) / SLOTS)

#define AG_PARTS(N) __shared__ __attribute__((aligned(16))) float part[(N) * Parts<DB, P, W>::FLOATS]

// ---- forward.  rope: q arrives un-rotated, is rotated on load and written back rotated.
template <typename T, int DB, int P, int W>
__global__ __launch_bounds__(W * 64) void attn_fwd_generic_k(T* q, const T* __restrict__ k, const T* __restrict__ v, T* __restrict__ o,
                                                                 float* __restrict__ lse, AgShape a, const float2* __restrict__ rope) {
  AG_PARTS(1);
  AG_WAVE_SETUP;
  __shared__ f32x4 sX[EXCHANGE<P, 1, W>];
  __shared__ float sM[SLOTS][16], sL[SLOTS][16], sF[SLOTS][16], sT[16];
  const int h = blockIdx.y, t0 = blockIdx.x * 16, kvh = h / (a.Hq / a.Hkv);
  const int kv_stride = a.Hkv * a.dh;
  const T *kb = k + (int64_t)kvh * a.dh, *vb = v + (int64_t)kvh * a.dh;
  const int t = min(t0 + li, a.c - 1), pos = a.q_start + t;                    // my query
  const int lo = first_key(a, pos), n_keys = a.q_start + min(t0 + 16, a.c);
  const int b0 = first_key(a, a.q_start + t0) / 16, b1 = (n_keys + 15) / 16;
  const int lo_last = first_key(a, a.q_start + min(t0 + 15, a.c - 1));
  auto q_row = [&](int row) { return q + ((int64_t)min(t0 + row, a.c - 1) * a.Hq + h) * a.dh; };
  typename Raw<T>::four kr[DB];
  typename Raw<T>::one vr[DB][4];
  auto load_k = [&](int u0) { load_row<T, DB>(kr, kb + (int64_t)u0 * kv_stride, min(li, n_keys - 1 - u0), kv_stride, FIRST, d0, lg4, a.dh); };
  auto load_v = [&](int u0) { load_across<T, DB>(vr, vb + (int64_t)u0 * kv_stride, lg4, n_keys - 1 - u0, kv_stride, FIRST, d0, li, a.dh); };
  f32x4 qf[DB];
  typename Raw<T>::four raw[DB];
  if (!rope) load_row<T, DB>(raw, q_row(0), min(li, a.c - 1 - t0), a.Hq * a.dh, FIRST, d0, lg4, a.dh);
  int b = b0 + slot;
  if (b < b1) { load_k(b * 16); load_v(b * 16); }      // the first block is under way before q is waited for
  if (rope) {
    const int half = a.dh / 2;
    constexpr int N = (16 * Pt::HEAD * 16 + Pt::THREADS - 1) / Pt::THREADS;
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const int i = n * Pt::THREADS + (int)threadIdx.x, row = i / (Pt::HEAD * 16), e = i % (Pt::HEAD * 16), ec = min(e, a.dh - 1), tr = min(t0 + row, a.c - 1);
      const T* p = q_row(row);
      const bool up = ec >= half;
      const float2 cs = rope[(int64_t)tr * half + (up ? ec - half : ec)];
      const float other = ldf(p + (up ? ec - half : ec + half));
      const float x = stored<T>(ldf(p + ec) * cs.x + (up ? other : -other) * cs.y);
      if (row < 16) part[row * Pt::ROW + e] = e < a.dh ? x : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const int i = n * Pt::THREADS + (int)threadIdx.x, row = i / (Pt::HEAD * 16), e = i % (Pt::HEAD * 16);
      if (row < 16 && e < a.dh && t0 + row < a.c) stf(q + ((int64_t)(t0 + row) * a.Hq + h) * a.dh + e, part[row * Pt::ROW + e]);
    }
#pragma unroll
    for (int d = 0; d < DB; ++d) {
      f32x4 x;
#pragma unroll
      for (int j = 0; j < 4; ++j) x[j] = part[li * Pt::ROW + max(0, min((d0 + d) * 16 + lg4, a.dh - 4) + j)];
      qf[d] = row_piece<T, DB>(x, FIRST, d0, d, lg4, a.dh) * a.scale;
    }
    __syncthreads();
  } else {
#pragma unroll
    for (int d = 0; d < DB; ++d) qf[d] = row_piece<T, DB>(Raw<T>::value(raw[d]), FIRST, d0, d, lg4, a.dh) * a.scale;
  }
  float m = -INFINITY, l = 0.f;
  f32x4 acc[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d) acc[d] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int rounds = AG_ROUNDS(b1 - b0);
  for (int n = 0; n < rounds; ++n, b += SLOTS) {
    const int u0 = b * 16, next = b + SLOTS;
    const bool on = P == 1 || b < b1;
    f32x4 sc[1] = {{0.f, 0.f, 0.f, 0.f}};
    f32x4& s = sc[0];
    if (on) {
#pragma unroll
      for (int d = 0; d < DB; ++d) {
        const f32x4 kd = row_piece<T, DB>(Raw<T>::value(kr[d]), FIRST, d0, d, lg4, a.dh);
#pragma unroll
        for (int j = 0; j < 4; ++j) s = AG_MFMA(kd[j], qf[d][j], s);
      }
      if (next < b1) load_k(next * 16);
    }
    exchange<P, 1, W>(sX, n, slot, share, on, sc);
    if (!on) continue;
    const bool edge = u0 + 15 > a.q_start + t0 || u0 < lo_last;
    bool seen[4];
    float mx = -INFINITY;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int u = u0 + lg4 + r;
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
    second_product<T, DB>(acc, d0, vr, s, edge, seen, a.dh, [&](int row, int e) { return ldf(vb + (int64_t)min(u0 + row, n_keys - 1) * kv_stride + e); });
    if (next < b1) load_v(next * 16);
  }
  // acc[d][r]: element (d0 + d) * 16 + 4 lg + r of O of query li
  l = over_groups(l);
  if (share == 0 && lg4 == 0) { sM[slot][li] = m; sL[slot][li] = l; }
  Pt::leave(part, slot, d0, acc, li, lg4);
  __syncthreads();
  // the slots' weights and the rows' denominators, once instead of for every element
  if (threadIdx.x < SLOTS * 16) {
    const int w = threadIdx.x >> 4, row = threadIdx.x & 15;
    float mt = sM[0][row], lt = 0.f;
#pragma unroll
    for (int x = 1; x < SLOTS; ++x) mt = fmaxf(mt, sM[x][row]);
#pragma unroll
    for (int x = 0; x < SLOTS; ++x) {
      const float f = sM[x][row] == -INFINITY ? 0.f : expf(sM[x][row] - mt);
      lt += sL[x][row] * f;
      if (x == w) sF[w][row] = f;
    }
    if (w == 0) {
      sT[row] = lt;
      if (t0 + row < a.c) lse[(int64_t)h * a.c + t0 + row] = lt > 0.f ? mt + logf(lt) : -INFINITY;
    }
  }
  __syncthreads();
  const int half = (a.dh + 1) / 2;
  float x[Pt::PAIRS], y[Pt::PAIRS];
  Pt::sums(part, half, x, y, [&](int w, int row) { return sF[w][row]; });
#pragma unroll
  for (int n = 0; n < Pt::PAIRS; ++n) {
    const auto p = Pt::pair(n, half);
    if (!p.in || t0 + p.row >= a.c) continue;
    const float lt = sT[p.row];
    T* out = o + ((int64_t)(t0 + p.row) * a.Hq + h) * a.dh + p.e;
    stf(out, lt > 0.f ? x[n] / lt : 0.f);
    if (p.e + half < a.dh) stf(out + half, lt > 0.f ? y[n] / lt : 0.f);
  }
}

// ---- dQ; also delta[h, t] = sum_j d_o[t,h,j] * o[t,h,j], which dK/dV reads.  rope: dq leaves rotated back.
template <typename T, int DB, int P, int W>
__device__ __forceinline__ void dq_block(float* part, int tile, int h, const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                                         const T* __restrict__ o, const T* __restrict__ d_o, const float* __restrict__ lse, float* __restrict__ delta,
                                         T* __restrict__ dq, const AgShape& a, const float2* __restrict__ rope) {
  AG_WAVE_SETUP;
  __shared__ f32x4 sX[EXCHANGE<P, 2, W>];
  __shared__ float sD[P][16];
  const int t0 = tile * 16, kvh = h / (a.Hq / a.Hkv);
  const int kv_stride = a.Hkv * a.dh;
  const T *kb = k + (int64_t)kvh * a.dh, *vb = v + (int64_t)kvh * a.dh;
  const int t = min(t0 + li, a.c - 1), pos = a.q_start + t;
  const int lo = first_key(a, pos), n_keys = a.q_start + min(t0 + 16, a.c);
  const int b0 = first_key(a, a.q_start + t0) / 16, b1 = (n_keys + 15) / 16;
  const int lo_last = first_key(a, a.q_start + min(t0 + 15, a.c - 1));
  const int64_t q0 = ((int64_t)t0 * a.Hq + h) * a.dh;
  const int row = min(li, a.c - 1 - t0), q_stride = a.Hq * a.dh;
  const float L = lse[(int64_t)h * a.c + t];
  f32x4 qf[DB], df[DB];
  typename Raw<T>::four raw_o[DB], raw_q[DB], raw_d[DB], kr[DB], vr[DB];
  typename Raw<T>::one kt[DB][4];
  load_row<T, DB>(raw_o, o + q0, row, q_stride, FIRST, d0, lg4, a.dh);
  load_row<T, DB>(raw_q, q + q0, row, q_stride, FIRST, d0, lg4, a.dh);
  load_row<T, DB>(raw_d, d_o + q0, row, q_stride, FIRST, d0, lg4, a.dh);
  auto load_rows = [&](int u0) {
    const int64_t at = (int64_t)u0 * kv_stride;
    const int key = min(li, n_keys - 1 - u0);
    load_row<T, DB>(kr, kb + at, key, kv_stride, FIRST, d0, lg4, a.dh);
    load_row<T, DB>(vr, vb + at, key, kv_stride, FIRST, d0, lg4, a.dh);
  };
  auto load_cols = [&](int u0) { load_across<T, DB>(kt, kb + (int64_t)u0 * kv_stride, lg4, n_keys - 1 - u0, kv_stride, FIRST, d0, li, a.dh); };
  int b = b0 + slot;
  if (b < b1) { load_rows(b * 16); load_cols(b * 16); }      // the first block is under way before q is waited for
  float D = 0.f;
#pragma unroll
  for (int d = 0; d < DB; ++d) {
    qf[d] = row_piece<T, DB>(Raw<T>::value(raw_q[d]), FIRST, d0, d, lg4, a.dh);
    df[d] = row_piece<T, DB>(Raw<T>::value(raw_d[d]), FIRST, d0, d, lg4, a.dh);
    const f32x4 of = row_piece<T, DB>(Raw<T>::value(raw_o[d]), FIRST, d0, d, lg4, a.dh);
#pragma unroll
    for (int j = 0; j < 4; ++j) D += df[d][j] * of[j];
  }
  D = over_groups(D);
  if constexpr (P > 1) {
    if (slot == 0 && lg4 == 0) sD[share][li] = D;
    __syncthreads();
    D = sD[0][li];
#pragma unroll
    for (int i = 1; i < P; ++i) D += sD[i][li];
  }
  if (delta && wave == 0 && lg4 == 0 && t0 + li < a.c) delta[(int64_t)h * a.c + t] = D;
  f32x4 acc[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d) acc[d] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int rounds = AG_ROUNDS(b1 - b0);
  for (int n = 0; n < rounds; ++n, b += SLOTS) {
    const int u0 = b * 16, next = b + SLOTS;
    const bool on = P == 1 || b < b1;
    f32x4 sc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    f32x4 &s = sc[0], &dp = sc[1];
    if (on) {
#pragma unroll
      for (int d = 0; d < DB; ++d) {
        const f32x4 kd = row_piece<T, DB>(Raw<T>::value(kr[d]), FIRST, d0, d, lg4, a.dh), vd = row_piece<T, DB>(Raw<T>::value(vr[d]), FIRST, d0, d, lg4, a.dh);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          s = AG_MFMA(kd[j], qf[d][j], s);
          dp = AG_MFMA(vd[j], df[d][j], dp);
        }
      }
      if (next < b1) load_rows(next * 16);
    }
    exchange<P, 2, W>(sX, n, slot, share, on, sc);
    if (!on) continue;
    const bool edge = u0 + 15 > a.q_start + t0 || u0 < lo_last;
    bool seen[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int u = u0 + lg4 + r;
      seen[r] = u <= pos && u >= lo;
      s[r] = seen[r] ? expf(s[r] * a.scale - L) * (dp[r] - D) * a.scale : 0.f;
    }
    second_product<T, DB>(acc, d0, kt, s, edge, seen, a.dh, [&](int row, int e) { return ldf(kb + (int64_t)min(u0 + row, n_keys - 1) * kv_stride + e); });
    if (next < b1) load_cols(next * 16);
  }
  const int half = (a.dh + 1) / 2;
  Pt::leave(part, slot, d0, acc, li, lg4);
  __syncthreads();
  float x[Pt::PAIRS], y[Pt::PAIRS];
  Pt::sums(part, half, x, y, [](int, int) { return 1.f; });
#pragma unroll
  for (int n = 0; n < Pt::PAIRS; ++n) {
    const auto p = Pt::pair(n, half);
    if (!p.in || t0 + p.row >= a.c) continue;
    T* out = dq + ((int64_t)(t0 + p.row) * a.Hq + h) * a.dh + p.e;
    if (rope) {                                                                // adjoint: rotation by the negative angle (an even head size)
      const float2 cs = rope[(int64_t)(t0 + p.row) * half + p.e];
      const float u = x[n] * cs.x + y[n] * cs.y, w = y[n] * cs.x + -x[n] * cs.y;
      x[n] = u; y[n] = w;
    }
    stf(out, x[n]);
    if (p.e + half < a.dh) stf(out + half, y[n]);
  }
}

template <typename T, int DB, int P, int W>
__global__ __launch_bounds__(W * 64) void attn_dq_generic_k(const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                                                                const T* __restrict__ o, const T* __restrict__ d_o, const float* __restrict__ lse,
                                                                float* __restrict__ delta, T* __restrict__ dq, AgShape a,
                                                                const float2* __restrict__ rope) {
  AG_PARTS(1);
  dq_block<T, DB, P, W>(part, blockIdx.x, blockIdx.y, q, k, v, o, d_o, lse, delta, dq, a, rope);
}

// ---- dK/dV (and dkc, dvc of the chunk's own rows, final with this call): 16 keys of one KV head; the slots walk blocks of 16 queries that see some of them, for every query head of the group
// DELTA: D of the queries from d_o and o, as dQ forms it, in place of reading what dQ has left.
template <typename T, int DB, int P, int W, bool DELTA>
__device__ __forceinline__ void dkv_block(float* part, int block, int kvh, const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                                          const T* __restrict__ o, const T* __restrict__ d_o, const float* __restrict__ lse, const float* __restrict__ delta,
                                          float* __restrict__ dk, float* __restrict__ dv, const AgShape& a, T* __restrict__ dkc, T* __restrict__ dvc,
                                          const float2* __restrict__ rope) {
  static_assert(!DELTA || P == 1, "a wave has whole rows of d_o and o");
  AG_WAVE_SETUP;
  __shared__ f32x4 sX[EXCHANGE<P, 2, W>];
  const int u0 = block * 16, G = a.Hq / a.Hkv;
  const int n_total = a.q_start + a.c, u = min(u0 + li, n_total - 1);          // my key
  const int kv_stride = a.Hkv * a.dh, q_stride = a.Hq * a.dh;
  const int t_first = max(0, u0 - a.q_start);                                  // rows before it see none of the keys, nor do rows from t_end on
  int t_end = a.c;
  if (a.window > 0) t_end = (int)min((int64_t)a.c, max((int64_t)0, (int64_t)u0 + 15 + a.window - a.q_start));
  if (u0 + 15 < a.kv_first) t_end = 0;
  const int b0 = t_first / 16, n_it = max(0, (t_end + 15) / 16 - b0) * G;
  typename Raw<T>::four qr[DB], dr[DB], orow[DELTA ? DB : 1], raw_k[DB], raw_v[DB];
  typename Raw<T>::one dt[DB][4], qt[DB][4];
  float L[4], D[4];
  auto head_of = [&](int it) { return kvh * G + it % G; };
  auto query_of = [&](int it) { return (b0 + it / G) * 16; };
  auto first_of = [&](int it) { return (int64_t)query_of(it) * q_stride + (int64_t)head_of(it) * a.dh; };
  auto load_rows = [&](int it) {
    const int row = min(li, a.c - 1 - query_of(it));
    load_row<T, DB>(qr, q + first_of(it), row, q_stride, FIRST, d0, lg4, a.dh);
    load_row<T, DB>(dr, d_o + first_of(it), row, q_stride, FIRST, d0, lg4, a.dh);
    if constexpr (DELTA) load_row<T, DB>(orow, o + first_of(it), row, q_stride, FIRST, d0, lg4, a.dh);
  };
  auto load_cols = [&](int it) {
    const int last = a.c - 1 - query_of(it);
    const int64_t at = (int64_t)head_of(it) * a.c + query_of(it);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      L[r] = (lse + at)[min(lg4 + r, last)];
      if constexpr (!DELTA) D[r] = (delta + at)[min(lg4 + r, last)];
    }
    load_across<T, DB>(dt, d_o + first_of(it), lg4, last, q_stride, FIRST, d0, li, a.dh);
    load_across<T, DB>(qt, q + first_of(it), lg4, last, q_stride, FIRST, d0, li, a.dh);
  };
  const int64_t k0 = (int64_t)u0 * kv_stride + (int64_t)kvh * a.dh;
  load_row<T, DB>(raw_k, k + k0, u - u0, kv_stride, FIRST, d0, lg4, a.dh);
  load_row<T, DB>(raw_v, v + k0, u - u0, kv_stride, FIRST, d0, lg4, a.dh);
  int it = slot;
  if (it < n_it) { load_rows(it); load_cols(it); }      // the first block is under way before k and v are waited for
  f32x4 kf[DB], vf[DB], ak[DB], av[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d) {
    kf[d] = row_piece<T, DB>(Raw<T>::value(raw_k[d]), FIRST, d0, d, lg4, a.dh);
    vf[d] = row_piece<T, DB>(Raw<T>::value(raw_v[d]), FIRST, d0, d, lg4, a.dh);
    ak[d] = av[d] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // Two slots instead of eight (P > 1): what four blocks gave goes to LDS, so that the sums stay as close to fp64 as eight shorter ones (bf16, 300 queries, heads of
  // 130: 4.5e-7 -> 3.5e-7; eight slots 3.9e-7).  Kept in registers the totals cost heads of 65 to 128 elements 20 to 50 %.
  bool left = false;
  auto leave = [&]() {
#pragma unroll
    for (int d = 0; d < DB; ++d) {
      f32x4 *pk = (f32x4*)(part + slot * Pt::SLOT + li * Pt::ROW + (d0 + d) * 16 + lg4), *pv = (f32x4*)((float*)pk + Pt::FLOATS);
      *pk = left ? *pk + ak[d] : ak[d];
      *pv = left ? *pv + av[d] : av[d];
      ak[d] = av[d] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    left = true;
  };
  const int rounds = AG_ROUNDS(n_it);
  for (int n = 0; n < rounds; ++n, it += SLOTS) {
    const int t0 = query_of(it), h = head_of(it), next = it + SLOTS;
    const bool on = P == 1 || it < n_it;
    f32x4 sc[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    f32x4 &s = sc[0], &dp = sc[1];
    if (on) {
      float dot = 0.f;
#pragma unroll
      for (int d = 0; d < DB; ++d) {
        const f32x4 qd = row_piece<T, DB>(Raw<T>::value(qr[d]), FIRST, d0, d, lg4, a.dh), dd = row_piece<T, DB>(Raw<T>::value(dr[d]), FIRST, d0, d, lg4, a.dh);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          s = AG_MFMA(qd[j], kf[d][j], s);
          dp = AG_MFMA(dd[j], vf[d][j], dp);
        }
        if constexpr (DELTA) {
          const f32x4 of = row_piece<T, DB>(Raw<T>::value(orow[d]), FIRST, d0, d, lg4, a.dh);
#pragma unroll
          for (int j = 0; j < 4; ++j) dot += dd[j] * of[j];
        }
      }
      if constexpr (DELTA) {
        dot = over_groups(dot);                // of query t0 + li
#pragma unroll
        for (int r = 0; r < 4; ++r) D[r] = __shfl(dot, lg4 + r, WAVE);
      }
      if (next < n_it) load_rows(next);
    }
    exchange<P, 2, W>(sX, n, slot, share, on, sc);
    if (!on) continue;
    const bool edge = u0 + 15 > a.q_start + t0 || u0 < first_key(a, a.q_start + t0 + 15) || t0 + 15 >= a.c || u0 + 15 >= n_total;
    bool seen[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int t = t0 + lg4 + r, pos = a.q_start + t;
      seen[r] = t < a.c && u0 + li < n_total && u <= pos && u >= first_key(a, pos);
      const float p = seen[r] ? expf(s[r] * a.scale - L[r]) : 0.f;
      s[r] = p;
      dp[r] = seen[r] ? p * (dp[r] - D[r]) * a.scale : 0.f;
    }
    auto at_row = [&](const T* __restrict__ p) { return [=](int row, int e) { return ldf(p + (int64_t)h * a.dh + (int64_t)min(t0 + row, a.c - 1) * q_stride + e); }; };
    second_product<T, DB>(av, d0, dt, s, edge, seen, a.dh, at_row(d_o));
    second_product<T, DB>(ak, d0, qt, dp, edge, seen, a.dh, at_row(q));
    if (next < n_it) load_cols(next);
    if (P > 1 && (n & 3) == 3) leave();
  }
  const int half = (a.dh + 1) / 2;
  float old[2][2][Pt::PAIRS];                  // of dk and dv
  auto at = [&](float* __restrict__ out, const typename Pt::Pair& p) { return out + ((int64_t)(u0 + p.row) * a.Hkv + kvh) * a.dh + p.e; };
#pragma unroll
  for (int which = 0; which < 2; ++which)
#pragma unroll
    for (int n = 0; n < Pt::PAIRS; ++n) {
      const auto p = Pt::pair(n, half);
      const bool in = p.in && u0 + p.row < n_total;
      float* x = at(which ? dv : dk, p);
      old[which][0][n] = in ? x[0] : 0.f;
      old[which][1][n] = in && p.e + half < a.dh ? x[half] : 0.f;
    }
  leave();
  __syncthreads();
  auto finish = [&](int which, float* __restrict__ out, T* __restrict__ fin) {
    float x[Pt::PAIRS], y[Pt::PAIRS];
    Pt::sums(part + which * Pt::FLOATS, half, x, y, [](int, int) { return 1.f; });
#pragma unroll
    for (int n = 0; n < Pt::PAIRS; ++n) {
      const auto p = Pt::pair(n, half);
      if (!p.in || u0 + p.row >= n_total) continue;
      const float r = old[which][0][n] + x[n], w = old[which][1][n] + y[n];
      at(out, p)[0] = r;
      if (p.e + half < a.dh) at(out, p)[half] = w;
      const int t = u0 + p.row - a.q_start;
      if (!fin || t < 0) continue;             // (an even head size: what the rotary embedding pairs)
      const float2 cs = which == 0 ? rope[(int64_t)t * half + p.e] : make_float2(1.f, 0.f);
      T* f = fin + ((int64_t)t * a.Hkv + kvh) * a.dh + p.e;
      stf(f, which == 0 ? r * cs.x + w * cs.y : r);             // rotation by the negative angle
      stf(f + half, which == 0 ? w * cs.x - r * cs.y : w);
    }
  };
  finish(0, dk, dkc);
  finish(1, dv, dvc);
}

// (Launch bounds: fp32 heads of 65 to 128 elements need 129 registers otherwise, one more than lets two workgroups share a CU.)
template <typename T, int DB, int P, int W>
__global__ __launch_bounds__(W * 64, DB * P == 8 ? 4 : 1) void attn_dkv_generic_k(const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v,
                                                                                  const T* __restrict__ d_o, const float* __restrict__ lse,
                                                                                  const float* __restrict__ delta, float* __restrict__ dk, float* __restrict__ dv,
                                                                                  AgShape a, T* __restrict__ dkc, T* __restrict__ dvc, const float2* __restrict__ rope) {
  AG_PARTS(2);
  dkv_block<T, DB, P, W, false>(part, blockIdx.x, blockIdx.y, q, k, v, nullptr, d_o, lse, delta, dk, dv, a, dkc, dvc, rope);
}
// dK/dV and dQ side by side, neither waiting for the other: the workgroups of dK/dV form delta themselves, the same sums in the same order.
template <typename T, int DB>
__global__ __launch_bounds__(512) void attn_bwd_narrow_k(const T* __restrict__ q, const T* __restrict__ k, const T* __restrict__ v, const T* __restrict__ o,
                                                          const T* __restrict__ d_o, const float* __restrict__ lse, T* __restrict__ dq, float* __restrict__ dk,
                                                          float* __restrict__ dv, AgShape a, T* __restrict__ dkc, T* __restrict__ dvc,
                                                          const float2* __restrict__ rope_q, const float2* __restrict__ rope_k, int n_first, bool dq_first) {
  constexpr int P = 1, W = 8;
  AG_PARTS(2);
  const bool first = (int)blockIdx.x < n_first;
  const int b = (int)blockIdx.x - (first ? 0 : n_first);
  if (first != dq_first) dkv_block<T, DB, P, W, true>(part, b / a.Hkv, b % a.Hkv, q, k, v, o, d_o, lse, nullptr, dk, dv, a, dkc, dvc, rope_k);
  else dq_block<T, DB, P, W>(part, b / a.Hq, b % a.Hq, q, k, v, o, d_o, lse, nullptr, dq, a, rope_q);
}

static AgShape shape_of(const AttnArgs& a) { return AgShape{a.Hq, a.Hkv, a.dh, a.q_start, a.q_len, a.scale, a.window, a.kv_first}; }
// Instances: pieces per wave, waves per block, waves.  Heads of up to 64 elements: one wave per block.  Wider ones, whose operands would not fit a wave's
// registers: two, or four - where there are few blocks, where the registers of two would spill (dK/dV, dQ of more than 160 elements), and, on sixteen waves, in
// the forward of more than 160.  Forward, 4 heads, 64 / 256 / 512 / 2112 keys, 64 queries, fp32, two per block and four, in us: heads of 80 7 11 17 58 and 8 15 27
// 100; 192 10 18 29 104 and 8 18 31 115; bf16 256 12 23 37 128 and 10 25 46 163, four of sixteen waves 12 22 34 115.
#define AG_CASE(DB, P, W) if (dh <= 16 * DB * P) return f(std::integral_constant<int, DB>{}, std::integral_constant<int, P>{}, std::integral_constant<int, W>{})
template <typename F> static void narrow_heads(int dh, F f) {
  AG_CASE(1, 1, 8);
  AG_CASE(2, 1, 8);
  AG_CASE(3, 1, 8);
  AG_CASE(4, 1, 8);
}
template <typename F> static void four_per_block(int dh, F f) {
  AG_CASE(2, 4, 8);
  AG_CASE(3, 4, 8);
  AG_CASE(4, 4, 8);
}
template <typename F> static void forward_long(int dh, F f) {
  AG_CASE(3, 2, 8);
  AG_CASE(4, 2, 8);
  AG_CASE(5, 2, 8);
  AG_CASE(3, 4, 16);
  AG_CASE(4, 4, 16);
}
template <typename F> static void dq_long(int dh, F f) {
  AG_CASE(3, 2, 8);
  AG_CASE(4, 2, 8);
  AG_CASE(5, 2, 8);
  AG_CASE(3, 4, 8);
  AG_CASE(4, 4, 8);
}
#undef AG_CASE
static bool few_keys(const AttnArgs& a) { return a.q_start + a.q_len <= (a.dh <= 128 ? 32 : a.dh <= 192 ? 128 : 256); }

template <typename T>
static hipError_t forward_t(const AttnArgs& a, hipStream_t st) {
  const AgShape s = shape_of(a);
  const dim3 grid((unsigned)cdiv(a.q_len, 16), (unsigned)a.Hq);
  auto go = [&](auto db, auto p, auto w) {
    attn_fwd_generic_k<T, decltype(db)::value, decltype(p)::value, decltype(w)::value><<<grid, decltype(w)::value * 64, 0, st>>>((T*)a.q, (const T*)a.k, (const T*)a.v, (T*)a.o, a.lse, s, a.rope_q);
  };
  if (a.dh <= 64) narrow_heads(a.dh, go); else if (few_keys(a)) four_per_block(a.dh, go); else forward_long(a.dh, go);
  return hipGetLastError();
}
template <typename T>
static hipError_t backward_t(const AttnArgs& a, hipStream_t st) {
  const AgShape s = shape_of(a);
  const dim3 gq((unsigned)cdiv(a.q_len, 16), (unsigned)a.Hq), gk((unsigned)cdiv((int64_t)a.q_start + a.q_len, 16), (unsigned)a.Hkv);
  const AttnNarrowPlan p = attn_narrow_plan(a);
  if (p.one_launch) {
    narrow_heads(a.dh, [&](auto db, auto, auto) {
      attn_bwd_narrow_k<T, decltype(db)::value><<<(unsigned)(p.n_dkv + p.n_dq), 512, 0, st>>>((const T*)a.q, (const T*)a.k, (const T*)a.v, (const T*)a.o, (const T*)a.d_o, a.lse, (T*)a.dq,
                                                                            a.dk, a.dv, s, (T*)a.dkc, (T*)a.dvc, a.rope_q, a.rope_k, (int)(p.dq_first ? p.n_dq : p.n_dkv), p.dq_first);
    });
    return hipGetLastError();
  }
  auto dq = [&](auto db, auto p, auto w) {
    attn_dq_generic_k<T, decltype(db)::value, decltype(p)::value, decltype(w)::value><<<gq, decltype(w)::value * 64, 0, st>>>((const T*)a.q, (const T*)a.k, (const T*)a.v, (const T*)a.o, (const T*)a.d_o,
                                                                                        a.lse, a.delta, (T*)a.dq, s, a.rope_q);
  };
  if (a.dh <= 64) narrow_heads(a.dh, dq); else if (few_keys(a)) four_per_block(a.dh, dq); else dq_long(a.dh, dq);
  auto dkv = [&](auto db, auto p, auto w) {
    attn_dkv_generic_k<T, decltype(db)::value, decltype(p)::value, decltype(w)::value><<<gk, decltype(w)::value * 64, 0, st>>>((const T*)a.q, (const T*)a.k, (const T*)a.v, (const T*)a.d_o, a.lse, a.delta,
                                                                                         a.dk, a.dv, s, (T*)a.dkc, (T*)a.dvc, a.rope_k);
  };
  if (a.dh <= 64) narrow_heads(a.dh, dkv); else four_per_block(a.dh, dkv);
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
