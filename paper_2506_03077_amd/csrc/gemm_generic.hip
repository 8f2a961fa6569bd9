// Shape-agnostic GEMM: any M, N, K, any of the three operand layouts, fp32 or
// bf16 storage, fp32 products and sums.  The path of the fp32 configuration and of
// shapes the bf16 MFMA kernels do not take.
#include "launch.h"
#include "device.h"

#include <algorithm>
#include <iterator>
#include <type_traits>

namespace sbp {

// 32 x 32 tiles, the reduction dealt to the eight waves of a workgroup in steps of 16, fp32 MFMAs (v_mfma_f32_16x16x4_f32) straight
// from registers.  What bounds the calls of the small fp32 configuration is latency - a handful of workgroups, each a chain of
// load -> barrier -> multiply per slice of the reduction - so there is no LDS staging and no barrier before the sum over the waves (a
// fixed order), and the loads of a wave's next step go out before it multiplies the present one.  Against 64 x 64 tiles staged
// through LDS (the earlier form): 64 x 64 x 64 10.7 -> 3.2 us, 64 x 64 x 512 67 -> 6.5, 256 x 1500 x 256 36 -> 7.4; what reads of the
// operands bound later is no worse: 1024^3 178 -> 35, 2048^3 416 -> 232 us (74 TFLOP/s).
// Lane l holds, of a 16-row block, row l % 16 at k 4 (l / 16) .. + 3 of the step; MFMA j of the step takes element j of both operands.
constexpr int TILE = GEMM_ROPE_COLS, WAVES = 8, KSTEP = 16;
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// An operand's four elements of a row and step, held as they were loaded until the product that takes them (a conversion would wait for them in front of the
// present step's products): bf16 in pairs where they lie side by side, else one by one.
template <typename TI> struct Held;
template <> struct Held<float> {
  typedef f32x4 type;
  typedef f32x4 four __attribute__((aligned(4)));      // rows may start anywhere
  static __device__ __forceinline__ type pack(f32x4 v) { return v; }
  static __device__ __forceinline__ float one(float x) { return x; }
  static __device__ __forceinline__ f32x4 value(type v, bool) { return v; }
};
template <> struct Held<bf16_t> {
  typedef u32x4 type;
  typedef uint32_t two __attribute__((ext_vector_type(2)));
  typedef two four __attribute__((aligned(2)));
  static __device__ __forceinline__ type pack(two v) { return type{v[0], v[1], 0u, 0u}; }
  static __device__ __forceinline__ uint32_t one(bf16_t x) { return (uint32_t)__builtin_bit_cast(uint16_t, x); }
  static __device__ __forceinline__ f32x4 value(type v, bool pairs) {
    f32x4 f;
    f[0] = __uint_as_float(v[0] << 16);
    f[1] = __uint_as_float(pairs ? v[0] & 0xffff0000u : v[1] << 16);
    f[2] = __uint_as_float(pairs ? v[1] << 16 : v[2] << 16);
    f[3] = __uint_as_float(pairs ? v[1] & 0xffff0000u : v[3] << 16);
    return f;
  }
};
// Both 16-row blocks of an operand for the step at k0: element (row, k + j), row-contiguous reductions at p[row * ld + k], reduction-major operands at
// p[k * ld + row]; past the last row: the last row again (its products are not stored); past the end of the reduction: its last element
// again (see step_values).  No load hangs on a lane condition, so that all of a step are under way at once: with one branch per element, the
// earlier form, each was waited for before the next (1025 x 4097 x 4097, fp32 NN 1000 -> 607 us, bf16 TN 1106 -> 640; 4097 x 4097 x 129, bf16 NN 155 -> 139;
// 4096^3 fp32 NN, which the L2 bounds, 2398 -> 2199).
template <typename TI>
__device__ __forceinline__ void load_step(typename Held<TI>::type (&v)[2], const TI* __restrict__ p, int64_t ld, bool k_major, int r0, int rows, int k0, int K,
                                          int li, int lg) {
  const bool whole = k0 + KSTEP <= K;
  const int k = k0 + 4 * lg;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = min(r0 + i * 16 + li, rows - 1);
    if (whole) {
      if (k_major) {
        const TI* q = p + (int64_t)k * ld + r;
#pragma unroll
        for (int j = 0; j < 4; ++j) v[i][j] = Held<TI>::one(q[j * ld]);
      } else {
        v[i] = Held<TI>::pack(*(const typename Held<TI>::four*)(p + (int64_t)r * ld + k));
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int64_t kk = min(k + j, K - 1);
        v[i][j] = Held<TI>::one(p[k_major ? kk * ld + r : (int64_t)r * ld + kk]);
      }
    }
  }
}
template <typename TI>
__device__ __forceinline__ f32x4 step_values(typename Held<TI>::type v, bool k_major, int k0, int K, int lg) {
  const bool whole = k0 + KSTEP <= K;
  f32x4 f = Held<TI>::value(v, whole && !k_major);
  if (!whole) {
#pragma unroll
    for (int j = 0; j < 4; ++j) f[j] = k0 + 4 * lg + j < K ? f[j] : 0.f;
  }
  return f;
}
// Several problems in one launch, each with its own layout, adding to its output or storing it, and one or more reduction segments (operand pairs whose products
// are summed into one output): a launch of the small configuration costs 4.8 us however little it does, its layer and head issued 86 of them.
// (NP problems, NS segments: the smallest of six sizes, as the arguments' cache lines are fetched one dependent miss after the other.  A 256-token fp32 layer with its
// head: GEMM launches 14 -> 12 and arguments of 2.6 KB -> 0.3 to 1.1: 108 -> 99 us.)
constexpr int GENERIC_PROBLEMS = 8, GENERIC_SEGMENTS = 56;
struct GenericSegment { const void* A; const void* B; const int* rows_dev; int K, lda, ldb; };
enum { GENERIC_TA = 1, GENERIC_TB = 2, GENERIC_ACC = 4 };
struct GenericProblem { void* C; int64_t ldc; int M, N, flags, seg0, nseg, tile0, tiles_n; };
template <int NP, int NS> struct GenericArgs { int n; GenericProblem p[NP]; GenericSegment s[NS]; };
using GenericAll = GenericArgs<GENERIC_PROBLEMS, GENERIC_SEGMENTS>;

// gate (optional; rows of ldc elements, like C, which is then not written): the product is the gradient wrt act = silu(gate) * up; act gets that
// value, gate and up their gradients, in place.
struct GenericSwiglu { void *gate, *up, *act; };
// tab (optional): the output of problem `problem` is rotated, heads of 2 * half columns, which divide a tile; the angles are fetched before the products.
// (As a pass over K: one launch more of a chain of 24, 96 us against 89.5 for a 256-token fp32 layer with its head.)
struct GenericRope { const float2* tab; int half, period, problem; };
// Launch bounds: 80 registers let three workgroups share a CU, and only the instance that rotates would take more, 82: with them in all fp32 instances of up to three
// problems two workgroups shared one, and 1024 x 2816 with K = 8, 2816 tiles, took 19.5 us instead of 15.0; with the rotation's code in the smaller instances, but 80 registers,
// the forward of 2 x 1133 rows at 264 / 2730 371 instead of 367 us, a head of 2036 rows, 16000 x 512, 1709 instead of 1674.
template <typename TI, typename TO, int NP, int NS>
__global__ __launch_bounds__(WAVES * 64, (!std::is_same_v<TI, bf16_t> && NP == 3 ? 6 : 1)) void gemm_generic_k(const GenericArgs<NP, NS> ga, const GenericSwiglu sw, const GenericRope rope) {
  constexpr bool ROPE = !std::is_same_v<TI, bf16_t> && NP == 3;      // (K beside V, or beside q and V)
  int pi = 0;
#pragma unroll
  for (int i = 1; i < NP; ++i)
    if (i < ga.n && (int)blockIdx.x >= ga.p[i].tile0) pi = i;
  const GenericProblem& g = ga.p[pi];
  const int tile = (int)blockIdx.x - g.tile0, m0 = tile / g.tiles_n * TILE, n0 = tile % g.tiles_n * TILE;
  // run-time row count (M for NT / NN, the reduction K for the dW form)
  auto rows = [&](const GenericSegment& q) { return q.rows_dev ? max(0, *q.rows_dev) : 0x7fffffff; };
  const bool ta = g.flags & GENERIC_TA, tb = g.flags & GENERIC_TB, acc_c = g.flags & GENERIC_ACC;
  const int M = ta ? g.M : min(g.M, rows(ga.s[g.seg0])), N = g.N;
  __shared__ float part[WAVES][TILE][TILE + 1];
  if (m0 >= M) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), li = threadIdx.x & 15, lg = (threadIdx.x & 63) >> 4;
  constexpr int OUT = TILE * TILE / (WAVES * 64);      // elements of C per thread
  const bool rotated = ROPE && rope.tab && pi == rope.problem;
  float2 cs[OUT];
  if (rotated) {
#pragma unroll
    for (int e = 0; e < OUT; ++e) {
      const int id = e * WAVES * 64 + (int)threadIdx.x;
      cs[e] = rope.tab[(int64_t)(min(m0 + id / TILE, M - 1) % rope.period) * rope.half + (id % TILE) % rope.half];
    }
  }
  f32x4 acc[2][2] = {};
  // The steps of all segments, one after the other, dealt to the waves: k0 = this wave's next one.  What a step reads by is kept in registers and
  // changes with the segment (NS == 1: never).
  int seg = -1, k0 = 0, dealt = 0;
  const TI *A = nullptr, *B = nullptr;
  int K = 0, lda = 0, ldb = 0;
  typename Held<TI>::type a[2], b[2];
  auto enter = [&]() {
    const GenericSegment& q = ga.s[NS == 1 ? 0 : g.seg0 + seg];
    A = (const TI*)q.A; B = (const TI*)q.B; lda = q.lda; ldb = q.ldb;
    K = ta ? min(q.K, rows(q)) : q.K;
    k0 = ((wave - dealt) & (WAVES - 1)) * KSTEP;
    dealt += (K + KSTEP - 1) / KSTEP;
  };
  auto next = [&]() {
    k0 += WAVES * KSTEP;
    while (k0 >= K) {
      if (NS == 1 || ++seg >= g.nseg) return false;
      enter();
    }
    return true;
  };
  auto load = [&]() {
    if (NS == 1) asm volatile("" : "+s"(lda), "+s"(ldb));      // (row times stride anew for each step: kept, all of them take 50 registers)
    load_step<TI>(a, A, lda, ta, m0, M, k0, K, li, lg);
    load_step<TI>(b, B, ldb, !tb, n0, N, k0, K, li, lg);
  };
  if (NS == 1) { enter(); k0 -= WAVES * KSTEP; }
  bool more = next();
  const bool any = more;
  if (more) load();
  while (more) {
    const f32x4 a0 = step_values<TI>(a[0], ta, k0, K, lg), a1 = step_values<TI>(a[1], ta, k0, K, lg);
    const f32x4 b0 = step_values<TI>(b[0], !tb, k0, K, lg), b1 = step_values<TI>(b[1], !tb, k0, K, lg);
    more = next();
    if (more) load();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[j], b0[j], acc[0][0], 0, 0, 0);
      acc[0][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[j], b1[j], acc[0][1], 0, 0, 0);
      acc[1][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[j], b0[j], acc[1][0], 0, 0, 0);
      acc[1][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[j], b1[j], acc[1][1], 0, 0, 0);
    }
  }
  const int waves = min(WAVES, dealt);      // the others had no step
  if (any) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) part[wave][i * 16 + 4 * lg + r][j * 16 + li] = acc[i][j][r];
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < OUT; ++e) {
    const int id = e * WAVES * 64 + (int)threadIdx.x, row = id / TILE, col = id % TILE;
    if (m0 + row >= M || n0 + col >= N) continue;
    float v = 0.f;
    for (int w = 0; w < waves; ++w) v += part[w][row][col];
    if (rotated) {
      const bool up = col % (2 * rope.half) >= rope.half;
      const int pair = up ? col - rope.half : col + rope.half;
      float x = 0.f;
      for (int w = 0; w < waves; ++w) x += part[w][row][pair];
      v = v * cs[e].x + (up ? x : -x) * cs[e].y;
    }
    const int64_t at = (int64_t)(m0 + row) * g.ldc + n0 + col;
    if (NP == 1 && sw.gate) {
      TO *gate = (TO*)sw.gate + at, *up = (TO*)sw.up + at;
      const float z = ldf(gate), u = ldf(up), s = 1.0f / (1.0f + __expf(-z));
      if (sw.act) stf((TO*)sw.act + at, z * s * u);
      stf(gate, v * u * s * (1.0f + z * (1.0f - s)));
      stf(up, v * z * s);
      continue;
    }
    TO* p = (TO*)g.C + at;
    stf(p, acc_c ? ldf(p) + v : v);
  }
}

// What one launch takes: problems of the same types.  Accumulated problems with the same C as an earlier one become segments of it (C is written once, and
// read if the first of them adds); sum: all n are segments of one stored output.  False: not in one launch.
static bool generic_args(const GemmArgs* gs, int n, bool sum, GenericAll& ga, int64_t& tiles) {
  ga.n = 0;
  tiles = 0;
  int seg_of[GENERIC_SEGMENTS], n_seg = 0;       // segments in the order given, and the problem each belongs to
  GenericSegment segs[GENERIC_SEGMENTS];
  for (int i = 0; i < n; ++i) {
    const GemmArgs& g = gs[i];
    if (g.M == 0 || g.N == 0) continue;
    if (g.in_dt != gs[0].in_dt || g.out_dt != gs[0].out_dt || g.lda > INT32_MAX || g.ldb > INT32_MAX) return false;
    const int layout = (g.ta ? GENERIC_TA : 0) | (g.tb ? GENERIC_TB : 0);
    int pi = -1;
    for (int j = 0; j < ga.n && pi < 0; ++j) {
      const GenericProblem& p = ga.p[j];
      if (p.C != g.C) continue;
      if (!(sum || g.acc) || p.M != g.M || p.N != g.N || p.ldc != g.ldc || ((p.flags ^ layout) & (GENERIC_TA | GENERIC_TB)) || (g.rows_dev && !g.ta)) return false;
      pi = j;
    }
    if (pi < 0) {
      if (ga.n == GENERIC_PROBLEMS || (sum && ga.n == 1)) return false;
      pi = ga.n++;
      ga.p[pi] = GenericProblem{g.C, g.ldc, g.M, g.N, layout | (g.acc && !sum ? GENERIC_ACC : 0), 0, 0, (int)tiles, (int)cdiv(g.N, TILE)};
      tiles += cdiv(g.M, TILE) * cdiv(g.N, TILE);
      if (tiles > INT32_MAX) return false;
    }
    for (int two = 0; two < (g.A2 ? 2 : 1); ++two) {
      if (n_seg == GENERIC_SEGMENTS) return false;
      const void *A = two ? g.A2 : g.A, *B = two ? g.B2 : g.B;
      segs[n_seg] = GenericSegment{A, B, g.rows_dev, g.K, (int)g.lda, (int)g.ldb};
      seg_of[n_seg++] = pi;
    }
  }
  int at = 0;
  for (int j = 0; j < ga.n; ++j) {
    ga.p[j].seg0 = at;
    for (int i = 0; i < n_seg; ++i)
      if (seg_of[i] == j) ga.s[at++] = segs[i];
    ga.p[j].nseg = at - ga.p[j].seg0;
  }
  return true;
}
// n problems in one launch (see generic_args); hipErrorInvalidValue where they do not fit one, with nothing launched
hipError_t gemm_generic(const GemmArgs* gs, int n, bool sum, hipStream_t st) {
  GenericAll ga;
  int64_t tiles;
  if (gs[0].swiglu_gate && (n != 1 || gs[0].acc || gs[0].A2)) return hipErrorInvalidValue;
  if (!generic_args(gs, n, sum, ga, tiles)) return hipErrorInvalidValue;
  if (ga.n == 0) return hipSuccess;
  const GemmArgs& g = gs[0];
  GenericRope rope{};
  for (int i = 0; i < n; ++i) {
    if (!gs[i].rope) continue;
    // (n problems without a shared or empty output: the i-th of them)
    if (rope.tab || ga.n != n || gs[i].in_dt == DT_BF16 || gs[i].acc || gs[i].ta || !gs[i].tb || gs[i].rope_dim < 2 || TILE % gs[i].rope_dim || gs[i].rope_dim % 2 ||
        gs[i].N % gs[i].rope_dim || gs[i].rope_period < 1)
      return hipErrorInvalidValue;
    rope = GenericRope{gs[i].rope, gs[i].rope_dim / 2, gs[i].rope_period, i};
  }
  int n_seg = 0;
  for (int i = 0; i < ga.n; ++i) n_seg += ga.p[i].nseg;
  if (rope.tab && n_seg > 3) return hipErrorInvalidValue;
  auto go = [&](auto kernel, auto args) {
    args.n = ga.n;
    std::copy_n(ga.p, std::min<size_t>(std::size(args.p), ga.n), args.p);
    std::copy_n(ga.s, std::min<size_t>(std::size(args.s), n_seg), args.s);
    kernel<<<(unsigned)tiles, WAVES * 64, 0, st>>>(args, GenericSwiglu{gs[0].swiglu_gate, gs[0].swiglu_up, gs[0].swiglu_act}, rope);
  };
#define GG(TI, TO)                                                                                             \
  do {                                                                                                         \
    if (ga.n == 1 && n_seg == 1 && !rope.tab) go(gemm_generic_k<TI, TO, 1, 1>, GenericArgs<1, 1>{});                        \
    else if (ga.n <= 2 && n_seg <= 3 && !rope.tab) go(gemm_generic_k<TI, TO, 2, 3>, GenericArgs<2, 3>{});                   \
    else if (ga.n <= 3 && n_seg <= 3) go(gemm_generic_k<TI, TO, 3, 3>, GenericArgs<3, 3>{});                   \
    else if (n_seg <= 8) go(gemm_generic_k<TI, TO, GENERIC_PROBLEMS, 8>, GenericArgs<GENERIC_PROBLEMS, 8>{});  \
    else if (n_seg <= 16) go(gemm_generic_k<TI, TO, GENERIC_PROBLEMS, 16>, GenericArgs<GENERIC_PROBLEMS, 16>{}); \
    else go(gemm_generic_k<TI, TO, GENERIC_PROBLEMS, GENERIC_SEGMENTS>, GenericAll{});                         \
  } while (0)
  if (g.in_dt != DT_BF16) GG(float, float);
  else if (g.out_dt == DT_BF16) GG(bf16_t, bf16_t);
  else GG(bf16_t, float);
#undef GG
  return hipGetLastError();
}

}  // namespace sbp
