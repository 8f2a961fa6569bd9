// Shape-agnostic GEMM: any M, N, K, any of the three operand layouts, fp32 or
// bf16 storage, fp32 products and sums.  The path of the fp32 configuration and of
// shapes the bf16 MFMA kernels do not take.
#include "launch.h"
#include "device.h"

#include <algorithm>
#include <iterator>

namespace sbp {

// 32 x 32 tiles, the reduction dealt to the eight waves of a workgroup in steps of 16, fp32 MFMAs (v_mfma_f32_16x16x4_f32) straight
// from registers.  What bounds the calls of the small fp32 configuration is latency - a handful of workgroups, each a chain of
// load -> barrier -> multiply per slice of the reduction - so there is no LDS staging and no barrier before the sum over the waves (a
// fixed order), and the loads of a wave's next step go out before it multiplies the present one.  Against 64 x 64 tiles staged
// through LDS (the earlier form): 64 x 64 x 64 10.7 -> 3.2 us, 64 x 64 x 512 67 -> 6.5, 256 x 1500 x 256 36 -> 7.4; what reads of the
// operands bound later is no worse: 1024^3 178 -> 35, 2048^3 416 -> 228 us (75 TFLOP/s).
// Lane l holds, of a 16-row block, row l % 16 at k 4 (l / 16) .. + 3 of the step; MFMA j of the step takes element j of both operands.
constexpr int TILE = 32, WAVES = 8, KSTEP = 16;
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <typename TI>
__device__ __forceinline__ f32x4 operand(const TI* __restrict__ p, bool k_major, int64_t ld, int row, int rows, int k, int K, bool vec) {
  // element (row, k + j): row-contiguous reductions at p[row * ld + k], reduction-major operands at p[k * ld + row]; past the end of
  // the reduction: zeros; past the last row: the last row again (its products are not stored)
  const int r = min(row, rows - 1);
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (!k_major) {
    const TI* q = p + (int64_t)r * ld + k;
    if (vec && k + 4 <= K) {
      if constexpr (sizeof(TI) == 4) v = *(const f32x4*)q;
      else {
        typedef bf16_t bf16x4 __attribute__((ext_vector_type(4)));
        const bf16x4 w = *(const bf16x4*)q;
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = (float)w[j];
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) if (k + j < K) v[j] = ldf(q + j);
    }
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) if (k + j < K) v[j] = ldf(p + (int64_t)(k + j) * ld + r);
  }
  return v;
}
// Several problems in one launch, each with its own layout and one or more reduction segments (operand pairs whose products are summed into
// one output): a launch of the small configuration costs 4.8 us however little it does, its layer and head issued 86 of them.
// (NP problems, NS segments: the smallest of three sizes, as the arguments' cache lines are fetched one dependent miss after the other.)
constexpr int GENERIC_PROBLEMS = 8, GENERIC_SEGMENTS = 56;
struct GenericSegment { const void* A; const void* B; const int* rows_dev; int K, lda, ldb, vec; };       // vec: bit 0 A, bit 1 B
struct GenericProblem { void* C; int64_t ldc; int M, N, ta, tb, seg0, nseg, tile0, tiles_n; };
template <int NP, int NS> struct GenericArgs { int n; GenericProblem p[NP]; GenericSegment s[NS]; };
using GenericAll = GenericArgs<GENERIC_PROBLEMS, GENERIC_SEGMENTS>;

// gate (optional; rows of ldc elements, like C, which is then not written): the product is the gradient wrt act = silu(gate) * up; act gets that
// value, gate and up their gradients, in place.
struct GenericSwiglu { void *gate, *up, *act; };
template <typename TI, typename TO, bool ACC, int NP, int NS>
__global__ __launch_bounds__(WAVES * 64) void gemm_generic_k(const GenericArgs<NP, NS> ga, const GenericSwiglu sw) {
  int pi = 0;
#pragma unroll
  for (int i = 1; i < NP; ++i)
    if (i < ga.n && (int)blockIdx.x >= ga.p[i].tile0) pi = i;
  const GenericProblem& g = ga.p[pi];
  const int tile = (int)blockIdx.x - g.tile0, m0 = tile / g.tiles_n * TILE, n0 = tile % g.tiles_n * TILE;
  // run-time row count (M for NT / NN, the reduction K for the dW form)
  auto rows = [&](const GenericSegment& q) { return q.rows_dev ? max(0, *q.rows_dev) : 0x7fffffff; };
  const int M = g.ta ? g.M : min(g.M, rows(ga.s[g.seg0])), N = g.N;
  __shared__ float part[WAVES][TILE][TILE + 1];
  if (m0 >= M) return;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), li = threadIdx.x & 15, lg = (threadIdx.x & 63) >> 4;
  f32x4 acc[2][2] = {};
  f32x4 a[2], b[2];
  // the steps of all segments, one after the other, dealt to the waves: seg, k0 = this wave's next one, K its segment's reduction
  int seg = -1, k0 = 0, K = 0, dealt = 0;
  auto next = [&]() {
    k0 += WAVES * KSTEP;
    while (k0 >= K) {
      dealt += (K + KSTEP - 1) / KSTEP;
      if (++seg >= g.nseg) return false;
      K = ga.s[g.seg0 + seg].K;
      if (g.ta) K = min(K, rows(ga.s[g.seg0 + seg]));
      k0 = ((wave - dealt) & (WAVES - 1)) * KSTEP;
    }
    return true;
  };
  auto load = [&]() {
    const GenericSegment& q = ga.s[g.seg0 + seg];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      a[i] = operand((const TI*)q.A, g.ta != 0, q.lda, m0 + i * 16 + li, M, k0 + 4 * lg, K, (q.vec & 1) != 0);
      b[i] = operand((const TI*)q.B, g.tb == 0, q.ldb, n0 + i * 16 + li, N, k0 + 4 * lg, K, (q.vec & 2) != 0);
    }
  };
  bool more = next();
  const bool any = more;
  if (more) load();
  while (more) {
    const f32x4 a0 = a[0], a1 = a[1], b0 = b[0], b1 = b[1];
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
  for (int e = 0; e < TILE * TILE / (WAVES * 64); ++e) {
    const int id = e * WAVES * 64 + (int)threadIdx.x, row = id / TILE, col = id % TILE;
    if (m0 + row >= M || n0 + col >= N) continue;
    float v = 0.f;
    for (int w = 0; w < waves; ++w) v += part[w][row][col];
    const int64_t at = (int64_t)(m0 + row) * g.ldc + n0 + col;
    if (NP == 1 && !ACC && sw.gate) {
      TO *gate = (TO*)sw.gate + at, *up = (TO*)sw.up + at;
      const float z = ldf(gate), u = ldf(up), s = 1.0f / (1.0f + __expf(-z));
      if (sw.act) stf((TO*)sw.act + at, z * s * u);
      stf(gate, v * u * s * (1.0f + z * (1.0f - s)));
      stf(up, v * z * s);
      continue;
    }
    TO* p = (TO*)g.C + at;
    if (ACC) stf(p, ldf(p) + v); else stf(p, v);
  }
}

// What one launch takes: problems of the same types that all add to their C or all store it.  Accumulated problems with the same C become
// segments of one (C is read and written once); sum: all n are segments of one stored output.  False: not in one launch.
static bool generic_args(const GemmArgs* gs, int n, bool sum, GenericAll& ga, int64_t& tiles) {
  ga.n = 0;
  tiles = 0;
  int seg_of[GENERIC_SEGMENTS], n_seg = 0;       // segments in the order given, and the problem each belongs to
  GenericSegment segs[GENERIC_SEGMENTS];
  const uintptr_t four = 4 * dtype_size(gs[0].in_dt) - 1;
  for (int i = 0; i < n; ++i) {
    const GemmArgs& g = gs[i];
    if (g.M == 0 || g.N == 0) continue;
    if (g.in_dt != gs[0].in_dt || g.out_dt != gs[0].out_dt || (!sum && g.acc != gs[0].acc) || g.lda > INT32_MAX || g.ldb > INT32_MAX) return false;
    int pi = -1;
    for (int j = 0; j < ga.n && pi < 0; ++j) {
      const GenericProblem& p = ga.p[j];
      if (p.C != g.C) continue;
      if (!(sum || g.acc) || p.M != g.M || p.N != g.N || p.ldc != g.ldc || p.ta != (g.ta ? 1 : 0) || p.tb != (g.tb ? 1 : 0) || (g.rows_dev && !g.ta)) return false;
      pi = j;
    }
    if (pi < 0) {
      if (ga.n == GENERIC_PROBLEMS || (sum && ga.n == 1)) return false;
      pi = ga.n++;
      ga.p[pi] = GenericProblem{g.C, g.ldc, g.M, g.N, g.ta ? 1 : 0, g.tb ? 1 : 0, 0, 0, (int)tiles, (int)cdiv(g.N, TILE)};
      tiles += cdiv(g.M, TILE) * cdiv(g.N, TILE);
      if (tiles > INT32_MAX) return false;
    }
    for (int two = 0; two < (g.A2 ? 2 : 1); ++two) {
      if (n_seg == GENERIC_SEGMENTS) return false;
      const void *A = two ? g.A2 : g.A, *B = two ? g.B2 : g.B;
      // four elements at a time where rows of a K-contiguous operand start at multiples of four
      segs[n_seg] = GenericSegment{A, B, g.rows_dev, g.K, (int)g.lda, (int)g.ldb, (g.lda % 4 == 0 && !((uintptr_t)A & four) ? 1 : 0) | (g.ldb % 4 == 0 && !((uintptr_t)B & four) ? 2 : 0)};
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
  int n_seg = 0;
  for (int i = 0; i < ga.n; ++i) n_seg += ga.p[i].nseg;
  auto go = [&](auto kernel, auto args) {
    args.n = ga.n;
    std::copy_n(ga.p, std::min<size_t>(std::size(args.p), ga.n), args.p);
    std::copy_n(ga.s, std::min<size_t>(std::size(args.s), n_seg), args.s);
    kernel<<<(unsigned)tiles, WAVES * 64, 0, st>>>(args, GenericSwiglu{gs[0].swiglu_gate, gs[0].swiglu_up, gs[0].swiglu_act});
  };
#define GG(TI, TO, ACC)                                                                                        \
  do {                                                                                                         \
    if (ga.n == 1 && n_seg == 1) go(gemm_generic_k<TI, TO, ACC, 1, 1>, GenericArgs<1, 1>{});                   \
    else if (ga.n <= 2 && n_seg <= 3) go(gemm_generic_k<TI, TO, ACC, 2, 3>, GenericArgs<2, 3>{});              \
    else go(gemm_generic_k<TI, TO, ACC, GENERIC_PROBLEMS, GENERIC_SEGMENTS>, GenericAll{});                    \
  } while (0)
  const bool acc = g.acc && !sum;
  if (g.in_dt == DT_BF16) {
    if (g.out_dt == DT_BF16 && acc) GG(bf16_t, bf16_t, true);
    else if (g.out_dt == DT_BF16) GG(bf16_t, bf16_t, false);
    else if (acc) GG(bf16_t, float, true);
    else GG(bf16_t, float, false);
  } else {
    if (acc) GG(float, float, true);
    else GG(float, float, false);
  }
#undef GG
  return hipGetLastError();
}

}  // namespace sbp
