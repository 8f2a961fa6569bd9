// Shape-agnostic GEMM: any M, N, K, any of the three operand layouts, fp32 or
// bf16 storage, fp32 products and sums.  The path of the fp32 configuration and of
// shapes the bf16 MFMA kernels do not take.
#include "launch.h"
#include "device.h"

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
template <typename TI, typename TO, bool ACC>
__global__ __launch_bounds__(WAVES * 64) void gemm_generic_k(const TI* __restrict__ A, const TI* __restrict__ B, TO* __restrict__ C, int M,
                                                              int N, int K, int64_t lda, int64_t ldb, int64_t ldc, int ta, int tb,
                                                              int vec_a, int vec_b, const int* __restrict__ rows_dev) {
  if (rows_dev) {   // run-time row count (M for NT / NN, the reduction K for the dW form)
    const int rows = max(0, *rows_dev);
    if (ta) K = min(K, rows); else M = min(M, rows);
  }
  __shared__ float part[WAVES][TILE][TILE + 1];
  const int m0 = blockIdx.y * TILE, n0 = blockIdx.x * TILE;
  if (m0 >= M) return;
  const int wave = threadIdx.x >> 6, li = threadIdx.x & 15, lg = (threadIdx.x & 63) >> 4;
  f32x4 acc[2][2] = {};
  f32x4 a[2], b[2];
  auto load = [&](int k0) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      a[i] = operand(A, ta != 0, lda, m0 + i * 16 + li, M, k0 + 4 * lg, K, vec_a != 0);
      b[i] = operand(B, tb == 0, ldb, n0 + i * 16 + li, N, k0 + 4 * lg, K, vec_b != 0);
    }
  };
  int k0 = wave * KSTEP;
  if (k0 < K) load(k0);
  while (k0 < K) {
    const f32x4 a0 = a[0], a1 = a[1], b0 = b[0], b1 = b[1];
    k0 += WAVES * KSTEP;
    if (k0 < K) load(k0);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      acc[0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[j], b0[j], acc[0][0], 0, 0, 0);
      acc[0][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[j], b1[j], acc[0][1], 0, 0, 0);
      acc[1][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[j], b0[j], acc[1][0], 0, 0, 0);
      acc[1][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[j], b1[j], acc[1][1], 0, 0, 0);
    }
  }
  const int waves = min(WAVES, (K + KSTEP - 1) / KSTEP);      // the others had no step
  if (wave < waves) {
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
    TO* p = C + (int64_t)(m0 + row) * ldc + n0 + col;
    if (ACC) stf(p, ldf(p) + v); else stf(p, v);
  }
}

hipError_t gemm_generic(const GemmArgs& g, hipStream_t st) {
  if (g.M == 0 || g.N == 0) return hipSuccess;
  const dim3 grid((unsigned)cdiv(g.N, TILE), (unsigned)cdiv(g.M, TILE));
  // four elements at a time where rows of a K-contiguous operand start at multiples of four
  const uintptr_t four = 4 * dtype_size(g.in_dt) - 1;
  const int vec_a = g.lda % 4 == 0 && !((uintptr_t)g.A & four), vec_b = g.ldb % 4 == 0 && !((uintptr_t)g.B & four);
#define GG(TI, TO, ACC)                                                                                                         \
  gemm_generic_k<TI, TO, ACC><<<grid, WAVES * 64, 0, st>>>((const TI*)g.A, (const TI*)g.B, (TO*)g.C, g.M, g.N, g.K, g.lda, g.ldb, \
                                                           g.ldc, g.ta ? 1 : 0, g.tb ? 1 : 0, vec_a, vec_b, g.rows_dev)
  if (g.in_dt == DT_BF16) {
    if (g.out_dt == DT_BF16 && g.acc) GG(bf16_t, bf16_t, true);
    else if (g.out_dt == DT_BF16) GG(bf16_t, bf16_t, false);
    else if (g.acc) GG(bf16_t, float, true);
    else GG(bf16_t, float, false);
  } else {
    if (g.acc) GG(float, float, true);
    else GG(float, float, false);
  }
#undef GG
  return hipGetLastError();
}

}  // namespace sbp
