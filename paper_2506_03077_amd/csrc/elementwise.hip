// Row-statistic and elementwise kernels: RMSNorm (forward / adjoint), RoPE,
// SwiGLU, residual adds, dK/dV finishing, embedding gather / scatter-add.
// All are HBM-bound: one pass over their operands, 128-bit accesses where the
// row width allows, fp32 arithmetic with wavefront (64-lane) reductions.
#include "launch.h"
#include "device.h"
#include <algorithm>

namespace sbp {

#define DISPATCH_DT(dt, T, ...)                      \
  do {                                               \
    if ((dt) == DT_BF16) { using T = bf16_t; __VA_ARGS__; } \
    else { using T = float; __VA_ARGS__; }           \
  } while (0)

// ------------------------------------------------------------------ RoPE --
// Rotate-half pairing (j, j + dh/2), angle (t + pos_offset) * theta^(-2j/dh).
// Angles go through fp64: an fp32 product pos*inv_freq has an absolute error of
// ~2e-3 rad at position 32768, which the fp32 path's tolerance cannot absorb.
static inline unsigned ew_grid(int64_t n) { return (unsigned)std::min<int64_t>(cdiv(n, 256), 256 * 16); }
// (the workgroups after the table's: zeros for what the call accumulates into, n16 pieces of 16 bytes)
__global__ void rope_table_k(float2* tab, int n_pos, int half, double theta, int pos_offset, unsigned table_blocks, uint4* zeros, int64_t n16) {
  if (blockIdx.x >= table_blocks) {
    const int64_t stride = (int64_t)(gridDim.x - table_blocks) * blockDim.x;
    for (int64_t i = (int64_t)(blockIdx.x - table_blocks) * blockDim.x + threadIdx.x; i < n16; i += stride) zeros[i] = make_uint4(0, 0, 0, 0);
    return;
  }
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)n_pos * half) return;
  int t = (int)(i / half), j = (int)(i % half);
  double inv_freq = pow(theta, -(double)j / (double)half);   // theta^(-2j/dh)
  double ang = ((double)t + (double)pos_offset) * inv_freq;
  double s, c;
  sincos(ang, &s, &c);
  tab[i] = make_float2((float)c, (float)s);
}

hipError_t rope_table(float2* tab, int n_pos, int dh, float theta, int pos_offset, void* zeros, size_t zero_bytes, hipStream_t st) {
  const int half = dh / 2;
  const unsigned table = (unsigned)cdiv((int64_t)n_pos * half, 256);
  if (((uintptr_t)zeros | zero_bytes) & 15) return hipErrorInvalidValue;      // (a region of the workspace)
  const int64_t n16 = (int64_t)(zero_bytes / 16);
  const unsigned fill = n16 > 0 ? ew_grid(n16) : 0;
  if (table + fill == 0) return hipSuccess;
  rope_table_k<<<table + fill, 256, 0, st>>>(tab, n_pos, half, (double)theta, pos_offset, table, (uint4*)zeros, n16);
  return hipGetLastError();
}

template <typename T>
__global__ void rope_apply_k(T* x, const float2* tab, int64_t n_pairs, int period, int H, int half, int inverse) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_pairs) return;
  int j = (int)(i % half);
  int64_t rh = i / half;              // row * H + head
  int row = (int)(rh / H) % period;
  float2 cs = tab[(int64_t)row * half + j];
  float sn = inverse ? -cs.y : cs.y;
  T* p = x + rh * (2 * half);
  float a = ldf(p + j), b = ldf(p + j + half);
  stf(p + j, a * cs.x - b * sn);
  stf(p + j + half, b * cs.x + a * sn);
}

hipError_t rope_apply(int dt, void* x, const float2* tab, int rows, int period, int H, int dh, bool inverse, hipStream_t st) {
  int64_t n = (int64_t)rows * H * (dh / 2);
  if (n == 0) return hipSuccess;
  DISPATCH_DT(dt, T, (rope_apply_k<T><<<(unsigned)cdiv(n, 256), 256, 0, st>>>((T*)x, tab, n, period, H, dh / 2, inverse ? 1 : 0)));
  return hipGetLastError();
}

// --------------------------------------------------------------- RMSNorm --
__device__ __forceinline__ void load8(const float* p, float (&v)[8]) {
  const float4 a = *(const float4*)p, b = *(const float4*)(p + 4);
  v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
}
__device__ __forceinline__ void load8(const bf16_t* p, float (&v)[8]) {
  typedef bf16_t bf16x8_t __attribute__((ext_vector_type(8)));
  const bf16x8_t a = *(const bf16x8_t*)p;
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = (float)a[e];
}
__device__ __forceinline__ void store8(float* p, const float (&v)[8]) {
  *(float4*)p = make_float4(v[0], v[1], v[2], v[3]);
  *(float4*)(p + 4) = make_float4(v[4], v[5], v[6], v[7]);
}
__device__ __forceinline__ void store8(bf16_t* p, const float (&v)[8]) {
  typedef bf16_t bf16x8_t __attribute__((ext_vector_type(8)));
  bf16x8_t a;
#pragma unroll
  for (int e = 0; e < 8; ++e) a[e] = (bf16_t)v[e];
  *(bf16x8_t*)p = a;
}
constexpr int RV_MAX_IT = 8;    // 64 lanes x 8 elements x 8 = 4096 columns (the backward's 4 x d floats of LDS stay under 64 KiB)
// Vectorised form for d % 8 == 0, d <= 4096: one wave per row, 8 elements per lane per access, the row stays in
// registers between the sum of squares and the scaling (one read of x instead of two).  IT = accesses per lane, a constant, lanes past
// the row read its last elements and count them as zero: without branches all loads of a row go out together.  With a branch per
// access the row cost one memory latency each: 512 rows of 3584 8.5 -> 5.7 us.
template <int IT, typename T>
__device__ __forceinline__ void load_row(const T* __restrict__ p, int d, int lane, float (&v)[IT][8]) {
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int j = it * 512 + lane * 8;
    load8(p + min(j, d - 8), v[it]);
  }
}
// One instance per number of accesses: a row pays for the 512-column blocks that it has and no more
#define VEC_ROW_IT(n_it, IT, ...)                        \
  do {                                                   \
    switch (n_it) {                                      \
      case 1: { constexpr int IT = 1; __VA_ARGS__; } break; \
      case 2: { constexpr int IT = 2; __VA_ARGS__; } break; \
      case 3: { constexpr int IT = 3; __VA_ARGS__; } break; \
      case 4: { constexpr int IT = 4; __VA_ARGS__; } break; \
      case 5: { constexpr int IT = 5; __VA_ARGS__; } break; \
      case 6: { constexpr int IT = 6; __VA_ARGS__; } break; \
      case 7: { constexpr int IT = 7; __VA_ARGS__; } break; \
      default: { constexpr int IT = RV_MAX_IT; __VA_ARGS__; } \
    }                                                    \
  } while (0)
template <int IT, typename T>
__global__ __launch_bounds__(256) void rmsnorm_fwd_vec_k(const T* __restrict__ x, const float* add,
                                                         const T* __restrict__ g, T* __restrict__ out,
                                                         float* sum_out, float* __restrict__ rstd,
                                                         int rows, int d, float eps) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  float v[IT][8], a[IT][8], gv[IT][8];
  load_row<IT>(x + row * d, d, lane, v);
  if (add) load_row<IT>(add + row * d, d, lane, a);
  if (out) load_row<IT>(g, d, lane, gv);
  float ss = 0.f;
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const bool in = it * 512 + lane * 8 < d;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if (add) v[it][e] += a[it][e];
      ss += in ? v[it][e] * v[it][e] : 0.f;
    }
  }
  ss = wave_sum(ss);
  const float r = 1.0f / sqrtf(ss / (float)d + eps);
  if (lane == 0 && rstd) rstd[row] = r;
  if (!out) return;
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int j = it * 512 + lane * 8;
    if (j < d) {
      float o[8];
      if (sum_out) store8(sum_out + row * d + j, v[it]);
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = gv[it][e] * v[it][e] * r;
      store8(out + row * d + j, o);
    }
  }
}

// One workgroup per row.  r = 1/sqrt(mean(v^2) + eps) with v = x (+ add).
template <typename T>
__global__ __launch_bounds__(256) void rmsnorm_fwd_k(const T* __restrict__ x, const float* add,
                                                     const T* __restrict__ g, T* __restrict__ out,
                                                     float* sum_out, float* __restrict__ rstd,
                                                     int d, float eps) {
  __shared__ float red[16];
  const int64_t row = blockIdx.x;
  const T* xr = x + row * d;
  const float* ar = add ? add + row * d : nullptr;
  float ss = 0.f;
  for (int j = threadIdx.x; j < d; j += blockDim.x) {
    float v = ldf(xr + j) + (ar ? ar[j] : 0.f);
    ss += v * v;
  }
  ss = block_sum(ss, red);
  const float r = 1.0f / sqrtf(ss / (float)d + eps);
  if (threadIdx.x == 0 && rstd) rstd[row] = r;
  if (!out) return;
  for (int j = threadIdx.x; j < d; j += blockDim.x) {
    float v = ldf(xr + j) + (ar ? ar[j] : 0.f);
    if (sum_out) sum_out[row * d + j] = v;
    stf(out + row * d + j, ldf(g + j) * v * r);
  }
}

hipError_t rmsnorm_fwd(int dt, const void* x, const float* add, const void* g, void* out, float* sum_out,
                       float* rstd, int rows, int d, float eps, hipStream_t st) {
  if (rows == 0) return hipSuccess;
  auto al = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
  const bool vec = d % 8 == 0 && d <= 512 * RV_MAX_IT && al(x) && al(add) && al(g) && al(out) && al(sum_out);
  DISPATCH_DT(dt, T, {
    if (vec) VEC_ROW_IT((d + 511) / 512, IT, rmsnorm_fwd_vec_k<IT, T><<<(unsigned)cdiv(rows, 4), 256, 0, st>>>((const T*)x, add, (const T*)g, (T*)out, sum_out, rstd, rows, d, eps));
    else rmsnorm_fwd_k<T><<<rows, 256, 0, st>>>((const T*)x, add, (const T*)g, (T*)out, sum_out, rstd, d, eps);
  });
  return hipGetLastError();
}

// Adjoint.  With u = dnorm * g and dot = <u, x>:  dx = u*r - x * r^3 * dot / d.
// A workgroup owns RB consecutive rows so that it can emit one partial row of
// dg = sum_rows dnorm * x * r; a second kernel adds the partial rows in a fixed
// order (no atomics: the result is reproducible run to run).  Four rows: one per wave
// in the vectorised form; the plain kernel, which walks its rows one after the other, gains from more and
// shorter workgroups what twice the partial rows of eight cost it, and more (whole adjoint, bf16, 512 rows of
// 5120 78 -> 45 us, 8192 rows of 8192 469 -> 283, with the column sums on sixteen waves).
constexpr int RB = 4;
template <typename T, typename XT, typename RT, typename DN = float>
__global__ __launch_bounds__(256) void rmsnorm_bwd_k(const DN* dnorm, const XT* __restrict__ xin,
                                                     const T* __restrict__ g, const float* __restrict__ rstd,
                                                     const RT* __restrict__ res, float* out_f32,
                                                     T* __restrict__ out_t, float* __restrict__ partial,
                                                     int rows, int d) {
  __shared__ float red[16];
  __shared__ float dots[RB];
  const int64_t row0 = (int64_t)blockIdx.x * RB;
  const int nr = (int)min((int64_t)RB, (int64_t)rows - row0);
  for (int r = 0; r < nr; ++r) {
    const int64_t row = row0 + r;
    float acc = 0.f;
    for (int j = threadIdx.x; j < d; j += blockDim.x)
      acc += ldf(dnorm + row * d + j) * ldf(g + j) * ldf(xin + row * d + j);
    acc = block_sum(acc, red);
    if (threadIdx.x == 0) dots[r] = acc;
  }
  __syncthreads();
  for (int j = threadIdx.x; j < d; j += blockDim.x) {
    const float gj = ldf(g + j);
    float dgj = 0.f;
    for (int r = 0; r < nr; ++r) {
      const int64_t row = row0 + r;
      const float rs = rstd[row];
      const float xv = ldf(xin + row * d + j);
      const float dn = ldf(dnorm + row * d + j);
      dgj += dn * xv * rs;
      const float v = (res ? ldf(res + row * d + j) : 0.f) + dn * gj * rs - xv * rs * rs * rs * dots[r] / (float)d;
      if (out_f32) out_f32[row * d + j] = v;
      if (out_t) stf(out_t + row * d + j, v);
    }
    if (partial) partial[(int64_t)blockIdx.x * d + j] = dgj;
  }
}

// Vectorised form for d % 8 == 0, d <= 4096: one wave per row (a workgroup takes RB rows), 8 elements (128 or 256 bits) per lane per
// access, the row's loads issued together and kept between the two passes; the four waves' shares of dg meet in LDS in a fixed
// order.  Same arithmetic and the same partial-sum layout as the plain kernel above.  (512 rows of 3584, with two rows per wave, a branch
// per access and both passes reading memory: 22 us, now 9; 1024 rows of 4096 28 -> 15.)
template <int IT, typename T, typename XT, typename RT, typename DN>
__global__ __launch_bounds__(256) void rmsnorm_bwd_vec_k(const DN* dnorm, const XT* __restrict__ xin,
                                                         const T* __restrict__ g, const float* __restrict__ rstd,
                                                         const RT* __restrict__ res, float* out_f32,
                                                         T* __restrict__ out_t, float* __restrict__ partial,
                                                         int rows, int d) {
  static_assert(RB == 4, "one row per wave");
  extern __shared__ float sdg[];   // [4][d]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t row = (int64_t)blockIdx.x * RB + wave;
  if (row < rows) {
    float dn[IT][8], xv[IT][8], gv[IT][8], rv[IT][8];
    load_row<IT>(dnorm + row * d, d, lane, dn);
    load_row<IT>(xin + row * d, d, lane, xv);
    load_row<IT>(g, d, lane, gv);
    if (res) load_row<IT>(res + row * d, d, lane, rv);
    const float rs = rstd[row];
    float dot = 0.f;
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const bool in = it * 512 + lane * 8 < d;
#pragma unroll
      for (int e = 0; e < 8; ++e) dot += in ? dn[it][e] * gv[it][e] * xv[it][e] : 0.f;
    }
    dot = wave_sum(dot);
    const float coef = rs * rs * rs * dot / (float)d;
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int j = it * 512 + lane * 8;
      if (j < d) {
        float o[8], dg[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          dg[e] = dn[it][e] * xv[it][e] * rs;
          o[e] = (res ? rv[it][e] : 0.f) + dn[it][e] * gv[it][e] * rs - xv[it][e] * coef;
        }
        if (out_f32) store8(out_f32 + row * d + j, o);
        if (out_t) store8(out_t + row * d + j, o);
        if (partial) store8(sdg + (int64_t)wave * d + j, dg);
      }
    }
  } else if (partial) {
    for (int j = lane; j < d; j += 64) sdg[(int64_t)wave * d + j] = 0.f;
  }
  if (!partial) return;
  __syncthreads();
  for (int j = threadIdx.x; j < d; j += blockDim.x)
    partial[(int64_t)blockIdx.x * d + j] = (sdg[j] + sdg[d + j]) + (sdg[2 * d + j] + sdg[3 * d + j]);
}
static bool rmsnorm_bwd_vec_ok(int d, const void* a, const void* b, const void* c, const void* e, const void* f, const void* h) {
  auto al = [](const void* p) { return ((uintptr_t)p & 15) == 0; };
  return d % 8 == 0 && d <= 512 * RV_MAX_IT && al(a) && al(b) && al(c) && al(e) && al(f) && al(h);
}

// dg[j] += sum over the given partial rows, in their order: 64 columns per workgroup, the rows of a buffer dealt to 16 waves, fixed summation
// order.  The buffers of a group of chunks and of both norms of a layer go in one launch (a launch per chunk and norm took 4 to 5 us each).
constexpr int CS_WAVES = 16;
__global__ __launch_bounds__(CS_WAVES * 64) void colsum_accum_k(const ColumnSums cs, int d) {
  __shared__ float red[CS_WAVES][64];
  const int j = blockIdx.x * 64 + (threadIdx.x & 63), part = threadIdx.x >> 6, which = blockIdx.y;
  float s = 0.f;
  if (j < d) {
    for (int i = 0; i < cs.n; ++i) {
      const float* partial = cs.partial[which][i];
      const int nblk = cs.blocks[i];
#pragma unroll 8
      for (int b = part; b < nblk; b += CS_WAVES) s += partial[(int64_t)b * d + j];
    }
  }
  red[part][threadIdx.x & 63] = s;
  __syncthreads();
  if (part == 0 && j < d) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < CS_WAVES; ++w) t += red[w][threadIdx.x];
    cs.dg[which][j] += t;
  }
}
hipError_t column_sums(const ColumnSums& cs, int n_dg, int d, hipStream_t st) {
  if (cs.n == 0) return hipSuccess;
  colsum_accum_k<<<dim3((unsigned)cdiv(d, 64), (unsigned)n_dg), CS_WAVES * 64, 0, st>>>(cs, d);
  return hipGetLastError();
}
int rmsnorm_bwd_partial_rows(int rows) { return (int)cdiv(rows, RB); }

size_t rmsnorm_bwd_partial_floats(int rows, int d) { return (size_t)cdiv(rows, RB) * (size_t)d; }

hipError_t rmsnorm_bwd(int dt, const float* dnorm, const void* xin, bool x_is_f32, const void* g,
                       const float* rstd, const void* res, bool res_is_f32, float* out_f32, void* out_t,
                       float* partial, int rows, int d, hipStream_t st) {
  if (rows == 0) return hipSuccess;
  const int nblk = (int)cdiv(rows, RB);
  const bool vec = rmsnorm_bwd_vec_ok(d, dnorm, xin, g, res, out_f32, out_t);
  const size_t shm = (size_t)4 * d * sizeof(float);
#define RB_LAUNCH(T, XT, RT)                                                                                     \
  do {                                                                                                           \
    if (vec)                                                                                                     \
      VEC_ROW_IT((d + 511) / 512, IT, rmsnorm_bwd_vec_k<IT, T, XT, RT, float><<<nblk, 256, shm, st>>>(dnorm, (const XT*)xin, (const T*)g, rstd, \
                                                                  (const RT*)res, out_f32, (T*)out_t, partial, rows, d)); \
    else                                                                                                         \
      rmsnorm_bwd_k<T, XT, RT><<<nblk, 256, 0, st>>>(dnorm, (const XT*)xin, (const T*)g, rstd, (const RT*)res,   \
                                                     out_f32, (T*)out_t, partial, rows, d);                      \
  } while (0)
  DISPATCH_DT(dt, T, {
    if (x_is_f32 && res_is_f32) RB_LAUNCH(T, float, float);
    else if (x_is_f32) RB_LAUNCH(T, float, T);
    else if (res_is_f32) RB_LAUNCH(T, T, float);
    else RB_LAUNCH(T, T, T);
  });
#undef RB_LAUNCH
  return hipGetLastError();
}

// Stand-alone norm adjoint with the incoming gradient in the storage type and no
// residual branch (the final norm between the layer stack and the LM head).
hipError_t rmsnorm_bwd_plain(int dt, const void* dy, const void* x, const void* g, const float* rstd, void* dx,
                             float* dg, float* partial, int rows, int d, hipStream_t st) {
  if (rows == 0) return hipSuccess;
  const int nblk = (int)cdiv(rows, RB);
  const bool vec = rmsnorm_bwd_vec_ok(d, dy, x, g, nullptr, nullptr, dx);
  const size_t shm = (size_t)4 * d * sizeof(float);
  DISPATCH_DT(dt, T, {
    if (vec)
      VEC_ROW_IT((d + 511) / 512, IT, rmsnorm_bwd_vec_k<IT, T, T, T, T><<<nblk, 256, shm, st>>>((const T*)dy, (const T*)x, (const T*)g, rstd, (const T*)nullptr,
                                                                                                nullptr, (T*)dx, partial, rows, d));
    else
      rmsnorm_bwd_k<T, T, T, T><<<nblk, 256, 0, st>>>((const T*)dy, (const T*)x, (const T*)g, rstd, (const T*)nullptr,
                                                      nullptr, (T*)dx, partial, rows, d);
  });
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  ColumnSums cs{};
  cs.n = 1; cs.partial[0][0] = partial; cs.blocks[0] = nblk; cs.dg[0] = dg;
  return column_sums(cs, 1, d, st);
}

// ---------------------------------------------------------------- SwiGLU --
__device__ __forceinline__ float sigmoidf_(float z) { return 1.0f / (1.0f + __expf(-z)); }

template <typename T>
__global__ void swiglu_fwd_k(const T* __restrict__ gate, const T* __restrict__ up, T* __restrict__ act, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) {
    float z = ldf(gate + i);
    stf(act + i, z * sigmoidf_(z) * ldf(up + i));
  }
}
template <typename T>
__global__ void swiglu_bwd_k(T* __restrict__ gate, T* __restrict__ up, const T* dact, T* act, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) {
    float z = ldf(gate + i), u = ldf(up + i), da = ldf(dact + i);
    float sg = sigmoidf_(z);
    if (act) stf(act + i, z * sg * u);
    stf(gate + i, da * u * sg * (1.0f + z * (1.0f - sg)));
    stf(up + i, da * z * sg);
  }
}
// 8 bf16 per lane (128-bit) variants for the wide MLP tensors
typedef bf16_t bf16x8 __attribute__((ext_vector_type(8)));
__global__ void swiglu_fwd_bf16x8_k(const bf16x8* __restrict__ gate, const bf16x8* __restrict__ up,
                                    bf16x8* __restrict__ act, int64_t n8) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n8; i += stride) {
    bf16x8 g = gate[i], u = up[i], a;
#pragma unroll
    for (int j = 0; j < 8; ++j) { float z = (float)g[j]; a[j] = (bf16_t)(z * sigmoidf_(z) * (float)u[j]); }
    act[i] = a;
  }
}
template <bool WITH_ACT>
__global__ void swiglu_bwd_bf16x8_k(bf16x8* __restrict__ gate, bf16x8* __restrict__ up,
                                    const bf16x8* dact, bf16x8* act, int64_t n8) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n8; i += stride) {
    bf16x8 g = gate[i], u = up[i], da = dact[i], dg, du, a;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      float z = (float)g[j], uu = (float)u[j], d = (float)da[j];
      float sg = sigmoidf_(z);
      if (WITH_ACT) a[j] = (bf16_t)(z * sg * uu);
      dg[j] = (bf16_t)(d * uu * sg * (1.0f + z * (1.0f - sg)));
      du[j] = (bf16_t)(d * z * sg);
    }
    if (WITH_ACT) act[i] = a;
    gate[i] = dg; up[i] = du;
  }
}


hipError_t swiglu_fwd(int dt, const void* gate, const void* up, void* act, int64_t n, hipStream_t st) {
  if (n == 0) return hipSuccess;
  if (dt == DT_BF16 && n % 8 == 0) {
    swiglu_fwd_bf16x8_k<<<ew_grid(n / 8), 256, 0, st>>>((const bf16x8*)gate, (const bf16x8*)up, (bf16x8*)act, n / 8);
  } else {
    DISPATCH_DT(dt, T, (swiglu_fwd_k<T><<<ew_grid(n), 256, 0, st>>>((const T*)gate, (const T*)up, (T*)act, n)));
  }
  return hipGetLastError();
}
hipError_t swiglu_bwd(int dt, void* gate, void* up, const void* dact, void* act, int64_t n, hipStream_t st) {
  if (n == 0) return hipSuccess;
  if (dt == DT_BF16 && n % 8 == 0) {
    if (act) swiglu_bwd_bf16x8_k<true><<<ew_grid(n / 8), 256, 0, st>>>((bf16x8*)gate, (bf16x8*)up, (const bf16x8*)dact, (bf16x8*)act, n / 8);
    else swiglu_bwd_bf16x8_k<false><<<ew_grid(n / 8), 256, 0, st>>>((bf16x8*)gate, (bf16x8*)up, (const bf16x8*)dact, nullptr, n / 8);
  } else {
    DISPATCH_DT(dt, T, (swiglu_bwd_k<T><<<ew_grid(n), 256, 0, st>>>((T*)gate, (T*)up, (const T*)dact, (T*)act, n)));
  }
  return hipGetLastError();
}

// ------------------------------------------------------------ small glue --
template <typename T>
__global__ void add_store_k(const float* __restrict__ a, const float* __restrict__ b, T* __restrict__ y, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n; i += stride) stf(y + i, a[i] + b[i]);
}
hipError_t add_store(int dt, const float* a, const float* b, void* y, int64_t n, hipStream_t st) {
  if (n == 0) return hipSuccess;
  DISPATCH_DT(dt, T, (add_store_k<T><<<ew_grid(n), 256, 0, st>>>(a, b, (T*)y, n)));
  return hipGetLastError();
}

template <typename T>
__global__ void kv_grad_finish_k(const float* __restrict__ dK, const float* __restrict__ dV,
                                 const float2* __restrict__ tab, T* __restrict__ dkc, T* __restrict__ dvc,
                                 int64_t n_pairs, int H, int half) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_pairs) return;
  int j = (int)(i % half);
  int64_t rh = i / half;
  int64_t row = rh / H;
  float2 cs = tab[row * half + j];
  int64_t base = rh * (2 * half);
  float a = dK[base + j], b = dK[base + j + half];
  stf(dkc + base + j, a * cs.x + b * cs.y);            // rotation by the negative angle
  stf(dkc + base + j + half, b * cs.x - a * cs.y);
  stf(dvc + base + j, dV[base + j]);
  stf(dvc + base + j + half, dV[base + j + half]);
}
hipError_t kv_grad_finish(int dt, const float* dK, const float* dV, const float2* tab, void* dkc, void* dvc,
                          int rows, int H, int dh, hipStream_t st) {
  int64_t n = (int64_t)rows * H * (dh / 2);
  if (n == 0) return hipSuccess;
  DISPATCH_DT(dt, T, (kv_grad_finish_k<T><<<(unsigned)cdiv(n, 256), 256, 0, st>>>(dK, dV, tab, (T*)dkc, (T*)dvc, n, H, dh / 2)));
  return hipGetLastError();
}

__global__ void fill_zero_k(uint4* p, int64_t n16) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n16; i += stride) p[i] = make_uint4(0, 0, 0, 0);
}
__global__ void fill_zero_bytes_k(unsigned char* p, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}
// A fill kernel rather than a memset node, so that callers may capture the stream into a graph.
hipError_t fill_zero(void* p, size_t bytes, hipStream_t st) {
  if (bytes == 0) return hipSuccess;
  size_t n16 = bytes / 16, tail = bytes - n16 * 16;
  if (((uintptr_t)p & 15) != 0) { n16 = 0; tail = bytes; }
  if (n16) fill_zero_k<<<ew_grid((int64_t)n16), 256, 0, st>>>((uint4*)p, (int64_t)n16);
  if (tail) fill_zero_bytes_k<<<(unsigned)cdiv((int64_t)tail, 256), 256, 0, st>>>((unsigned char*)p + n16 * 16, (int64_t)tail);
  return hipGetLastError();
}

// An id outside [0, vocab) is never used as an index: its row of x is zero and its row of dx is dropped.
__global__ void copy16_k(uint4* __restrict__ d, const uint4* __restrict__ s, int64_t n16) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (; i < n16; i += stride) d[i] = s[i];
}
__global__ void copy1_k(unsigned char* __restrict__ d, const unsigned char* __restrict__ s, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) d[i] = s[i];
}
hipError_t copy_bytes(void* dst, const void* src, size_t bytes, hipStream_t st) {
  if (bytes == 0) return hipSuccess;
  size_t n16 = bytes / 16, tail = bytes - n16 * 16;
  if ((((uintptr_t)dst | (uintptr_t)src) & 15) != 0) { n16 = 0; tail = bytes; }
  if (n16) copy16_k<<<ew_grid((int64_t)n16), 256, 0, st>>>((uint4*)dst, (const uint4*)src, (int64_t)n16);
  if (tail) copy1_k<<<(unsigned)cdiv((int64_t)tail, 256), 256, 0, st>>>((unsigned char*)dst + n16 * 16, (const unsigned char*)src + n16 * 16, (int64_t)tail);
  return hipGetLastError();
}

// 64 x 64 tiles through LDS, 16 bytes per lane on both sides (a tile's rows are 33 dwords apart).  2048 x 3584: 6.7 us, 4.4 TB/s read and written, next to
// the 4.9 of a large copy
__global__ __launch_bounds__(256) void transpose_rows_k(const bf16_t* __restrict__ src, const int32_t* __restrict__ rows_dev, int R, int C, bf16_t* __restrict__ dst, int64_t ld) {
  __shared__ bf16_t tile[64][66];
  const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64, t = threadIdx.x;
  if (rows_dev) R = min(R, *rows_dev);
  if (r0 >= R) return;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = (i * 256 + t) >> 3, col = (t & 7) * 8;
    bf16x8 v = {};
    if (r0 + row < R && c0 + col < C) v = *(const bf16x8*)(src + (int64_t)(r0 + row) * C + c0 + col);
#pragma unroll
    for (int e = 0; e < 8; ++e) tile[row][col + e] = v[e];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int col = (i * 256 + t) >> 3, row = (t & 7) * 8;
    bf16x8 v;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = tile[row + e][col];
    if (c0 + col < C) *(bf16x8*)(dst + (int64_t)(c0 + col) * ld + r0 + row) = v;
  }
}
hipError_t transpose_rows(const void* src, const int32_t* rows_dev, int R, int C, void* dst, int64_t ld, hipStream_t st) {
  if (R == 0 || C == 0) return hipSuccess;
  transpose_rows_k<<<dim3((unsigned)cdiv(C, 64), (unsigned)cdiv(R, 64)), 256, 0, st>>>((const bf16_t*)src, rows_dev, R, C, (bf16_t*)dst, ld);
  return hipGetLastError();
}

// element i of a launch over several jobs -> its job (they follow one another from job[x].begin on)
template <typename J> __device__ __forceinline__ int job_of(const J& jobs, int64_t i) {
  int x = 0;
  for (int k = 1; k < jobs.n; ++k)
    if (i >= jobs.job[k].begin) x = k;
  return x;
}
// What bounds these two: the accesses a thread makes, not their bytes (16 MB, 27 MB).  Eight and four elements a thread against one, seven adapters of rank 32 at 7B
// widths: 33 -> 14.4 and 20 -> 11.5 us.
template <typename T>
__global__ __launch_bounds__(256) void pad_matrices_k(const PadJobs jobs, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const PadJob& p = jobs.job[job_of(jobs, i)];
  const int64_t at = i - p.begin;
  const T* src = (const T*)p.src;
  T* dst = (T*)p.dst;
  float v[8];
  if (p.transposed) {      // eight rows of a column: neighbours in src, and the lanes' columns neighbours in dst
    const int r0 = (int)(at / p.C2) * 8, c = (int)(at % p.C2);
    if (c < p.C && r0 < p.R && p.R % 8 == 0 && !((uintptr_t)src & 15)) load8(src + (int64_t)c * p.R + r0, v);
    else {
#pragma unroll
      for (int k = 0; k < 8; ++k) v[k] = c < p.C && r0 + k < p.R ? ldf(src + (int64_t)c * p.R + r0 + k) : 0.f;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k)
      if (r0 + k < p.R2) stf(dst + (int64_t)(r0 + k) * p.C2 + c, r0 + k < p.R ? p.scale * v[k] : 0.f);
    return;
  }
  const int units = (p.C2 + 7) / 8, r = (int)(at / units), c0 = (int)(at % units) * 8;
  if (r < p.R && c0 + 8 <= p.C && p.C % 8 == 0 && p.C2 % 8 == 0 && !(((uintptr_t)src | (uintptr_t)dst) & 15)) {
    load8(src + (int64_t)r * p.C + c0, v);
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] *= p.scale;
    store8(dst + (int64_t)r * p.C2 + c0, v);
    return;
  }
#pragma unroll
  for (int k = 0; k < 8; ++k)
    if (c0 + k < p.C2) stf(dst + (int64_t)r * p.C2 + c0 + k, r < p.R && c0 + k < p.C ? p.scale * ldf(src + (int64_t)r * p.C + c0 + k) : 0.f);
}
hipError_t pad_matrices(int dt, PadJobs jobs, hipStream_t st) {
  int64_t n = 0;
  for (int k = 0; k < jobs.n; ++k) {      // a thread takes eight elements of a row of dst, or of a column (transposed)
    PadJob& p = jobs.job[k];
    p.begin = n;
    n += p.transposed ? cdiv(p.R2, 8) * p.C2 : (int64_t)p.R2 * cdiv(p.C2, 8);
  }
  if (n == 0) return hipSuccess;
  DISPATCH_DT(dt, T, (pad_matrices_k<T><<<(unsigned)cdiv(n, 256), 256, 0, st>>>(jobs, n)));
  return hipGetLastError();
}
__global__ __launch_bounds__(256) void add_scaled_blocks_k(const AddJobs jobs, float scale, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const AddJob& p = jobs.job[job_of(jobs, i)];
  const int64_t at = i - p.begin;
  const int units = (p.C + 3) / 4, r = (int)(at / units), c0 = (int)(at % units) * 4;
  float* dst = p.dst + (int64_t)r * p.C + c0;
  const float* src = p.src + (int64_t)r * p.ld + c0;
  if (p.C % 4 == 0 && p.ld % 4 == 0 && !(((uintptr_t)p.dst | (uintptr_t)p.src) & 15)) {
    float4 a = *(const float4*)dst;
    const float4 b = *(const float4*)src;
    a.x += scale * b.x; a.y += scale * b.y; a.z += scale * b.z; a.w += scale * b.w;
    *(float4*)dst = a;
    return;
  }
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (c0 + k < p.C) dst[k] += scale * src[k];
}
hipError_t add_scaled_blocks(AddJobs jobs, float scale, hipStream_t st) {
  int64_t n = 0;
  for (int k = 0; k < jobs.n; ++k) { jobs.job[k].begin = n; n += (int64_t)jobs.job[k].R * cdiv(jobs.job[k].C, 4); }      // a thread takes four elements of a row
  if (n == 0) return hipSuccess;
  add_scaled_blocks_k<<<(unsigned)cdiv(n, 256), 256, 0, st>>>(jobs, scale, n);
  return hipGetLastError();
}

template <typename T>
__global__ void embedding_fwd_k(const int32_t* __restrict__ ids, const T* __restrict__ emb, T* __restrict__ x, int d, int vocab) {
  const int64_t row = blockIdx.x;
  const int64_t id = ids[row];
  const bool ok = id >= 0 && id < vocab;
  for (int j = threadIdx.x; j < d; j += blockDim.x) x[row * d + j] = ok ? emb[id * d + j] : (T)0.0f;
}
template <typename T>
__global__ void embedding_bwd_k(const int32_t* __restrict__ ids, const T* __restrict__ dx, float* __restrict__ demb, int d, int vocab) {
  const int64_t row = blockIdx.x;
  const int64_t id = ids[row];
  if (id < 0 || id >= vocab) return;
  for (int j = threadIdx.x; j < d; j += blockDim.x) atomicAdd(demb + id * d + j, ldf(dx + row * d + j));
}
hipError_t embedding_fwd(int dt, const int32_t* ids, const void* emb, void* x, int64_t rows, int d, int vocab, hipStream_t st) {
  if (rows == 0) return hipSuccess;
  DISPATCH_DT(dt, T, (embedding_fwd_k<T><<<(unsigned)rows, 256, 0, st>>>(ids, (const T*)emb, (T*)x, d, vocab)));
  return hipGetLastError();
}
hipError_t embedding_bwd(int dt, const int32_t* ids, const void* dx, float* demb, int64_t rows, int d, int vocab, hipStream_t st) {
  if (rows == 0) return hipSuccess;
  DISPATCH_DT(dt, T, (embedding_bwd_k<T><<<(unsigned)rows, 256, 0, st>>>(ids, (const T*)dx, demb, d, vocab)));
  return hipGetLastError();
}

}  // namespace sbp
