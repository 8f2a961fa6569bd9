// bf16 MFMA chunk attention for gfx950 (head_dim DH = 128 or 64): forward, dQ and dK/dV.
//
// Query row t of the chunk sits at global position q_start + t and sees keys
// 0 .. q_start + t of the cached prefix (paper Sec. 3.2.2, partitioned attention;
// Property 3.1).  Key tiles that lie entirely above the diagonal are skipped,
// tiles on the diagonal are masked by an integer comparison of positions, rows
// past q_start + q_len of K/V are never read.  Two more mask rules are index
// arithmetic of the same kind (the paper's mask M covers "padding / sliding
// window"): window > 0 limits a query at position t to the keys t - window < u <= t,
// and kv_first hides the key positions before it (padding in front of the
// sequence); key tiles wholly outside a wave's range are skipped on the left edge
// just as on the right one, and a query that sees no key gets o = 0, lse = -inf
// and sends no gradient.
//
// All three kernels use the "transposed score" formulation: S^T[key, query] = K Q^T.
// The accumulator layout then gives every lane ONE query and several keys of a
// block, so row max / row sum are in-register plus one or two lane exchanges, and
// exp(S^T) is already in the register layout of the B operand of the next product
// (P^T as [key, query] with keys as the reduction index).  The reduction-index
// permutation this implies is matched on the A side by the transposing LDS load
// (ds_read_b64_tr_b16) that fetches V^T / K^T / Q^T / dO^T fragments from tiles
// kept in their natural [row][head_dim] layout.
//
//  forward : 256 (or 128) queries of one query head per workgroup, 16x16x32 MFMAs,
//            8 waves x 32 queries; K and V tiles of 64 keys stream HBM -> LDS
//            (direct-to-LDS); online softmax in the exp2 domain; multiply and
//            softmax slots of two wave groups alternate.
//  dQ      : same decomposition, slots and MFMAs; recomputes P from the
//            saved log-sum-exp; dQ^T += K^T dS^T.
//  dK/dV   : workgroup = 128 keys of one KV head, 4 key blocks x 2 roles: one wave of
//            a block computes P and dV^T += dO^T P, its partner dP, dS and
//            dK^T += Q^T dS (P crosses through LDS); loops over the query
//            tiles at or below the diagonal and over the query heads of the group, Q
//            and dO tiles of 64 queries stream through four LDS stages; results are
//            added to the fp32 prefix accumulators (every element has one owner, or
//            its parts are summed in a fixed order: no atomics, reproducible).
#include "launch.h"
#include "attn_plan.h"
#include "device.h"

#include <type_traits>

#include <algorithm>

namespace sbp {

typedef bf16_t bf16x8 __attribute__((ext_vector_type(8)));
typedef bf16_t bf16x4 __attribute__((ext_vector_type(4)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef short short8v __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int AT_THREADS = 512;          // 8 waves (forward, dQ): 2 per SIMD
constexpr int TQ = ATTN_TILE_Q;          // queries per workgroup (fwd, dQ): 8 waves x 32
constexpr int TK = ATTN_TILE_K;          // 64 keys per step (fwd, dQ)
constexpr int KV_TILE = ATTN_KV_TILE;    // keys per workgroup (dK/dV): 4 key blocks x 2 roles = 8 waves
constexpr int KV_THREADS = 512;
constexpr int QT = ATTN_KV_QUERIES;      // queries per step (dK/dV)
// Workgroups of a backward that runs as one launch (four rounds of the chip; six behind a prefix), which fills what dQ's last workgroups leave.  dQ and dK/dV in
// one launch / in two: 238 sizes of up to 1024 workgroups 0.59-1.00 (mean 0.75), 19 of up to 1536 0.72-1.01 (0.91), 13 beyond 0.88-1.01 (0.96).  With dQ first, behind a
// prefix, there is no limit: 164 sizes 0.56-0.99 (0.72).
constexpr int MERGED_MAX = 1024;
constexpr int MERGED_MAX_PREFIX = 1536;
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

// LDS tile [64 rows][DH bf16], 16 (DH = 64: 8) chunks of 16 B per row, chunk ^= f(row): conflict-free both for 128-bit
// row-fragment reads (16 consecutive rows, same chunk) and for the transposing 64-bit reads (4 consecutive rows x 64 B, or 8 x 32 B).
template <int DH> constexpr int TILE64 = 64 * DH * 2;      // bytes: 16 or 8 KiB
template <int DH>
__device__ __forceinline__ int swz(int row) {
  static_assert(DH == 128 || DH == 64, "head sizes of the MFMA kernels");
  if (DH == 128) return ((row & 3) << 2) | ((((row >> 2) ^ (row >> 3)) & 1) << 1) | ((row >> 3) & 1);
  return (((row >> 1) & 1) << 2) | (((row >> 2) & 1) << 1) | ((row >> 3) & 1);      // (two rows per 256 bytes of banks)
}
template <int DH>
__device__ __forceinline__ int tile_off(int row, int chunk) { return row * DH * 2 + ((chunk ^ swz<DH>(row)) << 4); }

// Probabilities and dS are operands of the second products.  DH = 128 rounds them to bf16; DH = 64 keeps them as a sum of bf16 terms, at
// the price of a further MFMA each: two (2^-17 relative) where the result is rounded to bf16, o and dq, three (exact) for dv = P^T dO
// and dk = dS^T Q, which leave as fp32.  The statistics of DH = 64 keep fp32 as well: the denominator sums the fp32 probabilities
// (not the terms, by one more product), P goes to the dK role in fp32, and exponents are differences in the natural domain, scaled
// to base 2 last (one multiply per score more), so that log-sum-exp and probabilities are rounded where the shape-agnostic kernels
// round them.  Norm-wise error against fp64, these / the shape-agnostic fp32 kernels, 16 / 4 heads, 512 queries: log-sum-exp 4.3e-8 /
// 4.5e-8, dv 6.1e-7 / 1.03e-6, dk 6.41e-4 / 6.43e-4, o 1.596e-3 and dq 1.795e-3 both (statistics from the terms, in base 2: log-sum-exp
// 7.1e-8, at two visible keys 7.2e-7 instead of 4.4e-8).  A 1024-wide two-layer step pays 0.6 % for it.
template <int DH> constexpr int TERMS = DH == 64 ? 2 : 1;
template <int DH> constexpr int KV_TERMS = DH == 64 ? 3 : 1;
template <int DH> constexpr bool FP32_STATS = DH == 64;

// Two values rounded to bf16 by one instruction, and what that leaves of them.  Element by element the conversions were a fifth of the vector work of DH = 64
// (dQ and dK/dV of 1840 queries behind 5360 keys, 12 / 2 heads, 327 -> 304 us); DH = 128, which has no rests to form, is 0.5 % slower this way.
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef bf16_t bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ bf16x2 round2(f32x2 x) { return __builtin_convertvector(x, bf16x2); }
__device__ __forceinline__ f32x2 rest2(f32x2 x, bf16x2 w) { return f32x2{x[0] - (float)w[0], x[1] - (float)w[1]}; }

// exp(x * scale + c): c in log2 units, or in natural ones where the statistics keep fp32
template <int DH>
__device__ __forceinline__ float exp_of(float x, float scale, float sl, float c) {
  if (FP32_STATS<DH>) return __builtin_amdgcn_exp2f(__builtin_fmaf(x, scale, c) * LOG2E);
  return __builtin_amdgcn_exp2f(__builtin_fmaf(x, sl, c));
}

// ---- address work hoisted out of the tile loops --------------------------------------------------------------
// In the tile loops every vector-ALU instruction competes with the softmax arithmetic for the SIMD's VALU issue
// slots, so nothing there computes an address: the per-lane byte offsets of the fragment reads inside a 64-row
// tile and of the direct-to-LDS loads are computed once per kernel, every row block is reached with an immediate
// offset, the addresses move on from stage to stage by one addition each, and the global side is an SGPR base plus
// those per-lane offsets.
__device__ __forceinline__ bf16x8 lds_b128(uint32_t addr) {
  return *(const bf16x8*)(__attribute__((address_space(3))) const char*)(uintptr_t)addr;
}
__device__ __forceinline__ bf16x8 lds_tr(uint32_t lo_addr, uint32_t hi_addr) {
  short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)(uintptr_t)lo_addr);
  short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)(uintptr_t)hi_addr);
  short8v r = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, r);
}

// Direct-to-LDS load of a 64-row tile by NT threads: rows 0..63 of a [*, stride] bf16 matrix starting at `g`
// (uniform pointer to the tile's first row, first of its DH columns).  rows_valid = rows that exist from `g` on:
// a tile that runs past the end (only the last one) clamps its row indices so that nothing out of range is read.
template <int DH, int NT>
struct TileLoad { uint32_t voff[8 * DH / NT]; };
template <int DH, int NT>
__device__ __forceinline__ uint32_t tile_load_offset(int i, int64_t stride, int rows_valid) {
  const int id = i * NT + (int)threadIdx.x % NT;      // (NT = half the workgroup: each half loads tiles of its own)
  const int row = id / (DH / 8), pc = id % (DH / 8);
  const int chunk = pc ^ swz<DH>(row);
  return (uint32_t)(((int64_t)min(row, rows_valid - 1) * stride + chunk * 8) * 2);
}
template <int DH, int NT>
__device__ __forceinline__ TileLoad<DH, NT> tile_load_pre(int64_t stride) {
  TileLoad<DH, NT> t;
#pragma unroll
  for (int i = 0; i < 8 * DH / NT; ++i) t.voff[i] = pin(tile_load_offset<DH, NT>(i, stride, 64));
  return t;
}
template <int DH, int NT>
__device__ __forceinline__ void dma_tile64(const TileLoad<DH, NT>& t, const bf16_t* g, int64_t stride, int rows_valid, uint32_t lds_tile) {
  const uint32_t dst = __builtin_amdgcn_readfirstlane(lds_tile + (uint32_t)(threadIdx.x % NT & ~63) * 16u);
  if (rows_valid >= 64) {
#pragma unroll
    for (int i = 0; i < 8 * DH / NT; ++i) dma16((const char*)g, t.voff[i], dst + (uint32_t)(i * NT * 16));
  } else {
#pragma unroll
    for (int i = 0; i < 8 * DH / NT; ++i) dma16((const char*)g, tile_load_offset<DH, NT>(i, stride, rows_valid), dst + (uint32_t)(i * NT * 16));
  }
}

// A chain of N steps, an MFMA or two each, whose A operands come from LDS: the fragment of step i+DEPTH is requested before the MFMAs of
// step i issue (ring of DEPTH+1 fragments), and scheduling barriers keep that order - left alone, the compiler
// sinks every LDS read to just before its MFMA and the wave eats one LDS latency per MFMA.
template <int N, int DEPTH = 3, typename LoadF, typename MmaF>
__device__ __forceinline__ void mfma_chain(LoadF load, MmaF mma) {
  bf16x8 f[DEPTH + 1];
#pragma unroll
  for (int i = 0; i < DEPTH && i < N; ++i) f[i] = load(i);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (i + DEPTH < N) f[(i + DEPTH) % (DEPTH + 1)] = load(i + DEPTH);
    __builtin_amdgcn_sched_barrier(0);
    mma(i, f[i % (DEPTH + 1)]);
    __builtin_amdgcn_sched_barrier(0);
  }
}
#define WAIT_VM0() __builtin_amdgcn_s_waitcnt(0x0f70)

// ---- 16x16x32 MFMA building blocks -----------------------------------------------------------------------------
// A product of 16 x 16 x 32 reads and writes its accumulators half as often as one of 32 x 32 x 16, and the chip is at its power limit: from registers alone, on
// random data, the one holds 2020 TFLOP/s here, the other 1370 (1800 in the first 0.1 s).
// S^T blocks of 16 keys x 16 queries: lane l holds query l % 16 and keys 4 (l / 16) + r.  Two such blocks (32 keys) are the B operand
// of the next product with slot 8 (l / 16) + j <-> key 16 (j >> 2) + 4 (l / 16) + (j & 3), matched on the A side by two
// transposing reads 16 rows apart.
#define MFMA16(a, b, c) __builtin_amdgcn_mfma_f32_16x16x32_bf16((a), (b), (c), 0, 0, 0)
// fragment of 16 rows x 32 elements (one k32 step): row l % 16, elements 8 (l / 16) .. + 7   (row block b: + b * 16 rows)
template <int DH>
__device__ __forceinline__ uint32_t frag16_rows(int kk) {
  const int l = threadIdx.x & 63;
  return (uint32_t)tile_off<DH>(l & 15, kk * 4 + (l >> 4));
}
// transposed fragment of 16 columns (head_dim block d) x 32 rows: rows 4 (l / 16) .. + 3 here, and 16 rows further
template <int DH>
__device__ __forceinline__ uint32_t frag16_tr(int d) {
  const int l = threadIdx.x & 63, p = l & 15, g = l >> 4;
  const int col = d * 16 + 4 * (p & 3), row = 4 * g + (p >> 2);
  return (uint32_t)(tile_off<DH>(row, col >> 3) + ((col & 7) << 1));
}
// maximum over the four lanes that share a query (l % 16)
__device__ __forceinline__ float max_raw(float a, float b) {      // v_max_f32 without the quieting moves fmaxf adds for unknown operands
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
  return r;
}
__device__ __forceinline__ float max_over_quads(float x) {
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  u32x2 r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false));
  x = max_raw(__uint_as_float(r[0]), __uint_as_float(r[1]));
  r = __builtin_bit_cast(u32x2, __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false));
  return max_raw(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
#define AT_WAIT_VM(n) asm volatile("s_waitcnt vmcnt(%0)" ::"i"(n) : "memory")
#define AT_SLOT_BARRIER()                     \
  do {                                        \
    __builtin_amdgcn_sched_barrier(0);        \
    asm volatile("s_barrier" ::: "memory");   \
    __builtin_amdgcn_sched_barrier(0);        \
  } while (0)
// Workgroup `id` -> (query tile, head of a sequence).  An XCD gets a contiguous run of (head, tile) pairs, so that the heads of one K/V group run on one XCD
// and share its stream through that L2, and walks them tile by tile, all of its heads side by side, the tiles with the most keys first: the heads
// of a group are then in step, and what comes last is short.  Forward and dQ of more than a round, against head after head and tile after tile over all heads:
// 32k layer at 7B widths 68.7 -> 67.8 ms, 8192 tokens, 32 / 8 heads, 11.01 -> 10.92.
__device__ __forceinline__ void query_tile_of(int id, int n_qt, int heads, int& qt, int& h) {
  const int n = n_qt * heads, x = id % 8, q = n / 8, r = n % 8, first = x * q + min(x, r), last = first + q + (x < r ? 1 : 0) - 1;
  if (n <= 256) {      // one round: no order
    const int c = first + id / 8;
    h = c / n_qt;
    qt = n_qt - 1 - c % n_qt;
    return;
  }
  const int h0 = first / n_qt, row0 = first % n_qt, h1 = last / n_qt, row1 = last % n_qt;      // the run: from row row0 of head h0 to row row1 of head h1
  int k = id / 8, row = 0;
  for (;; ++row) {
    const int from = h0 + (row < row0 ? 1 : 0), heads_in = h1 - (row > row1 ? 1 : 0) - from + 1;
    if (k < heads_in) { h = from + k; break; }
    k -= heads_in;
  }
  qt = n_qt - 1 - row;
}

// ------------------------------------------------------------------ forward --
// 8 waves in two groups of four; waves w and w + 4 share a SIMD.  A key tile costs a wave two slots, each closed by a barrier:
// multiply (O += P V of the previous tile, S = K Q^T of this one: 68 MFMAs, the softmax denominator - at DH = 128 one product against
// an all-ones operand - among them; then the maxima of S) and softmax (and the loads of later tiles, spread between the exponentials).  Group 1 runs one
// slot behind group 0, so on every SIMD one wave multiplies while the other does its exponentials.
//   SPLIT = false: 256 queries, 32 per wave; all waves walk all key tiles, four K and four V stages (128 KB), loads two to three
//                  tiles ahead.
//   SPLIT = true : 128 queries, for launches that would leave CUs idle: the groups take the even / odd key tiles of the same
//                  queries, each with two stages of its own, and meet in LDS at the end.  They exchange their running
//                  maxima tile by tile (a group reads what the other left one slot ago), so that every probability is rounded
//                  against the maximum it has in the sequential walk.
// What bounds it: a slot takes about 1600 cycles at 2.0 GHz where the 68 MFMAs take 1088 - the vector instructions of one wave (about
// 160, 32 of them exponentials) and the MFMAs of the other share the SIMD's issue port and delay each other; without the vector
// work a slot takes 1050 cycles, without the MFMAs 1150.  Last 2048-query chunk of 32k, 28 heads: 1110 -> 957 us, by the steps below 806 to 820.
// The masks and the rows' maxima close the multiply slot, which is the shorter one where few workgroups leave the clock high: 128 queries behind 4096 keys,
// 28 heads, 69.1 -> 64.9 us, 1024 from the first on 23.8 -> 22.6, 16 heads of 64 23.3 -> 21.5; the same where the chip is full.
// A wave's tiles are one loop whose LDS stages move with the addresses, as in dQ: 16 registers fewer than four steps unrolled, a quarter of the code, 820 -> 813 us on
// that chunk, 777 windowed queries 31.9 -> 31.1.  Half of its LDS reads left out 739, its exponentials 789, a quarter of the products 710.
// Tried with a maximum that lags by up to 2^8, itself 921 us but another rounding of every probability: 32x32x16 MFMAs in the same
// schedule 965, loads in the multiply slot 954, the next slot's first fragments read early 958.
template <int DH, bool SPLIT>
__global__ __launch_bounds__(AT_THREADS) void attn_fwd_mfma_k(bf16_t* q, const bf16_t* __restrict__ k,
                                                                 const bf16_t* __restrict__ v, bf16_t* __restrict__ o,
                                                                 float* __restrict__ lse, int Hq, int Hkv, int q_start,
                                                                 int c, float scale, const float2* __restrict__ rope,
                                                                 int window, const AttnSeqs seqs) {
  __shared__ __attribute__((aligned(1024))) char sT[8 * TILE64<DH>];   // K stages, then V stages
  __shared__ float sM[SPLIT ? 2 : 1][4][32];                  // SPLIT: the running maxima of the groups' queries
  constexpr int QW = SPLIT ? TQ / 2 : TQ;                     // queries of the workgroup
  constexpr int STAGES = SPLIT ? 2 : 4, K_AHEAD = SPLIT ? 2 : 3, V_AHEAD = SPLIT ? 1 : 2;
  constexpr int LOADERS = SPLIT ? AT_THREADS / 2 : AT_THREADS, LOADS = 8 * DH / LOADERS;   // threads that load a tile, 16-byte loads of each

  int qt, bh;
  query_tile_of(blockIdx.x, (c + QW - 1) / QW, Hq * seqs.n, qt, bh);
  const int b = bh / Hq, h = bh - b * Hq, kv_first = seqs.first[b];
  q += (int64_t)b * c * Hq * DH; o += (int64_t)b * c * Hq * DH; lse += (int64_t)b * c * Hq;
  k += (int64_t)b * c * Hkv * DH; v += (int64_t)b * c * Hkv * DH;
  const int q0 = qt * QW, kvh = h / (Hq / Hkv);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
  const int grp = wave >> 2;
  const int qw0 = q0 + (SPLIT ? wave & 3 : wave) * 32;
  const int64_t kv_stride = (int64_t)Hkv * DH;
  const bf16_t* kbase = k + (int64_t)kvh * DH;
  const bf16_t* vbase = v + (int64_t)kvh * DH;
  const int n_total = q_start + c;                                    // rows of K/V that exist for this chunk
  const int n_keys = q_start + min(q0 + QW, c);                       // keys visible to the workgroup
  const int n_tiles = (n_keys + TK - 1) / TK;
  const int wave_last_key = q_start + min(qw0 + 32, c) - 1;           // last key any query of this wave sees
  const int wave_first_qpos = q_start + qw0;
  // left edge of the visible range: first visible key of a query at position p
  auto first_key = [&](int p) { return max(kv_first, window > 0 ? p - window + 1 : 0); };
  const int wave_lo_min = first_key(wave_first_qpos);                 // lowest first key in the wave (its first query)
  const int wave_lo_max = first_key(wave_last_key);                   // highest one (its last query)
  const int kt0 = first_key(q_start + q0) / TK;                       // first key tile any query of the workgroup sees
  const int n_it = SPLIT ? (max(0, n_tiles - kt0) + 1) / 2 : max(0, n_tiles - kt0);
  auto tile_of = [&](int i) { return SPLIT ? kt0 + 2 * i + grp : kt0 + i; };

  constexpr int KS = DH / 32, DB = DH / 16;                   // k32 steps of a score, 16-row blocks of the output
  bf16x8 bq[2][KS];      // [16-query block][k32 step]: B operands of S^T = K Q^T
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int q_row = min(qw0 + b * 16 + li, c - 1);
    const bf16_t* qp = q + ((int64_t)q_row * Hq + h) * DH + lg * 8;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) bq[b][kk] = *(const bf16x8*)(qp + kk * 32);
  }
  if (rope) {
    // Rotary embedding of the query on load: the rotate-half partner of element j < DH / 2 is j + DH / 2, i.e. the same element of
    // fragment kk + KS / 2, in the same lane.  The rotated row is written back so that the backward kernels, which read q
    // through LDS, find it rotated.
    if (SPLIT) __syncthreads();      // both groups hold the un-rotated rows
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int my_q = qw0 + b * 16 + li, q_row = min(my_q, c - 1);
      const float2* tr = rope + (int64_t)q_row * (DH / 2) + lg * 8;
#pragma unroll
      for (int kk = 0; kk < KS / 2; ++kk)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float2 cs = tr[kk * 32 + e];
          const float x1 = (float)bq[b][kk][e], x2 = (float)bq[b][kk + KS / 2][e];
          bq[b][kk][e] = (bf16_t)(x1 * cs.x - x2 * cs.y);
          bq[b][kk + KS / 2][e] = (bf16_t)(x2 * cs.x + x1 * cs.y);
        }
      if (my_q < c && (!SPLIT || grp == 0)) {
        bf16_t* qp = q + ((int64_t)my_q * Hq + h) * DH + lg * 8;
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) *(bf16x8*)(qp + kk * 32) = bq[b][kk];
      }
    }
  }
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) asm volatile("" : "+v"(bq[b][kk]));   // (arrived: the compiler must not wait for them in the loop)
  AT_WAIT_VM(0);     // from here on the loop counts its own loads only

  // ---- addresses, computed once: LDS fragments (+ stage, the only part that moves), global loads
  const uint32_t lds0 = lds_addr(sT);
  const uint32_t lds_k = lds0 + (SPLIT ? (uint32_t)grp * STAGES * TILE64<DH> : 0u), lds_v = lds_k + 4 * TILE64<DH>;
  const int tid = SPLIT ? (int)threadIdx.x & (LOADERS - 1) : (int)threadIdx.x;
  auto load_offset = [&](int i, int rows_valid) {
    const int id = i * LOADERS + tid, row = id / (DH / 8), chunk = (id % (DH / 8)) ^ swz<DH>(row);
    return (uint32_t)(((int64_t)min(row, rows_valid - 1) * kv_stride + chunk * 8) * 2);
  };
  // loads of tile i of this wave's sequence; past the end the last tile is loaded again, so that the wait counts stay the same.
  // The last tile may be short: its rows past the end re-read the last one.
  const int t_max = n_tiles - 1;
  uint32_t voff[LOADS], voff_last[LOADS];
#pragma unroll
  for (int j = 0; j < LOADS; ++j) { voff[j] = pin(load_offset(j, TK)); voff_last[j] = pin(load_offset(j, min(TK, n_total - t_max * TK))); }
  const uint32_t dst_k = __builtin_amdgcn_readfirstlane(lds_k + (uint32_t)(tid & ~63) * 16u), tile_bytes = (uint32_t)(TK * kv_stride * 2);
  // load p (of PIECES) of the pair V(i + V_AHEAD), K(i + K_AHEAD)
  constexpr int PIECES = 2 * LOADS;
  auto issue_piece = [&](int p, int i) __attribute__((always_inline)) {
    const bool is_k = p >= LOADS;
    const int j = p % LOADS, ahead = is_k ? K_AHEAD : V_AHEAD, t = min(tile_of(i + ahead), t_max);
    const char* src = (const char*)(is_k ? kbase : vbase) + (uint64_t)tile_bytes * (uint32_t)t;
    dma16(src, t == t_max ? voff_last[j] : voff[j],
          dst_k + (uint32_t)(((is_k ? 0 : 4) + (i + ahead) % STAGES) * TILE64<DH> + j * LOADERS * 16));
  };

  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (bf16_t)1.0f;
  asm volatile("" : "+v"(ones));
  f32x4 acc[2][DB], acc_l[2], s[2][4];     // O^T [query block][16 head_dim rows], denominator, S^T [query block][16 keys]
  bf16x8 pb[TERMS<DH>][2][2];             // P^T: [term][query block][k32 step]
  float m_floor = -INFINITY;
  asm volatile("" : "+v"(m_floor));
  float m_raw[2] = {-INFINITY, -INFINITY}, m_neg[2] = {0.f, 0.f};   // maximum of the raw scores; what the exponent adds (see exp_of)
  if (SPLIT) {
    if (lane < 32) sM[grp][wave & 3][lane] = -INFINITY;
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  }
#pragma unroll
  for (int b = 0; b < 2; ++b) {
#pragma unroll
    for (int d = 0; d < DB; ++d) acc[b][d] = f32x4{0.f, 0.f, 0.f, 0.f};
    acc_l[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const float sl = scale * LOG2E;
  // steps in which some (query, key) pair of the wave is visible: tiles wave_lo_min / TK .. wave_last_key / TK
  const int step_t = SPLIT ? 2 : 1, first_t = tile_of(0);
  const int act0 = max(0, (wave_lo_min / TK - first_t + step_t - 1) / step_t);
  const int act1 = qw0 < c && wave_last_key >= 0 ? min(n_it, (wave_last_key / TK - first_t + step_t) / step_t) : 0;

  // LDS addresses of fragments, one step after the other: of K rows of the present tile, of V transposed of the previous one
  uint32_t fr[KS], ft[DB];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) fr[kk] = pin(lds_k + frag16_rows<DH>(kk) + (uint32_t)(act0 % STAGES) * TILE64<DH>);
#pragma unroll
  for (int d = 0; d < DB; ++d) ft[d] = pin(lds_v + frag16_tr<DH>(d) + (uint32_t)(act0 % STAGES) * TILE64<DH>);
  auto to_next = [&](int i) { return i % STAGES == STAGES - 1 ? (uint32_t)-(int)((STAGES - 1) * TILE64<DH>) : (uint32_t)TILE64<DH>; };      // from the stage of tile i

  // fragment reads run RING - 1 fragments (two MFMAs each) ahead of the products
  constexpr int RING = 8;
  constexpr uint32_t ROWS16 = 16 * DH * 2;
  bf16x8 f[RING];
  auto v_frag = [&](int n) {      // n = k32 step * DB + head_dim block
    return lds_tr(ft[n % DB] + (uint32_t)(n / DB) * 2 * ROWS16, ft[n % DB] + ((uint32_t)(n / DB) * 2 * ROWS16 + ROWS16));
  };
  auto k_frag = [&](int n) { return lds_b128(fr[n >> 2] + (uint32_t)(n & 3) * ROWS16); };   // n = k32 step * 4 + key block
  auto pv = [&](int i) __attribute__((always_inline)) {
#pragma unroll
    for (int n = 0; n < RING - 1; ++n) f[n] = v_frag(n);
#pragma unroll
    for (int n = 0; n < 2 * DB; ++n) {
      if (n + RING - 1 < 2 * DB) f[(n + RING - 1) % RING] = v_frag(n + RING - 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int b = 0; b < 2; ++b) {
#pragma unroll
        for (int t = 0; t < TERMS<DH>; ++t) {
          acc[b][n % DB] = MFMA16(f[n % RING], pb[t][b][n / DB], acc[b][n % DB]);
          if (!FP32_STATS<DH> && n % DB == DB - 1) acc_l[b] = MFMA16(ones, pb[t][b][n / DB], acc_l[b]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    const uint32_t move = to_next(i);
#pragma unroll
    for (int d = 0; d < DB; ++d) ft[d] = pin(ft[d] + move);
  };
  auto qk = [&](int i) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) s[b][kb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int n = 0; n < RING - 1; ++n) f[n] = k_frag(n);
#pragma unroll
    for (int n = 0; n < 4 * KS; ++n) {
      if (n + RING - 1 < 4 * KS) f[(n + RING - 1) % RING] = k_frag(n + RING - 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int b = 0; b < 2; ++b) s[b][n & 3] = MFMA16(f[n % RING], bq[b][n >> 2], s[b][n & 3]);
      __builtin_amdgcn_sched_barrier(0);
    }
    const uint32_t move = to_next(i);
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) fr[kk] = pin(fr[kk] + move);
  };
  auto row_max = [&](int i, float (&mx)[2]) __attribute__((always_inline)) {      // masks, and the maxima of the raw scores (scale > 0 keeps the order)
    const int k0 = tile_of(i) * TK;
    if (k0 + TK - 1 > wave_first_qpos || k0 < wave_lo_max) {   // only tiles on an edge of the visible range pay for the mask
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        // key 4 lg + e of the tile is visible for first <= e < first + n: one unsigned comparison
        const int qpos = q_start + min(qw0 + b * 16 + li, c - 1), lo = first_key(qpos);
        const int first = lo - k0 - 4 * lg;
        const uint32_t n = (uint32_t)max(0, qpos - lo + 1);
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
#pragma unroll
          for (int r = 0; r < 4; ++r) s[b][kb][r] = (uint32_t)(kb * 16 + r - first) < n ? s[b][kb][r] : -INFINITY;
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      float m2[2];
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        m2[x] = m_floor;
#pragma unroll
        for (int e = 0; e < 8; ++e) m2[x] = fmaxf(m2[x], s[b][2 * x + (e >> 2)][e & 3]);
      }
      mx[b] = max_raw(m2[0], m2[1]);
    }
#pragma unroll
    for (int b = 0; b < 2; ++b) mx[b] = max_over_quads(mx[b]);
  };
  auto softmax = [&](int i, float (&mx)[2]) __attribute__((always_inline)) {
    if constexpr (SPLIT) {
#pragma unroll
      for (int b = 0; b < 2; ++b) mx[b] = max_raw(mx[b], sM[grp ^ 1][wave & 3][b * 16 + li]);
    }
    // The maximum (and with it the rescale of O) only moves when some query of the wave sees a new one.
    if (__builtin_amdgcn_ballot_w64(mx[0] > m_raw[0] || mx[1] > m_raw[1]) != 0) {
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        const float m_new = mx[b] > m_raw[b] ? mx[b] : m_raw[b];
        const float neg = m_new == -INFINITY ? 0.0f : -(m_new * (FP32_STATS<DH> ? scale : sl));   // all scores so far masked: exp2(-inf - 0) = 0, not exp2(-inf + inf)
        // a query that has seen no key yet keeps its zeros
        const float alpha = FP32_STATS<DH> ? (m_raw[b] == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f((neg - m_neg[b]) * LOG2E))
                                           : (m_new == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f(m_raw[b] * sl - m_new * sl));
        m_raw[b] = m_new;
        m_neg[b] = neg;
#pragma unroll
        for (int r = 0; r < 4; ++r) acc_l[b][r] *= alpha;
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[b][d][r] *= alpha;
      }
      if (SPLIT && lg < 2) {       // (lanes 0 .. 15 query block 0, 16 .. 31 block 1)
        sM[grp][wave & 3][lane] = lg == 0 ? m_raw[0] : m_raw[1];
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      }
    }
#pragma unroll
    for (int x = 0; x < 4; ++x) {        // eight probabilities at a time, the loads spread between them
      const int b = x >> 1, kk = x & 1;
#pragma unroll
      for (int p = x * PIECES / 4; p < (x + 1) * PIECES / 4; ++p) issue_piece(p, i);
      __builtin_amdgcn_sched_barrier(0);
      float pe[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        pe[e] = exp_of<DH>(s[b][2 * kk + (e >> 2)][e & 3], scale, sl, m_neg[b]);
        pb[0][b][kk][e] = (bf16_t)pe[e];
        if (TERMS<DH> == 2) pb[TERMS<DH> - 1][b][kk][e] = (bf16_t)(pe[e] - (float)pb[0][b][kk][e]);
      }
      if (FP32_STATS<DH>) acc_l[b][0] += ((pe[0] + pe[1]) + (pe[2] + pe[3])) + ((pe[4] + pe[5]) + (pe[6] + pe[7]));
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  if (n_it > 0) {
    // loads are issued in the order K(0) | V(0) K(1) | V(1) K(2) ...: per softmax slot i, V(i + V_AHEAD) and K(i + K_AHEAD)
#pragma unroll
    for (int j = 0; j <= V_AHEAD; ++j)
#pragma unroll
      for (int p = j == 0 ? LOADS : 0; p < PIECES; ++p) issue_piece(p, j - 1 - V_AHEAD);
    AT_WAIT_VM(PIECES * V_AHEAD);
    AT_SLOT_BARRIER();
    if (grp == 1) AT_SLOT_BARRIER();        // group 1 falls one slot behind ...
    // Before a tile is read every wave has waited for its own share of it and a barrier has passed: V(i), K(i + 1) by group 0 in
    // its softmax slot, by group 1, one slot behind, at the end of its multiply slot (the two later pairs of tiles issued by
    // then stay in flight, one for group 1 and if SPLIT).
    int i = 0;
    auto into_softmax = [&]() __attribute__((always_inline)) {
      if (!SPLIT && grp == 1) AT_WAIT_VM(PIECES * (V_AHEAD - 1));
      AT_SLOT_BARRIER();
    };
    auto into_multiply = [&]() __attribute__((always_inline)) {
      if (SPLIT || grp == 0) AT_WAIT_VM(PIECES * V_AHEAD);
      AT_SLOT_BARRIER();
      ++i;
    };
    auto skip = [&]() __attribute__((always_inline)) {      // a tile that no query of the wave sees
      into_softmax();
#pragma unroll
      for (int p = 0; p < PIECES; ++p) issue_piece(p, i);
      into_multiply();
    };
    while (i < min(act0, n_it)) skip();
    if (i < act1) {      // the wave's tiles: one run of steps, without a branch around the products
      __builtin_amdgcn_s_setprio(1);
      do {
        float mx[2];
        qk(i);
        __builtin_amdgcn_s_setprio(0);
        row_max(i, mx);
        into_softmax();
        softmax(i, mx);
        into_multiply();
        __builtin_amdgcn_s_setprio(1);
        pv(i - 1);
      } while (i < act1);
      __builtin_amdgcn_s_setprio(0);
    }
    while (i < n_it) skip();
    AT_WAIT_VM(0);
    if (grp == 0) AT_SLOT_BARRIER();        // ... and group 0 waits for it here: both execute the same number of barriers
  }

  if constexpr (FP32_STATS<DH>) {      // the four lanes that share a query hold a quarter of its keys each
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      acc_l[b][0] += __shfl_xor(acc_l[b][0], 16, 64);
      acc_l[b][0] += __shfl_xor(acc_l[b][0], 32, 64);
    }
  }
  if constexpr (SPLIT) {
    // the two halves of the keys meet in LDS: group 1 leaves (maximum, denominator, O), group 0 merges
    __syncthreads();
    float* mine = (float*)(sT + (wave & 3) * ((4 * DB + 4) * 2 * 256)) + lane;      // [float][lane]
    if (grp == 1) {
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        mine[(b * (4 * DB + 4) + 0) * 64] = m_raw[b];
        mine[(b * (4 * DB + 4) + 1) * 64] = acc_l[b][0];
        if (FP32_STATS<DH>) mine[(b * (4 * DB + 4) + 2) * 64] = m_neg[b];
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
          for (int r = 0; r < 4; ++r) mine[(b * (4 * DB + 4) + 4 + d * 4 + r) * 64] = acc[b][d][r];
      }
    }
    __syncthreads();
    if (grp == 1) return;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const float m1 = mine[(b * (4 * DB + 4) + 0) * 64], l1 = mine[(b * (4 * DB + 4) + 1) * 64];
      const float m_new = fmaxf(m_raw[b], m1);
      float e0 = (m_raw[b] - m_new) * sl, e1 = (m1 - m_new) * sl;
      if (FP32_STATS<DH>) {      // what the exponents added, as it was rounded
        const float neg1 = mine[(b * (4 * DB + 4) + 2) * 64], neg = m1 > m_raw[b] ? neg1 : m_neg[b];
        e0 = (neg - m_neg[b]) * LOG2E;
        e1 = (neg - neg1) * LOG2E;
        m_neg[b] = neg;
      }
      const float f0 = m_raw[b] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(e0);
      const float f1 = m1 == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(e1);
      m_raw[b] = m_new;
      acc_l[b][0] = acc_l[b][0] * f0 + l1 * f1;
#pragma unroll
      for (int d = 0; d < DB; ++d)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[b][d][r] = acc[b][d][r] * f0 + mine[(b * (4 * DB + 4) + 4 + d * 4 + r) * 64] * f1;
    }
  }
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int my_q = qw0 + b * 16 + li;
    if (my_q >= c) continue;
    const float l_tot = acc_l[b][0];
    const float inv = l_tot > 0.f ? 1.0f / l_tot : 0.0f;      // a query that saw no key: o = 0, lse = -inf
    bf16_t* op = o + ((int64_t)my_q * Hq + h) * DH + 4 * lg;
#pragma unroll
    for (int d = 0; d < DB; ++d) {
      bf16x4 w;
#pragma unroll
      for (int r = 0; r < 4; ++r) w[r] = (bf16_t)(acc[b][d][r] * inv);
      *(bf16x4*)(op + d * 16) = w;
    }
    if (lg == 0) lse[(int64_t)h * c + my_q] = !(l_tot > 0.f) ? -INFINITY : FP32_STATS<DH> ? logf(l_tot) - m_neg[b] : (m_raw[b] * sl + log2f(l_tot)) * LN2;
  }
}

// ----------------------------------------------------------------------- dQ --
// The slots of the forward kernel: multiply (dQ^T += K^T dS of the previous tile, S = K Q^T and dP = V dO^T of this one) and vector work (dS, and
// the loads of a later tile), group 1 of the waves one slot behind group 0, four K and V stages.
//   SPLIT = false: 256 queries, tiles of 64 keys.  A tile is loaded by all waves; group 0 loads two tiles ahead, group 1 three.
//   SPLIT = true : 128 queries per workgroup for launches that would leave CUs idle, as in the forward kernel: the groups take the even /
//                  odd tiles, of 32 keys, of the same queries and add up in LDS (1024 queries, 32 heads: 128 workgroups of 256 queries).
// What bounds it: the clock that the power limit leaves.  The slots keep the matrix pipe busier than two stages behind one barrier per tile did, and the
// clock falls by most of what that gives: backward and forward of the last 2048-query chunk of 32k, 28 heads, 3.68 -> 3.64 ms; a 32k layer at 7B widths
// 69.5 -> 67.9; 777 windowed queries 141.5 -> 139.0 us.  Tiles of 32 keys without SPLIT: 3.66 ms, the layer 70.0 (a slot of 24 MFMAs does not cover its start).
// 16x16x32 MFMAs take less of that power than 32x32x16 ones: the kernel itself on that chunk 1123 -> 1050 us (1002 to 1013 on other cards since).
// A wave's tiles are one loop without branches around the products, the stages moving with the addresses: with four steps unrolled, each skipping its products by a
// branch, the accumulators of four registers are moved about and 130 registers spill (1925 us).
// With few workgroups it is a step's instructions, slot by slot: the groups' slots are as long as the longer of the two, so what need not be in that one is in
// the other.  DH = 128 multiplies longer, and moves its fragments' addresses on in the vector slot; DH = 64 has the longer vector slot, and SPLIT loads at the start of the
// multiply slot.  27 queries behind 8877 keys, 12 / 2 heads of 128, backward 130.9 -> 129.9 us with the addresses moved, -> 122.5 with loads that pick their row offsets
// without a branch (the 32x32x16 kernel, steps unrolled, 126.4); 19 behind 4601, 16 / 4 heads of 64, 73.6 -> 71.2 without the branch, -> 69.5 with the loads moved,
// -> 65.5 with conversions two at a time (69.0).  More fragments requested ahead (7) or the two halves of the vector work not kept apart: no faster.
template <int DH, bool SPLIT>
struct DqShared { char sT[8][TILE64<DH>]; };      // K and V of stage after stage; SPLIT: of group 0, then of group 1
constexpr int DQ_CHAIN = 5;                       // LDS fragments requested ahead of the products (4: the same within 0.3 %)
template <int DH, bool SPLIT>
__device__ __forceinline__ void dq_tile(DqShared<DH, SPLIT>& sh, int q_block, int bh, const bf16_t* __restrict__ q, const bf16_t* __restrict__ k,
                                        const bf16_t* __restrict__ v, const bf16_t* __restrict__ d_o, const float* __restrict__ lse,
                                        const float* __restrict__ delta, bf16_t* __restrict__ dq, int Hq, int Hkv, int q_start, int c,
                                        float scale, const float2* __restrict__ rope, int window, const AttnSeqs& seqs) {
  auto& sT = sh.sT;
  const int b = bh / Hq, h = bh - b * Hq, kv_first = seqs.first[b];
  q += (int64_t)b * c * Hq * DH; d_o += (int64_t)b * c * Hq * DH; dq += (int64_t)b * c * Hq * DH;
  k += (int64_t)b * c * Hkv * DH; v += (int64_t)b * c * Hkv * DH;
  lse += (int64_t)b * c * Hq; delta += (int64_t)b * 2 * c * Hq;
  constexpr int QW = SPLIT ? TQ / 2 : TQ, NK = SPLIT ? TK / 2 : TK, NB = NK / 16;      // queries of the workgroup; keys of a tile, its 16-key blocks
  constexpr int STAGES = 4, TILE = NK * DH * 2;
  constexpr int LOADERS = SPLIT ? AT_THREADS / 2 : AT_THREADS, LOADS = NK * DH / 8 / LOADERS;      // threads that load a tile, 16-byte loads of each
  // Which slot a step's addresses and loads lie in (see above)
  constexpr bool MOVE_LATE = DH == 128, LOAD_LATE = SPLIT && DH == 64;

  const int q0 = q_block * QW, kvh = h / (Hq / Hkv);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), grp = wave >> 2, lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
  const int qw0 = q0 + (SPLIT ? wave & 3 : wave) * 32;      // a lane has the queries li and 16 + li from there on
  const int64_t kv_stride = (int64_t)Hkv * DH;
  const bf16_t* kbase = k + (int64_t)kvh * DH;
  const bf16_t* vbase = v + (int64_t)kvh * DH;
  const int n_total = q_start + c;
  const int n_keys = q_start + min(q0 + QW, c);
  const int n_tiles = (n_keys + NK - 1) / NK;
  const int wave_last_key = q_start + min(qw0 + 32, c) - 1;
  const int wave_first_qpos = q_start + qw0;
  auto first_key = [&](int p) { return max(kv_first, window > 0 ? p - window + 1 : 0); };   // left edge of the visible range
  const int wave_lo_min = first_key(wave_first_qpos), wave_lo_max = first_key(wave_last_key);
  const int kt0 = first_key(q_start + q0) / NK;
  // tile i of this wave's sequence
  auto tile_of = [&](int i) { return SPLIT ? kt0 + 2 * i + grp : kt0 + i; };
  const int n_it = SPLIT ? (max(0, n_tiles - kt0) + 1) / 2 : max(0, n_tiles - kt0);

  constexpr int KS = DH / 32, DB = DH / 16;      // k32 steps of a score, 16-row blocks of the output
  bf16x8 bq[2][KS], bdo[2][KS];                  // [16-query block][k32 step]
  float lse2[2], dlt[2];
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int q_row = min(qw0 + b * 16 + li, c - 1);
    const int64_t off = ((int64_t)q_row * Hq + h) * DH + lg * 8;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) { bq[b][kk] = *(const bf16x8*)(q + off + kk * 32); bdo[b][kk] = *(const bf16x8*)(d_o + off + kk * 32); }
    const float lse_q = lse[(int64_t)h * c + q_row];
    lse2[b] = lse_q == -INFINITY ? 0.0f : FP32_STATS<DH> ? lse_q : lse_q * LOG2E;    // a query that saw no key: every score is masked, p = exp2(-inf) = 0
    dlt[b] = delta[(int64_t)h * c + q_row];
  }
#pragma unroll
  for (int b = 0; b < 2; ++b) {
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) asm volatile("" : "+v"(bq[b][kk]), "+v"(bdo[b][kk]));      // (arrived: the compiler must not wait for them in the loop)
    asm volatile("" : "+v"(lse2[b]), "+v"(dlt[b]));
  }
  AT_WAIT_VM(0);     // from here on the loop counts its own loads only
  const float sl = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(scale * LOG2E)));

  // ---- addresses, computed once
  const uint32_t lds_k = lds_addr(&sT[0][0]) + (SPLIT ? (uint32_t)grp * 2 * STAGES * TILE : 0u);
  constexpr uint32_t STAGE = 2 * TILE;           // K, then V
  const uint32_t tid = threadIdx.x % LOADERS;
  auto load_offset = [&](uint32_t id, uint32_t row) { return (row * (uint32_t)kv_stride + ((id % (DH / 8)) ^ (uint32_t)swz<DH>((int)(id / (DH / 8)))) * 8) * 2; };      // (within a tile)
  // loads of tile i; past the end the last tile is loaded again, so that the wait counts stay the same.  The last tile may be short: its rows
  // past the end re-read the last one.  (Load j: LOADERS / (DH / 8) rows, a multiple of 16, further.)
  constexpr int ROWS_J = LOADERS / (DH / 8);
  const int t_max = n_tiles - 1, row_last = n_total - 1 - t_max * NK;
  const uint32_t voff = pin(load_offset(tid, tid / (DH / 8)));
  uint32_t voff_of[SPLIT ? LOADS : 1], voff_last[SPLIT ? LOADS : 1];      // SPLIT has registers for every load's offset, and no branch then
#pragma unroll
  for (int j = 0; j < (SPLIT ? LOADS : 0); ++j) {
    const uint32_t row = tid / (DH / 8) + j * ROWS_J;
    voff_of[j] = pin(load_offset(tid, row));
    voff_last[j] = pin(load_offset(tid, min(row, (uint32_t)row_last)));
  }
  const uint32_t dst = __builtin_amdgcn_readfirstlane(lds_k + (uint32_t)(tid & ~63) * 16u), tile_bytes = (uint32_t)(NK * kv_stride * 2);
  auto issue = [&](int i) __attribute__((always_inline)) {
    const int t = min(tile_of(i), t_max);
    const char *ks = (const char*)kbase + (uint64_t)tile_bytes * (uint32_t)t, *vs = (const char*)vbase + (uint64_t)tile_bytes * (uint32_t)t;
    const uint32_t to = dst + (uint32_t)(i % STAGES) * STAGE;
    if constexpr (SPLIT) {
#pragma unroll
      for (int j = 0; j < LOADS; ++j) {
        const uint32_t off = t == t_max ? voff_last[j] : voff_of[j];
        dma16(ks, off, to + (uint32_t)(j * LOADERS * 16));
        dma16(vs, off, to + (uint32_t)(TILE + j * LOADERS * 16));
      }
    } else if (t < t_max || row_last >= NK - 1) {
#pragma unroll
      for (int j = 0; j < LOADS; ++j) {
        const int64_t rows = (int64_t)j * ROWS_J * kv_stride * 2;
        dma16(ks + rows, voff, to + (uint32_t)(j * LOADERS * 16));
        dma16(vs + rows, voff, to + (uint32_t)(TILE + j * LOADERS * 16));
      }
    } else {
#pragma unroll
      for (int j = 0; j < LOADS; ++j) {
        const uint32_t id = pin(threadIdx.x) % LOADERS;      // (opaque: nothing of this is kept in a register from tile to tile)
        const uint32_t off = load_offset(id, min(id / (DH / 8) + j * ROWS_J, (uint32_t)row_last));
        dma16(ks, off, to + (uint32_t)(j * LOADERS * 16));
        dma16(vs, off, to + (uint32_t)(TILE + j * LOADERS * 16));
      }
    }
  };
  // steps in which some (query, key) pair of the wave is visible
  const int step_t = SPLIT ? 2 : 1, first_t = tile_of(0);
  const int act0 = max(0, (wave_lo_min / NK - first_t + step_t - 1) / step_t);
  const int act1 = qw0 < c && wave_last_key >= 0 ? min(n_it, (wave_last_key / NK - first_t + step_t) / step_t) : 0;

  // LDS addresses of fragments, one step after the other: of K (and V) rows of the present tile, of K transposed of the previous one
  uint32_t fr[KS], ft[DB];
#pragma unroll
  for (int kk = 0; kk < KS; ++kk) fr[kk] = pin(lds_k + frag16_rows<DH>(kk) + (uint32_t)(act0 % STAGES) * STAGE);
#pragma unroll
  for (int d = 0; d < DB; ++d) ft[d] = pin(lds_k + frag16_tr<DH>(d) + (uint32_t)((act0 + (MOVE_LATE ? STAGES - 1 : 0)) % STAGES) * STAGE);
  auto to_next = [&](int i) { return i % STAGES == STAGES - 1 ? (uint32_t)-(int)((STAGES - 1) * STAGE) : STAGE; };      // from the stage of tile i
  auto move_rows = [&](int i) __attribute__((always_inline)) {
    const uint32_t move = to_next(i);
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) fr[kk] = pin(fr[kk] + move);
  };
  auto move_tr = [&](int i) __attribute__((always_inline)) {
    const uint32_t move = to_next(i);
#pragma unroll
    for (int d = 0; d < DB; ++d) ft[d] = pin(ft[d] + move);
  };

  struct Scores { f32x4 s[2][NB], dp[2][NB]; };        // S^T, dP^T [query block][16 keys]
  struct Operand { bf16x8 w[TERMS<DH>][2][NB / 2]; };  // dS^T: [term][query block][k32 step]
  f32x4 acc[2][DB];                                    // dQ^T [query block][16 head_dim rows]
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int d = 0; d < DB; ++d) acc[b][d] = f32x4{0.f, 0.f, 0.f, 0.f};
  constexpr uint32_t ROWS16 = 16 * DH * 2;
  auto second = [&](const Operand& ds, int i) __attribute__((always_inline)) {
    // n = k32 step * DB + head_dim block
    mfma_chain<NB / 2 * DB, DQ_CHAIN>(
        [&](int n) { const uint32_t o = (uint32_t)(n / DB) * 2 * ROWS16; return lds_tr(ft[n % DB] + o, ft[n % DB] + (o + ROWS16)); },
        [&](int n, const bf16x8& f) {
#pragma unroll
          for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int t = 0; t < TERMS<DH>; ++t) acc[b][n % DB] = MFMA16(f, ds.w[t][b][n / DB], acc[b][n % DB]);
        });
    if (!MOVE_LATE) move_tr(i);
  };
  auto first = [&](Scores& x, int i) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int kb = 0; kb < NB; ++kb) { x.s[b][kb] = f32x4{0.f, 0.f, 0.f, 0.f}; x.dp[b][kb] = f32x4{0.f, 0.f, 0.f, 0.f}; }
    // n = k32 step * 2 NB + which: S of the key blocks, then dP of the key blocks
    mfma_chain<2 * NB * KS, DQ_CHAIN>(
        [&](int n) { const int kb = n % (2 * NB); return lds_b128(fr[n / (2 * NB)] + (kb >= NB ? (uint32_t)TILE : 0u) + (uint32_t)(kb % NB) * ROWS16); },
        [&](int n, const bf16x8& f) {
          const int kb = n % (2 * NB), kk = n / (2 * NB);
#pragma unroll
          for (int b = 0; b < 2; ++b)
            if (kb < NB) x.s[b][kb] = MFMA16(f, bq[b][kk], x.s[b][kb]); else x.dp[b][kb - NB] = MFMA16(f, bdo[b][kk], x.dp[b][kb - NB]);
        });
    if (!MOVE_LATE) move_rows(i);
  };
  auto vector = [&](Scores& x, Operand& ds, int i) __attribute__((always_inline)) {
    const int k0 = tile_of(i) * NK;
    if (k0 + NK - 1 > wave_first_qpos || k0 < wave_lo_max) {      // only tiles on an edge of the visible range pay for the mask
      const int l = (int)pin(threadIdx.x) & 63;
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        // key 4 lg + e of the tile is visible for first <= e < first + n: one unsigned comparison
        const int qpos = q_start + min(qw0 + b * 16 + (l & 15), c - 1), lo = first_key(qpos), from = lo - k0 - 4 * (l >> 4);
        const uint32_t n = (uint32_t)max(0, qpos - lo + 1);
#pragma unroll
        for (int kb = 0; kb < NB; ++kb) {
#pragma unroll
          for (int r = 0; r < 4; ++r) x.s[b][kb][r] = (uint32_t)(kb * 16 + r - from) < n ? x.s[b][kb][r] : -INFINITY;     // exp2(-inf) = 0
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int ks = 0; ks < NB / 2; ++ks) {
        __builtin_amdgcn_sched_barrier(0);
        auto grad = [&](int e) __attribute__((always_inline)) {      // dS^T (the factor `scale` is applied at the end)
          const int kb = 2 * ks + (e >> 2), r = e & 3;
          const float p = exp_of<DH>(x.s[b][kb][r], scale, sl, -lse2[b]);
          return p * (x.dp[b][kb][r] - dlt[b]);
        };
        if constexpr (TERMS<DH> == 1) {
#pragma unroll
          for (int e = 0; e < 8; ++e) ds.w[0][b][ks][e] = (bf16_t)grad(e);
        } else {
#pragma unroll
          for (int e = 0; e < 8; e += 2) {
            const f32x2 y = {grad(e), grad(e + 1)};
            const bf16x2 w0 = round2(y), w1 = round2(rest2(y, w0));
#pragma unroll
            for (int u = 0; u < 2; ++u) { ds.w[0][b][ks][e + u] = w0[u]; ds.w[1][b][ks][e + u] = w1[u]; }
          }
        }
      }
    __builtin_amdgcn_sched_barrier(0);
  };

  if (n_it > 0) {
    // Before a tile is read every wave has waited for its own share of it and a barrier has passed: tile j + 1 by the end of vector slot j, or,
    // where group 1 loads for group 0 as well, by the end of its multiply slot j; what was issued after it stays in flight.  A stage is
    // loaded again once the slot is over in which its K was last read, for the second product: by group 0 two tiles ahead, as group 1 reads
    // K of tile j - 2 in the slot before vector slot j of group 0; else three.
    constexpr int PAIR = 2 * LOADS;
    const bool late = !SPLIT && grp == 1;
    const int ahead = SPLIT || late ? 3 : 2;
    auto wait_late = [&]() __attribute__((always_inline)) { if (late) AT_WAIT_VM(PAIR); };
    auto wait_early = [&]() __attribute__((always_inline)) {
      if (SPLIT) AT_WAIT_VM((LOAD_LATE ? 1 : 2) * PAIR);
      else if (!late) AT_WAIT_VM(PAIR);
    };
    for (int j = 0; j < ahead; ++j) issue(j);
    if (SPLIT || late) AT_WAIT_VM(2 * PAIR);
    else AT_WAIT_VM(PAIR);
    AT_SLOT_BARRIER();
    if (grp == 1) AT_SLOT_BARRIER();
    int i = 0;
    auto into_vector = [&]() __attribute__((always_inline)) {
      __builtin_amdgcn_s_setprio(0);
      wait_late();
      AT_SLOT_BARRIER();
      if (!LOAD_LATE) issue(i + ahead);
    };
    auto into_multiply = [&]() __attribute__((always_inline)) {
      wait_early();
      AT_SLOT_BARRIER();
      if (LOAD_LATE) issue(i + ahead);      // (the stage of tile i - 1, whose K every wave of the group has read by the barrier before)
      ++i;
    };
    auto skip = [&]() __attribute__((always_inline)) { into_vector(); into_multiply(); };      // a tile that no query of the wave sees
    while (i < min(act0, n_it)) skip();
    if (i < act1) {
      __builtin_amdgcn_s_setprio(1);
      do {
        Scores x;
        Operand ds;
        first(x, i);
        into_vector();
        if (MOVE_LATE) { move_rows(i); move_tr(i + STAGES - 1); }
        vector(x, ds, i);
        into_multiply();
        __builtin_amdgcn_s_setprio(1);
        second(ds, i - 1);
      } while (i < act1);
      __builtin_amdgcn_s_setprio(0);
    }
    while (i < n_it) skip();
    AT_WAIT_VM(0);
    if (grp == 0) AT_SLOT_BARRIER();        // both groups execute the same number of barriers
  }

  if constexpr (SPLIT) {
    __syncthreads();
    float* mine = (float*)&sT[0][0] + (wave & 3) * (DB * 8 * 64) + lane;      // [float][lane]
    if (grp == 1) {
#pragma unroll
      for (int i = 0; i < DB * 8; ++i) mine[i * 64] = acc[i / (DB * 4)][(i >> 2) % DB][i & 3];
    }
    __syncthreads();
    if (grp == 1) return;
#pragma unroll
    for (int i = 0; i < DB * 8; ++i) acc[i / (DB * 4)][(i >> 2) % DB][i & 3] += mine[i * 64];
  }
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const int my_q = qw0 + b * 16 + li;
    if (my_q >= c) continue;
    bf16_t* op = dq + ((int64_t)my_q * Hq + h) * DH + 4 * lg;
    if (rope) {
      // adjoint of the rotary embedding on the way out: element j < DH / 2 (accumulator block d < DB / 2) pairs with
      // j + DH / 2 (block d + DB / 2, same register of the same lane); rotation by the negative angle
      const float2* tr = rope + (int64_t)my_q * (DH / 2) + 4 * lg;
#pragma unroll
      for (int d = 0; d < DB / 2; ++d) {
        bf16x4 w1, w2;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float2 cs = tr[d * 16 + r];
          const float d1 = acc[b][d][r] * scale, d2 = acc[b][d + DB / 2][r] * scale;
          w1[r] = (bf16_t)(d1 * cs.x + d2 * cs.y);
          w2[r] = (bf16_t)(d2 * cs.x - d1 * cs.y);
        }
        *(bf16x4*)(op + d * 16) = w1;
        *(bf16x4*)(op + (d + DB / 2) * 16) = w2;
      }
    } else {
#pragma unroll
      for (int d = 0; d < DB; ++d) {
        bf16x4 w;
#pragma unroll
        for (int r = 0; r < 4; ++r) w[r] = (bf16_t)(acc[b][d][r] * scale);
        *(bf16x4*)(op + d * 16) = w;
      }
    }
  }
}

template <int DH, bool SPLIT>
__global__ __launch_bounds__(AT_THREADS) void attn_bwd_dq_mfma_k(const bf16_t* __restrict__ q, const bf16_t* __restrict__ k,
                                                                    const bf16_t* __restrict__ v, const bf16_t* __restrict__ d_o,
                                                                    const float* __restrict__ lse, const float* __restrict__ delta,
                                                                    bf16_t* __restrict__ dq, int Hq, int Hkv, int q_start, int c,
                                                                    float scale, const float2* __restrict__ rope, int window,
                                                                    const AttnSeqs seqs, int q_blocks) {
  __shared__ __attribute__((aligned(1024))) DqShared<DH, SPLIT> sh;
  int qt = blockIdx.x % q_blocks, bh = blockIdx.x / q_blocks;
  if ((int)gridDim.x > 256) query_tile_of(blockIdx.x, q_blocks, Hq * seqs.n, qt, bh);
  dq_tile<DH, SPLIT>(sh, qt, bh, q, k, v, d_o, lse, delta, dq, Hq, Hkv, q_start, c, scale, rope, window, seqs);
}

// -------------------------------------------------------------------- dK/dV --
// Workgroup = 128 keys of one KV head, 8 waves = 4 key blocks of 32 x 2 roles, so that each SIMD holds the two
// waves of one key block:
//   role P (waves 0-3): S = Q K^T -> P = exp(S*scale - lse) (masked), DH = 128: rounded to bf16 -> leaves P in LDS for its
//                       partner -> dV^T += dO^T P
//   role S (waves 4-7): dP = dO V^T -> takes P -> dS = P * (dP - delta) -> dK^T += Q^T dS
// Each role keeps only its own operand fragments (K or V) and its own accumulator (dV or dK) in registers: half the registers of a
// do-everything wave, so two waves fit per SIMD.  As in the forward kernel a tile costs a wave two slots, each closed by a barrier:
// multiply (dV += dO^T P resp. dK += Q^T dS of the previous tile, S = Q K^T resp. dP = dO V^T of this one) and vector work; role S runs
// one slot behind role P - it then finds the P of its tile in LDS - so on every SIMD one wave multiplies while the other works on
// exponentials or dS.  Four stages of the Q / dO tiles; role P loads two tiles ahead, role S three.
// What bounds it: as in the forward kernel, vector work and MFMAs of a SIMD's two waves share the issue port, and the power limit leaves 2.0 GHz.  Last
// 2048-query chunk of 32k, 28 / 4 heads: dQ + dK/dV 3.08 -> 2.95 ms, all of it here (about 1.85 -> 1.72), against one barrier per tile and each wave doing its
// products and its vector work in any order; 1740 -> 1655 us with 16x16x32 MFMAs in place of 32x32x16, -> 1610 with a loop whose stages move with the
// addresses in place of four steps unrolled (a quarter of the code); 1494 to 1518 us on other cards since.  What parts of it cost cannot be told by leaving them out: other values
// are multiplied then, at another power (without exponentials 1406; the kernel on 32x32x16 MFMAs took 1745, 1630 with half of its LDS reads, 1705 without exponentials).
// The loop walks the query tiles at or below the diagonal and, for each, the query heads of the group.
//
// Its steps come in `slices` shares, whose sums are added to dK / dV in their order.  Where there is room for them a workgroup takes each share
// and leaves its sum in `part`.  Without that room a workgroup takes one share after the other, with the same sums in the same order.  It empties
// its pipeline between them, which costs about three steps each time; IN_TURN, for the chunks of few key blocks that come in many shares,
// walks them without a break and keeps the total beside the present sum, in registers.  Both only fit for half of the head's columns, so two
// workgroups share a key block, each with all scores and half of the second product.  Whole backward, without / with a break | one share, dQ
// apart | with room, 28 / 4 heads: 512 queries from 0 228 / 123 | 143 | 41 us, 2048 from 0 401 / 357 | 459 | 177; 512 from 2560 (96 blocks) 135 /
// 124 | 184 | 123, from 2816 (104 blocks, whose 208 workgroups leave dQ too few CUs) 136 / 152 | 188 | 127, from 3500 145 / 198 | 205 | 146.
constexpr int KV_STAGES = 4;
constexpr int CHAIN = 6;                 // LDS fragments requested ahead of the products (dK/dV)

template <int DH>
struct DkvShared {
  char sQD[2][KV_STAGES][TILE64<DH>];             // [Q | dO][stage]
  // P of the tile, [key block][slot][lane]: bf16, slot = query block * 2 + k16 step; FP32_STATS: fp32, slot = query block * 4 + r / 4
  bf16x8 sP[4][FP32_STATS<DH> ? 8 : 4][64];
  float sL[KV_STAGES][QT];                        // (log2-domain) log-sum-exp of the tile's queries
  float sDl[KV_STAGES][QT];                       // delta of the tile's queries
};
template <int DH, bool IN_TURN>
__device__ __forceinline__ void dkv_block(DkvShared<DH>& sh, int key_block, int bh, int slice, const bf16_t* __restrict__ q,
                                          const bf16_t* __restrict__ k, const bf16_t* __restrict__ v, const bf16_t* __restrict__ d_o,
                                          const float* __restrict__ lse2, const float* __restrict__ delta, float* __restrict__ dk,
                                          float* __restrict__ dv, int Hq, int Hkv, int q_start, int c, float scale, int window, const AttnSeqs& seqs,
                                          int key_block0, int slices, float* __restrict__ part) {
  const int sq = bh / Hkv, kvh = bh - sq * Hkv, kv_first = seqs.first[sq];
  {
    const int64_t nq = (int64_t)sq * c * Hq, nk = (int64_t)sq * c * Hkv * DH;
    q += nq * DH; d_o += nq * DH; lse2 += 2 * nq; delta += 2 * nq;
    k += nk; v += nk; dk += nk; dv += nk;
    if (part) part += (int64_t)sq * slices * 2 * (q_start + c - key_block0 * KV_TILE) * Hkv * DH;
  }
  auto& sQD = sh.sQD;
  auto& sP = sh.sP;
  auto& sL = sh.sL;
  auto& sDl = sh.sDl;

  const int G = Hq / Hkv;
  const int key0 = (key_block0 + key_block) * KV_TILE;   // key blocks before key_block0 are visible to no query
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
  const int kb = wave & 3;
  const bool role_p = wave < 4;
  const int n_total = q_start + c;
  const int kw0 = key0 + kb * 32;      // a lane has the keys li and 16 + li from there on
  auto key_of = [&](int b) { return kw0 + b * 16 + li; };
  auto key_row = [&](int b) { return (int64_t)min(key_of(b), n_total - 1); };
  const int64_t kv_stride = (int64_t)Hkv * DH;
  const int64_t q_stride = (int64_t)Hq * DH;

  // Fragment addresses: one set reaches all stages of its operand with immediate offsets.  Role P reads Q row-wise and dO
  // transposed, role S the other way round; only the half of each set that the role uses stays live.
  const uint32_t lds0 = lds_addr(&sQD[0][0][0]), lds_do = lds0 + KV_STAGES * TILE64<DH>;
  constexpr int KS = DH / 32, DB = DH / 16 / (IN_TURN ? 2 : 1);      // k32 steps of a score, 16-row blocks of the output
  const int col0 = IN_TURN ? slice * (DH / 2) : 0;       // IN_TURN: `slice` is the half of the columns
  const TileLoad<DH, KV_THREADS> tl = tile_load_pre<DH, KV_THREADS>(q_stride);
  const uint32_t sp_lane = pin(lds_addr(&sP[kb][0][lane]));                      // + slot * 1024
  const uint32_t stat_lane = pin(lds_addr(role_p ? &sL[0][4 * lg] : &sDl[0][4 * lg]));   // + stage * 256 + query block * 64

  // what this lane's keys grow by, rows = head_dim col0 + 16 d + 4 lg .. + 3
  auto out_of = [&](int b) { return (role_p ? dv : dk) + key_row(b) * kv_stride + (int64_t)kvh * DH + col0 + 4 * lg; };
  f32x4 sum[2][IN_TURN ? DB : 1];
  if constexpr (IN_TURN) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int d = 0; d < DB; ++d) sum[b][d] = *(const f32x4*)(out_of(b) + d * 16);
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int d = 0; d < DB; ++d) asm volatile("" : "+v"(sum[b][d]));
  }
  bf16x8 breg[2][KS];   // B operand of the first product: K rows (role P) or V rows (role S) of my keys
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    const bf16_t* src = (role_p ? k : v) + key_row(b) * kv_stride + (int64_t)kvh * DH + lg * 8;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) breg[b][kk] = *(const bf16x8*)(src + kk * 32);
  }
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) asm volatile("" : "+v"(breg[b][kk]));   // (arrived: the compiler must not wait for them in the loop)
  AT_WAIT_VM(0);
  const float sl = scale * LOG2E;

  // query tiles that can see at least one key of this workgroup: query position >= key0
  // ... and, under a sliding window, query position <= last key of the workgroup + window - 1
  const int qt_first = max(0, key0 - q_start) / QT;
  int n_qt = (c + QT - 1) / QT;
  if (window > 0) n_qt = min(n_qt, max(0, key0 + KV_TILE - 1 + window - 1 - q_start) / QT + 1);
  const int n_all = key0 + KV_TILE <= kv_first ? 0 : max(0, n_qt - qt_first) * G;      // (a sequence of several may hide blocks that others see)
  auto share = [&](int z) { return (int)((int64_t)n_all * z / slices); };      // first step of share z
  for (int z = part ? slice : 0, z_last = IN_TURN ? 0 : part ? slice : slices - 1; z <= z_last; ++z) {
  const int it0 = IN_TURN ? 0 : share(z), n_iter = (IN_TURN ? n_all : share(z + 1)) - it0;

  // Loads of the next tile (query tile lq, head lh of the group); past the end the last one again, so that the wait counts
  // stay the same.
  int lq = qt_first + it0 / G, lh = it0 % G, left = n_iter;
  auto issue = [&](int stage) {
    const int qt = lq, hh = kvh * G + lh;
    if (--left > 0 && ++lh == G) { lh = 0; ++lq; }
    const int64_t corner = (int64_t)qt * QT * q_stride + (int64_t)hh * DH;
    dma_tile64(tl, q + corner, q_stride, c - qt * QT, lds0 + (uint32_t)(stage * TILE64<DH>));
    dma_tile64(tl, d_o + corner, q_stride, c - qt * QT, lds_do + (uint32_t)(stage * TILE64<DH>));
    // 64 log-sum-exp values (role P) or deltas (role S), 4 B per lane, also direct to LDS (by every wave of the role, the same
    // values, so that all waves count the same number of loads)
    const int row = min(qt * QT + lane, c - 1);
    dma4(uniform_ptr((role_p ? lse2 : delta) + (int64_t)hh * c), (uint32_t)row * 4u,
         __builtin_amdgcn_readfirstlane(lds_addr(role_p ? &sL[stage][0] : &sDl[stage][0])));
  };
  // One 64-query tile = two 32-query blocks.  `active`: the wave has a valid key and some query of the tile is
  // at or after its first key (the same answer for both waves of a key block).
  auto tile_active = [&](int qbase) {
    return kw0 < n_total && q_start + min(qbase + QT, c) - 1 >= kw0 && kw0 + 31 >= kv_first &&
           (window == 0 || q_start + qbase - window < kw0 + 31);     // the tile's first query still reaches the wave's last key
  };
  auto lds_f4 = [](uint32_t addr) { return *(const float4*)(__attribute__((address_space(3))) const char*)(uintptr_t)addr; };

  constexpr int LOADS = 2 * (8 * DH / KV_THREADS) + 1;       // vector-memory operations of one issue
  auto run = [&](auto role_c) __attribute__((always_inline)) {
    constexpr bool RP = decltype(role_c)::value;
    constexpr int NT = KV_TERMS<DH>;
    f32x4 acc[2][DB];        // dV^T (role P) or dK^T (role S): [16-key block][16 head_dim rows], column = my key
    f32x4 t[2][4];           // S or dP of the tile: [key block][16-query block], rows = queries 4 lg + r of the block
    bf16x8 w[NT][2][2];      // P or dS: [term][key block][k32 step]
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int d = 0; d < DB; ++d) acc[b][d] = f32x4{0.f, 0.f, 0.f, 0.f};
    const float f = RP ? 1.0f : scale;
    int present = 0, present_end = IN_TURN ? share(1) : 0;      // IN_TURN: the share that is being summed, and the step after it
    auto close = [&]() __attribute__((always_inline)) {         // total += the share's sum
#pragma unroll
      for (int i = 0; i < (IN_TURN ? 2 * DB : 0); ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
#pragma clang fp contract(off)      // product and sum rounded separately, with or without parts
          sum[i / DB][i % DB][r] += acc[i / DB][i % DB][r] * f;
          acc[i / DB][i % DB][r] = 0.f;
        }
    };
    int j = 0, qbase = (qt_first + it0 / G) * QT, head = it0 % G;      // the present step, of its tile
    // LDS addresses of fragments, one step after the other: of the row-wise operand of the present tile, Q (P) / dO (S), and of the transposed
    // one, dO (P) / Q (S), of the previous tile
    uint32_t fr[KS], gt[DB];
    auto to_next = [&](int step) { return step % KV_STAGES == KV_STAGES - 1 ? (uint32_t)-(int)((KV_STAGES - 1) * TILE64<DH>) : (uint32_t)TILE64<DH>; };      // from its stage
    constexpr uint32_t ROWS16 = 16 * DH * 2;
    auto second = [&]() __attribute__((always_inline)) {
      // n = k32 step * DB + head_dim block
      mfma_chain<2 * DB, CHAIN>(
          [&](int n) { const uint32_t o = (uint32_t)(n / DB) * 2 * ROWS16; return lds_tr(gt[n % DB] + o, gt[n % DB] + (o + ROWS16)); },
          [&](int n, const bf16x8& g) {
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
              for (int u = 0; u < NT; ++u) acc[b][n % DB] = MFMA16(g, w[u][b][n / DB], acc[b][n % DB]);
          });
      const uint32_t move = to_next(j - 1);
#pragma unroll
      for (int d = 0; d < DB; ++d) gt[d] = pin(gt[d] + move);
    };
    auto first = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int qb = 0; qb < 4; ++qb) t[b][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
      // n = k32 step * 4 + query block
      mfma_chain<4 * KS, CHAIN>([&](int n) { return lds_b128(fr[n >> 2] + (uint32_t)(n & 3) * ROWS16); },
                                [&](int n, const bf16x8& g) {
#pragma unroll
                                  for (int b = 0; b < 2; ++b) t[b][n & 3] = MFMA16(g, breg[b][n >> 2], t[b][n & 3]);
                                });
      const uint32_t move = to_next(j);
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) fr[kk] = pin(fr[kk] + move);
    };
    auto terms = [&](int b, int ks) __attribute__((always_inline)) {      // P resp. dS as operands of the second product
      auto value = [&](int e) __attribute__((always_inline)) { return t[b][2 * ks + (e >> 2)][e & 3]; };
      if constexpr (NT == 1) {
#pragma unroll
        for (int e = 0; e < 8; ++e) w[0][b][ks][e] = (bf16_t)value(e);
      } else {
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
          const f32x2 x = {value(e), value(e + 1)};
          const bf16x2 w0 = round2(x);
          const f32x2 r0 = rest2(x, w0);
          const bf16x2 w1 = round2(r0), w2 = round2(rest2(r0, w1));
#pragma unroll
          for (int u = 0; u < 2; ++u) { w[0][b][ks][e + u] = w0[u]; w[1][b][ks][e + u] = w1[u]; w[2][b][ks][e + u] = w2[u]; }
        }
      }
    };
    auto vector = [&]() __attribute__((always_inline)) {
      const uint32_t stat = stat_lane + (uint32_t)(j % KV_STAGES) * QT * 4;
      if constexpr (RP) {
        const bool diag = (q_start + qbase < kw0 + 31) || (qbase + QT > c) || kw0 < kv_first ||   // some pair masked, or ragged query tile
                          (window > 0 && q_start + qbase + QT - 1 - window >= kw0);
        if (diag) {
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            // query 4 lg + e of the tile sees the key for from <= e < from + n: one unsigned comparison
            const int key = key_of(b), lo = max(0, key - q_start), hi = window > 0 ? min(c, key + min(window, n_total) - q_start) : c;
            const uint32_t n = key < kv_first ? 0u : (uint32_t)max(0, hi - lo);
            const int from = lo - qbase - 4 * lg;
#pragma unroll
            for (int qb = 0; qb < 4; ++qb) {
#pragma unroll
              for (int r = 0; r < 4; ++r) t[b][qb][r] = (uint32_t)(qb * 16 + r - from) < n ? t[b][qb][r] : -INFINITY;      // exp2(-inf) = 0
              __builtin_amdgcn_sched_barrier(0);
            }
          }
        }
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
          for (int x = 0; x < 2; ++x) {
            const int qb = 2 * ks + x;
            const float4 l4 = lds_f4(stat + qb * 64);
            const float lv[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
              for (int r = 0; r < 4; ++r) t[b][qb][r] = exp_of<DH>(t[b][qb][r], scale, sl, -lv[r]);
          }
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            terms(b, ks);
            if constexpr (!FP32_STATS<DH>)
              *(bf16x8*)(__attribute__((address_space(3))) char*)(uintptr_t)(sp_lane + (b * 2 + ks) * 1024) = w[0][b][ks];
            else {
#pragma unroll
              for (int x = 0; x < 2; ++x)
                *(f32x4*)(__attribute__((address_space(3))) char*)(uintptr_t)(sp_lane + (b * 4 + 2 * ks + x) * 1024) = t[b][2 * ks + x];
            }
          }
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // P is in LDS before the barrier
      } else {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          const float4 d0 = lds_f4(stat + ks * 128), d1 = lds_f4(stat + ks * 128 + 64);
          const float dl[8] = {d0.x, d0.y, d0.z, d0.w, d1.x, d1.y, d1.z, d1.w};
#pragma unroll
          for (int b = 0; b < 2; ++b) {
            float pv[8];
            if constexpr (FP32_STATS<DH>) {
              const float4 p0 = lds_f4(sp_lane + (b * 4 + 2 * ks) * 1024), p1 = lds_f4(sp_lane + (b * 4 + 2 * ks + 1) * 1024);
              pv[0] = p0.x; pv[1] = p0.y; pv[2] = p0.z; pv[3] = p0.w; pv[4] = p1.x; pv[5] = p1.y; pv[6] = p1.z; pv[7] = p1.w;
            } else {
              const bf16x8 p8 = lds_b128(sp_lane + (b * 2 + ks) * 1024);
#pragma unroll
              for (int e = 0; e < 8; ++e) pv[e] = (float)p8[e];
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              f32x4& x = t[b][2 * ks + (e >> 2)];
              x[e & 3] = pv[e] * (x[e & 3] - dl[e]);     // dS (the softmax scale is applied once at the end)
            }
            terms(b, ks);
          }
        }
      }
    };
    if (n_iter > 0) {
      // Role P loads tile j + 2 in its vector slot j, role S tile j + 3 in its own: the stage was last read at least one slot before.
      // Tile j + 1 has landed for everyone before role P multiplies it: role P waits at the end of vector slot j, role S, one slot
      // behind, at the end of multiply slot j; the one tile issued after it stays in flight.
      constexpr int AHEAD = RP ? 2 : 3;
#pragma unroll
      for (int a = 0; a < AHEAD; ++a) issue(a);
      AT_WAIT_VM(LOADS * (AHEAD - 1));
      AT_SLOT_BARRIER();
      if (!RP) AT_SLOT_BARRIER();
      auto into_vector = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_s_setprio(0);
        if (!RP) AT_WAIT_VM(LOADS);
        AT_SLOT_BARRIER();
        issue((j + AHEAD) % KV_STAGES);
      };
      auto into_multiply = [&]() __attribute__((always_inline)) {
        if (++head == G) { head = 0; qbase += QT; }
        if (RP) AT_WAIT_VM(LOADS);
        AT_SLOT_BARRIER();
        ++j;
      };
      auto boundary = [&]() __attribute__((always_inline)) {
        if (IN_TURN && j == present_end) {
          close();
          while (present_end == j && present + 1 < slices) present_end = share(++present + 1);      // (shares without steps add nothing)
        }
      };
      auto skip = [&]() __attribute__((always_inline)) { into_vector(); into_multiply(); boundary(); };      // a tile that the wave has no pair of
      boundary();            // (the first shares may be empty)
      while (j < n_iter && !tile_active(qbase)) skip();
      if (j < n_iter) {      // the wave's tiles: one run of steps
#pragma unroll
        for (int kk = 0; kk < KS; ++kk) fr[kk] = pin((RP ? lds0 : lds_do) + frag16_rows<DH>(kk) + (uint32_t)(j % KV_STAGES) * TILE64<DH>);
#pragma unroll
        for (int d = 0; d < DB; ++d) gt[d] = pin((RP ? lds_do : lds0) + frag16_tr<DH>(col0 / 16 + d) + (uint32_t)(j % KV_STAGES) * TILE64<DH>);
        __builtin_amdgcn_s_setprio(1);
        do {
          first();
          into_vector();
          vector();
          into_multiply();
          __builtin_amdgcn_s_setprio(1);
          second();
          boundary();
        } while (j < n_iter && tile_active(qbase));
        __builtin_amdgcn_s_setprio(0);
      }
      while (j < n_iter) skip();
      AT_WAIT_VM(0);
      if (RP) AT_SLOT_BARRIER();        // both roles execute the same number of barriers
    }
    if constexpr (IN_TURN) close();
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      if (key_of(b) >= n_total) continue;
      if constexpr (IN_TURN) {
#pragma unroll
        for (int d = 0; d < DB; ++d) *(f32x4*)(out_of(b) + d * 16) = sum[b][d];
      } else {
        // several workgroups per key block: each leaves its sum in its own slice [workgroup][dk | dv][key][kv head][DH]
        const int64_t first = (int64_t)key_block0 * KV_TILE;
        float* to = part ? part + ((int64_t)z * 2 + (RP ? 1 : 0)) * (n_total - first) * kv_stride + (key_of(b) - first) * kv_stride + (int64_t)kvh * DH + 4 * lg : out_of(b);
#pragma unroll
        for (int d = 0; d < DB; ++d) {
          f32x4 u = part ? f32x4{0.f, 0.f, 0.f, 0.f} : *(f32x4*)(to + d * 16);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
#pragma clang fp contract(off)
            u[r] += acc[b][d][r] * f;
          }
          *(f32x4*)(to + d * 16) = u;
        }
      }
    }
  };
  if (role_p) run(std::true_type{});
  else run(std::false_type{});
  if (z < z_last) __syncthreads();      // the next share loads into the stages of this one
  }
}

template <int DH>
__global__ __launch_bounds__(KV_THREADS) void attn_bwd_dkv_mfma_k(const bf16_t* __restrict__ q, const bf16_t* __restrict__ k,
                                                                  const bf16_t* __restrict__ v, const bf16_t* __restrict__ d_o,
                                                                  const float* __restrict__ lse2, const float* __restrict__ delta,
                                                                  float* __restrict__ dk, float* __restrict__ dv, int Hq, int Hkv,
                                                                  int q_start, int c, float scale, int window, const AttnSeqs seqs,
                                                                  int key_block0, int slices, float* __restrict__ part) {
  __shared__ __attribute__((aligned(1024))) DkvShared<DH> sh;
  dkv_block<DH, false>(sh, blockIdx.x, blockIdx.y, blockIdx.z, q, k, v, d_o, lse2, delta, dk, dv, Hq, Hkv, q_start, c, scale, window,
                       seqs, key_block0, slices, part);
}

// dK/dV and dQ in one launch, the longer workgroups first: for chunks that are a few rounds of the chip, where each
// launch on its own leaves CUs idle at its end (AttnBackwardPlan).
template <int DH, bool SPLIT, bool IN_TURN>
__device__ __forceinline__ void bwd_block(const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v,
                                          const bf16_t* __restrict__ d_o, const float* __restrict__ lse, const float* __restrict__ lse2,
                                          const float* __restrict__ delta, bf16_t* __restrict__ dq, float* __restrict__ dk, float* __restrict__ dv,
                                          int Hq, int Hkv, int q_start, int c, float scale, const float2* __restrict__ rope, int window,
                                          const AttnSeqs& seqs, int key_block0, int key_blocks, int slices, float* __restrict__ part, int q_blocks, bool dq_first, bool side_by_side) {
  static_assert(AT_THREADS == KV_THREADS, "one workgroup shape");
  __shared__ __attribute__((aligned(1024))) union { DkvShared<DH> dkv; DqShared<DH, SPLIT> dq; } sh;
  const int kv_heads = Hkv * seqs.n, heads = Hq * seqs.n, n_dkv = key_blocks * kv_heads * (IN_TURN ? 2 : part ? slices : 1), n_dq = q_blocks * heads;
  const int b = dq_first ? ((int)blockIdx.x < n_dq ? (int)blockIdx.x + n_dkv : (int)blockIdx.x - n_dq) : (int)blockIdx.x;
  if (b < n_dkv) {
    // The key blocks that most queries see first (AttnBackwardPlan: side_by_side)
    const int of = side_by_side ? key_blocks : n_dkv / key_blocks, slow = __builtin_amdgcn_readfirstlane(b / of), fast = b - slow * of;
    const int r = side_by_side ? slow : fast;
    dkv_block<DH, IN_TURN>(sh.dkv, side_by_side ? fast : slow, r % kv_heads, r / kv_heads, q, k, v, d_o, lse2, delta, dk, dv, Hq, Hkv, q_start, c, scale, window, seqs,
                           key_block0, slices, part);
  } else {
    const int i = b - n_dkv;
    int qt = q_blocks - 1 - i / heads, bh = i % heads;      // less than a round: the tiles with the most keys first
    if (q_blocks * heads > 256) query_tile_of(i, q_blocks, heads, qt, bh);
    dq_tile<DH, SPLIT>(sh.dq, qt, bh, q, k, v, d_o, lse, delta, dq, Hq, Hkv, q_start, c, scale, rope, window, seqs);
  }
}
#define BWD_PARAMS const bf16_t *__restrict__ q, const bf16_t *__restrict__ k, const bf16_t *__restrict__ v, const bf16_t *__restrict__ d_o, \
                   const float *__restrict__ lse, const float *__restrict__ lse2, const float *__restrict__ delta, bf16_t *__restrict__ dq, \
                   float *__restrict__ dk, float *__restrict__ dv, int Hq, int Hkv, int q_start, int c, float scale, \
                   const float2 *__restrict__ rope, int window, const AttnSeqs seqs, int key_block0, int key_blocks, int slices, float *__restrict__ part, int q_blocks, bool dq_first, bool side_by_side
#define BWD_ARGS q, k, v, d_o, lse, lse2, delta, dq, dk, dv, Hq, Hkv, q_start, c, scale, rope, window, seqs, key_block0, key_blocks, slices, part, q_blocks, dq_first, side_by_side
template <int DH, bool SPLIT> __global__ __launch_bounds__(AT_THREADS) void attn_bwd_mfma_k(BWD_PARAMS) { bwd_block<DH, SPLIT, false>(BWD_ARGS); }
template <int DH, bool SPLIT> __global__ __launch_bounds__(AT_THREADS) void attn_bwd_in_turn_k(BWD_PARAMS) { bwd_block<DH, SPLIT, true>(BWD_ARGS); }
#undef BWD_PARAMS
#undef BWD_ARGS

// dk / dv += sum over the slices of the split form, in their order, keys from `first` on (blockIdx.y: sequence).  A thread takes elements e .. e + 3 and e + DH / 2 .. of a
// (key, head): what the rotary embedding pairs, so that the chunk's own rows, final with this call, leave as dkc = RoPE^T(dk) and dvc = dv
// too (optional).
template <int DH>
__global__ __launch_bounds__(256) void attn_dkv_sum_k(const float* __restrict__ part, int slices, int64_t pairs, int first, int Hkv, float* __restrict__ dk,
                                                      float* __restrict__ dv, int q_start, bf16_t* __restrict__ dkc, bf16_t* __restrict__ dvc,
                                                      const float2* __restrict__ rope) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;      // dk, then dv
  if (i >= 2 * pairs) return;
  const int64_t keys = first + pairs * 8 / ((int64_t)Hkv * DH), sq = blockIdx.y;      // of a sequence
  part += sq * slices * 2 * pairs * 8;
  dk += sq * keys * Hkv * DH; dv += sq * keys * Hkv * DH;
  if (dkc) { dkc += sq * (keys - q_start) * Hkv * DH; dvc += sq * (keys - q_start) * Hkv * DH; }
  const bool is_dk = i < pairs;
  const int64_t p = is_dk ? i : i - pairs, rh = p / (DH / 8);
  const int e = (int)(p % (DH / 8)) * 4;
  const int64_t at = rh * DH + e, n = pairs * 8;                  // floats of dk (and of dv)
  float* out = (is_dk ? dk : dv) + (int64_t)first * Hkv * DH + at;
  f32x4 x = *(const f32x4*)out, y = *(const f32x4*)(out + DH / 2);
  const float* src = part + (is_dk ? 0 : n) + at;
#pragma unroll 4
  for (int z = 0; z < slices; ++z) {
    x += *(const f32x4*)(src + z * 2 * n);
    y += *(const f32x4*)(src + z * 2 * n + DH / 2);
  }
  *(f32x4*)out = x;
  *(f32x4*)(out + DH / 2) = y;
  const int64_t row = first + rh / Hkv - q_start;
  if (!dkc || row < 0) return;
  bf16x4 u, w;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float2 cs = is_dk ? rope[row * (DH / 2) + e + r] : make_float2(1.f, 0.f);
    u[r] = (bf16_t)(is_dk ? x[r] * cs.x + y[r] * cs.y : x[r]);    // rotation by the negative angle
    w[r] = (bf16_t)(is_dk ? y[r] * cs.x - x[r] * cs.y : y[r]);
  }
  bf16_t* fin = (is_dk ? dkc : dvc) + (row * Hkv + rh % Hkv) * DH + e;
  *(bf16x4*)fin = u;
  *(bf16x4*)(fin + DH / 2) = w;
}

// delta[h, t] = sum_j d_o[t,h,j] * o[t,h,j]  (DH / 8 lanes per (t, h), 16 bytes of each tensor per lane)
// also lse2[h, t] = lse[h, t] * log2(e), the form the dK/dV kernel's exp2 wants (one multiply per (t, h) here
// instead of one per score there); 64-wide heads, whose exponents are natural differences: lse[h, t] itself
template <int DH>
__global__ __launch_bounds__(256) void attn_delta_mfma_k(const bf16_t* __restrict__ o, const bf16_t* __restrict__ d_o,
                                                         const float* __restrict__ lse, float* __restrict__ delta,
                                                         int Hq, int c) {
  constexpr int LANES = DH / 8;
  const int64_t first = (int64_t)blockIdx.y * c * Hq;      // blockIdx.y: sequence
  const int64_t pair = (int64_t)blockIdx.x * (256 / LANES) + threadIdx.x / LANES;      // t * Hq + h
  if (pair >= (int64_t)c * Hq) return;
  o += first * DH; d_o += first * DH; lse += first; delta += 2 * first;
  float* lse2 = delta + (int64_t)c * Hq;      // second half of the [2, Hq, c] scratch
  const int lane = threadIdx.x % LANES;
  const bf16x8 x = *(const bf16x8*)(o + pair * DH + lane * 8), y = *(const bf16x8*)(d_o + pair * DH + lane * 8);
  float s = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) s += (float)x[e] * (float)y[e];
#pragma unroll
  for (int off = LANES / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, WAVE);
  if (lane == 0) {
    const int t = (int)(pair / Hq), h = (int)(pair % Hq);
    delta[(int64_t)h * c + t] = s;
    const float l = lse[(int64_t)h * c + t];
    lse2[(int64_t)h * c + t] = l == -INFINITY ? 0.0f : FP32_STATS<DH> ? l : l * LOG2E;   // a query that saw no key: its scores are all masked anyway
  }
}

bool attn_mfma_eligible(int dt, int dh, int Hq, int Hkv) { return dt == DT_BF16 && (dh == 128 || dh == 64) && Hq % Hkv == 0; }

static bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

// the MFMA kernels move 16 bytes per lane: every tensor they touch must be 16-byte aligned
bool attn_mfma_aligned(const AttnArgs& a, bool backward) {
  if (!aligned16(a.q) || !aligned16(a.k) || !aligned16(a.v) || !aligned16(a.o) || !aligned16(a.dkv_scratch) || ((uintptr_t)a.rope_q & 7)) return false;
  return !backward || (aligned16(a.d_o) && aligned16(a.dq) && aligned16(a.dk) && aligned16(a.dv) && aligned16(a.dkc) && aligned16(a.dvc));
}

// Several sequences in one launch: with their first keys in its arguments, from the first position on.  A sequence of a batch of short ones is a
// fraction of a round of the chip: four of 640 tokens, 28 / 4 heads, forward, backward, delta and the sum of the parts 320 -> 210 us; with 2 x 1023
// tokens and 16 / 4 heads of 64 a stack of two layers 2290 -> 2130 us.
bool attn_sequences_fit(const AttnArgs& a) { return a.batch <= ATTN_MAX_SEQS && a.q_start == 0; }

static AttnSeqs sequences(const AttnArgs& a) {
  AttnSeqs s{};
  s.n = a.batch;
  for (int b = 0; b < a.batch; ++b) s.first[b] = a.kv_firsts ? a.kv_firsts[b] : a.kv_first;
  return s;
}
template <int DH>
static hipError_t forward_dh(const AttnArgs& a, hipStream_t st) {
  if (a.q_len == 0) return hipSuccess;
  const int64_t heads = (int64_t)a.Hq * a.batch, full = cdiv(a.q_len, TQ) * heads, halves = cdiv(a.q_len, TQ / 2) * heads;
  auto launch = [&](auto kernel, int64_t n) {
    kernel<<<(unsigned)n, AT_THREADS, 0, st>>>((bf16_t*)a.q, (const bf16_t*)a.k, (const bf16_t*)a.v, (bf16_t*)a.o, a.lse, a.Hq, a.Hkv,
                                               a.q_start, a.q_len, a.scale, a.rope_q, a.window, sequences(a));
  };
  if (attn_half_tiles_faster(a, attn_half_step_forward(DH))) launch(attn_fwd_mfma_k<DH, true>, halves);
  else launch(attn_fwd_mfma_k<DH, false>, full);
  return hipGetLastError();
}

template <int DH>
static hipError_t backward_dh(const AttnArgs& a, hipStream_t st) {
  if (a.q_len == 0) return hipSuccess;
  const int64_t pairs = (int64_t)a.q_len * a.Hq;
  const float* lse2 = a.delta + pairs;   // second half of the [2, Hq, c] scratch
  const AttnSeqs seqs = sequences(a);
  attn_delta_mfma_k<DH><<<dim3((unsigned)cdiv(pairs, 256 / (DH / 8)), a.batch), 256, 0, st>>>((const bf16_t*)a.o, (const bf16_t*)a.d_o, a.lse, a.delta, a.Hq,
                                                                                               a.q_len);
  const AttnBackwardPlan p = attn_backward_plan(a, MERGED_MAX, MERGED_MAX_PREFIX);
  const int slices = std::max(1, a.dkv_slices);
  float* part = p.parts ? a.dkv_scratch : nullptr;
  const bf16_t *q = (const bf16_t*)a.q, *k = (const bf16_t*)a.k, *v = (const bf16_t*)a.v, *d_o = (const bf16_t*)a.d_o;
  if (p.one_launch) {
    auto launch = [&](auto kernel) {
      kernel<<<(unsigned)(p.n_dkv + p.n_dq), AT_THREADS, 0, st>>>(q, k, v, d_o, a.lse, lse2, a.delta, (bf16_t*)a.dq, a.dk, a.dv, a.Hq, a.Hkv, a.q_start,
                                                                         a.q_len, a.scale, a.rope_q, a.window, seqs, p.key_block0, p.key_blocks, slices,
                                                                         part, p.q_blocks, p.dq_first, p.side_by_side);
    };
    if (p.in_turn && p.halves) launch(attn_bwd_in_turn_k<DH, true>);
    else if (p.in_turn) launch(attn_bwd_in_turn_k<DH, false>);
    else if (p.halves) launch(attn_bwd_mfma_k<DH, true>);
    else launch(attn_bwd_mfma_k<DH, false>);
  } else {
    auto launch_dq = [&](auto kernel) {
      kernel<<<(unsigned)p.n_dq, AT_THREADS, 0, st>>>(q, k, v, d_o, a.lse, a.delta, (bf16_t*)a.dq, a.Hq, a.Hkv, a.q_start, a.q_len, a.scale,
                                                                    a.rope_q, a.window, seqs, p.q_blocks);
    };
    if (p.halves) launch_dq(attn_bwd_dq_mfma_k<DH, true>);
    else launch_dq(attn_bwd_dq_mfma_k<DH, false>);
    if (p.n_dkv > 0)
      attn_bwd_dkv_mfma_k<DH><<<dim3((unsigned)p.key_blocks, a.Hkv * a.batch, part ? (unsigned)slices : 1u), KV_THREADS, 0, st>>>(
          q, k, v, d_o, lse2, a.delta, a.dk, a.dv, a.Hq, a.Hkv, a.q_start, a.q_len, a.scale, a.window, seqs, p.key_block0, slices, part);
  }
  if (part) {
    const int first = p.key_block0 * KV_TILE;
    const int64_t pairs = (int64_t)(a.q_start + a.q_len - first) * a.Hkv * (DH / 8);
    attn_dkv_sum_k<DH><<<dim3((unsigned)cdiv(2 * pairs, 256), a.batch), 256, 0, st>>>(part, slices, pairs, first, a.Hkv, a.dk, a.dv, a.q_start, (bf16_t*)a.dkc, (bf16_t*)a.dvc,
                                                                       a.rope_k);
    if (first <= a.q_start) return hipGetLastError();
  }
  if (a.dkc) {      // (also where some of the chunk's own keys, all hidden, come before the first visible block)
    hipError_t e = hipGetLastError();
    const int64_t own = (int64_t)a.q_len * a.Hkv * DH, keys = own + (int64_t)a.q_start * a.Hkv * DH;      // elements of a sequence's rows of the chunk, of all its keys
    for (int b = 0; b < a.batch && e == hipSuccess; ++b)
      e = kv_grad_finish(a.dt, a.dk + b * keys + (keys - own), a.dv + b * keys + (keys - own), a.rope_k, (bf16_t*)a.dkc + b * own, (bf16_t*)a.dvc + b * own, a.q_len, a.Hkv,
                         DH, st);
    return e;
  }
  return hipGetLastError();
}

hipError_t attn_forward_mfma(const AttnArgs& a, hipStream_t st) { return a.dh == 64 ? forward_dh<64>(a, st) : forward_dh<128>(a, st); }
hipError_t attn_backward_mfma(const AttnArgs& a, hipStream_t st) { return a.dh == 64 ? backward_dh<64>(a, st) : backward_dh<128>(a, st); }

}  // namespace sbp
