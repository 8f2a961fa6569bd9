// bf16 MFMA GEMM for outputs of few tiles, fp32 accumulation: C = sum over segments of A B^T (NT) or A B (NN), stored in fp32 or bf16.
//
// Where an output has fewer 256 x 256 tiles than the chip has CUs, gemm_mfma.hip splits the reduction over workgroups, and the
// fp32 partial tiles cost more than the product: 28 tiles split nine ways write and read 64 MB for a 512 x 3584 output, and
// a second launch adds them up.  Here the tiles are smaller (TM x TN of 64 or 128) and the reduction is split over the two
// halves of one workgroup, which meet in LDS.
#include "launch.h"
#include "gemm_tile.h"

#include <algorithm>

namespace sbp {

constexpr int FEW_THREADS = 512;       // two groups of four waves; waves w and w + 4 share a SIMD
constexpr int FEW_SEG = 3, FEW_PROBLEMS = 8;
struct FewSegment { const bf16_t* A; const bf16_t* B; int K, lda, ldb; };
struct FewProblem { FewSegment seg[FEW_SEG]; void* C; int nseg, M, N, tile_begin, tiles_m, tiles_n; int64_t ldc; };
struct FewArgs { FewProblem p[FEW_PROBLEMS]; int n, tiles; };

// Reduction-major operand of W = 128 or 64 columns: [64 k][W], 32-byte groups, group ^= f(k-row) (64 columns: two k-rows per 256 bytes)
template <int W> __device__ __forceinline__ int few_mn_swz(int krow) {
  return W == 128 ? mnmaj_swz(krow) : (((krow >> 1) & 1) | (((krow >> 3) & 1) << 1));
}

// One TM x TN tile.  Group g takes the K steps (BK = 64 or, for the smallest tile, 128 wide) t = g, g + 2, ...; a step is two slots, each closed by a barrier: fetch (LDS reads of
// all its fragments, the DMA of a later step) and multiply.  Group 1 runs one slot behind, so on every SIMD one wave multiplies while
// the other fetches, and a slot takes one K step forward.  The stages form a ring of NS steps (128 KB; 128 x 64 tiles: 144); step t + AHEAD is
// loaded in the fetch slot of step t, into the stage that the other group has left (its reads were waited for before the barrier in
// between), and has AHEAD - 1 slots to land.  Wave w of a group owns rows (w / 2) * TM / 2 and columns (w % 2) * TN / 2 of the tile.
template <int TM, int TN> constexpr int FEW_BK = TM * TN == 64 * 64 ? 128 : 64;

template <bool TB, int MODE, int TM, int TN>
__global__ __launch_bounds__(FEW_THREADS) void gemm_few_k(const FewArgs fa) {
  constexpr bool BMN = !TB;
  constexpr int BK = FEW_BK<TM, TN>, SUB = BK / 64;       // a step is SUB pieces of 64, each with its own layout
  constexpr int A_BYTES = TM * 64 * 2, B_BYTES = TN * 64 * 2, PIECE = A_BYTES + B_BYTES, STEP = SUB * PIECE;
  constexpr int NS = STEP == 32768 ? 4 : 6, AHEAD = NS - 1, NEWER = (AHEAD - 1) / 2;
  static_assert(AHEAD % 2 == 1, "a step is waited for by the group that loads it, one slot before it is read");
  constexpr int IA = TM / 32, JB = TN / 32;              // 16-row and 16-column blocks of a wave
  constexpr int LA = TM / 32, LB = TN / 32, LOADS = SUB * (LA + LB);   // 16-byte loads per thread of a group and piece / step
  constexpr int OUT_BYTES = MODE == 1 ? TM * TN * 2 : TM * TN * 4;
  constexpr int SMEM = std::max(NS * STEP, TM * TN * 4 + OUT_BYTES);
  __shared__ __attribute__((aligned(1024))) char smem[SMEM];

  const int id = xcd_contiguous_id((int)blockIdx.x, fa.tiles);
  int pi = 0;
#pragma unroll
  for (int i = 1; i < FEW_PROBLEMS; ++i)
    if (i < fa.n && id >= fa.p[i].tile_begin) pi = i;
  const FewProblem& g = fa.p[pi];
  int tm, tn;
  band_coords(id - g.tile_begin, g.tiles_m, g.tiles_n, band_height(g.tiles_m, g.tiles_m * g.tiles_n, true), tm, tn);
  const int m0 = tm * TM, n0 = tn * TN;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int grp = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1, tid = threadIdx.x & 255;

  const uint32_t lds0 = lds_addr(smem);
  const uint32_t dst = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)(tid & ~63) * 16u);
  // fragment addresses in stage 0: rows l % 16 of a 16-row block, k 8 (l / 16) .. + 7 of k32 step kk
  uint32_t fa_[2], fb[BMN ? JB * 2 : 2];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
    const int row = wm * (TM / 2) + (lane & 15);
    fa_[kk] = pin(lds0 + (uint32_t)(row * 128 + (((kk * 4 + (lane >> 4)) ^ kmaj_swz(row)) << 4)));
    if (!BMN) {
      const int rb = wn * (TN / 2) + (lane & 15);
      fb[kk] = pin(lds0 + A_BYTES + (uint32_t)(rb * 128 + (((kk * 4 + (lane >> 4)) ^ kmaj_swz(rb)) << 4)));
    }
  }
  if constexpr (BMN) {
#pragma unroll
    for (int x = 0; x < JB * 2; ++x) {      // [16-column block][k-rows + 0 / + 4]
      const int p = lane & 15, col = wn * (TN / 2) + (x >> 1) * 16 + 4 * (p & 3), krow = 8 * (lane >> 4) + (p >> 2) + 4 * (x & 1), c16 = col >> 3;
      const int p16 = (((c16 >> 1) ^ few_mn_swz<TN>(krow)) << 1) | (c16 & 1);
      fb[x] = pin(lds0 + A_BYTES + (uint32_t)(krow * TN * 2 + (p16 << 4) + ((col & 7) << 1)));
    }
  }

  // The loads of this group: every second step, one cursor over the segments
  const char *gA = nullptr, *gB = nullptr;
  uint32_t offA[LA], offB[LB];
  int seg = -1, ks = 0, nk = 0;               // segment, K step within it, its K steps
  int64_t pieceB = 128;                       // bytes
  auto enter = [&](int s) {
    seg = s;
    const FewSegment& q = g.seg[s];
    nk = q.K / BK;
    const int r_max = g.M - 1, c_max = g.N - 1;
#pragma unroll
    for (int i = 0; i < LA; ++i) {
      const int slot = i * 256 + tid, row = slot >> 3;
      offA[i] = (uint32_t)(((int64_t)(min(m0 + row, r_max) - m0) * q.lda + ((slot & 7) ^ kmaj_swz(row)) * 8) * 2);
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      const int slot = i * 256 + tid;
      if (!BMN) {
        const int row = slot >> 3;
        offB[i] = (uint32_t)(((int64_t)(min(n0 + row, c_max) - n0) * q.ldb + ((slot & 7) ^ kmaj_swz(row)) * 8) * 2);
      } else {
        const int krow = slot / (TN / 8), p16 = slot % (TN / 8), c16 = (((p16 >> 1) ^ few_mn_swz<TN>(krow)) << 1) | (p16 & 1);
        offB[i] = (uint32_t)(((int64_t)krow * q.ldb + min(c16 * 8, c_max - n0 - 7)) * 2);
      }
    }
    gA = uniform_ptr(q.A + (int64_t)m0 * q.lda);
    gB = uniform_ptr(q.B + (BMN ? (int64_t)n0 : (int64_t)n0 * q.ldb));
    if (BMN) pieceB = (int64_t)128 * q.ldb;
  };
  // move the cursor `by` steps on; false: past the end
  auto advance = [&](int by) {
    ks += by;
    while (ks >= nk) {
      ks -= nk;
      if (seg + 1 >= g.nseg) return false;
      enter(seg + 1);
    }
    return true;
  };
  auto issue = [&](uint32_t stage) {
#pragma unroll
    for (int u = 0; u < SUB; ++u) {
      const char* a = gA + (int64_t)(ks * SUB + u) * 128;
      const char* b = gB + (int64_t)(ks * SUB + u) * pieceB;
#pragma unroll
      for (int i = 0; i < LA; ++i) dma16(a, offA[i], dst + stage * STEP + u * PIECE + i * 4096);
#pragma unroll
      for (int i = 0; i < LB; ++i) dma16(b, offB[i], dst + stage * STEP + u * PIECE + A_BYTES + i * 4096);
    }
  };

  f32x4 acc[IA][JB];
#pragma unroll
  for (int i = 0; i < IA; ++i)
#pragma unroll
    for (int j = 0; j < JB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  int steps = 0;
  for (int i = 0; i < g.nseg; ++i) steps += g.seg[i].K / BK;
  // Prologue: steps 0 .. AHEAD - 1 as if loaded in slots -AHEAD .. -1, so group g loads the steps of parity 1 - g.
  const int first = 1 - grp;
  enter(0);
  bool more = advance(first);
#pragma unroll
  for (int t = 0; t < AHEAD; t += 2) {
    if (t + first < AHEAD && more) {
      issue((uint32_t)(t + first));
      more = advance(2);
    }
  }
  // at most `n` of this group's steps may still be in flight
  auto wait_newer = [&](int n) {
    if (n >= NEWER) WAIT_VMCNT(LOADS * NEWER);
    else if (NEWER > 2 && n == 2) WAIT_VMCNT(LOADS * 2);
    else if (NEWER > 1 && n == 1) WAIT_VMCNT(LOADS);
    else WAIT_VMCNT(0);
  };
  if (grp == 1) wait_newer(max(0, (steps - 1) / 2));     // step 0; newer: 2, 4, ..
  SLOT_BARRIER();
  if (grp == 1) SLOT_BARRIER();                           // group 1 falls one slot behind
  bf16x8 a[SUB][IA][2], b[SUB][JB][2];
  uint32_t rd = (uint32_t)grp, wr = (uint32_t)((grp + AHEAD) % NS);      // stages of the step fetched and of the step loaded
  for (int t = grp; t < steps; t += 2) {
    const uint32_t O = rd * STEP;
#pragma unroll
    for (int u = 0; u < SUB; ++u)
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const uint32_t P = O + u * PIECE;
#pragma unroll
        for (int i = 0; i < IA; ++i) a[u][i][kk] = lds_read_b128(fa_[kk] + P + i * 2048);
#pragma unroll
        for (int j = 0; j < JB; ++j)
          b[u][j][kk] = BMN ? lds_read_tr(fb[(j * 2) % (BMN ? JB * 2 : 2)] + P + kk * (32 * TN * 2), fb[(j * 2 + 1) % (BMN ? JB * 2 : 2)] + P + kk * (32 * TN * 2))
                            : lds_read_b128(fb[kk] + P + j * 2048);
      }
    if (more) {
      issue(wr);
      more = advance(2);
    }
    // step t + 1 was loaded by this group and is read by the other in the next slot; newer: t + 3, t + 5, .. as far as they exist
    wait_newer(max(0, (steps - 2 - t) / 2));
    WAIT_LDS();                                           // before the other group may refill the stage
    SLOT_BARRIER();
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int u = 0; u < SUB; ++u)
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int i = 0; i < IA; ++i)
#pragma unroll
          for (int j = 0; j < JB; ++j)                    // operands swapped: C^T blocks, a lane owns one row and four consecutive columns
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[u][j][kk], a[u][i][kk], acc[i][j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    SLOT_BARRIER();
    rd = (rd + 2) % NS;
    wr = (wr + 2) % NS;
  }
  if (grp == (steps & 1)) SLOT_BARRIER();                 // both groups have executed the same number of barriers

  // The halves of the reduction meet in LDS: a group keeps the row blocks i / (IA / 2) == g and gives the others away.
  constexpr int IH = IA / 2;
  f32x4* give = (f32x4*)smem + ((1 - grp) * 4 + (wave & 3)) * (IH * JB * 64) + lane;
  const f32x4* take = (const f32x4*)smem + (grp * 4 + (wave & 3)) * (IH * JB * 64) + lane;
#pragma unroll
  for (int i = 0; i < IH; ++i)
#pragma unroll
    for (int j = 0; j < JB; ++j) give[(i * JB + j) * 64] = grp == 0 ? acc[IH + i][j] : acc[i][j];
  __syncthreads();
  char* out = smem + TM * TN * 4;
#pragma unroll
  for (int i = 0; i < IH; ++i) {
    const int row = wm * (TM / 2) + (grp * IH + i) * 16 + (lane & 15);
#pragma unroll
    for (int j = 0; j < JB; ++j) {
      const f32x4 v = (grp == 0 ? acc[i][j] : acc[IH + i][j]) + take[(i * JB + j) * 64];
      const int col = wn * (TN / 2) + j * 16 + 4 * (lane >> 4);
      if constexpr (MODE == 1) {
        bf16x4 o;
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r] = (bf16_t)v[r];
        *(bf16x4*)(out + row * (TN * 2) + (((col >> 3) ^ (row & (TN / 8 - 1))) << 4) + ((col & 4) << 1)) = o;
      } else {
        *(f32x4*)(out + row * (TN * 4) + (((col >> 2) ^ (row & 15)) << 4)) = v;
      }
    }
  }
  __syncthreads();
  // whole rows, 16 bytes per lane
  constexpr int PER_ROW = MODE == 1 ? TN / 8 : TN / 4, PASSES = TM * PER_ROW / FEW_THREADS;
#pragma unroll
  for (int p = 0; p < PASSES; ++p) {
    const int slot = p * FEW_THREADS + (int)threadIdx.x, row = slot / PER_ROW, c = slot % PER_ROW;
    const int col = n0 + c * (MODE == 1 ? 8 : 4);
    const i32x4 v = *(const i32x4*)(out + row * (PER_ROW * 16) + ((c ^ (row & (MODE == 1 ? TN / 8 - 1 : 15))) << 4));
    if (m0 + row < g.M && col < g.N) {
      if constexpr (MODE == 1) *(i32x4*)((bf16_t*)g.C + (int64_t)(m0 + row) * g.ldc + col) = v;
      else *(i32x4*)((float*)g.C + (int64_t)(m0 + row) * g.ldc + col) = v;
    }
  }
}

// What gemm_few_k takes: C = A B^T or A B in bf16, whole K steps, 16-byte rows; C in fp32 or bf16
static bool few_operands_ok(const GemmArgs& g) {
  return g.in_dt == DT_BF16 && !g.ta && g.M >= 1 && g.N >= 8 && g.N % 8 == 0 && g.K >= 64 && g.K % 64 == 0 && g.lda % 8 == 0 && g.ldb % 8 == 0 &&
         g.lda < (1 << 22) && g.ldb < (1 << 22) && !((uintptr_t)g.A & 15) && !((uintptr_t)g.B & 15) && !((uintptr_t)g.C & 15) &&
         g.ldc % (g.out_dt == DT_BF16 ? 8 : 4) == 0;
}
static bool few_plain(const GemmArgs& g) { return !g.rows_dev && !g.row_stats && !g.numer_targets && !g.swiglu_gate && !g.glu_up && !g.C0; }
static bool few_segment(FewProblem& p, const GemmArgs& g, const void* A, const void* B) {
  if (p.nseg == FEW_SEG) return false;
  p.seg[p.nseg++] = FewSegment{(const bf16_t*)A, (const bf16_t*)B, g.K, (int)g.lda, (int)g.ldb};
  return true;
}

// sum = false: n <= 8 independent products (A2 / B2: a second reduction segment); sum = true: one product with n reduction segments, the
// first of which is stored and the others accumulated to the same C.
static bool few_args(const GemmArgs* gs, int n, bool sum, FewArgs& fa) {
  fa = FewArgs{};
  if (n < 1 || (!sum && n > FEW_PROBLEMS)) return false;
  for (int i = 0; i < n; ++i) {
    const GemmArgs& g = gs[i];
    if (!few_operands_ok(g) || !few_plain(g) || g.tb != gs[0].tb || g.out_dt != gs[0].out_dt) return false;
    if (sum ? g.A2 || g.acc != (i > 0) || g.C != gs[0].C || g.M != gs[0].M || g.N != gs[0].N || g.ldc != gs[0].ldc : g.acc) return false;
    if (g.A2 && (((uintptr_t)g.A2 & 15) || ((uintptr_t)g.B2 & 15))) return false;
    FewProblem& p = fa.p[sum ? 0 : i];
    if (!sum || i == 0) { p.C = g.C; p.M = g.M; p.N = g.N; p.ldc = g.ldc; }
    if (!few_segment(p, g, g.A, g.B) || (g.A2 && !few_segment(p, g, g.A2, g.B2))) return false;
  }
  fa.n = sum ? 1 : n;
  return true;
}
static int few_tiles(FewArgs& fa, int TM, int TN) {
  fa.tiles = 0;
  for (int i = 0; i < fa.n; ++i) {
    FewProblem& p = fa.p[i];
    p.tiles_m = (int)cdiv(p.M, TM); p.tiles_n = (int)cdiv(p.N, TN); p.tile_begin = fa.tiles;
    fa.tiles += p.tiles_m * p.tiles_n;
  }
  return fa.tiles;
}

// Which tile, and what it takes in us; tm = 0: not for these kernels.  A launch costs `fixed`, a 64-wide piece of the reduction `piece` where the
// weights (B, up to 8 MB) stay in the caches and `piece_mem` where they come from memory: the loads' latency, not their rate (511 x 1024
// outputs, K 1024 and 2816: 7.1 and 12.1 us with 64 x 64 tiles, 9.5 / 17.6 with 128 x 64, 11.3 / 21.0 with 128 x 128; 512 x 3584, K 3584, 25 MB of
// weights: 35.4 / 26.5 / 34.8; 1024 x 4096, K 4096: 75 / 57 / 39).
FewChoice gemm_few_choice(const GemmArgs* gs, int n, bool sum) {
  FewArgs fa;
  FewChoice best{0, 0, 0.0};
  for (int i = 0; i < n; ++i)
    if (!gs[i].few_ok) return best;
  if (!few_args(gs, n, sum, fa)) return best;
  int pieces = 0;
  bool even = true;
  double b_bytes = 0.0;
  for (int i = 0; i < fa.n; ++i) {
    int k = 0;
    for (int s = 0; s < fa.p[i].nseg; ++s) { k += fa.p[i].seg[s].K / 64; even = even && fa.p[i].seg[s].K % 128 == 0; }
    pieces = std::max(pieces, k);
    b_bytes = std::max(b_bytes, 128.0 * k * fa.p[i].N);
  }
  static const struct { int tm, tn; double fixed, piece, piece_mem; } forms[3] = {{128, 128, 5.8, 0.35, 0.52}, {128, 64, 4.9, 0.29, 0.385}, {64, 64, 4.3, 0.175, 0.265}};
  for (const auto& f : forms) {
    if (f.tm == 64 && !even) continue;
    const int tiles = few_tiles(fa, f.tm, f.tn), rounds = (int)cdiv(tiles, N_CU);
    const double us = f.fixed + rounds * pieces * (b_bytes > 8e6 ? f.piece_mem : f.piece) + 3.0 * (rounds - 1);
    if (!best.tm || us < best.us) best = FewChoice{f.tm, f.tn, us};
  }
  return best;
}

hipError_t gemm_few(const GemmArgs* gs, int n, bool sum, int TM, int TN, hipStream_t st) {
  FewArgs fa;
  if (!few_args(gs, n, sum, fa)) return hipErrorInvalidValue;
  if (!(TM == 128 && TN == 128) && !(TM == 128 && TN == 64) && !(TM == 64 && TN == 64)) return hipErrorInvalidValue;
  for (int i = 0; i < n; ++i)
    if (TM == 64 && gs[i].K % FEW_BK<64, 64> != 0) return hipErrorInvalidValue;
  const unsigned tiles = (unsigned)few_tiles(fa, TM, TN);
  auto go = [&](auto kernel) { kernel<<<tiles, FEW_THREADS, 0, st>>>(fa); };
#define FEW_TILE(TB, MODE)                                                \
  do {                                                                    \
    if (TM == 128 && TN == 128) go(gemm_few_k<TB, MODE, 128, 128>);       \
    else if (TM == 128) go(gemm_few_k<TB, MODE, 128, 64>);                \
    else go(gemm_few_k<TB, MODE, 64, 64>);                                \
  } while (0)
  const bool tb = gs[0].tb, bf = gs[0].out_dt == DT_BF16;
  if (tb && bf) FEW_TILE(true, 1);
  else if (tb) FEW_TILE(true, 0);
  else if (bf) FEW_TILE(false, 1);
  else FEW_TILE(false, 0);
#undef FEW_TILE
  return hipGetLastError();
}

}  // namespace sbp
