// bf16 MFMA GEMM for gfx950, fp32 accumulation, four operand layouts:
//   NT  C[M,N] = A[M,K] B[N,K]^T     (forward projections: both operands K-contiguous)
//   NN  C[M,N] = A[M,K] B[K,N]       (input gradients dX = dY W)
//   TN  C[M,N] = A[K,M]^T B[K,N]     (weight gradients dW += dY^T X; K = chunk rows)
//   TT  C[M,N] += A[K,M]^T B[N,K]^T  (the same from a transposed copy of X, where the caller keeps one)
//
// Design (CDNA4):
//  * 256x256 output tile per workgroup, 8 wavefronts in two groups of four that alternate between fetching and multiplying
//    (gemm_tile below); accumulators are 32 v_mfma_f32_16x16x32_bf16 blocks per wave (128 registers).
//  * Operand tiles (256 x 64 bf16 each) go HBM -> LDS with 128-bit direct-to-LDS loads (no VGPR staging), in halves of 128
//    rows, up to 80 KB of them in flight.
//  * K-contiguous operands are read from LDS with ds_read_b128; operands whose
//    reduction index is the slow dimension in memory are kept in their natural
//    [k][m|n] layout in LDS and fetched with the transposing LDS load
//    (ds_read_b64_tr_b16), so no transposed copy has to exist in HBM.
//  * Both LDS layouts are XOR-swizzled (at 16-byte / 32-byte granularity) so that
//    the fragment reads are bank-conflict free; because a direct-to-LDS load
//    writes lane-linear, the swizzle is applied on the global-address side.
//  * Workgroups are renumbered so that each XCD (own L2) works on a contiguous
//    band of output tiles that share operand panels.
//  * Ragged M (last chunk) and ragged N (an output width that is a multiple of 8 but not of 256, e.g. a 151936-word
//    vocabulary) are handled by clamping loads and masking stores;
//    ragged K (dW with a ragged chunk) by writing zeros instead of loading.
//  * Output tiles leave through LDS, so that C is written (or read, added to and written) in whole rows, 16 bytes per lane.
//  * Split-K for problems with too few output tiles to fill the chip: partial tiles go to
//    fp32 scratch and a small kernel sums them in a fixed order (deterministic) into C; the workgroups of a K slice are
//    numbered consecutively, so that an XCD holds one slice or a few.
//  * Weight gradients: C += acc, fp32 or bf16 C; several reduction segments (operand pairs) per output tile; grouped launches.
#include "launch.h"
#include "gemm_tile.h"

#include <algorithm>
#include <type_traits>

namespace sbp {

constexpr int BM = 256, BN = 256, BK = 64;
constexpr int NWAVE_N = 4;                             // waves along N; the two waves along M are the two groups of the main loop
constexpr int NTHREADS = 512;
constexpr int HALF_BYTES = 128 * BK * 2;               // 16 KiB: 128 rows (columns) of one operand, one K step
constexpr int STAGE_BYTES = 2 * HALF_BYTES;            // one operand, one K step
constexpr int OPERAND_BYTES = 2 * STAGE_BYTES;         // two K steps: 64 KiB, the reach of an LDS read's immediate offset
constexpr int SMEM_BYTES = 2 * OPERAND_BYTES;          // [operand][K step parity][half]

// Byte offset, relative to the tile's corner element, of load i (0, 1) of this thread's share of half h.
//   KMAJ : corner = (row r0, column k0); rows clamped so that r0 + row <= r_max
//   MNMAJ: corner = (k-row k0, column r0); columns clamped so that r0 + col <= r_max
template <bool MNMAJ>
__device__ __forceinline__ uint32_t load_offset(int i, int h, int64_t ld, int r0, int r_max) {
  const int id = i * NTHREADS + (int)threadIdx.x;   // 16-byte slot in the half tile, lane-linear within a wave
  if (!MNMAJ) {
    const int row = id >> 3, pc = id & 7;
    return (uint32_t)(((int64_t)(min(r0 + h * 128 + row, r_max) - r0) * ld + (pc ^ kmaj_swz(row)) * 8) * 2);
  } else {
    const int krow = id >> 4, p16 = id & 15;
    const int c16 = (((p16 >> 1) ^ mnmaj_swz(krow)) << 1) | (p16 & 1);
    // columns past the operand's last one (a ragged last tile; widths are multiples of 8) re-read its last 8 columns:
    // finite duplicates whose products land in rows / columns of C that the epilogue masks
    const int col = min(h * 128 + c16 * 8, r_max - r0 - 7);
    return (uint32_t)(((int64_t)krow * ld + col) * 2);
  }
}

// LDS byte offset (within a half tile) of this lane's fragment read of the 16 rows from row_base on.  A fragment is 16 rows x 32
// k: lane l holds row l % 16, k 8 (l / 16) .. + 7.  K-major: one 128-bit read per k32 step kk (row blocks 2048 B apart).
// Reduction-major: two transposing 64-bit reads (k-rows +0 and +4; k32 steps 8192 B apart).
__device__ __forceinline__ uint32_t frag_off_kmaj(int row_base, int kk) {
  const int l = threadIdx.x & 63, row = row_base + (l & 15);
  return (uint32_t)(row * (BK * 2) + (((kk * 4 + (l >> 4)) ^ kmaj_swz(row)) << 4));
}
__device__ __forceinline__ uint32_t frag_off_mnmaj(int col_base, int hi) {
  const int l = threadIdx.x & 63, p = l & 15, g = l >> 4;
  const int col = col_base + 4 * (p & 3), krow = 8 * g + (p >> 2) + 4 * hi, c16 = col >> 3;
  const int p16 = (((c16 >> 1) ^ mnmaj_swz(krow)) << 1) | (c16 & 1);
  return (uint32_t)(krow * 256 + (p16 << 4) + ((col & 7) << 1));
}
// One 256x256 output tile: K range [k_begin, k_end).
// MODE: 0 = store fp32, 1 = store bf16, 2 = accumulate fp32 (C +=),
//       4 = accumulate into a bf16 C (read, add in fp32, round once; weight-gradient form only),
//       5 = store fp32 and emit per-row (max, sum of exp) pairs over the tile's columns (`stats`)
//       6 = C is not stored: the tile is the gradient wrt act = silu(gate) * up and the epilogue writes act, d gate, d up
//       8 = C (bf16) receives silu(A B^T) * (A B2^T): 128 columns of each product per tile, in the halves of B
//       7 = like 5, but C (bf16) receives exp(c - block max) instead of c, and the value of each row's target column is kept
//       9 = like 2, through the caches (weight-gradient form of few tiles)
constexpr bool mode_accumulates(int mode) { return mode == 2 || mode == 4 || mode == 9; }
constexpr bool mode_splits(int mode) { return mode <= 2 || mode == 9; }      // forms whose reduction may be split over workgroups
// Floats of a partial tile: an output of fewer than 256 rows has partial tiles of as many (the scratch and its traffic shrink with it)
__host__ __device__ __forceinline__ int partial_floats(int max_m) { return (max_m < BM ? max_m : BM) * BN; }
struct SwigluFuse { bf16_t* gate; bf16_t* up; bf16_t* act; };
struct NumerFuse { const int32_t* targets; const int32_t* row_index; float* target_value; };
// The reduction may come in several segments (operand pairs of the same shape and leading dimensions whose products
// are summed into the same output tile): one accumulator, one epilogue.
constexpr int64_t NUMERATORS_CACHED = (256 << 20) / 2;      // elements of C (bf16) that the memory-side cache holds
// Up to so many tiles C += goes through the caches: an XCD then has four of them at most, 2 MB of its 4 MB L2, and the next launch that adds to C may find it there.  Past /
// through them, whole call, heads of 520 x 999, 12 tiles, 132 rows 60.8 / 59.1 us, a layer of 520 / 1378, products of 4 to 18 tiles, 264 / 259; of 5003 x 1024, 80 tiles, 118 / 126,
// of 16000 x 256, 63 tiles, 98 / 100.
constexpr int FEW_TILES = 32;
constexpr int MAX_SEG = 8;
struct KSegment {
  const bf16_t* A; const bf16_t* B;
  int k_begin, k_end;     // range of the reduction this tile works on
};

// Main loop.  The eight waves are two groups of four (waves w and w + 4 share a SIMD); wave (g, n) owns rows g*64 .. +63 and
// columns n*32 .. +31 of each of the four 128 x 128 quadrants of the tile.  A K step has four phases, one quadrant each (16
// v_mfma_f32_16x16x32_bf16 per wave), in the order (A0,B0) (A0,B1) (A1,B1) (A1,B0), so that each phase needs only one new operand
// half.  A phase is two slots, each closed by a barrier: fetch (LDS reads of the phase's fragments, the DMA of one half tile) and
// multiply.  Group 1 runs one slot behind group 0, so on every SIMD one wave multiplies while the other fetches: the matrix pipe
// does not wait for LDS reads, load issue or barriers.  The half read in phase p is refilled two phases later for the K step after
// next: five half tiles (80 KB) stay in flight and a load has six phases to land (a two-stage loop with one barrier and one burst
// of loads per K step waits for a whole tile's latency each time).  A refill may only be issued when both groups' reads of the half
// have returned, in a slot after a barrier that follows their waits.  A0, B1 and A1 are consumed, and with that waited for, in the
// multiply slot after their fetch.  B0 is fetched a phase early (phase 3, used in phase 0 of the next K step), where group 1 would
// wait for it in the very slot in which group 0 refills it: phase 0 therefore opens with a wait for it (two slots after the reads
// went out: nothing stalls).
// What bounds it: the matrix pipe at its power-limited clock.  8192^3 bf16, same card: NT 1265 -> 1556, NN 1256 -> 1546, TN 1199
// -> 1440 TFLOP/s (vendor library 1614 / 1390 / 1202); half of the gain is the slot schedule (1410 with 32x32x16 MFMAs), half the
// 16x16x32 MFMA.  With the wait for B0, on another card: 1559 / 1459 / 1329 (library 1550 / 1327 / 1180).
// The TN form is closest to the LDS limit (transposing reads of both operands); with B stored [N, K] (TT) 8192^3 takes 868 us against 909.
// No vector-ALU address work: global addresses are an SGPR base plus per-lane offsets computed once, LDS fragment
// addresses are computed once and reached with immediate offsets.
template <bool TA, bool TB, int MODE, typename SegmentF>
__device__ __forceinline__ void gemm_tile(int n_segments, SegmentF segment, void* __restrict__ Cv, int M, int N, int64_t lda,
                                          int64_t ldb, int64_t ldc, int tm, int tn, char* smem,
                                          float* __restrict__ partial = nullptr, int partial_bytes = 0, void* __restrict__ stats_out = nullptr,
                                          SwigluFuse sw = SwigluFuse{}, NumerFuse nf = NumerFuse{}, const void* __restrict__ C0 = nullptr,
                                          const bf16_t* __restrict__ Bu = nullptr) {
  constexpr bool AMN = TA, BMN = !TB;     // operand kept reduction-major in LDS (B stored [N,K] is the K-contiguous case)
  constexpr bool GLU = MODE == 8;
  const int m0 = tm * BM, n0 = tn * (GLU ? BN / 2 : BN);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int grp = wave / NWAVE_N, wn = wave % NWAVE_N;

  f32x4 acc[2][2][4][2];   // [A half][B half][16-row block][16-column block]: C^T blocks, lane l = row l % 16, columns 4 (l / 16) .. + 3
#pragma unroll
  for (int x = 0; x < 32; ++x)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[x >> 4][(x >> 3) & 1][(x >> 1) & 3][x & 1][r] = 0.f;

  // ---- global side: per-lane byte offsets (rows clamped once); the uniform 64-bit bases walk along K
  const int64_t stepA = (AMN ? (int64_t)BK * lda : (int64_t)BK) * 2, stepB = (BMN ? (int64_t)BK * ldb : (int64_t)BK) * 2;
  uint32_t offA[2][2], offB[2][2];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      offA[h][i] = pin(load_offset<AMN>(i, h, lda, m0, (AMN ? (M + 7) & ~7 : M) - 1));   // (padded A: whole 8-column granules)
      offB[h][i] = pin(load_offset<BMN>(i, GLU ? 0 : h, ldb, n0, N - 1));
    }
  const uint32_t lds0 = lds_addr(smem);
  const uint32_t lds_wave = __builtin_amdgcn_readfirstlane(lds0 + (uint32_t)(threadIdx.x & ~63) * 16u);

  // ---- LDS side: fragment addresses, computed once
  constexpr int NA = AMN ? 8 : 2, NB = BMN ? 4 : 2;
  uint32_t fa[NA], fb[NB];
#pragma unroll
  for (int x = 0; x < NA; ++x) fa[x] = pin(lds0 + (AMN ? frag_off_mnmaj(grp * 64 + (x >> 1) * 16, x & 1) : frag_off_kmaj(grp * 64, x)));
#pragma unroll
  for (int x = 0; x < NB; ++x)
    fb[x] = pin(lds0 + OPERAND_BYTES + (BMN ? frag_off_mnmaj(wn * 32 + (x >> 1) * 16, x & 1) : frag_off_kmaj(wn * 32, x)));
  bf16x8 a[4][2], bx[2][2], by[2][2];     // [16-row block][k32 step]; bx / by swap roles every K step
  using S0 = std::integral_constant<int, 0>;
  using S1 = std::integral_constant<int, 1>;

  for (int sg = 0; sg < n_segments; ++sg) {
    const KSegment seg = segment(sg);
    const int k_begin = seg.k_begin, k_end = seg.k_end;
    const int nk = (k_end - k_begin + BK - 1) / BK;
    if (nk <= 0) continue;
    const char* gA = uniform_ptr(seg.A + (AMN ? (int64_t)k_begin * lda + m0 : (int64_t)m0 * lda + k_begin));
    const char* gB = uniform_ptr(seg.B + (BMN ? (int64_t)k_begin * ldb + n0 : (int64_t)n0 * ldb + k_begin));
    const char* gB1 = GLU ? uniform_ptr(Bu + (int64_t)n0 * ldb + k_begin) : gB;      // second half
    // DMA of half h of K step kt (two 16-byte slots per thread).  Reduction rows past the end (the last K step of a ragged
    // reduction) are not loaded: the lane writes zeros into its slot instead.
    auto issue_half = [&](const char* base, const uint32_t (&off)[2], bool mnmaj, int kt, uint32_t dst) {
      const int k0 = k_begin + kt * BK;
      if (mnmaj && k0 + BK > k_end) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          if (k0 + i * 32 + (int)(threadIdx.x >> 4) < k_end) dma16(base, off[i], dst + i * (HALF_BYTES / 2));
          else *(__attribute__((address_space(3))) i32x4*)(uintptr_t)(dst + i * (HALF_BYTES / 2) + (threadIdx.x & 63) * 16) = i32x4{0, 0, 0, 0};
        }
      } else {
        dma16(base, off[0], dst);
        dma16(base, off[1], dst + HALF_BYTES / 2);
      }
    };
    const bool ragged = (AMN || BMN) && (k_end - k_begin) % BK != 0;
    const int n_tail = ragged ? 3 : 2;
    auto issue_a = [&](int h, int kt) {
      issue_half(gA + (int64_t)kt * stepA, offA[h], AMN, kt, lds_wave + (uint32_t)((kt & 1) * STAGE_BYTES + h * HALF_BYTES));
    };
    auto issue_b = [&](int h, int kt) {
      issue_half((h ? gB1 : gB) + (int64_t)kt * stepB, offB[h], BMN, kt, lds_wave + (uint32_t)(OPERAND_BYTES + (kt & 1) * STAGE_BYTES + h * HALF_BYTES));
    };
    auto read_a = [&](auto stage, int h) {
      const uint32_t O = decltype(stage)::value * STAGE_BYTES + h * HALF_BYTES;
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          a[i][kk] = AMN ? lds_read_tr(fa[(i * 2) % NA] + O + kk * 8192, fa[(i * 2 + 1) % NA] + O + kk * 8192)
                         : lds_read_b128(fa[kk] + O + i * 2048);
    };
    auto read_b = [&](auto stage, int h, bf16x8 (&b)[2][2]) {
      const uint32_t O = decltype(stage)::value * STAGE_BYTES + h * HALF_BYTES;
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          b[j][kk] = BMN ? lds_read_tr(fb[(j * 2) % NB] + O + kk * 8192, fb[(j * 2 + 1) % NB] + O + kk * 8192)
                         : lds_read_b128(fb[kk] + O + j * 2048);
    };
    auto multiply = [&](int ha, int hb, bf16x8 (&b)[2][2]) {
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)     // operands swapped: C^T blocks, a lane owns one row and four consecutive columns
            acc[ha][hb][i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j][kk], a[i][kk], acc[ha][hb][i][j], 0, 0, 0);
    };
    // A half is waited for one phase before it is read (each wave waits for its own share, the barriers in between cover the
    // others'): in the steady state the ten youngest loads (five halves) may still be outstanding; the last two K steps
    // issue no more loads and count down.  A wave may skip loads of a ragged last K step, so from their issue on nothing is counted.
    auto k_step = [&](auto stage, int kt, bf16x8 (&bc)[2][2], bf16x8 (&bn)[2][2]) __attribute__((always_inline)) {
      constexpr int S = decltype(stage)::value;
      using Next = std::integral_constant<int, 1 - S>;
      const int rem = nk - 1 - kt;
#define WAIT_TAIL(penultimate, last)                  \
  do {                                                \
    if (rem >= n_tail) WAIT_VMCNT(10);                \
    else if (ragged) WAIT_VMCNT(0);                   \
    else if (rem == 1) WAIT_VMCNT(penultimate);       \
    else WAIT_VMCNT(last);                            \
  } while (0)
      WAIT_LDS();                         // B0 is in registers: the other group refills its half in the slot after next
      read_a(stage, 0);
      if (rem >= 1) issue_a(1, kt + 1);
      WAIT_TAIL(10, 2);
      SLOT_BARRIER(); multiply(0, 0, bc); SLOT_BARRIER();
      read_b(stage, 1, bn);
      if (rem >= 2) issue_b(0, kt + 2);
      WAIT_TAIL(8, 0);
      SLOT_BARRIER(); multiply(0, 1, bn); SLOT_BARRIER();
      read_a(stage, 1);
      if (rem >= 2) issue_a(0, kt + 2);
      WAIT_TAIL(6, 0);
      SLOT_BARRIER(); multiply(1, 1, bn); SLOT_BARRIER();
      read_b(Next{}, 0, bn);              // B0 of the next K step (a harmless read after the last one)
      if (rem >= 2) issue_b(1, kt + 2);
      WAIT_TAIL(4, 0);
      SLOT_BARRIER(); multiply(1, 0, bc); SLOT_BARRIER();
#undef WAIT_TAIL
    };
    if (sg > 0) __syncthreads();     // everyone is done reading the stages of the previous segment
    issue_b(0, 0); issue_a(0, 0); issue_b(1, 0); issue_a(1, 0);
    if (nk > 1) { issue_b(0, 1); issue_a(0, 1); issue_b(1, 1); if (nk > 2 || !ragged) WAIT_VMCNT(10); } else WAIT_VMCNT(4);
    if (ragged && nk <= 2) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");   // (lgkmcnt: the zeros written in place of rows past the end)
    SLOT_BARRIER();
    read_b(S0{}, 0, bx);
    if (grp == 1) SLOT_BARRIER();    // group 1 falls one slot behind ...
    const int nk_even = nk & ~1;
    for (int kt = 0; kt < nk_even; kt += 2) {
      k_step(S0{}, kt, bx, by);
      k_step(S1{}, kt + 1, by, bx);
    }
    if (nk & 1) k_step(S0{}, nk - 1, bx, by);
    WAIT_LDS();                      // (the read of B0 past the last K step: the next segment's loads refill the stage)
    if (grp == 0) SLOT_BARRIER();    // ... and group 0 waits for it here: both execute the same number of barriers
  }

  // Epilogue.  A lane holds, per (A half ha, block i), row ha*128 + grp*64 + i*16 + l%16 of the tile and, per (B half hb, block j),
  // its columns hb*128 + wn*32 + j*16 + 4 (l/16) .. + 3.
  float* Cf = (float*)Cv;
  bf16_t* Cb = (bf16_t*)Cv;
  auto row_of = [&](int ha, int i) { return ha * 128 + grp * 64 + i * 16 + (lane & 15); };
  auto col_of = [&](int hb, int j) { return hb * 128 + wn * 32 + j * 16 + 4 * (lane >> 4); };
  // Plain stores go through LDS (free once every wave has left the main loop), so that a wave writes whole rows of C, 16 bytes
  // per lane: storing from the accumulator layout directly (32-byte pieces of 16 rows per instruction) measured 2-5 % slower
  // over the whole product at K = 3584.
  if constexpr (mode_splits(MODE)) {
    if (partial) {     // a slice of the reduction: the fp32 tile, masked and combined by splitk_tail_k
      // stores past the end of a partial tile of fewer than 256 rows fall outside the buffer and are dropped: a branch per row
      // in their place made every split product 0.5 us slower (small model, 64 of 16 us each)
      __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(partial, 0, partial_bytes, 0x00027000);
#pragma unroll
      for (int ha = 0; ha < 2; ++ha) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int hb = 0; hb < 2; ++hb)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
              const int row = row_of(0, i), col = col_of(hb, j);
              *(f32x4*)(smem + row * 1024 + (((col >> 2) ^ (row & 15)) << 4)) = acc[ha][hb][i][j];
            }
        __syncthreads();
        const int c4 = threadIdx.x & 63;
        // an output narrower than a tile: without the columns that it does not have (2048 x 32 x 18944, 176 tiles 32.4 -> 29.8 us); a wider one's are few tiles of many
        const int past = N < BN && c4 * 4 >= N ? 0x40000000 : 0;
#pragma unroll
        for (int p = 0; p < 16; ++p) {
          const int row_l = p * 8 + (threadIdx.x >> 6);
          const f32x4 v = *(const f32x4*)(smem + row_l * 1024 + ((c4 ^ (row_l & 15)) << 4));
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), out, past + ((ha * 128 + row_l) * BN + c4 * 4) * 4, 0, 0);
        }
      }
      return;
    }
  }
  if constexpr (MODE == 1) {
    __syncthreads();
#pragma unroll
    for (int ha = 0; ha < 2; ++ha)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int hb = 0; hb < 2; ++hb)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int row = row_of(ha, i), col = col_of(hb, j);
            bf16x4 o;
#pragma unroll
            for (int r = 0; r < 4; ++r) o[r] = (bf16_t)acc[ha][hb][i][j][r];
            *(bf16x4*)(smem + row * 512 + (((col >> 3) ^ (row & 15)) << 4) + ((col & 4) << 1)) = o;
          }
      }
    __syncthreads();
    const int c16 = threadIdx.x & 31, col = n0 + c16 * 8;
#pragma unroll
    for (int p = 0; p < 16; ++p) {
      const int row = p * 16 + (threadIdx.x >> 5);
      const i32x4 v = *(const i32x4*)(smem + row * 512 + ((c16 ^ (row & 15)) << 4));
      if (m0 + row < M && col < N) *(i32x4*)(Cb + (int64_t)(m0 + row) * ldc + col) = v;
    }
    return;
  }
  if constexpr (GLU) {
    // Gate and up of a column are the same registers of the two halves.  Against storing both and reading them again (2048 x 18944 x 3584: 430 us
    // and 37 for the elementwise pass) the product is bound as before and the pass is gone: forward of 8192 rows, four chunks, 4.02 -> 3.81 ms.
    __syncthreads();
#pragma unroll
    for (int ha = 0; ha < 2; ++ha)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int row = row_of(ha, i), col = col_of(0, j);
          bf16x4 o;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float z = acc[ha][0][i][j][r];
            o[r] = (bf16_t)(z / (1.0f + __expf(-z)) * acc[ha][1][i][j][r]);
          }
          *(bf16x4*)(smem + row * 256 + (((col >> 3) ^ (row & 15)) << 4) + ((col & 4) << 1)) = o;
        }
    __syncthreads();
    const int c16 = threadIdx.x & 15, col = n0 + c16 * 8;
#pragma unroll
    for (int p = 0; p < 8; ++p) {
      const int row = p * 32 + (threadIdx.x >> 4);
      const i32x4 v = *(const i32x4*)(smem + row * 256 + ((c16 ^ (row & 15)) << 4));
      if (m0 + row < M && col < N) *(i32x4*)(Cb + (int64_t)(m0 + row) * ldc + col) = v;
    }
    return;
  }
  if constexpr (MODE == 0 || MODE == 4) {
    // fp32 rows: one half of the tile's rows at a time (128 KB)
#pragma unroll
    for (int ha = 0; ha < 2; ++ha) {
      __syncthreads();
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int hb = 0; hb < 2; ++hb)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int row = row_of(0, i), col = col_of(hb, j);
            *(f32x4*)(smem + row * 1024 + (((col >> 2) ^ (row & 15)) << 4)) = acc[ha][hb][i][j];
          }
      __syncthreads();
      if constexpr (MODE == 4) {
        // bf16 C += acc: every element has exactly one owner per launch; the sum is formed in fp32 and rounded once.  The loads
        // of C (16 bytes per lane), or of the C0 that it starts from, go out before the first use.  (C0: a copy of 24 us before and 39 us of
        // product per 18944 x 3584 matrix, 222 us for seven matrices in one launch now.)
        const bf16_t* from = C0 ? (const bf16_t*)C0 : Cb;
        const int c8 = threadIdx.x & 31, col = n0 + c8 * 8;
        bf16x8 old[8];
#pragma unroll
        for (int p = 0; p < 8; ++p) {
          const int row = m0 + ha * 128 + p * 16 + (threadIdx.x >> 5);
          if (row < M && col < N) old[p] = *(const bf16x8*)(from + (int64_t)row * ldc + col);
        }
#pragma unroll
        for (int p = 0; p < 8; ++p) {
          const int row_l = p * 16 + (threadIdx.x >> 5), row = m0 + ha * 128 + row_l;
          const f32x4 lo = *(const f32x4*)(smem + row_l * 1024 + (((c8 * 2) ^ (row_l & 15)) << 4));
          const f32x4 hi = *(const f32x4*)(smem + row_l * 1024 + (((c8 * 2 + 1) ^ (row_l & 15)) << 4));
          bf16x8 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) { o[e] = (bf16_t)((float)old[p][e] + lo[e]); o[e + 4] = (bf16_t)((float)old[p][e + 4] + hi[e]); }
          if (row < M && col < N) *(bf16x8*)(Cb + (int64_t)row * ldc + col) = o;
        }
      } else {
        const int c4 = threadIdx.x & 63, col = n0 + c4 * 4;
#pragma unroll
        for (int p = 0; p < 16; ++p) {
          const int row_l = p * 8 + (threadIdx.x >> 6), row = m0 + ha * 128 + row_l;
          const f32x4 v = *(const f32x4*)(smem + row_l * 1024 + ((c4 ^ (row_l & 15)) << 4));
          if (row < M && col < N) *(f32x4*)(Cf + (int64_t)row * ldc + col) = v;
        }
      }
    }
    return;
  }
  if constexpr (MODE == 2 || MODE == 9) {
    // fp32 C += acc, half of the tile's rows at a time: a plain read-modify-write, every element has one owner per launch.  What bounds it is
    // the latency of the reads of C, not their rate: those of a half (16 accesses of 16 bytes per lane) all go out before the half is
    // staged, the second half's before the first is added.  Against eight at a time behind the staging: 18944 x 3584, K = 128 134 -> 103
    // us, K = 1024 253 -> 227; 152064 x 3584, K = 1536 2207 -> 2108, K = 16384 14.90 -> 14.74 ms.  (fp32 atomic adds without return cost 1721
    // instead of 1139 us where the pass over C dominates - 152064 x 3584, K = 512 - and the same at K >= 8192; the same form for bf16
    // C, which has half the bytes to wait for: 2 % faster at K = 512, 1-4 % slower from K = 4096 on.)
    // C is touched once: the accesses are non-temporal, so that its 512 KB per tile do not push the operand panels that the XCD's other tiles share out
    // of the L2.  Seven gradients of a 7B layer, 0.93 GB, K = 2048 1040 -> 997 us, 2560 1264 -> 1238, 8192 the same; 152064 x 3584, K = 1536 1996
    // -> 1921 (the loads alone 1001, 1937).  The bf16 form, the plain stores and the elementwise passes gain nothing or lose (SwiGLU adjoint 70 -> 79 us: its
    // tensors are in the memory-side cache).  A dword of every 128 bytes of C asked for two K steps ahead: 1040 -> 1130.
    const int c4 = threadIdx.x & 63, r0 = threadIdx.x >> 6;
    const char* base = uniform_ptr(Cf + (int64_t)m0 * ldc + n0);
    const uint32_t lane_off = (uint32_t)((r0 * ldc + c4 * 4) * 4);
    const bool col_in = n0 + c4 * 4 < N;
    const int rows_in = M - m0 - r0;      // rows of this lane's passes that exist
    f32x4 old[2][16];
    auto at = [&](int ha, int p) { return (f32x4*)(base + (int64_t)(ha * 128 + p * 8) * ldc * 4 + lane_off); };
    auto inside = [&](int ha, int p) { return ha * 128 + p * 8 < rows_in && col_in; };
    auto fetch = [&](int ha) {
#pragma unroll
      for (int p = 0; p < 16; ++p)
        if (inside(ha, p)) old[ha][p] = MODE == 2 ? __builtin_nontemporal_load(at(ha, p)) : *at(ha, p);
    };
    fetch(0);
#pragma unroll
    for (int ha = 0; ha < 2; ++ha) {
      WAIT_LDS();
      SLOT_BARRIER();
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int hb = 0; hb < 2; ++hb)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int row = row_of(0, i), cl = col_of(hb, j);
            *(f32x4*)(smem + row * 1024 + (((cl >> 2) ^ (row & 15)) << 4)) = acc[ha][hb][i][j];
          }
      WAIT_LDS();
      SLOT_BARRIER();
      if (ha == 0) fetch(1);
#pragma unroll
      for (int p = 0; p < 16; ++p) {
        const int row_l = p * 8 + r0;
        const f32x4 v = *(const f32x4*)(smem + row_l * 1024 + ((c4 ^ (row_l & 15)) << 4));
        if (!inside(ha, p)) continue;
        if (MODE == 2) __builtin_nontemporal_store(old[ha][p] + v, at(ha, p));
        else *at(ha, p) = old[ha][p] + v;
      }
    }
    return;
  }
  if constexpr (MODE == 5 || MODE == 7) {
    float2* stats = (float2*)stats_out;
    // Row statistics for a softmax over the columns of C: every row of the tile gets (max, sum of exp(c - max)) over
    // the tile's 256 columns - in-lane over the lane's 16 columns, two lane exchanges, and the NWAVE_N waves that share a row
    // meet in LDS (free once every wave has left the main loop).
    // MODE 5 stores C in fp32.  MODE 7 stores softmax numerators (Sec. 5 names fused backward operators as the way to cut the
    // per-chunk HBM passes): what the row kernel after the logits GEMM needs of a row is exp(c - lse), and exp(c - max of the
    // 256-column block) differs from it by one factor per block - so the tile stores that, in bf16; the sum is taken from the
    // unrounded values.  The logit of each row's target column, which the loss needs exactly, is kept in fp32 on the side.
    // The numerators leave through LDS in whole rows, 16 bytes per lane, as the plain stores do, and the target columns are looked up for all
    // of a lane's rows at once: 2048 x 152064 x 3584 1.75 -> 1.64 ms against 8-byte stores from the accumulator layout and a
    // dependent pair of loads per row.
    __syncthreads();
    float* pmax = (float*)(smem + (MODE == 7 ? SMEM_BYTES : 0));      // [NWAVE_N][BM]
    float* psum = pmax + NWAVE_N * BM;         // [NWAVE_N][BM]
    constexpr float LOG2E = 1.4426950408889634f;
    int d[2][4];                               // MODE 7: target column of the lane's rows, relative to the tile
    if constexpr (MODE == 7) {
#pragma unroll
      for (int x = 0; x < 8; ++x) {
        const int row = min(m0 + row_of(x >> 2, x & 3), M - 1);
        d[x >> 2][x & 3] = nf.row_index ? nf.row_index[row] : row;
      }
#pragma unroll
      for (int x = 0; x < 8; ++x) d[x >> 2][x & 3] = nf.targets[d[x >> 2][x & 3]] - n0;
    }
#pragma unroll
    for (int ha = 0; ha < 2; ++ha)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row_l = row_of(ha, i), row = m0 + row_l;
        float mx = -INFINITY;
#pragma unroll
        for (int hb = 0; hb < 2; ++hb)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int col = col_of(hb, j);
            if (MODE == 5 && row < M && n0 + col < N) *(f32x4*)(Cf + (int64_t)row * ldc + n0 + col) = acc[ha][hb][i][j];
            if (n0 + col + 3 >= N) {           // ragged last column tile: columns past N take no part
#pragma unroll
              for (int r = 0; r < 4; ++r) acc[ha][hb][i][j][r] = n0 + col + r < N ? acc[ha][hb][i][j][r] : -INFINITY;
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) mx = fmaxf(mx, acc[ha][hb][i][j][r]);
            if constexpr (MODE == 7) {
              const int r = d[ha][i] - col;    // which of the four, if any, is the target's
              if (row < M && (uint32_t)r < 4u && n0 + d[ha][i] < N) {
                const f32x4 v = acc[ha][hb][i][j];
                nf.target_value[row] = r == 0 ? v[0] : r == 1 ? v[1] : r == 2 ? v[2] : v[3];
              }
            }
          }
        mx = fmaxf(mx, __shfl_xor(mx, 16, WAVE));
        mx = fmaxf(mx, __shfl_xor(mx, 32, WAVE));
        if (lane < 16) pmax[wn * BM + row_l] = mx;
      }
    __syncthreads();
#pragma unroll
    for (int ha = 0; ha < 2; ++ha)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row_l = row_of(ha, i);
        float m = pmax[row_l];
#pragma unroll
        for (int w = 1; w < NWAVE_N; ++w) m = fmaxf(m, pmax[w * BM + row_l]);   // finite: wave 0 always holds valid columns
        float se = 0.f;
#pragma unroll
        for (int hb = 0; hb < 2; ++hb)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int col = col_of(hb, j);
            bf16x4 o;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float ex = __builtin_amdgcn_exp2f((acc[ha][hb][i][j][r] - m) * LOG2E);   // difference first: exact near the maximum
              se += ex;
              o[r] = (bf16_t)ex;
            }
            if (MODE == 7) *(bf16x4*)(smem + row_l * 512 + (((col >> 3) ^ (row_l & 15)) << 4) + ((col & 4) << 1)) = o;
          }
        se += __shfl_xor(se, 16, WAVE);
        se += __shfl_xor(se, 32, WAVE);
        if (lane < 16) psum[wn * BM + row_l] = se;
      }
    __syncthreads();
    if constexpr (MODE == 7) {
      const int c16 = threadIdx.x & 31, col = n0 + c16 * 8;
      // Past the caches, as for C += above, where the memory-side cache does not hold all of C for the pass that reads it next: 2048 rows of 152064 1627 -> 1605 us.
      // Where it does, the pass finds it there, whole call, past / into the caches: 100352 columns, hidden 256, 100 rows (20 MB) 199 / 192 us, 1000 (200 MB) 447 / 425; 50256,
      // hidden 1024, 1000 rows 500 / 490, 2048 (206 MB) 783 / 790; 151936, hidden 3584, 1000 (304 MB) 3706 / 3720.
      const bool past_caches = (int64_t)M * ldc > NUMERATORS_CACHED;
#pragma unroll
      for (int p = 0; p < 16; ++p) {
        const int row = p * 16 + (threadIdx.x >> 5);
        const i32x4 v = *(const i32x4*)(smem + row * 512 + ((c16 ^ (row & 15)) << 4));
        if (m0 + row < M && col < N) {
          if (ldc % 8 == 0 && past_caches) __builtin_nontemporal_store(v, (i32x4*)(Cb + (int64_t)(m0 + row) * ldc + col));
          else if (ldc % 8 == 0) *(i32x4*)(Cb + (int64_t)(m0 + row) * ldc + col) = v;
          else {                               // (rows that start between 16-byte boundaries: half of them at a time)
            typedef int i32x2 __attribute__((ext_vector_type(2)));
            *(i32x2*)(Cb + (int64_t)(m0 + row) * ldc + col) = i32x2{v[0], v[1]};
            *(i32x2*)(Cb + (int64_t)(m0 + row) * ldc + col + 4) = i32x2{v[2], v[3]};
          }
        }
      }
    }
    if ((int)threadIdx.x < BM && m0 + (int)threadIdx.x < M) {
      float m = pmax[threadIdx.x], sum = psum[threadIdx.x];
#pragma unroll
      for (int w = 1; w < NWAVE_N; ++w) { m = fmaxf(m, pmax[w * BM + threadIdx.x]); sum += psum[w * BM + threadIdx.x]; }
      stats[(int64_t)(m0 + (int)threadIdx.x) * ((N + BN - 1) / BN) + tn] = make_float2(m, sum);
    }
    return;
  }
  if constexpr (MODE == 6) {
    // SwiGLU adjoint on the accumulators (Sec. 5 names fused backward operators as the way to cut the per-chunk HBM
    // passes): 8-byte accesses to gate / up / act.  Every element has exactly one owner, so gate and up are rewritten in place.
#pragma unroll
    for (int ha = 0; ha < 2; ++ha)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = m0 + row_of(ha, i);
        if (row >= M) continue;
        bf16x4 gv[2][2], uv[2][2];
#pragma unroll
        for (int hb = 0; hb < 2; ++hb)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int col = n0 + col_of(hb, j);
            gv[hb][j] = col < N ? *(const bf16x4*)(sw.gate + (int64_t)row * ldc + col) : bf16x4{};
            uv[hb][j] = col < N ? *(const bf16x4*)(sw.up + (int64_t)row * ldc + col) : bf16x4{};
          }
#pragma unroll
        for (int hb = 0; hb < 2; ++hb)
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const int col = n0 + col_of(hb, j);
            if (col >= N) continue;
            bf16x4 a4, dg4, du4;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float z = (float)gv[hb][j][e], u = (float)uv[hb][j][e], d = acc[ha][hb][i][j][e];
              const float sg = 1.0f / (1.0f + __expf(-z));
              a4[e] = (bf16_t)(z * sg * u);
              dg4[e] = (bf16_t)(d * u * sg * (1.0f + z * (1.0f - sg)));
              du4[e] = (bf16_t)(d * z * sg);
            }
            const int64_t idx = (int64_t)row * ldc + col;
            if (sw.act) *(bf16x4*)(sw.act + idx) = a4;
            *(bf16x4*)(sw.gate + idx) = dg4;
            *(bf16x4*)(sw.up + idx) = du4;
          }
      }
  }
}

// How the tiles of a launch are spread over the 256 CUs (one workgroup each): whole rounds of 256 tiles first, each tile by one
// workgroup; the reduction of the tiles that are left over (or of all of them, where there are fewer than 256) is split
// `splits` ways, so that the last round is not mostly idle.  Split tiles go to fp32 scratch and are summed in a fixed order.
// The number of splits weighs the K steps saved against what the partial tiles cost: about 3.5 K steps for the extra launch
// and 0.09 K step per partial tile (256 KB written and read back at ~4.5 TB/s against 1.45 us per K step).  Up to 27 splits: eight
// tiles with the reduction of a 50257-word vocabulary, or 28 with that of two MLP widths, would keep most CUs idle with four.
constexpr int MAX_SPLITS = 27;        // the numbers tried: 2 .. 8, 10, 12, 15, 18, 22, 27
struct Schedule { int tiles, full, tail, splits; };
__host__ __device__ __forceinline__ Schedule make_schedule(int tiles, int k_steps, int scratch_tiles) {
  const int tail = tiles % N_CU;
  int best = 1;
  if (tail > 0) {
    float gain = 0.f;
    for (int s = 2; s <= MAX_SPLITS && s * tail <= N_CU && s * tail <= scratch_tiles && k_steps / s >= 4; s += s < 8 ? 1 : s / 4) {
      const float g = (float)(k_steps - (k_steps + s - 1) / s) - 3.5f - 0.09f * (float)(s * tail);
      if (g > gain) { gain = g; best = s; }
    }
  }
  return best > 1 ? Schedule{tiles, tiles - tail, tail, best} : Schedule{tiles, tiles, 0, 1};
}
// The other way to fill the last round, for fp32 stores whose sizes the host knows and 129 to 160 tiles left over, which no whole number of splits
// fits: each of these `tail` tiles keeps a workgroup of its own, which stops after `main` K steps and stores to C, and the `helpers` CUs without
// a tile form the `rest` of the reductions.  First of a tile each, in step with their neighbours, so that they share operand panels in their L2;
// then of the `last` tiles, in `parts` pieces each.  Each piece is a workgroup, dispatched as CUs become free, and leaves a partial tile
// (at most one per CU in all), which shared_tail_k adds to C in the order of the reduction.
// What bounds it: the clock, which falls as more CUs multiply (a K step of 140 tiles takes 1.18 us, of 252 1.52), and the sum.  Whole product, tiles
// unshared / shared, 3584 columns, K = 2 x 18944: 140 tiles 683 / 570 us, 154 691 / 628, 406 1615 / 1521 (126, in two splits, 575); K = 18944: 140 319 /
// 274, 154 326 / 307; 4096 columns, K = 2 x 14336: 144 530 / 445, 160 537 / 500; 2048 columns, K = 2 x 5632: 136 215 / 195.  From 168 tiles on, where
// a helper takes the rest of two tiles and more, it loses: 168 724 / 814, 196 780 / 846.
struct SharedTail { int full, tail, main, rest, helpers, last, parts; };
constexpr int SHARED_TAIL_MAX = 160, SHARED_PARTS = 8;
__host__ __device__ __forceinline__ int shared_pieces(const SharedTail& sh) { return sh.helpers + sh.last * sh.parts; }
// Cost in K steps as for the splits above: 5 for the start and the end of the second piece, 3.5 for the launch of the sum and 0.09 per tile written
// and read, C itself among them.
static bool shared_schedule(int tiles, int k_steps, int scratch_tiles, SharedTail& sh) {
  const int tail = tiles % N_CU;
  if (2 * tail <= N_CU || tail > SHARED_TAIL_MAX || scratch_tiles < N_CU) return false;
  sh.full = tiles - tail; sh.tail = tail;
  sh.helpers = N_CU - tail; sh.last = tail - sh.helpers;
  sh.parts = std::min(sh.helpers / sh.last, SHARED_PARTS);
  sh.rest = (int)((k_steps - 5) / (2.0 + 1.0 / sh.parts));
  sh.main = k_steps - sh.rest;
  if (sh.rest < 32) return false;
  sh.parts = (int)cdiv(sh.rest, cdiv(sh.rest, sh.parts));      // as many as pieces of that length make: none without a step (33 steps: seven of five, not eight)
  return sh.rest - 3.5 - 0.09 * (shared_pieces(sh) + tail) > 0.0;
}
// Workgroup -> (tile, split); false: nothing to do
__device__ __forceinline__ bool scheduled_tile(const Schedule& sc, int block, bool interleaved, int& tile, int& split) {
  split = 0;
  if (block < sc.full) { tile = interleaved ? block : xcd_contiguous_id(block, sc.full); return true; }
  const int q = block - sc.full;
  if (q >= sc.tail * sc.splits) return false;
  const int c = xcd_contiguous_id(q, sc.tail * sc.splits);      // an XCD works on one slice of the reduction (its share of K stays in its L2)
  split = c / sc.tail;
  tile = sc.full + c % sc.tail;
  return true;
}

template <bool TA, bool TB, int MODE>
__global__ __launch_bounds__(NTHREADS) void gemm_mfma_k(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B,
                                                        void* __restrict__ Cv, int M, int N, int K, int64_t lda,
                                                        int64_t ldb, int64_t ldc, const int* __restrict__ rows_dev,
                                                        const bf16_t* __restrict__ A2, const bf16_t* __restrict__ B2,
                                                        float* __restrict__ scratch, int scratch_tiles, void* __restrict__ row_stats,
                                                        SwigluFuse sw, NumerFuse nf, const void* __restrict__ C0) {
  __shared__ __attribute__((aligned(1024))) char smem[SMEM_BYTES + (MODE == 7 ? 2 * NWAVE_N * BM * 4 : 0)];
  const int part = partial_floats(M);
  if (rows_dev) {                     // run-time row count: rows are M (NT / NN) or the reduction K (dW form)
    const int rows = max(0, *rows_dev);
    if (TA) K = min(K, rows); else M = min(M, rows);
  }
  constexpr int WIDE = MODE == 8 ? BN / 2 : BN;
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + WIDE - 1) / WIDE, k_steps = (K + BK - 1) / BK;
  const int all_steps = A2 ? 2 * k_steps : k_steps;          // two operand pairs: their reductions follow one another
  if (mode_accumulates(MODE) && all_steps == 0) return;      // nothing to add
  const Schedule sc = make_schedule(tiles_m * tiles_n, all_steps, mode_splits(MODE) ? scratch_tiles : 0);
  int tile, split, tm, tn;
  if (!scheduled_tile(sc, blockIdx.x, mode_accumulates(MODE), tile, split)) return;
  band_coords(tile, tiles_m, tiles_n, band_height(tiles_m, sc.tiles, !mode_accumulates(MODE)), tm, tn);
  int s0 = 0, s1 = all_steps;
  float* partial = nullptr;
  if (tile >= sc.full) {
    const int per = (all_steps + sc.splits - 1) / sc.splits;
    s0 = split * per;
    s1 = min(all_steps, s0 + per);
    partial = scratch + ((int64_t)split * sc.tail + (tile - sc.full)) * part;
  }
  auto segment = [&](int i) {
    const int b = max(s0 - i * k_steps, 0) * BK, e = min(min(s1 - i * k_steps, k_steps) * BK, K);
    return KSegment{i ? A2 : A, i ? B2 : B, b, e};
  };
  gemm_tile<TA, TB, MODE>(A2 ? 2 : 1, segment, Cv, M, N, lda, ldb, ldc, tm, tn, smem, partial, part * 4, row_stats, sw, nf, C0, MODE == 8 ? B2 : nullptr);
}

// C = A B (TB: B^T stored), fp32, the last round of tiles shared (SharedTail)
template <bool TB>
__global__ __launch_bounds__(NTHREADS) void gemm_mfma_shared_k(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, float* __restrict__ C, int M, int N, int K,
                                                               int64_t lda, int64_t ldb, int64_t ldc, const bf16_t* __restrict__ A2,
                                                               const bf16_t* __restrict__ B2, float* __restrict__ scratch, const SharedTail sh) {
  __shared__ __attribute__((aligned(1024))) char smem[SMEM_BYTES];
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN, k_steps = (K + BK - 1) / BK, part = partial_floats(M);
  const int all_steps = A2 ? 2 * k_steps : k_steps, q = (int)blockIdx.x - sh.full, p = q - sh.tail;
  int tile, s0 = 0, s1 = all_steps;
  float* partial = nullptr;
  if (q < 0) tile = xcd_contiguous_id(blockIdx.x, sh.full);
  else if (p < 0) { tile = sh.full + xcd_contiguous_id(q, sh.tail); s1 = sh.main; }
  else {
    int t, slot;
    s0 = sh.main;
    if (p < sh.helpers) t = slot = xcd_contiguous_id(p, sh.helpers);
    else {      // piece of a last tile
      const int i = p - sh.helpers, u = i % sh.last, piece = i / sh.last, per = (sh.rest + sh.parts - 1) / sh.parts;
      t = sh.helpers + u;
      slot = sh.helpers + u * sh.parts + piece;
      s0 += piece * per;
      s1 = min(all_steps, s0 + per);
    }
    tile = sh.full + t;
    partial = scratch + (int64_t)slot * part;
  }
  int tm, tn;
  band_coords(tile, tiles_m, tiles_n, band_height(tiles_m, tiles_m * tiles_n, true), tm, tn);
  auto segment = [&](int i) {
    const int b = max(s0 - i * k_steps, 0) * BK, e = min(min(s1 - i * k_steps, k_steps) * BK, K);
    return KSegment{i ? A2 : A, i ? B2 : B, b, e};
  };
  gemm_tile<false, TB, 0>(A2 ? 2 : 1, segment, C, M, N, lda, ldb, ldc, tm, tn, smem, partial, part * 4);
}
// C += the pieces of its tiles (64 workgroups each) in the order of the reduction
__global__ __launch_bounds__(256) void shared_tail_k(const SharedTail sh, const float* __restrict__ scratch, float* __restrict__ C, int M, int N, int64_t ldc) {
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN, part = partial_floats(M);
  const int t = blockIdx.x / 64, u = t - sh.helpers;
  int tm, tn;
  band_coords(sh.full + t, tiles_m, tiles_n, band_height(tiles_m, tiles_m * tiles_n, true), tm, tn);
  const int row_l = (blockIdx.x % 64) * 4 + (threadIdx.x >> 6), col_l = 4 * (threadIdx.x & 63), row = tm * BM + row_l, col = tn * BN + col_l;
  if (row >= M || col >= N) return;
  const int first = u < 0 ? t : sh.helpers + u * sh.parts, n = u < 0 ? 1 : sh.parts;
  float* c = C + (int64_t)row * ldc + col;
  const float* src = scratch + (int64_t)first * part + row_l * BN + col_l;
  f32x4 v = *(const f32x4*)c, in[SHARED_PARTS];
#pragma unroll
  for (int z = 0; z < SHARED_PARTS; ++z)
    if (z < n) in[z] = *(const f32x4*)(src + (int64_t)z * part);
#pragma unroll
  for (int z = 0; z < SHARED_PARTS; ++z)
    if (z < n) v += in[z];
  *(f32x4*)c = v;
}

// Weight-gradient form with a segmented reduction: C += sum_s A_s^T B_s (TB: B_s^T stored), every segment with its own run-time row
// count.  One pass over C for several chunks' worth of rows.
struct SegLaunch { const bf16_t* A[MAX_SEG]; const bf16_t* B[MAX_SEG]; const int* rows_dev[MAX_SEG]; int K[MAX_SEG]; int n; };
template <bool C_BF16, bool TB>
__global__ __launch_bounds__(NTHREADS) void gemm_mfma_seg_k(const SegLaunch sl, void* __restrict__ C, int M, int N, int64_t lda,
                                                            int64_t ldb, int64_t ldc) {
  __shared__ __attribute__((aligned(1024))) char smem[SMEM_BYTES];
  const int tiles_m = (M + BM - 1) / BM, tiles_n = (N + BN - 1) / BN;
  int tm, tn;
  band_coords((int)blockIdx.x, tiles_m, tiles_n, band_height(tiles_m, tiles_m * tiles_n, false), tm, tn);
  auto rows = [&](int i) { return sl.rows_dev[i] ? min(sl.K[i], max(0, *sl.rows_dev[i])) : sl.K[i]; };
  int total = 0;
  for (int i = 0; i < sl.n; ++i) total += rows(i);
  if (total == 0) return;   // nothing to add
  gemm_tile<true, TB, C_BF16 ? 4 : 2>(sl.n, [&](int i) { return KSegment{sl.A[i], sl.B[i], 0, rows(i)}; }, C, M, N, lda, ldb,
                                         ldc, tm, tn, smem);
}

// Several independent GEMMs of one layout / output mode in a single launch: the tiles of all problems form one
// grid, so small problems fill the tail of large ones instead of each paying its own partial last round.
constexpr int MAX_GROUP = 8;
constexpr int MAX_GSEG = MAX_SEG;   // reduction segments per grouped problem (accumulate form: several chunks' operands)
struct GroupProblem {
  const bf16_t* A[MAX_GSEG]; const bf16_t* B[MAX_GSEG]; void* C; const void* C0;
  int M, N, K[MAX_GSEG], nseg;
  int64_t lda, ldb, ldc;
  int tile_begin, tiles_m, tiles_n;
};
struct GroupArgs { GroupProblem p[MAX_GROUP]; int n; Schedule sched; float* scratch; int part; };     // part: floats of a partial tile

template <bool TA, bool TB, int MODE>
__global__ __launch_bounds__(NTHREADS) void gemm_mfma_group_k(const GroupArgs ga) {
  __shared__ __attribute__((aligned(1024))) char smem[SMEM_BYTES];
  int id, split;
  if (!scheduled_tile(ga.sched, blockIdx.x, mode_accumulates(MODE), id, split)) return;
  int pi = 0;
#pragma unroll
  for (int i = 1; i < MAX_GROUP; ++i)
    if (i < ga.n && id >= ga.p[i].tile_begin) pi = i;
  const GroupProblem& g = ga.p[pi];
  int tm, tn;
  band_coords(id - g.tile_begin, g.tiles_m, g.tiles_n, band_height(g.tiles_m, g.tiles_m * g.tiles_n, !mode_accumulates(MODE)), tm, tn);
  int b = 0, e = 0x7fffffff;
  float* partial = nullptr;
  if (mode_splits(MODE) && id >= ga.sched.full) {     // (split launches have one reduction segment per problem)
    const int k_steps = (g.K[0] + BK - 1) / BK, per = (k_steps + ga.sched.splits - 1) / ga.sched.splits;
    b = split * per * BK;
    e = b + per * BK;
    partial = ga.scratch + ((int64_t)split * ga.sched.tail + (id - ga.sched.full)) * ga.part;
  }
  gemm_tile<TA, TB, MODE>(mode_accumulates(MODE) ? g.nseg : 1, [&](int i) { return KSegment{g.A[i], g.B[i], b, min(e, g.K[i])}; }, g.C, g.M, g.N,
                          g.lda, g.ldb, g.ldc, tm, tn, smem, partial, ga.part * 4, nullptr, SwigluFuse{}, NumerFuse{}, MODE == 4 ? g.C0 : nullptr);
}

// The tiles whose reduction was split: C (=|+=) sum of the partial tiles in a fixed order, rounded once.  Few tiles of many parts are bound by the
// latency of the parts' reads: up to TAIL_AHEAD of them are under way at once, and a tile is dealt to 64 workgroups (one access per lane and part)
// where 16 per tile, four accesses per lane one after the other, would leave CUs idle (8 tiles of 27 parts 34.8 -> 12.5 us; 112 of 2: 15.7 both).
constexpr int TAIL_AHEAD = 8;
struct TailProblem { void* C; int M, N; int64_t ldc; int tile_begin, tiles_m, tiles_n; };
struct TailArgs {
  TailProblem p[MAX_GROUP];
  int n;
  Schedule sched;
  const int* rows_dev;          // run-time row count of p[0] (single problems): the schedule is then made again from it
  int K;                        // > 0: rows_dev counts the reduction, of at most K rows (weight gradients)
  int k_steps, scratch_tiles;
  const float* scratch;
  int part;                     // floats of a partial tile
  int blocks;                   // workgroups per tile: 16 or 64
};
template <int MODE>
__global__ __launch_bounds__(256) void splitk_tail_k(const TailArgs ta) {
  Schedule sc = ta.sched;
  int M0 = ta.p[0].M, tiles_m0 = ta.p[0].tiles_m;
  if (ta.rows_dev) {
    int k_steps = ta.k_steps;
    if (ta.K > 0) k_steps = (min(ta.K, max(0, *ta.rows_dev)) + BK - 1) / BK;
    else M0 = min(M0, max(0, *ta.rows_dev));
    tiles_m0 = (M0 + BM - 1) / BM;
    sc = make_schedule(tiles_m0 * ta.p[0].tiles_n, k_steps, ta.scratch_tiles);
  }
  const int t = blockIdx.x / ta.blocks, block = blockIdx.x % ta.blocks;
  if (t >= sc.tail) return;
  const int id = sc.full + t;
  int pi = 0;
  for (int i = 1; i < ta.n; ++i)
    if (id >= ta.p[i].tile_begin) pi = i;
  const TailProblem& g = ta.p[pi];
  const int M = pi == 0 ? M0 : g.M, tiles_m = pi == 0 ? tiles_m0 : g.tiles_m;
  int tm, tn;
  band_coords(id - g.tile_begin, tiles_m, g.tiles_n, band_height(tiles_m, tiles_m * g.tiles_n, !mode_accumulates(MODE)), tm, tn);
  const int col_l = 4 * (threadIdx.x & 63), col = tn * BN + col_l;
  for (int row_l = block * 4 + (threadIdx.x >> 6); row_l < BM; row_l += ta.blocks * 4) {
    const int row = tm * BM + row_l;
    if (row >= M || col >= g.N) continue;
    const float* src = ta.scratch + (int64_t)t * ta.part + row_l * BN + col_l;
    const int64_t step = (int64_t)sc.tail * ta.part;
    f32x4 v = {0.f, 0.f, 0.f, 0.f}, in[TAIL_AHEAD];
    for (int z0 = 0; z0 < sc.splits; z0 += TAIL_AHEAD) {
#pragma unroll
      for (int z = 0; z < TAIL_AHEAD; ++z)
        if (z0 + z < sc.splits) in[z] = *(const f32x4*)(src + (z0 + z) * step);
#pragma unroll
      for (int z = 0; z < TAIL_AHEAD; ++z)
        if (z0 + z < sc.splits) v = z0 + z == 0 ? in[z] : v + in[z];
    }
    if constexpr (MODE == 1) {
      bf16x4 o;
#pragma unroll
      for (int r = 0; r < 4; ++r) o[r] = (bf16_t)v[r];
      *(bf16x4*)((bf16_t*)g.C + (int64_t)row * g.ldc + col) = o;
    } else {
      f32x4* c = (f32x4*)((float*)g.C + (int64_t)row * g.ldc + col);
      if (MODE == 2) v += *c;
      *c = v;
    }
  }
}

bool gemm_mfma_eligible(const GemmArgs& g) {
  if (g.in_dt != DT_BF16) return false;
  if (g.acc && g.out_dt != DT_F32 && !(g.out_dt == DT_BF16 && g.ta)) return false;   // bf16 C += : dW forms only
  // Output widths need not be multiples of the 256-wide tile: a ragged last tile clamps its loads and masks its stores
  // (16-byte granules: multiples of 8 elements), e.g. a 151936-word vocabulary = 593.5 tiles.
  if (g.M < 1 || g.N < 1 || g.K < 1) return false;
  if (g.N % 8 != 0 && !(g.c_padded && !g.ta && g.tb && !g.acc && g.ldc % 8 == 0 && g.ldc >= g.N)) return false;
  if (g.ta && !g.tb) {                       // TN: both operands reduction-major; ragged K allowed
    if (g.M % 8 != 0 && !g.a_padded) return false;
  } else if (!g.ta) {                        // NT / NN; a ragged K needs B reduction-major and A's rows padded with zeros
    if (g.K % BK != 0 && (g.tb || !g.a_padded)) return false;
  } else {                                   // TT: weight gradients only, B^T stored; a ragged K needs B's rows padded
    if (!g.acc || g.A2 || (g.M % 8 != 0 && !g.a_padded) || (g.K % BK != 0 && !g.b_padded)) return false;
  }
  if (g.lda % 8 || g.ldb % 8) return false;
  if (g.lda >= (1 << 22) || g.ldb >= (1 << 22)) return false;   // per-lane byte offsets within a tile are 32-bit
  if (((uintptr_t)g.A & 15) || ((uintptr_t)g.B & 15) || ((uintptr_t)g.C & 15) || ((uintptr_t)g.C0 & 15)) return false;
  if (g.C0 && !(g.acc && g.out_dt == DT_BF16)) return false;
  // fp32 rows, the softmax numerators and the fused SwiGLU adjoint move 4 elements at a time, plain and accumulated bf16 rows 8
  return g.ldc % (g.out_dt == DT_BF16 && !g.numer_targets && !g.swiglu_gate ? 8 : 4) == 0;
}

// the operand-pair form: two reductions, one after the other, in one accumulator
bool gemm_mfma_pair_ok(const GemmArgs& g) { return g.A2 && g.B2 && !g.ta && !((uintptr_t)g.A2 & 15) && !((uintptr_t)g.B2 & 15); }

// the fused SwiGLU adjoint exists for the store form C = A B (input-gradient layout), bf16 tensors that share C's layout
bool gemm_mfma_swiglu_ok(const GemmArgs& g) {
  return g.swiglu_gate && g.swiglu_up && !g.ta && !g.tb && !g.acc && !g.A2 && !g.row_stats && g.ldc % 4 == 0 &&
         !((uintptr_t)g.swiglu_gate & 7) && !((uintptr_t)g.swiglu_up & 7) && !((uintptr_t)g.swiglu_act & 7);
}

// the row-statistics epilogue exists for the fp32 store form of C = A B^T
bool gemm_mfma_stats_ok(const GemmArgs& g) {
  return !g.ta && g.tb && g.out_dt == DT_F32 && !g.acc && !g.A2 && !((uintptr_t)g.row_stats & 7) && !g.numer_targets;
}

// ... and its softmax-numerator variant for a bf16 C
bool gemm_mfma_numer_ok(const GemmArgs& g) {
  return !g.ta && g.tb && g.out_dt == DT_BF16 && !g.acc && !g.A2 && g.row_stats && !((uintptr_t)g.row_stats & 7) &&
         g.numer_targets && g.numer_target_value && !g.swiglu_gate;
}

size_t gemm_scratch_bytes(int max_m, int max_n) {
  // partial tiles: at most one per CU is ever useful
  const int64_t tiles = cdiv(max_m, BM) * cdiv(max_n, BN);
  return (size_t)std::min<int64_t>(N_CU, tiles * MAX_SPLITS) * partial_floats(max_m) * sizeof(float);
}
static int scratch_tiles_of(const GemmArgs& g, int max_m) {
  return g.scratch && !((uintptr_t)g.scratch & 15) ? (int)std::min<size_t>(N_CU, g.scratch_bytes / (partial_floats(max_m) * sizeof(float))) : 0;
}
// fp32 store of one product (or pair) with the sizes on the host
static bool shares_tail(const GemmArgs& g, int scratch_tiles, SharedTail& sh) {
  return !g.ta && !g.acc && g.out_dt == DT_F32 && !g.rows_dev && !g.glu_up && !g.numer_targets && !g.row_stats && !g.swiglu_gate &&
         shared_schedule((int)(cdiv(g.M, BM) * cdiv(g.N, BN)), (int)cdiv(g.K, BK) * (g.A2 ? 2 : 1), scratch_tiles, sh);
}
static hipError_t launch_tail(int mode, TailArgs t, int max_tail, hipStream_t st) {
  t.blocks = max_tail < 64 ? 64 : 16;
  const unsigned blocks = (unsigned)(max_tail * t.blocks);
  if (mode == 0) splitk_tail_k<0><<<blocks, 256, 0, st>>>(t);
  else if (mode == 1) splitk_tail_k<1><<<blocks, 256, 0, st>>>(t);
  else splitk_tail_k<2><<<blocks, 256, 0, st>>>(t);
  return hipGetLastError();
}

// Estimated time in us of a launch of `tiles` 256 x 256 tiles, for the choice between these kernels and those of gemm_few.hip: a K step takes
// 1.2 us (1.35 where all CUs multiply), a launch 5 us; one with split tiles 14, 0.3 per split and 0.055 per partial tile of 256
// rows that is written and read.  Measured / estimated: 511 x 1024 x 1024 20.5 / 21.9, 512 x 3584 x 3584 35.0 / 38.9, 1024 x 4096 x 4096 48.8 / 50.9,
// 2048 x 3584 x 3584 61.1 / 64.7, 512 x 18944 x 3584 85 / 78.
static double launch_us(int tiles, int k_steps, int scratch_tiles, int max_m) {
  const Schedule sc = make_schedule(tiles, k_steps, scratch_tiles);
  const double step = 1.2 + 0.15 * std::min(1.0, (double)tiles * sc.splits / N_CU);
  const double whole = (double)cdiv(sc.full, N_CU) * k_steps * step;
  return sc.splits == 1 ? 5.0 + whole
                        : 14.0 + 0.3 * sc.splits + whole + (double)cdiv(k_steps, sc.splits) * step + 0.055 * sc.tail * sc.splits * partial_floats(max_m) / (BM * BN);
}
double gemm_mfma_us(const GemmArgs* gs, int n) {      // n > 1: one grouped launch
  int tiles = 0, k = 0, max_m = 0;
  for (int i = 0; i < n; ++i) {
    tiles += (int)(cdiv(gs[i].M, BM) * cdiv(gs[i].N, BN));
    k = std::max(k, (int)cdiv(gs[i].K, BK) * (gs[i].A2 ? 2 : 1));
    max_m = std::max(max_m, gs[i].M);
  }
  const int scratch_tiles = scratch_tiles_of(gs[0], max_m);
  if (SharedTail sh; n == 1 && shares_tail(gs[0], scratch_tiles, sh))
    return 14.0 + 1.35 * ((double)(sh.full / N_CU) * k + sh.main) + 0.055 * (shared_pieces(sh) + sh.tail);
  return launch_us(tiles, k, scratch_tiles, max_m);
}

// C = silu(A B^T) * (A glu_up^T): from as many tiles on as a grouped launch of both products takes.  Whole forward of a layer in one chunk, this form / the
// products apart: 44 tiles 1.09, 88 0.95-0.97, 112 0.97-1.06, 132 to 198 0.84-0.87, 220 to 444 0.95-1.065 (512 rows at 3584 x 18944, 296 tiles in two rounds, 356
// us against 335; before this form 386).
bool gemm_mfma_glu_ok(const GemmArgs& g) {
  return g.glu_up && !g.ta && g.tb && !g.acc && g.out_dt == DT_BF16 && !g.A2 && !g.row_stats && !g.numer_targets && !g.swiglu_gate && !g.rows_dev &&
         !((uintptr_t)g.glu_up & 15) && cdiv(g.M, BM) * cdiv(g.N, BN / 2) >= 200;
}

hipError_t gemm_mfma(const GemmArgs& g, hipStream_t st) {
  const int tiles_m = (int)cdiv(g.M, BM), tiles_n = (int)cdiv(g.N, g.glu_up ? BN / 2 : BN);
  const int k_steps = (int)cdiv(g.K, BK) * (g.A2 ? 2 : 1);
  const int mode = g.glu_up ? 8 : g.numer_targets ? 7 : g.row_stats ? 5 : g.swiglu_gate ? 6
                 : g.acc ? (g.out_dt == DT_BF16 ? 4 : 2) : (g.out_dt == DT_BF16 ? 1 : 0);
  const bool dev_rows = g.rows_dev != nullptr;
  int scratch_tiles = mode_splits(mode) ? scratch_tiles_of(g, g.M) : 0;
  // (a run-time reduction: split at most where its largest length is)
  if (g.ta && dev_rows && make_schedule(tiles_m * tiles_n, k_steps, scratch_tiles).splits == 1) scratch_tiles = 0;
  if (SharedTail sh; shares_tail(g, scratch_tiles, sh)) {
    {
      prof::Scope sc_time(prof::GEMM_SINGLE + (g.tb ? 0 : 4), 2.0 * g.M * g.N * g.K * (g.A2 ? 2 : 1), false, st);
      auto launch = [&](auto kernel) {
        kernel<<<(unsigned)(sh.full + sh.tail + shared_pieces(sh)), NTHREADS, 0, st>>>((const bf16_t*)g.A, (const bf16_t*)g.B, (float*)g.C, g.M, g.N, g.K, g.lda, g.ldb, g.ldc,
                                                                (const bf16_t*)g.A2, (const bf16_t*)g.B2, g.scratch, sh);
      };
      if (g.tb) launch(gemm_mfma_shared_k<true>);
      else launch(gemm_mfma_shared_k<false>);
    }
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) shared_tail_k<<<(unsigned)sh.tail * 64, 256, 0, st>>>(sh, g.scratch, (float*)g.C, g.M, g.N, g.ldc);
    return e != hipSuccess ? e : hipGetLastError();
  }
  const Schedule sc = make_schedule(tiles_m * tiles_n, k_steps, scratch_tiles);
  // with a run-time row count the schedule is made on the device: room for any tail
  const unsigned grid = dev_rows && scratch_tiles ? (unsigned)(tiles_m * tiles_n + N_CU) : (unsigned)(sc.full + sc.tail * sc.splits);
  const bool may_split = dev_rows ? scratch_tiles >= 2 : sc.splits > 1;
#define LAUNCH(TA, TB, MODE) \
  gemm_mfma_k<TA, TB, MODE><<<grid, NTHREADS, 0, st>>>((const bf16_t*)g.A, (const bf16_t*)g.B, g.C, g.M, g.N, g.K, g.lda, g.ldb, g.ldc, g.rows_dev, \
                                                       (const bf16_t*)g.A2, (const bf16_t*)(g.glu_up ? g.glu_up : g.B2), g.scratch, scratch_tiles, \
                                                       (void*)g.row_stats, \
                                                       SwigluFuse{(bf16_t*)g.swiglu_gate, (bf16_t*)g.swiglu_up, (bf16_t*)g.swiglu_act}, \
                                                       NumerFuse{g.numer_targets, g.numer_row_index, g.numer_target_value}, g.C0)
#define LAUNCH_LAYOUT(MODE)                       \
  do {                                            \
    if (!g.ta && g.tb) LAUNCH(false, true, MODE); \
    else if (!g.ta && !g.tb) LAUNCH(false, false, MODE); \
    else LAUNCH(true, false, MODE);               \
  } while (0)
  const int layout = g.ta ? 2 : (g.tb ? 0 : 1);
  const int kind = mode == 8 ? (int)prof::GEMM_GLU : mode == 7 ? (int)prof::GEMM_NUMER : mode == 5 ? (int)prof::GEMM_STATS : mode == 6 ? (int)prof::GEMM_SWIGLU
                 : prof::GEMM_SINGLE + layout * 4 + (mode == 4 ? 2 : mode);   // (both accumulate forms are timed as one kind)
  {
    prof::Scope sc_time(kind, 2.0 * g.M * g.N * g.K * (g.A2 || g.glu_up ? 2 : 1), dev_rows, st);   // times the GEMM kernel, not the sum of the partial tiles after it
    if (mode == 8) LAUNCH(false, true, 8);
    else if (mode == 7) LAUNCH(false, true, 7);
    else if (mode == 5) LAUNCH(false, true, 5);
    else if (mode == 6) LAUNCH(false, false, 6);
    else if (g.ta && g.tb && mode == 4) LAUNCH(true, true, 4);
    else if (g.ta && g.tb) LAUNCH(true, true, 2);
    else if (g.ta && mode == 2 && tiles_m * tiles_n <= FEW_TILES) LAUNCH(true, false, 9);
    else if (mode == 4) LAUNCH(true, false, 4);
    else if (mode == 1) LAUNCH_LAYOUT(1);
    else if (mode == 2) LAUNCH_LAYOUT(2);
    else LAUNCH_LAYOUT(0);
  }
#undef LAUNCH_LAYOUT
#undef LAUNCH
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !may_split) return e;
  TailArgs t{};
  t.n = 1;
  t.p[0] = TailProblem{g.C, g.M, g.N, g.ldc, 0, tiles_m, tiles_n};
  t.sched = sc; t.rows_dev = g.rows_dev; t.k_steps = k_steps; t.scratch_tiles = scratch_tiles; t.scratch = g.scratch;
  t.part = partial_floats(g.M);
  t.K = g.ta ? g.K : 0;
  return launch_tail(mode, t, dev_rows && !g.ta ? std::min(N_CU / 2, tiles_m * tiles_n) : sc.tail, st);
}

// Grouped launch.  Requires every problem to be eligible, of the same layout / output type / accumulate mode.
// Accumulate-form problems that write the same C (same shape and leading dimensions) are folded into one grouped
// problem with several reduction segments: one pass over that C.
static bool same_output(const GemmArgs& a, const GemmArgs& b) {
  return !a.C0 && !b.C0 && a.C == b.C && a.M == b.M && a.N == b.N && a.lda == b.lda && a.ldb == b.ldb && a.ldc == b.ldc;
}
static int group_fold(const GemmArgs* gs, int n, int* owner /* [n]: index of the first problem with the same output */) {
  int n_out = 0;
  for (int i = 0; i < n; ++i) {
    owner[i] = i;
    if (gs[i].acc)
      for (int j = 0; j < i; ++j)
        if (owner[j] == j && same_output(gs[j], gs[i])) { owner[i] = j; break; }
    if (owner[i] == i) ++n_out;
  }
  return n_out;
}
constexpr int MAX_BATCH = MAX_GROUP * MAX_GSEG;
// separate_us: estimated time of the problems on their own
bool gemm_mfma_group_eligible(const GemmArgs* gs, int n, bool small_ok, double separate_us) {
  if (n < 2 || n > MAX_BATCH) return false;
  int64_t tiles = 0;
  int owner[MAX_BATCH], nseg[MAX_BATCH] = {0};
  const int n_out = group_fold(gs, n, owner);
  if (n_out > MAX_GROUP) return false;
  for (int i = 0; i < n; ++i) {
    if (!gemm_mfma_eligible(gs[i]) || gs[i].rows_dev || gs[i].A2 || (gs[i].ta && gs[i].tb)) return false;
    if (gs[i].ta != gs[0].ta || gs[i].tb != gs[0].tb || gs[i].out_dt != gs[0].out_dt || gs[i].acc != gs[0].acc) return false;
    if (++nseg[owner[i]] > MAX_GSEG) return false;
    if (owner[i] == i) tiles += cdiv(gs[i].M, BM) * cdiv(gs[i].N, BN);
  }
  if (tiles >= (1 << 30)) return false;
  // Few tiles: launches of their own, each split over the chip, may fill it better - where the reductions are long enough to make up for a launch and a
  // sum of partial tiles each, which the estimates say.  The seven weight gradients of a 1024-wide layer, 172 tiles: 2046 rows 244 us apart, 86 in
  // one launch, 660 rows 208 and 48.  Problems that share an output are one pass over it in one launch, and several
  // passes apart.  (small_ok: many skinny problems, none of which could fill the chip alone either)
  return tiles >= 200 || n_out < n || small_ok || gemm_mfma_us(gs, n) < separate_us;
}

hipError_t gemm_mfma_group(const GemmArgs* gs, int n, hipStream_t st) {
  GroupArgs ga{};
  int owner[MAX_BATCH], slot[MAX_BATCH];
  group_fold(gs, n, owner);
  int tiles = 0, np = 0;
  for (int i = 0; i < n; ++i) {
    if (owner[i] == i) {
      slot[i] = np;
      GroupProblem& p = ga.p[np++];
      p.C = gs[i].C; p.C0 = gs[i].C0; p.M = gs[i].M; p.N = gs[i].N; p.lda = gs[i].lda; p.ldb = gs[i].ldb; p.ldc = gs[i].ldc;
      p.nseg = 0;
      p.tiles_m = (int)cdiv(gs[i].M, BM); p.tiles_n = (int)cdiv(gs[i].N, BN); p.tile_begin = tiles;
      tiles += p.tiles_m * p.tiles_n;
    }
    GroupProblem& p = ga.p[slot[owner[i]]];
    p.A[p.nseg] = (const bf16_t*)gs[i].A; p.B[p.nseg] = (const bf16_t*)gs[i].B; p.K[p.nseg] = gs[i].K;
    ++p.nseg;
  }
  ga.n = np;
  const GemmArgs& g = gs[0];
  const int mode = g.acc ? (g.out_dt == DT_BF16 ? 4 : 2) : (g.out_dt == DT_BF16 ? 1 : 0);
  int min_k = g.K, max_m = g.M;
  for (int i = 1; i < n; ++i) { min_k = std::min(min_k, gs[i].K); max_m = std::max(max_m, gs[i].M); }
  ga.sched = make_schedule(tiles, (int)cdiv(min_k, BK), mode_splits(mode) && np == n ? scratch_tiles_of(g, max_m) : 0);
  ga.scratch = g.scratch;
  ga.part = partial_floats(max_m);
  const unsigned grid = (unsigned)(ga.sched.full + ga.sched.tail * ga.sched.splits);
  double work = 0.0;
  for (int i = 0; i < n; ++i) work += 2.0 * gs[i].M * gs[i].N * gs[i].K;
  const int layout = g.ta ? 2 : (g.tb ? 0 : 1);
  {
  prof::Scope sc(prof::GEMM_GROUP + layout * 4 + (mode == 4 ? 2 : mode), work, false, st);
#define GLAUNCH(TA, TB, MODE) gemm_mfma_group_k<TA, TB, MODE><<<grid, NTHREADS, 0, st>>>(ga)
#define GLAUNCH_LAYOUT(MODE)                     \
  do {                                           \
    if (!g.ta && g.tb) GLAUNCH(false, true, MODE); \
    else if (!g.ta && !g.tb) GLAUNCH(false, false, MODE); \
    else GLAUNCH(true, false, MODE);             \
  } while (0)
  if (g.out_dt == DT_BF16 && g.acc) GLAUNCH(true, false, 4);
  else if (g.out_dt == DT_BF16) GLAUNCH_LAYOUT(1);
  else if (g.acc) GLAUNCH_LAYOUT(2);
  else GLAUNCH_LAYOUT(0);
#undef GLAUNCH_LAYOUT
#undef GLAUNCH
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || ga.sched.splits == 1) return e;
  TailArgs t{};
  t.n = np;
  for (int i = 0; i < np; ++i) t.p[i] = TailProblem{ga.p[i].C, ga.p[i].M, ga.p[i].N, ga.p[i].ldc, ga.p[i].tile_begin, ga.p[i].tiles_m, ga.p[i].tiles_n};
  t.sched = ga.sched; t.scratch = ga.scratch; t.part = ga.part;
  return launch_tail(mode, t, ga.sched.tail, st);
}

// Segmented weight-gradient launch: gs[0..n) are accumulate-form (TN, fp32 or bf16 C +=) problems that share C, M, N and the
// leading dimensions and differ in A, B, K and rows_dev.
bool gemm_mfma_seg_eligible(const GemmArgs* gs, int n) {
  if (n < 2 || n > MAX_SEG) return false;
  for (int i = 0; i < n; ++i) {
    const GemmArgs& g = gs[i];
    if (!gemm_mfma_eligible(g) || !g.ta || g.tb != gs[0].tb || !g.acc || g.out_dt != gs[0].out_dt || g.A2) return false;
    if (g.C0 || g.C != gs[0].C || g.M != gs[0].M || g.N != gs[0].N || g.lda != gs[0].lda || g.ldb != gs[0].ldb || g.ldc != gs[0].ldc) return false;
  }
  return true;
}
hipError_t gemm_mfma_seg(const GemmArgs* gs, int n, hipStream_t st) {
  SegLaunch sl{};
  sl.n = n;
  double work = 0.0;
  bool bounded = false;
  for (int i = 0; i < n; ++i) {
    sl.A[i] = (const bf16_t*)gs[i].A; sl.B[i] = (const bf16_t*)gs[i].B; sl.rows_dev[i] = gs[i].rows_dev; sl.K[i] = gs[i].K;
    work += 2.0 * gs[i].M * gs[i].N * gs[i].K;
    bounded = bounded || gs[i].rows_dev != nullptr;
  }
  const GemmArgs& g = gs[0];
  const int tiles = (int)cdiv(g.M, BM) * (int)cdiv(g.N, BN);
  prof::Scope sc(prof::GEMM_SEG, work, bounded, st);
  auto go = [&](auto kernel) { kernel<<<tiles, NTHREADS, 0, st>>>(sl, g.C, g.M, g.N, g.lda, g.ldb, g.ldc); };
  if (g.out_dt == DT_BF16) g.tb ? go(gemm_mfma_seg_k<true, true>) : go(gemm_mfma_seg_k<true, false>);
  else g.tb ? go(gemm_mfma_seg_k<false, true>) : go(gemm_mfma_seg_k<false, false>);
  return hipGetLastError();
}

// ---- what the matrix pipe sustains on its own -------------------------------------------------------------
// Eight independent 32x32x16 products per round, two waves per SIMD, no global memory traffic.  R of the eight A fragments
// of a round are re-read from LDS (one conflict-free ds_read_b128 = 1 KB per wave each, the way the GEMM and attention
// kernels feed their MFMAs: the GEMM main loop reads 6 fragments per 8 products, the attention backward 8); the others
// and the B fragments never change.  The rate depends on the VALUES of the fragments (power management), which is why
// the caller supplies them.
template <int R>
__global__ __launch_bounds__(NTHREADS) void mfma_rate_probe_k(const bf16x8* __restrict__ operands, float* __restrict__ sink, int iters) {
  __shared__ __attribute__((aligned(1024))) bf16x8 frag[R > 0 ? 2 * NTHREADS * 8 : 1];   // two rounds' worth: 128 KB
  if (R > 0) {
    for (int i = threadIdx.x; i < 2 * NTHREADS * 8; i += NTHREADS) frag[i] = operands[i % 4096];
    __syncthreads();
  }
  const uint32_t base = lds_addr(&frag[0]) + (threadIdx.x & 63) * 16 + (threadIdx.x >> 6) * 8 * 1024;
  bf16x8 a[8], b[2];
#pragma unroll
  for (int i = 0; i < 8; ++i) a[i] = operands[(threadIdx.x + i * NTHREADS) % 4096];
#pragma unroll
  for (int j = 0; j < 2; ++j) b[j] = operands[(threadIdx.x + (8 + j) * NTHREADS) % 4096];
  f32x16 acc[8];
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
  for (int it = 0; it < iters; ++it) {
    const uint32_t off = (uint32_t)(it & 1) * (NTHREADS * 8 * 16);
#pragma unroll
    for (int i = 0; i < R; ++i) a[i] = lds_read_b128(base + off + i * 1024);
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[i & 1], acc[i], 0, 0, 0);
  }
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) s += acc[i][r];
  sink[(int64_t)blockIdx.x * NTHREADS + threadIdx.x] = s;
}
hipError_t mfma_rate_probe(const void* operands, float* sink, int workgroups, int iters, int lds_reads, hipStream_t st) {
  if (workgroups <= 0 || iters < 0) return hipErrorInvalidValue;
  if (lds_reads == 0) mfma_rate_probe_k<0><<<workgroups, NTHREADS, 0, st>>>((const bf16x8*)operands, sink, iters);
  else if (lds_reads == 6) mfma_rate_probe_k<6><<<workgroups, NTHREADS, 0, st>>>((const bf16x8*)operands, sink, iters);
  else if (lds_reads == 8) mfma_rate_probe_k<8><<<workgroups, NTHREADS, 0, st>>>((const bf16x8*)operands, sink, iters);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace sbp
