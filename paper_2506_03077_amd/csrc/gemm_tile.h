// What the bf16 MFMA GEMM kernels share: operand layouts in LDS, fragment reads, the order of output tiles, waits.
#pragma once
#include "device.h"

namespace sbp {

typedef bf16_t bf16x8 __attribute__((ext_vector_type(8)));
typedef bf16_t bf16x4 __attribute__((ext_vector_type(4)));
typedef short short4v __attribute__((ext_vector_type(4)));
typedef short short8v __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int N_CU = 256;

// ---- LDS layouts of a half tile.  K-contiguous operand: [128 rows][64 k], 128 B per row = 8 chunks of 16 B, chunk ^= (row>>1)&7:
//      16 consecutive rows at one logical chunk cover all 64 banks exactly once.
__device__ __forceinline__ int kmaj_swz(int row) { return (row >> 1) & 7; }
// ---- reduction-major operand: [64 k][128 rows], 256 B per k-row = 8 groups of 32 B, group ^= f(krow): the 32 lanes of a
//      transposing read touch k-rows {0..3, 8..11} (+ 4 or + 16) at one logical group; f tells those eight apart.
__device__ __forceinline__ int mnmaj_swz(int krow) { return (krow & 3) | (((krow >> 3) & 1) << 2); }

__device__ __forceinline__ bf16x8 lds_read_b128(uint32_t addr) {
  return *(const bf16x8*)(__attribute__((address_space(3))) const char*)(uintptr_t)addr;
}
__device__ __forceinline__ bf16x8 lds_read_tr(uint32_t lo_addr, uint32_t hi_addr) {
  short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)(uintptr_t)lo_addr);
  short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) short4v*)(uintptr_t)hi_addr);
  short8v r = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, r);
}

// Tile id -> (tile_m, tile_n): walk tiles in column bands of group_m row tiles so that the workgroups resident
// together share A row panels and B column panels in their XCD's L2.
__device__ __forceinline__ void band_coords(int id, int tiles_m, int tiles_n, int group_m, int& tm, int& tn) {
  const int band = group_m * tiles_n;
  const int g = id / band;
  const int first_m = g * group_m;
  const int gsz = min(tiles_m - first_m, group_m);
  const int r = id % band;
  tm = first_m + r % gsz;
  tn = r / gsz;
}
// Band height.  With XCD-contiguous ids each XCD works on a run of n_tiles/8 consecutive ids, i.e. a block of
// group_m rows x run/group_m columns of tiles; the fabric traffic of that XCD is proportional to rows + columns,
// so the block is made as square as the problem allows.  (Interleaved ids, used by the accumulate form, give
// every XCD one row of each band and all columns; 8 rows per band suit that.)
__device__ __forceinline__ int band_height_for_run(int tiles_m, int run) {
  int h = (int)(sqrtf((float)max(1, run)) + 0.5f);
  return max(1, min(h, min(tiles_m, 8)));
}
__device__ __forceinline__ int band_height(int tiles_m, int n_tiles, bool xcd_contiguous) {
  if (!xcd_contiguous) return 8;
  return band_height_for_run(tiles_m, n_tiles / 8);
}
// Hardware deals consecutive workgroups round-robin to the 8 XCDs (each with its own L2); undo that so each
// XCD gets a contiguous run of tile ids.  Measured: +3-4% for the store-only forms; the accumulate form is up to 3 % faster with
// the hardware's interleaved order, so it keeps that.
__device__ __forceinline__ int xcd_contiguous_id(int id, int n_tiles) {
  constexpr int NXCD = 8;
  const int x = id % NXCD, q = n_tiles / NXCD, r = n_tiles % NXCD;   // XCD x owns q (+1 if x < r) consecutive ids
  return x * q + min(x, r) + id / NXCD;
}

// Counted wait / workgroup barrier of the main loop.  Inline assembly (with a memory clobber) so that the compiler neither adds
// waits of its own nor moves LDS reads across; the scheduling barriers keep the machine scheduler from doing the same.
#define WAIT_VMCNT(n) asm volatile("s_waitcnt vmcnt(%0)" ::"i"(n) : "memory")
#define WAIT_LDS() asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory")
#define SLOT_BARRIER()                        \
  do {                                        \
    __builtin_amdgcn_sched_barrier(0);        \
    asm volatile("s_barrier" ::: "memory");   \
    __builtin_amdgcn_sched_barrier(0);        \
  } while (0)

}  // namespace sbp
