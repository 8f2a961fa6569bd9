// How a call of the MFMA attention kernels is dealt to workgroups: sizes of the query tiles, launches, order.  Host code, results of the sizes alone.
#pragma once

#include <algorithm>

#include "launch.h"

namespace sbp {

// Time of a launch in key steps: its query tiles, those with the most keys first, dealt to 256 CUs as they become free.  A tile takes a step for every `keys`
// keys that it sees and six more for its start and end.  More than eight rounds: their mean.
inline double attn_launch_steps(const AttnArgs& a, int tile, int keys) {
  const int64_t heads = (int64_t)a.Hq * a.batch, rows = cdiv(a.q_len, tile);
  auto steps_of = [&](int64_t row) {
    const int64_t first_q = a.q_start + row * tile, last = std::min<int64_t>(a.q_start + a.q_len, first_q + tile);
    const int64_t first = std::max<int64_t>(a.kv_first, a.window > 0 ? first_q - a.window + 1 : 0);
    return cdiv(std::max<int64_t>(last - first, 0), keys) + 6;
  };
  if (rows * heads > 8 * 256) {
    double sum = 0.0;
    for (int64_t row = 0; row < rows; ++row) sum += (double)steps_of(row) * (double)heads;
    return sum / 256.0;
  }
  struct Free { int64_t at; int n; } cus[258];      // CUs by the time they become free, the earliest first: at most 256 different times and a new one
  int n_times = 1;
  int64_t end = 0;
  cus[0] = {0, 256};
  for (int64_t row = rows - 1; row >= 0; --row) {
    const int64_t len = steps_of(row);
    for (int64_t left = heads; left > 0;) {
      const int take = (int)std::min<int64_t>(cus[0].n, left);
      const int64_t at = cus[0].at + len;
      left -= take;
      if ((cus[0].n -= take) == 0) std::copy(cus + 1, cus + n_times--, cus);
      int i = n_times;
      while (i > 0 && cus[i - 1].at > at) --i;
      if (i > 0 && cus[i - 1].at == at) cus[i - 1].n += take;
      else {
        std::copy_backward(cus + i, cus + n_times, cus + n_times + 1);
        cus[i] = {at, take};
        ++n_times;
      }
      end = std::max(end, at);
    }
  }
  return (double)end;
}
// Query tiles of 128, whose two wave groups take even and odd key tiles, or of 256.  A step of 128 keys costs a half tile `cost` times what one of 64 costs a whole
// one.  Forward, heads of 128: 2.1 against 1.95 us; heads of 64, where the vector work of 128 keys is the longer part, 0.94 times (2398 queries from 0, 32 / 8
// heads, whole / half tiles 75 / 66 us, 3302 under a window of 124, 28 / 4, 36 / 32; 3613 behind 927, 32 / 8, 175 / 187).  dQ, whose half tiles have 32 keys, more.  Whole / half tiles,
// measured, forward of 2048 queries, 28 heads of 128, from 0 73 / 62 us (whole: as long as the longest tile), from 2048 132 / 123, 4096 from 4096 403 / 437; four
// sequences of 640 tokens 52 / 59, with the backward 81 / 85; 2048 queries, 32 heads: backward from 0 352 / 362, from 4096 600 / 580, from 6144 768 / 789.
constexpr double ATTN_HALF_STEP_DQ = 1.15;
inline double attn_half_step_forward(int dh) { return dh == 64 ? 0.94 : 1.08; }
inline bool attn_half_tiles_faster(const AttnArgs& a, double cost) {
  return cost * attn_launch_steps(a, ATTN_TILE_Q / 2, 2 * ATTN_TILE_K) < attn_launch_steps(a, ATTN_TILE_Q, ATTN_TILE_K);
}

constexpr int ATTN_IN_TURN_BLOCKS = 96;       // key blocks times K/V heads up to which shares are taken without a break
constexpr int ATTN_DQ_FIRST = 192;
struct AttnBackwardPlan {
  bool halves;                        // dQ: tiles of 128 queries
  int key_block0, key_blocks;         // key blocks that some query of the chunk sees; the others' dK/dV are zero and not launched
  bool parts, in_turn;                // the slices of a key block: a workgroup each, whose sums meet in the scratch; or in turn, the columns halved between two workgroups
  int q_blocks;
  int64_t n_dkv, n_dq;                // workgroups
  bool one_launch, dq_first;          // dK/dV and dQ in one launch; those of dQ first
  bool side_by_side;                  // one launch: the key blocks of a head side by side, else the heads of a key block
};
// most, most_prefix: workgroups up to which a call, one behind a prefix, is one launch where dK/dV comes first
inline AttnBackwardPlan attn_backward_plan(const AttnArgs& a, int most, int most_prefix) {
  AttnBackwardPlan p{};
  p.halves = attn_half_tiles_faster(a, ATTN_HALF_STEP_DQ);
  p.key_block0 = attn_first_key_block(a);
  p.key_blocks = std::max(0, (int)cdiv((int64_t)a.q_start + a.q_len, ATTN_KV_TILE) - p.key_block0);
  const int slices = std::max(1, a.dkv_slices), tile = p.halves ? ATTN_TILE_Q / 2 : ATTN_TILE_Q;
  const int64_t blocks = (int64_t)p.key_blocks * a.Hkv * a.batch;
  p.parts = slices > 1 && a.dkv_scratch;
  p.in_turn = slices > 1 && !p.parts && blocks > 0 && blocks <= ATTN_IN_TURN_BLOCKS;
  p.n_dkv = blocks * (p.in_turn ? 2 : p.parts ? slices : 1);
  p.q_blocks = (int)cdiv(a.q_len, tile);
  p.n_dq = (int64_t)p.q_blocks * a.Hq * a.batch;
  // The longer workgroups first, by their steps: last, they are a tail on a chip that is otherwise done.  A dQ tile sees at most its own keys and a window before them.
  // dQ comes first only where it leaves a quarter of the CUs to dK/dV: with more workgroups its key tiles are shared in the L2 no better than the queries of
  // dK/dV.  Backward, dQ last / first: 283 queries behind 4775 keys, 32 / 32 heads 190 / 149 us, 129 behind 6926, window 697, 64 / 8, 64 / 56, 640 behind
  // 8000, 32 / 8, 303 / 295; 224 workgroups (2048 behind 30720, 28 / 4) 2521 / 2617 us.  One step as long as the other: 383 behind 3704, 40 / 8, 3 % and 777
  // behind 3000, 16 / 4, 6 % faster with dQ first, 907 behind 12397, window 430, 12 / 2, 4 %, 1228 from 0, window 230, 16 / 4 heads of 64, 6 % slower.
  const int64_t first_visible = std::max<int64_t>(a.kv_first, a.window > 0 ? (int64_t)a.q_start - a.window + 1 : 0);
  const int64_t visible = std::max<int64_t>((int64_t)a.q_start + a.q_len - first_visible, 0);
  const int64_t seen = a.window > 0 ? std::min<int64_t>(visible, (int64_t)a.window + std::min(tile, a.q_len)) : visible;
  const int64_t seen_by = a.window > 0 ? std::min<int64_t>(a.q_len, (int64_t)a.window + ATTN_KV_TILE) : a.q_len;
  const int64_t dq_steps = cdiv(seen, p.halves ? 2 * ATTN_TILE_K : ATTN_TILE_K);
  const int64_t dkv_steps = cdiv(seen_by, ATTN_KV_QUERIES) * (a.Hq / a.Hkv) / (p.parts ? slices : 1);
  p.dq_first = dq_steps > dkv_steps && p.n_dq <= ATTN_DQ_FIRST;
  const int64_t n = p.n_dkv + p.n_dq;
  p.one_launch = p.n_dkv > 0 && (p.in_turn || (p.dq_first && a.q_start > 0) || n <= (a.q_start > 0 ? most_prefix : most));
  // Workgroup b runs on XCD b % 8.  With the key blocks side by side an XCD has every eighth of them: where the chunk's own blocks, which ever fewer queries see, are
  // many, up to 2.4 times the work of another (2048 queries from 0, 28 / 4 heads 182 us, the heads of a block side by side 133, from 2048 344 / 328; 32 / 8 heads
  // 385 / 352 from 0, 790 / 769 from 6144).  Where they are an eighth or less, or each workgroup has a CU of its own, there is nothing to even out, and a head's
  // queries are shared by more of the chip: 4096 queries behind 28672 keys, 28 / 4, 1 and 2 % faster than the heads side by side, 117 behind 1183, 16 / 4, 1 %,
  // 719 from 0, 8 / 8, 4 %.  With dQ first, which takes most of the first round, the heads side by side are as fast or up to 7 % faster.
  const int own = (int)(cdiv((int64_t)a.q_start + a.q_len, ATTN_KV_TILE) - a.q_start / ATTN_KV_TILE);
  p.side_by_side = n <= 256 || (!p.dq_first && (int64_t)own * 8 <= p.key_blocks);
  return p;
}

// The shape-agnostic kernels.
// dQ and dK/dV of heads of up to 64 elements in one launch: without a prefix, up to 1024 workgroups, or with few of dQ behind a long prefix, which come first as
// the longer ones (so do they wherever a key block has fewer query blocks than the other way round).  Backward apart / in one, fp32, us: 256 queries from 0, 4 heads
// of 16 10.9 / 6.6, 8 of 64 24.2 / 14.6, 16 of 64, 512 queries, 71.6 / 54.9; 2048 queries, 8 of 64 330 / 268, 16 of 32 297 / 228, bf16 4096, 8 of 16 336 / 262; 64 from
// 3000, 2 of 16 30.2 / 25.2; 128 from 30000, 16 of 32 741 / 534.  Behind a prefix with more workgroups the loads of o, which dK/dV reads as well, outweigh it: 256 from
// 8000, 16 of 64 442 / 464, 2048 from 8000 3785 / 3840.
constexpr int64_t ATTN_NARROW_MAX = 1024, ATTN_NARROW_DQ = 192;
struct AttnNarrowPlan { bool one_launch, dq_first; int64_t n_dkv, n_dq; };
inline AttnNarrowPlan attn_narrow_plan(const AttnArgs& a) {
  const int64_t q_blocks = cdiv(a.q_len, 16), key_blocks = cdiv((int64_t)a.q_start + a.q_len, 16);
  AttnNarrowPlan p{};
  p.n_dkv = key_blocks * a.Hkv;
  p.n_dq = q_blocks * a.Hq;
  p.dq_first = key_blocks > q_blocks * (a.Hq / a.Hkv);
  const int64_t n = p.n_dkv + p.n_dq;
  // (dq may take o's place: dK/dV then has to be a launch that does not read o)
  p.one_launch = a.dh <= 64 && a.dq != a.o && n <= INT32_MAX && (a.q_start == 0 || n <= ATTN_NARROW_MAX || (p.dq_first && p.n_dq <= ATTN_NARROW_DQ));
  return p;
}

}  // namespace sbp
