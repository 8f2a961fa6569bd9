// How the MFMA attention kernels deal a call to workgroups (csrc/attn_plan.h).  Each line of standard input is a call,
//   dh n_q_heads n_kv_heads q_start q_len window kv_first sequences room most most_prefix
// (room: for the slices of dK/dV side by side), each line of standard output its plan as JSON: of the MFMA kernels and, narrow_*, of the shape-agnostic ones for
// heads of up to 64 elements (narrow_in_place: one launch also where dq takes o's place).
#include "attn_plan.h"

#include <cstdint>
#include <cstdio>
#include <iostream>

int main() {
  sbp::AttnArgs a{};
  int room, most, most_prefix;
  static float scratch[1];
  while (std::cin >> a.dh >> a.Hq >> a.Hkv >> a.q_start >> a.q_len >> a.window >> a.kv_first >> a.batch >> room >> most >> most_prefix) {
    a.dt = sbp::DT_BF16;
    a.o = &a;
    a.dkv_slices = sbp::attn_dkv_slices(a, SIZE_MAX);
    a.dkv_scratch = room ? scratch : nullptr;
    const sbp::AttnBackwardPlan p = sbp::attn_backward_plan(a, most, most_prefix);
    std::printf("{\"forward_halves\": %d, \"halves\": %d, \"key_blocks\": %d, \"slices\": %d, \"parts\": %d, \"in_turn\": %d, \"n_dkv\": %lld, \"n_dq\": %lld, \"one_launch\": %d, "
                "\"dq_first\": %d, \"side_by_side\": %d, ",
                sbp::attn_half_tiles_faster(a, sbp::attn_half_step_forward(a.dh)), p.halves, p.key_blocks, a.dkv_slices, p.parts, p.in_turn, (long long)p.n_dkv, (long long)p.n_dq, p.one_launch,
                p.dq_first, p.side_by_side);
    const sbp::AttnNarrowPlan g = sbp::attn_narrow_plan(a);
    std::printf("\"narrow_one_launch\": %d, \"narrow_dq_first\": %d, \"narrow_n\": %lld, ", g.one_launch, g.dq_first, (long long)(g.n_dkv + g.n_dq));
    a.dq = a.o;
    std::printf("\"narrow_in_place\": %d}\n", sbp::attn_narrow_plan(a).one_launch);
    a.dq = nullptr;
  }
  return 0;
}
