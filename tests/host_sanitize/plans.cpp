// How the host layer deals the rows of a layer call to passes, as its calls of the kernel launchers show it (stub_launch.cpp).
// Each line of standard input is a configuration,
//   dtype grad_dtype batch seq_len chunk dw_group_rows hidden n_q_heads n_kv_heads head_dim mlp_width window padded first[0 .. batch)
// (padded 0: no list), each line of standard output its calls as JSON: "forward" / "backward" the attention calls of the two entry points as
// [sequences, q_start, rows, slices of a key block, slices side by side], "dw" the weight-gradient launches as lists of [first row, rows].
#include "../../include/streambp.h"
#include "launch.h"

#include <cstdio>
#include <cstdlib>
#include <functional>
#include <iostream>
#include <string>
#include <vector>

namespace sbp {
extern std::function<void(const AttnArgs&, bool)> stub_on_attn;
extern std::function<void(const GemmArgs*, int)> stub_on_gemm_batch;
}

int main() {
  sbp_layer_cfg c{};
  int padded;
  while (std::cin >> c.dtype >> c.grad_dtype >> c.batch >> c.seq_len >> c.chunk >> c.dw_group_rows >> c.hidden >> c.n_q_heads >> c.n_kv_heads >> c.head_dim >>
         c.mlp_width >> c.window >> padded) {
    std::vector<int32_t> first(c.batch, 0);
    if (padded) for (int32_t& f : first) std::cin >> f;
    c.seq_first = padded ? first.data() : nullptr;
    c.rms_eps = 1e-6f; c.rope_theta = 1e4f;
    const size_t es = c.dtype == SBP_BF16 ? 2 : 4, d = c.hidden, F = c.mlp_width, qd = (size_t)c.n_q_heads * c.head_dim, kd = (size_t)c.n_kv_heads * c.head_dim;
    std::vector<void*> owned;
    auto take = [&](size_t bytes) {      // (calloc: pages that no call touches cost nothing)
      void* p = std::calloc(bytes + 512, 1);
      owned.push_back(p);
      return (void*)(((uintptr_t)p + 255) & ~(uintptr_t)255);
    };
    void* wm[9]; void* gm[9];
    const size_t sizes[9] = {qd * d, kd * d, kd * d, d * qd, F * d, F * d, d * F, d, d};
    for (int i = 0; i < 9; ++i) { wm[i] = take(sizes[i] * es); gm[i] = take(sizes[i] * 4); }
    sbp_layer_weights w{wm[0], wm[1], wm[2], wm[3], wm[4], wm[5], wm[6], wm[7], wm[8]};
    sbp_layer_grads g{gm[0], gm[1], gm[2], gm[3], gm[4], gm[5], gm[6], (float*)gm[7], (float*)gm[8]};
    const size_t act = (size_t)c.batch * c.seq_len * d * es;
    char *x = (char*)take(act), *dy = (char*)take(act), *dx = (char*)take(act), *y = (char*)take(act);
    const size_t need = streambp_layer_workspace_bytes(&c);
    void* ws = take(need);
    std::string attn[2], dw;
    int entry = 0;
    sbp::stub_on_attn = [&](const sbp::AttnArgs& a, bool bwd) {
      if (entry == 0 && !bwd) return;      // (the backward's reforward: the same rows again)
      char s[128];
      std::snprintf(s, sizeof s, "%s[%d, %d, %d, %d, %d]", attn[entry].empty() ? "" : ", ", a.batch, a.q_start, a.q_len, a.dkv_slices, a.dkv_scratch != nullptr);
      attn[entry] += s;
    };
    sbp::stub_on_gemm_batch = [&](const sbp::GemmArgs* gs, int n) {
      std::string rows;
      for (int i = 0; i < n; ++i)
        if (gs[i].C == g.wdown) rows += (rows.empty() ? "[" : ", [") + std::to_string(((const char*)gs[i].A - dy) / (ptrdiff_t)(d * es)) + ", " + std::to_string(gs[i].K) + "]";
      if (!rows.empty()) dw += (dw.empty() ? "[" : ", [") + rows + "]";
    };
    int32_t rc = streambp_layer_backward(&c, &w, x, dy, dx, &g, ws, need, nullptr);
    entry = 1;
    if (rc == SBP_OK) rc = streambp_layer_forward(&c, &w, x, y, ws, need, nullptr);
    if (rc != SBP_OK) { std::printf("{\"error\": %d}\n", rc); return 1; }
    std::printf("{\"backward\": [%s], \"forward\": [%s], \"dw\": [%s]}\n", attn[0].c_str(), attn[1].c_str(), dw.c_str());
    for (void* p : owned) std::free(p);
  }
  return 0;
}
