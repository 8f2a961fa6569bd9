"""The copies of adapter operands and the sums of adapter gradients (csrc/elementwise.hip), their kernels run thread by thread on the CPU over exactly sized
allocations under -fsanitize=address,undefined, against the definition."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2506_03077_amd", "csrc")

SHIM = r"""
#include <cassert>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include "launch.h"
#define __launch_bounds__(x)
struct Dim { unsigned x; };
static Dim blockIdx, threadIdx;
struct float4 { float x, y, z, w; };
struct bf16_t {      // (small whole numbers only: the upper half of the fp32 value)
  uint16_t u;
  bf16_t() = default;
  explicit bf16_t(float f) { uint32_t b; memcpy(&b, &f, 4); assert((b & 0xffff) == 0); u = b >> 16; }
  explicit operator float() const { uint32_t b = (uint32_t)u << 16; float f; memcpy(&f, &b, 4); return f; }
};
template <typename T> float ldf(const T* p) { return (float)*p; }
template <typename T> void stf(T* p, float v) { *p = (T)v; }
template <typename T> void load8(const T* p, float (&v)[8]) { assert(!((uintptr_t)p & 15)); for (int k = 0; k < 8; ++k) v[k] = ldf(p + k); }
template <typename T> void store8(T* p, const float (&v)[8]) { assert(!((uintptr_t)p & 15)); for (int k = 0; k < 8; ++k) stf(p + k, v[k]); }
inline hipError_t hipGetLastError() { return hipSuccess; }
#define DISPATCH_DT(dt, T, ...) do { if ((dt) == DT_BF16) { using T = bf16_t; __VA_ARGS__; } else { using T = float; __VA_ARGS__; } } while (0)
template <typename F> void launch(unsigned grid, F f) {
  for (blockIdx.x = 0; blockIdx.x < grid; ++blockIdx.x)
    for (threadIdx.x = 0; threadIdx.x < 256; ++threadIdx.x) f();
}
namespace sbp {
"""

MAIN = r"""
}  // namespace sbp
using namespace sbp;
template <typename T> int pad_case(int dt, int R, int C, int R2, int C2, int transposed, int shift) {
  const size_t n = (size_t)R * C;
  T* src = (T*)malloc((n + shift) * sizeof(T)) + shift;      // (the allocation ends where the source does)
  for (size_t i = 0; i < n; ++i) src[i] = (T)(float)(1 + i % 100);
  T* dst = (T*)malloc((size_t)R2 * C2 * sizeof(T));
  for (size_t i = 0; i < (size_t)R2 * C2; ++i) dst[i] = (T)-7.0f;
  PadJobs jobs{};
  jobs.n = 2;      // two jobs, the second behind the first
  T one = (T)3.0f, one_out = (T)0.0f;
  jobs.job[0] = PadJob{&one, &one_out, 1, 1, 0, 1, 1, 1.0f, 0};
  jobs.job[1] = PadJob{src, dst, R, C, transposed, R2, C2, 2.0f, 0};
  pad_matrices(dt, jobs, nullptr);
  int bad = (float)one_out != 3.0f;
  for (int r = 0; r < R2; ++r)
    for (int c = 0; c < C2; ++c) {
      const float want = r < R && c < C ? 2.0f * (float)src[transposed ? (size_t)c * R + r : (size_t)r * C + c] : 0.0f;
      bad += (float)dst[(size_t)r * C2 + c] != want;
    }
  free(src - shift); free(dst);
  return bad;
}
static int add_case(int R, int C, int ld, int shift_src, int shift_dst) {
  const size_t n = (size_t)(R - 1) * ld + C, m = (size_t)R * C;
  float* src = (float*)malloc((n + shift_src) * 4) + shift_src;
  float* dst = (float*)malloc((m + shift_dst) * 4) + shift_dst;
  for (size_t i = 0; i < n; ++i) src[i] = (float)(i % 97);
  for (size_t i = 0; i < m; ++i) dst[i] = (float)(i % 31);
  AddJobs jobs{};
  jobs.n = 2;
  float a = 1.0f, b = 5.0f;
  jobs.job[0] = AddJob{&a, 1, &b, 1, 1, 0};
  jobs.job[1] = AddJob{src, ld, dst, R, C, 0};
  add_scaled_blocks(jobs, 2.0f, nullptr);
  int bad = b != 7.0f;
  for (int r = 0; r < R; ++r)
    for (int c = 0; c < C; ++c) bad += dst[(size_t)r * C + c] != (float)(((size_t)r * C + c) % 31) + 2.0f * src[(size_t)r * ld + c];
  free(src - shift_src); free(dst - shift_dst);
  return bad;
}
int main(int, char** argv) {
  int bad = 0;
  const int dt = argv[2][0] == 'b' ? DT_BF16 : DT_F32;
  const int v[7] = {0, atoi(argv[3]), atoi(argv[4]), atoi(argv[5]), atoi(argv[6]), atoi(argv[7]), atoi(argv[8])};
  if (argv[1][0] == 'p') bad = dt == DT_BF16 ? pad_case<bf16_t>(dt, v[1], v[2], v[3], v[4], v[5], v[6]) : pad_case<float>(dt, v[1], v[2], v[3], v[4], v[5], v[6]);
  else bad = add_case(v[1], v[2], v[3], v[4], v[5]);
  std::printf("%d wrong\n", bad);
  return bad != 0;
}
"""


@pytest.fixture(scope="module")
def binary(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    with open(os.path.join(CSRC, "elementwise.hip")) as f:
        text = f.read()
    code = text[text.index("// element i of a launch over several jobs"):text.index("template <typename T>\n__global__ void embedding_fwd_k")]
    code, launches = re.subn(r"([\w<>]+)<<<(.+?), 256, 0, st>>>\(([^()]*)\)", r"launch(\2, [&] { \1(\3); })", code)
    assert launches == 2
    d = tmp_path_factory.mktemp("adapter_copies")
    src, out = str(d / "copies.cpp"), str(d / "copies")
    with open(src, "w") as f:
        f.write(SHIM + code + MAIN)
    p = subprocess.run([gxx, "-std=c++17", "-O1", "-g", "-w", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-I", os.path.join(ROOT, "tests", "host_sanitize"),
                        "-I", CSRC, src, "-o", out], capture_output=True, text=True)
    assert p.returncode == 0, p.stderr[-4000:]

    def run(*args):
        env = dict(os.environ, ASAN_OPTIONS="detect_leaks=0")
        env.pop("LD_PRELOAD", None)
        p = subprocess.run([out, *map(str, args)], capture_output=True, text=True, env=env, timeout=60)
        assert p.returncode == 0 and p.stdout == "0 wrong\n", (p.stdout, p.stderr[-2000:])
    return run


# rows, columns, padded rows, padded columns
@pytest.mark.parametrize("R,C,R2,C2", [(32, 40, 32, 40), (8, 5, 24, 5), (16, 9, 16, 16), (32, 3, 40, 8), (12, 16, 16, 16), (7, 33, 8, 40), (1, 1, 8, 8), (3, 24, 8, 27), (8, 8, 9, 8)])
@pytest.mark.parametrize("transposed", [0, 1])
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_copies_stay_inside_their_source(binary, dtype, shift, transposed, R, C, R2, C2):
    binary("pad", dtype, R, C, R2, C2, transposed, shift)


@pytest.mark.parametrize("R,C,ld", [(5, 8, 8), (3, 8, 12), (4, 7, 8), (2, 1, 4), (6, 12, 13), (1, 4, 4)])
@pytest.mark.parametrize("shifts", [(0, 0), (1, 0), (0, 1), (2, 2)])
def test_sums_stay_inside_their_blocks(binary, shifts, R, C, ld):
    binary("add", "f32", R, C, ld, *shifts, 0)
