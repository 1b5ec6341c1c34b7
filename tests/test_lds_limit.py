"""The raising of kernels' dynamic-LDS limits (host code): once per kernel and size, whatever their signatures."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

# The runtime's calls are replaced by counters, so the program needs no GPU.
SOURCE = r"""
#include <hip/hip_runtime.h>
#include <atomic>
#include <cstdio>
#include <thread>
#include <vector>
static std::atomic<int> calls{0};
static std::atomic<size_t> limit_a{0}, limit_d{0};
template <typename T>
static hipError_t count_set(T fn, hipFuncAttribute, int bytes);
#define hipFuncSetAttribute count_set
#include "fused_common.h"
__global__ void ka(int) {}
__global__ void kb(int) {}
__global__ void kd(int) {}
__global__ void kc(float*) {}
template <typename T>
static hipError_t count_set(T fn, hipFuncAttribute, int bytes) {
  ++calls;
  if ((const void*)fn == (const void*)ka) limit_a = bytes;
  if ((const void*)fn == (const void*)kd) limit_d = bytes;
  return hipSuccess;
}
using dark::fz::allow_lds;
int main() {
  const size_t K = 1024;
  int bad = 0;
  for (int i = 0; i < 5; ++i) bad += allow_lds(ka, 60 * K) + allow_lds(kb, 100 * K) + allow_lds(kc, 50 * K) + allow_lds(kc, 48 * K);
  printf("%d", calls.load());
  for (int i = 0; i < 5; ++i) bad += allow_lds(ka, (i % 2 ? 60 : 70) * K);   // raised, never lowered again
  printf(" %d %zu", calls.load(), limit_a.load() / K);
  const int before = calls;
  std::vector<std::thread> t;
  for (int i = 0; i < 8; ++i)
    t.emplace_back([&, i] {
      const size_t need = (i % 2 ? 150 : 90) * K;
      for (int j = 0; j < 1000; ++j)
        if (allow_lds(kd, need) != DARK_OK || limit_d < need) _Exit(1);
    });
  for (auto& x : t) x.join();
  printf(" %d %zu %d %d\n", calls.load() - before <= 2, limit_d.load() / K, bad, allow_lds(ka, 161 * K) == DARK_EUNSUPPORTED);
}
"""


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="needs hipcc")
def test_limits_are_raised_once(tmp_path):
    src, exe = tmp_path / "limits.hip", tmp_path / "limits"
    src.write_text(SOURCE)
    subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-std=c++17", "-O1", "-pthread", "-Wno-unused-function",
                           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2603_04127_amd", "csrc"),
                           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", str(src), "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60, check=True).stdout
    assert out.split() == ["3", "4", "70", "1", "150", "0", "1"], out
