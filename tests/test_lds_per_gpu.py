"""Kernels with more than 64 KiB of LDS have to be announced to every GPU that a process uses, on the CPU: the helper of kernels.h on a runtime
of two GPUs that counts the calls."""
import os
import subprocess

from paper_2405_16283_amd import build

MAIN = r"""
#include <cassert>
#include <cstdio>
#include <map>
#include <mutex>
#include <thread>
#include <vector>
#include "kernels.h"
static thread_local int device = 0;
static std::mutex mu;
static std::map<std::pair<int, const void*>, int> calls;
static bool failing = false;
extern "C" hipError_t hipGetDevice(int* d) { *d = device; return hipSuccess; }
extern "C" hipError_t hipFuncSetAttribute(const void* f, hipFuncAttribute, int) {
  std::lock_guard<std::mutex> lock(mu);
  ++calls[{device, f}];
  return failing ? hipErrorInvalidValue : hipSuccess;
}
static char kernels[2];
static hipError_t launch(int k) {
  static std::atomic<uint64_t> allowed[2] = {};
  return tn::allow_lds(allowed[k], kernels + k, 131072);
}
int main() {
  failing = true;
  if (launch(0) != hipErrorInvalidValue) return 1;
  failing = false;
  for (int d : {0, 1, 0, 70, 1})
    for (int k = 0; k < 2; ++k)
      for (int n = 0; n < 3; ++n) {
        device = d;
        if (launch(k) != hipSuccess) return 2;
      }
  if (calls[{0, kernels}] != 2 || calls[{0, kernels + 1}] != 1 || calls[{1, kernels}] != 1 || calls[{1, kernels + 1}] != 1) return 3;
  if (calls[{70, kernels}] != 3) return 4;  // not among those that are remembered
  std::vector<std::thread> all;
  for (int d = 2; d < 10; ++d)
    all.emplace_back([d] { device = d; for (int n = 0; n < 1000; ++n) if (launch(n & 1) != hipSuccess) std::abort(); });
  for (auto& t : all) t.join();
  for (int d = 2; d < 10; ++d)
    for (int k = 0; k < 2; ++k) if (calls[{d, kernels + k}] != 1) return 5;
  return 0;
}
"""


def test_every_gpu_is_told_once(tmp_path):
    (tmp_path / "main.cpp").write_text(MAIN)
    exe = str(tmp_path / "main")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", os.path.join(build.ROOT, "include"),
                    "-I", build.CSRC, "-o", exe, str(tmp_path / "main.cpp"), "-lpthread"], check=True)
    assert subprocess.run([exe], timeout=60).returncode == 0


def test_no_kernel_is_announced_to_one_gpu_only():
    for f in os.listdir(build.CSRC):
        text = open(os.path.join(build.CSRC, f)).read()
        assert text.count("hipFuncSetAttribute(") == (f == "kernels.h"), f
