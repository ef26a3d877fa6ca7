"""The per-device LDS limit of a kernel, against a HIP runtime of the test's own: raised once on every
device, also by several threads, and tried again after a failure."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2607_03441_amd", "csrc")
PROGRAM = r"""
#include <cstdio>
#include <thread>
#include <vector>
#include "lds_limit.hpp"

static thread_local int device = 0;
static std::atomic<int> calls[70];
static bool fail = false;
extern "C" hipError_t hipGetDevice(int* d) { *d = device; return hipSuccess; }
extern "C" hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int value) {
  if (fail || value != 81920) return hipErrorInvalidValue;
  ++calls[device];
  return hipSuccess;
}

int main() {
  attt::LdsLimit limit, other;
  int kernel = 0;
  fail = true;
  if (limit.raise(&kernel, 81920) == hipSuccess) return 1;
  fail = false;
  for (int d : {0, 1, 0, 1, 7, 7, 66, 66}) {
    device = d;
    if (limit.raise(&kernel, 81920) != hipSuccess) return 2;
  }
  if (calls[0] != 1 || calls[1] != 1 || calls[7] != 1 || calls[66] != 2) return 3;
  device = 0;
  if (other.raise(&kernel, 81920) != hipSuccess || calls[0] != 2) return 4;
  attt::LdsLimit shared;
  std::vector<std::thread> threads;
  for (int t = 0; t < 8; ++t)
    threads.emplace_back([&, t] {
      device = 20 + t % 2;
      for (int i = 0; i < 100; ++i) shared.raise(&kernel, 81920);
    });
  for (auto& t : threads) t.join();
  for (int d : {20, 21})
    if (calls[d] < 1 || calls[d] > 4) return 5;  // at most once per thread that found it unset
  std::puts("ok");
  return 0;
}
"""


@pytest.mark.skipif(not shutil.which("g++"), reason="no host compiler")
def test_raised_once_per_device(tmp_path):
    src, exe = tmp_path / "limit.cpp", tmp_path / "limit"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I", CSRC, str(src),
                    "-o", str(exe)], check=True, capture_output=True, text=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout == "ok\n", r


def test_every_launcher_uses_it():
    """No launcher keeps a flag of its own for the whole process."""
    for name in os.listdir(CSRC):
        if name.endswith(".hip"):
            text = open(os.path.join(CSRC, name)).read()
            assert "hipFuncSetAttribute" not in text, name
