"""The device code's division by a host-known divisor, against the
processor's own, on the CPU: every divisor up to 3000 and others over the
32-bit range, at the multiples' edges and at random values."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = r"""
#include <hip/hip_runtime.h>
#include <cstdio>
#include <random>
#include "%s"
thread_local Dim3 threadIdx, blockIdx, blockDim, gridDim;
using namespace pcsdf;
int main() {
  std::mt19937_64 r(1);
  long bad = 0;
  auto check = [&](uint32_t d) {
    const FastDiv f = fast_div(d);
    auto one = [&](uint32_t n) { bad += quotient(n, f) != n / d; };
    for (uint32_t k : {0u, 1u, 2u, 1000u, 0xFFFFFFFFu / d})
      for (int e = -2; e <= 2; ++e) one(k * d + (uint32_t)e);
    one(0xFFFFFFFFu);
    for (int q = 0; q < 200; ++q) one((uint32_t)r() >> (q %% 32));
  };
  for (uint32_t d = 1; d <= 3000; ++d) check(d);
  for (int q = 0; q < 20000; ++q) check(((uint32_t)r() >> (q %% 32)) | 1u);
  for (int s = 0; s < 32; ++s)
    for (int e = -1; e <= 1; ++e)
      if ((1u << s) + (uint32_t)e) check((1u << s) + (uint32_t)e);
  check(0xFFFFFFFFu);
  printf("bad %%ld\n", bad);
}
"""


def test_fast_division(tmp_path):
    head = os.path.join(HERE, "..", "paper_2201_05058_amd", "csrc",
                        "device_common.h")
    src, exe = str(tmp_path / "d.cpp"), str(tmp_path / "d")
    with open(src, "w") as f:
        f.write(SRC % os.path.abspath(head))
    subprocess.run(["g++", "-O1", "-std=c++20",
                    "-I" + os.path.join(HERE, "cpu_device"), "-o", exe, src],
                   check=True)
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0 and "bad 0" in out.stdout, out.stdout
