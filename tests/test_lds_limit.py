"""The helper that raises a kernel's LDS limit, compiled here against a stand-in for the HIP
runtime that records the calls (CPU only)."""
import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_06434_amd", "csrc")

RUNTIME = """#pragma once
#include <map>
enum hipError_t { hipSuccess };
enum hipFuncAttribute { hipFuncAttributeMaxDynamicSharedMemorySize };
inline int device = 0;
inline std::map<std::pair<int, const void *>, int> limits;
inline hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute, int v) {
  limits[{device, f}] = v;
  return hipSuccess;
}
"""

PROGRAM = """#include "lds_limit.h"
template <int TILE> void kernel(const float *, int tile) { (void)tile; }
int main() {
  using bomp::lds_limit;
  auto set = [](int dev, void (*k)(const float *, int)) { return limits[{dev, reinterpret_cast<const void *>(k)}]; };
  // two kernels of one type, the smaller one first
  lds_limit(kernel<1>, 66 * 1024);
  lds_limit(kernel<2>, 130 * 1024);
  if (set(0, kernel<1>) != 66 * 1024 || set(0, kernel<2>) != 130 * 1024) return 1;
  device = 1;  // the limit of one device says nothing about another
  lds_limit(kernel<1>, 66 * 1024);
  if (set(1, kernel<1>) != 66 * 1024) return 2;
  lds_limit(kernel<2>, 64 * 1024);  // within every kernel's own limit
  return set(1, kernel<2>) == 0 ? 0 : 3;
}
"""


def test_every_kernel_and_device_gets_its_limit(tmp_path):
    (tmp_path / "hip").mkdir()
    (tmp_path / "hip" / "hip_runtime.h").write_text(RUNTIME)
    (tmp_path / "program.cpp").write_text(PROGRAM)
    exe = tmp_path / "program"
    subprocess.run(["g++", "-std=c++17", "-I", str(tmp_path), "-I", CSRC, str(tmp_path / "program.cpp"), "-o", str(exe)],
                   check=True)
    assert subprocess.run([str(exe)]).returncode == 0
