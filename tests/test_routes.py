"""Which kernels a call is sent to, where a rule by sizes decides it: the library's own host
functions, called from a small C++ program built here (CPU only, nothing is launched)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PREC = {"fp32": 0, "bf16": 1, "fp64": 2, "fp16": 3}

PROBE = r"""
#include "omp_internal.h"
#include <cstdio>
using namespace bomp;
int main() {
  long M, N, B;
  int S, prec;
  char *mem = reinterpret_cast<char *>(1 << 20);  // addresses only, nothing is read
  while (std::scanf("%d %ld %ld %ld %d", &prec, &M, &N, &B, &S) == 5) {
    const WorkView w = work_view(mem, M, N, B, S, prec, 0);
    std::printf("%d %d\n", w.tile_cfg, solve_loop_signals(dict_view(mem, M, N, prec), w, prec));
  }
}
"""


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    """Function from [(precision, M, N, B, S)] to [(tile configuration chosen by shape,
    signals per workgroup of the one-launch solve or 0)]."""
    pkg = os.path.join(ROOT, "paper_2407_06434_amd")
    d = tmp_path_factory.mktemp("routes")
    (d / "probe.cpp").write_text(PROBE)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    lib = os.path.join(pkg, "libbatched_omp.so")
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"), "-I",
                    os.path.join(pkg, "csrc"), str(d / "probe.cpp"), lib, "-L", os.path.join(rocm, "lib"), "-lamdhip64",
                    f"-Wl,-rpath,{pkg}:{os.path.join(rocm, 'lib')}", "-o", str(d / "probe")], check=True)

    def ask(cases):
        text = "".join(f"{PREC[p]} {M} {N} {B} {S}\n" for p, M, N, B, S in cases)
        out = subprocess.run([str(d / "probe")], input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]

    return ask


def test_half_tiles_only_where_they_relieve_the_fullest_cu(routes):
    """128 x 64 tiles run where the CU with the most work has less of it with them (or both
    halves of its one tile); with 641 to 767 whole tiles they were up to 15% slower."""
    up = lambda x: (x + 255) // 256 * 2  # 128-wide tiles of the padded size
    cases = [(p, M, N, B, 12) for p in ("fp32", "bf16", "fp16") for M in (64, 3000) for N in (200, 500, 1024, 2304, 4864)
             for B in range(256, 25000, 509)]
    for (p, M, N, B, _), (cfg, _) in zip(cases, routes(cases)):
        t = up(N) * up(B)
        if t // 4 >= 192:
            assert cfg == 3, (p, M, N, B)
            continue
        most_whole, most_half = -(-t // 256), -(-2 * t // 256)
        if 128 < t <= 256:
            assert cfg == (1 if p == "fp32" and M == 3000 else 5), (p, M, N, B)
        else:
            assert cfg == (5 if most_half < 2 * most_whole else 1), (p, M, N, B, t)
    assert [c for c, _ in routes([("bf16", 1024, 1024, 11000, 12), ("bf16", 2500, 2304, 5120, 12),
                                  ("bf16", 256, 1024, 9984, 12)])] == [1, 1, 5]
