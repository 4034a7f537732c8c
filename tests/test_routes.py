"""Which kernels a call is sent to, where a rule by sizes decides it: the library's own host
functions, called from a small C++ program built here (CPU only, nothing is launched)."""
import ctypes
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PREC = {"fp32": 0, "bf16": 1, "fp64": 2, "fp16": 3}

PROBE = r"""
#include "batched_omp.h"
#include "omp_internal.h"
#include "mlp_internal.h"
#include <cstdio>
using namespace bomp;
int main(int argc, char **) {
  long M, N, B;
  int S, prec;
  if (argc > 1) {  // problems side by side
    omp_problem_t p[OMP_MAX_PROBLEMS] = {};
    omp_dict_t d[OMP_MAX_PROBLEMS] = {};
    int n = 0;
    for (; std::scanf("%d %ld %ld %ld %d", &prec, &M, &N, &B, &S) == 5; ++n) {
      d[n].precision = prec;
      d[n].M = M;
      d[n].N = N;
      p[n].dict = &d[n];
      p[n].B = B;
    }
    fill_schedule(p, n, 8192);
    for (int i = 0; i < n; ++i) std::printf("%d %d\n", p[i].tile_config, p[i].slots);
    return 0;
  }
  char *mem = reinterpret_cast<char *>(1 << 20);  // addresses only, nothing is read
  while (std::scanf("%d %ld %ld %ld %d", &prec, &M, &N, &B, &S) == 5) {
    const WorkView w = work_view(mem, M, N, B, S, prec, 0);
    std::printf("%d %d %d %ld\n", w.tile_cfg, solve_loop_signals(dict_view(mem, M, N, prec), w, prec),
                work_view(mem, M, N, B, S, prec, 1).tile_cfg, (long)loss_blocks(round_up(B, BPAD), N));
  }
}
"""


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    """Function from [(precision, M, N, B, S)] to [(tile configuration chosen by shape,
    signals per workgroup of the one-launch solve or 0, tile that configuration 1 stands
    for, workgroups of a network's loss product of B rows and N columns)], and with `multi` to the (tile configuration or 0 for the choice by shape, slots) of
    these problems run side by side."""
    pkg = os.path.join(ROOT, "paper_2407_06434_amd")
    d = tmp_path_factory.mktemp("routes")
    (d / "probe.cpp").write_text(PROBE)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    lib = os.path.join(pkg, "libbatched_omp.so")
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"), "-I",
                    os.path.join(pkg, "csrc"), "-I", os.path.join(ROOT, "include"), str(d / "probe.cpp"), lib, "-L", os.path.join(rocm, "lib"), "-lamdhip64",
                    f"-Wl,-rpath,{pkg}:{os.path.join(rocm, 'lib')}", "-o", str(d / "probe")], check=True)

    def ask(cases, multi=False):
        text = "".join(f"{PREC[p]} {M} {N} {B} {S}\n" for p, M, N, B, S in cases)
        out = subprocess.run([str(d / "probe")] + ["multi"] * multi, input=text, capture_output=True, text=True, check=True).stdout
        return [tuple(map(int, line.split())) for line in out.splitlines()]

    return ask


def test_half_tiles_only_where_they_relieve_the_fullest_cu(routes):
    """128 x 64 tiles run where the CU with the most work has less of it with them (or both
    halves of its one tile); with 641 to 767 whole tiles they were up to 15% slower."""
    up = lambda x: (x + 255) // 256 * 2  # 128-wide tiles of the padded size
    cases = [(p, M, N, B, 12) for p in ("fp32", "bf16", "fp16") for M in (64, 3000) for N in (200, 500, 1024, 2304, 4864)
             for B in range(256, 25000, 509)]
    for (p, M, N, B, _), (cfg, _, one, _) in zip(cases, routes(cases)):
        t = up(N) * up(B)
        if t // 4 >= 192:
            assert cfg == 3, (p, M, N, B)
            continue
        assert one == cfg  # what a schedule that names configuration 1 (the tuner's) gets
        most_whole, most_half = -(-t // 256), -(-2 * t // 256)
        if 128 < t <= 256:
            assert cfg == (1 if p == "fp32" and M == 3000 else 5), (p, M, N, B)
        else:
            assert cfg == (5 if most_half < 2 * most_whole else 1), (p, M, N, B, t)
    assert [r[0] for r in routes([("bf16", 1024, 1024, 11000, 12), ("bf16", 2500, 2304, 5120, 12),
                                  ("bf16", 256, 1024, 9984, 12)])] == [1, 1, 5]


def test_one_launch_solve_where_it_is_the_faster_one(routes):
    """The one-launch solve has every workgroup read the whole dictionary at each step: not
    beyond 4 MiB in FP32 (up to 7% slower than the steps at 1024 x 2048), nor over wide
    dictionaries with fewer signals than CUs would share their atoms."""
    yes = [("fp32", 1000, 1000, 1, 24), ("fp32", 1000, 1000, 1024, 24), ("fp32", 512, 2048, 256, 24),
           ("fp32", 256, 2048, 512, 24), ("fp32", 64, 256, 100, 8), ("fp32", 1024, 200, 1500, 24),
           ("bf16", 256, 1000, 1, 20), ("bf16", 64, 2000, 1, 16), ("fp16", 128, 2000, 64, 20), ("bf16", 60, 100, 8192, 20)]
    no = [("fp32", 1024, 2048, 1, 24), ("fp32", 1024, 2048, 512, 24), ("fp32", 900, 1900, 256, 24),
          ("fp32", 512, 2000, 300, 16), ("bf16", 128, 2000, 1, 20), ("fp16", 128, 2000, 15, 16),
          ("fp32", 256, 1024, 2049, 24), ("bf16", 1000, 500, 40, 20), ("fp64", 64, 256, 100, 8)]
    got = [r[1] for r in routes(yes + no)]
    for case, g in zip(yes + no, got):
        assert (g > 0) == (case in yes), (case, g)
        assert g in (0, -(-case[3] // 256)), (case, g)


def test_default_slots_by_the_work_of_an_iteration():
    """Problems that name no slots get 8192 only where an iteration over them costs little
    more than over 4096: an FP32 product over 1024 x 4096 made that default up to half as
    slow again. Read off the workspace the problems ask for."""
    from paper_2407_06434_amd import omp
    lib = omp.load()
    o = omp.OmpMultiOptsStruct()

    def size(prec, shapes, slots):
        arr = (omp.OmpProblemStruct * len(shapes))()
        keep = []
        for p, (M, N, B) in zip(arr, shapes):
            d = omp.OmpDictStruct(0x4F4D5044, PREC[prec], M, N, 0, 0, 1 << 20, 1 << 20, 1 << 40)
            keep.append(d)
            p.dict = ctypes.pointer(d)
            p.Y = p.support_out = 1 << 20
            p.B, p.ldy, p.S, p.slots = B, M, 16, slots
        o.precision = PREC[prec]
        return lib.omp_multi_workspace_size(arr, len(shapes), ctypes.byref(o))

    for prec, M, N, B, slots in (
            ("fp32", 64, 256, 5000, 8192), ("fp32", 128, 768, 20000, 8192), ("fp32", 200, 768, 20000, 8192),
            ("fp32", 1000, 100, 20000, 8192), ("fp32", 256, 1024, 20000, 4096), ("fp32", 512, 2048, 20000, 4096),
            ("fp32", 1024, 4096, 5000, 4096), ("fp32", 32, 4096, 20000, 4096), ("fp32", 64, 2048, 6500, 4096),
            ("bf16", 256, 1024, 20000, 8192), ("bf16", 512, 2048, 10000, 8192), ("fp16", 1024, 2048, 6500, 8192),
            ("bf16", 256, 2048, 5000, 4096), ("bf16", 512, 4096, 20000, 4096), ("fp16", 1024, 2500, 20000, 4096)):
        one = [(M, N, B)]
        assert size(prec, one, 4096) < size(prec, one, 8192)
        assert size(prec, one, 0) == size(prec, one, slots), (prec, M, N, B)
    # problems run side by side: one that does better with 4096 holds the others to it
    for prec, slots in (("fp32", 4096), ("bf16", 8192)):
        two = [(128, 512, 10000), (512, 2048, 10000)]
        assert size(prec, two, 0) == size(prec, two, slots), prec


def test_half_tiles_beside_other_problems(routes):
    """FP32 problems side by side whose products are more than two 128 x 128 tiles a CU keep
    whole tiles, also where one of them alone would run on halves (8% slower then)."""
    pair = [("fp32", 128, 512, 10000, 32), ("fp32", 512, 2048, 10000, 32)]
    assert routes(pair, multi=True) == [(6, 4096), (0, 4096)]  # 6: whole 128 x 128 tiles
    assert routes(pair[:1], multi=True) == [(0, 8192)]
    assert routes([("fp32", 64, 256, 10000, 16), ("fp32", 256, 1024, 10000, 32)], multi=True) == [(0, 4096)] * 2
    assert routes(pair[:1] + [("fp32", 512, 2048, 0, 32)], multi=True) == [(0, 8192)] * 2
    assert routes([("bf16", *c[1:]) for c in pair], multi=True) == [(0, 8192)] * 2


def test_loss_products_keep_128_wide_tiles(routes):
    """The loss epilogue on 256 x 256 tiles spilled its registers: four times slower than on
    128 x 128, which large products run on; small ones run on 64 x 64."""
    for B, n, t in ((5000, 4096, 128), (16384, 1024, 128), (20000, 4096, 128), (1024, 1024, 64), (100, 256, 64)):
        Bp = -(-B // 256) * 256
        assert routes([("bf16", 64, n, B, 8)])[0][3] == (Bp // t) * (n // t), (B, n)
