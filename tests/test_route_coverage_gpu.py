"""The kernels that larger calls run, on sizes where small calls take the one-launch solve: a
named tile configuration keeps a call on the step-by-step kernels and their graphs."""
import numpy as np
import pytest

from tests import parity

pytestmark = pytest.mark.gpu
KEYS = ("support", "coef", "status", "rnorm")


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def _solve(omp, A, Y, S, prec, d, tile, **kw):
    return omp.solve(A, Y, S, precision=prec, dictionary=d, tile_config=tile, **kw)


@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp16"])
def test_step_graph_replays_match_direct_launches(prec):
    """The residual-vector forms' replayed graph against the direct launches, on every replay,
    with other eager work, a timed call and synchronisations between."""
    torch = _torch()
    from paper_2407_06434_amd import omp, workloads
    w = workloads.batched_256x1024(B=300)
    A, Y = torch.from_numpy(w.A).cuda(), torch.from_numpy(w.Y).cuda()
    d = omp.Dictionary(A, prec)
    print(f"case step graph replays {prec}", flush=True)
    ref = _solve(omp, A, Y, w.S, prec, d, 1, graph=False)
    ref = {k: getattr(ref, k).clone() for k in KEYS + ("X",)}
    ws = torch.empty(omp.workspace_bytes(w.M, w.N, w.B, w.S, prec, with_dict=True, tile_config=1), dtype=torch.uint8,
                     device="cuda")
    out = None
    for rep in range(5):
        out = _solve(omp, A, Y, w.S, prec, d, 1, workspace=ws, out=out, timing={} if rep == 2 else None)
        torch.cuda.synchronize()
        for k in ref:
            assert torch.equal(getattr(out, k), ref[k]), (rep, k)
        _solve(omp, A, Y[:50], 8, prec, d, 3, graph=False)
        out.X.zero_()
        out.support.fill_(-7)
        torch.cuda.synchronize()


def test_step_graph_eviction_with_solves_in_flight():
    """24 argument sets, more than the 16 cached graphs, enqueued without a host
    synchronisation: an evicted graph goes only after its last launch."""
    torch = _torch()
    from paper_2407_06434_amd import omp, workloads
    w = workloads.custom(96, 320, 150, 12, seed=19, k_true=12)
    A, Y = torch.from_numpy(w.A).cuda(), torch.from_numpy(w.Y).cuda()
    d = omp.Dictionary(A, "fp32")
    print("case step graph eviction", flush=True)
    ref = _solve(omp, A, Y, w.S, "fp32", d, 1, graph=False)
    outs = [_solve(omp, A, Y, w.S, "fp32", d, 1) for _ in range(24)]  # fresh outputs: a new argument set each
    torch.cuda.synchronize()
    for i, o in enumerate(outs):
        for k in KEYS + ("X",):
            assert torch.equal(getattr(o, k), getattr(ref, k)), (i, k)


@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("M,N,B,S", [(200, 700, 48, 30), (1000, 500, 44, 40), (640, 700, 50, 64), (512, 1000, 40, 24)])
def test_residual_formed_in_the_step_solve(orc, M, N, B, S, prec):
    """The step solve that forms the residual itself, with the former residual in registers for
    512 < M <= 1024: every signal against the oracle."""
    torch = _torch()
    from paper_2407_06434_amd import omp, workloads
    w = workloads.custom(M, N, B, S, seed=3 * M + N, k_true=S)
    A, Y = torch.from_numpy(w.A).cuda(), torch.from_numpy(w.Y).cuda()
    print(f"case residual in the step solve M={M} N={N} B={B} S={S} {prec}", flush=True)
    r = _solve(omp, A, Y, S, prec, None, 1)
    rep = parity.check(w, {k: getattr(r, k).cpu().numpy() for k in KEYS + ("X",)}, orc)
    assert rep["passed"] == w.B


@pytest.mark.parametrize("prec,M,N,B,S", [("fp32", 640, 700, 300, 20), ("fp32", 1000, 500, 44, 40), ("fp32", 1000, 1000, 1000, 6),
                                          ("fp32", 513, 257, 513, 33), ("bf16", 1000, 200, 500, 24),
                                          ("fp16", 1000, 200, 100, 24), ("bf16", 700, 300, 2048, 9),
                                          ("bf16", 64, 2048, 8192, 6), ("fp16", 50, 2000, 7900, 12),
                                          ("bf16", 128, 1000, 5000, 7), ("fp16", 180, 700, 6000, 7)])
def test_one_launch_solve_equals_the_steps(prec, M, N, B, S):
    """Signals of more than 512 samples, where the steps hold the residual in registers, and
    batches whose own tiles would be 256 x 256."""
    torch = _torch()
    from paper_2407_06434_amd import omp
    g = torch.Generator(device="cuda").manual_seed(M + B)
    A = torch.randn((N, M), generator=g, device="cuda") * (0.5 + torch.rand((N, 1), generator=g, device="cuda"))
    Y = torch.randn((B, M), generator=g, device="cuda")
    caps = torch.randint(0, S + 1, (B,), generator=g, device="cuda", dtype=torch.int32)
    d = omp.Dictionary(A, prec)
    print(f"case one launch against steps {prec} M={M} N={N} B={B} S={S}", flush=True)
    one, steps = (_solve(omp, A, Y, S, prec, d, t, S_per_signal=caps) for t in (0, 1))
    for k in KEYS + ("X",):
        assert torch.equal(getattr(one, k), getattr(steps, k)), k


@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("M,N,B", [(512, 2048, 600), (1100, 300, 1200), (40, 1000, 6300), (100, 1000, 9900)])
def test_tiles_chosen_by_shape_equal_the_others(prec, M, N, B):
    """128 x 64 tiles (the third shape: 128 x 128) against 256 x 256 and 256 x 128, beyond the
    one-launch solve."""
    torch = _torch()
    from paper_2407_06434_amd import omp
    g = torch.Generator(device="cuda").manual_seed(N + B)
    A = torch.randn((N, M), generator=g, device="cuda")
    Y = torch.randn((B, M), generator=g, device="cuda")
    d = omp.Dictionary(A, prec)
    print(f"case tiles {prec} M={M} N={N} B={B}", flush=True)
    ref = _solve(omp, A, Y, 10, prec, d, 0)
    for t in (1, 2, 3, 4):
        got = _solve(omp, A, Y, 10, prec, d, t)
        for k in ("support", "coef", "rnorm"):
            assert torch.equal(getattr(ref, k), getattr(got, k)), (t, k)
