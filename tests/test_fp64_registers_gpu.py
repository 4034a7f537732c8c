"""The FP64 form's whole solve with D in registers against its parts with D in memory
(which a timed call launches one by one): supports, coefficients and status bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("M,N,B,S,eps", [(3, 5, 3, 3, 0.0), (40, 256, 9, 8, 0.0), (64, 257, 33, 9, 0.2), (50, 513, 20, 16, 0.0),
                                         (130, 700, 65, 17, 0.1), (200, 1024, 300, 32, 0.0), (150, 500, 40, 33, 0.0),
                                         (90, 512, 21, 64, 0.0), (64, 1000, 12, 40, 0.0), (256, 1500, 30, 20, 0.05)])
def test_registers_equal_memory_bit_for_bit(M, N, B, S, eps, ties):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_06434_amd import omp
    g = np.random.default_rng(M + N + B)
    A = g.normal(size=(N, M)).astype(np.float32)
    if N > 8:
        A[N // 2] = A[1]               # an exact tie
        A[N - 1] = 0.0                 # never selectable
        A[N // 3] = A[2] * (1 + 1e-7)  # dependent once its twin is in
    Y = g.normal(size=(B, M)).astype(np.float32)
    Y[B // 2] = 0.0
    Y[0] = A[2] + A[0] if N > 2 else Y[0]  # explained exactly: the residual is formed explicitly
    At, Yt = torch.from_numpy(A).cuda(), torch.from_numpy(Y).cuda()
    caps = torch.from_numpy(g.integers(0, S + 1, B).astype(np.int32)).cuda()
    caps[0] = S
    e = torch.from_numpy((eps * np.linalg.norm(Y.astype(np.float64), axis=1)).astype(np.float32)).cuda()
    d = omp.Dictionary(At, "fp64")
    print(f"case fp64 registers M={M} N={N} B={B} S={S} eps={eps} ties={ties}", flush=True)
    whole, parts = (omp.solve(At, Yt, S, precision="fp64", dictionary=d, S_per_signal=caps, eps_per_signal=e,
                              flag_near_ties=ties, timing=t) for t in (None, {}))
    # signal 0's last residuals are rounding noise: its later picks follow the norm's summation order
    for a, b in ((whole.support, parts.support), (whole.status, parts.status), (whole.coef, parts.coef)):
        assert torch.equal(a[1:], b[1:])
    assert torch.equal(whole.support[0, :2].sort().values, parts.support[0, :2].sort().values)
    assert torch.allclose(whole.rnorm[1:], parts.rnorm[1:], rtol=1e-6, atol=0.0)


@pytest.mark.parametrize("M,N,B,S", [(16, 30, 37, 16), (30, 600, 50, 30), (64, 256, 40, 60), (100, 900, 33, 32),
                                     (300, 500, 20, 64)])
def test_residual_norms_bit_for_bit(M, N, B, S):
    """Both paths give the same norms for every signal, also where they are rounding noise
    (S = M, or signals that 5 atoms explain: there a stop near eps hangs on the last bits)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_06434_amd import omp
    g = np.random.default_rng(M + N)
    A = (g.normal(size=(N, M)) / np.sqrt(M)).astype(np.float32)
    Y = g.normal(size=(B, M)).astype(np.float32)
    Y[: B // 3] = A[np.argsort(g.random((B // 3, N)), axis=1)[:, :5]].sum(axis=1)
    At, Yt = torch.from_numpy(A).cuda(), torch.from_numpy(Y).cuda()
    d = omp.Dictionary(At, "fp64")
    print(f"case fp64 norms M={M} N={N} B={B} S={S}", flush=True)
    for eps in (0.0, 1e-7, 0.3):
        whole, parts = (omp.solve(At, Yt, S, eps, precision="fp64", dictionary=d, timing=t) for t in (None, {}))
        for k in ("support", "status", "coef", "rnorm", "X"):
            assert torch.equal(getattr(whole, k), getattr(parts, k)), (eps, k)
