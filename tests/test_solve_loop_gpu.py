"""The one-launch solve of small batches against the step-by-step kernels (which a call
that names a tile configuration runs): supports, coefficients and status bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("M,N,B,S,eps", [(1, 3, 4, 1, 0.0), (16, 32, 1, 5, 0.0), (31, 64, 256, 31, 0.0),
                                         (65, 65, 257, 12, 0.3), (100, 300, 37, 12, 0.1), (200, 513, 513, 64, 0.0),
                                         (64, 250, 1500, 9, 0.2), (256, 1024, 771, 40, 0.0), (129, 512, 2048, 20, 0.05),
                                         (200, 1024, 300, 33, 0.0), (60, 2048, 100, 16, 0.0),
                                         (64, 1000, 4100, 8, 0.0), (30, 2048, 2049, 25, 0.1), (300, 301, 7937, 11, 0.2)])
def test_loop_equals_steps_bit_for_bit(M, N, B, S, eps, prec):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_06434_amd import omp
    g = np.random.default_rng(M + N + B)
    A = (g.normal(size=(N, M)) * g.uniform(0.5, 2.0, (N, 1))).astype(np.float32)
    if N > 8:
        A[N // 2] = A[1]      # an exact tie
        A[N - 1] = 0.0        # never selectable
        A[N // 3] *= 1e-12    # a tiny atom
    Y = g.normal(size=(B, M)).astype(np.float32)
    Y[B // 2] = 0.0
    if B > 5:
        Y[4, M // 2] = np.nan
        Y[3] *= 1e15
    At, Yt = torch.from_numpy(A).cuda(), torch.from_numpy(Y).cuda()
    caps = torch.from_numpy(g.integers(max(0, S - 3), S + 1, B).astype(np.int32)).cuda()
    e = torch.from_numpy((eps * np.linalg.norm(np.nan_to_num(Y).astype(np.float64), axis=1)).astype(np.float32)).cuda()
    d = omp.Dictionary(At, prec)
    print(f"case loop M={M} N={N} B={B} S={S} eps={eps} {prec}", flush=True)
    loop, steps = (omp.solve(At, Yt, S, precision=prec, dictionary=d, S_per_signal=caps, eps_per_signal=e, tile_config=c)
                   for c in (0, 1))
    assert torch.equal(loop.support, steps.support)
    assert torch.equal(loop.status, steps.status)
    assert torch.equal(loop.coef, steps.coef) and torch.equal(loop.X, steps.X)
    # ||r||^2 is summed over the lanes in another order where the steps keep r in slices
    assert torch.allclose(loop.rnorm, steps.rnorm, rtol=1e-6, atol=0.0)
