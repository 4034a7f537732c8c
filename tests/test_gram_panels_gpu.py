"""The Gram-domain select through panels of G in LDS against the select through the caches:
a batch is solved whole (panels) and in parts of under 512 signals (caches)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("M,N,B,S", [(16, 32, 512, 3), (64, 250, 515, 9), (100, 300, 1021, 17), (300, 1024, 777, 40),
                                     (128, 1000, 2053, 70)])
def test_panels_equal_slices_bit_for_bit(M, N, B, S, ties):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_06434_amd import omp
    g = np.random.default_rng(M + B)
    A = g.normal(size=(N, M)).astype(np.float32)
    A[N // 2] = A[1]  # an exact tie, decided by the index
    A[N - 1] = 0.0    # never selectable
    Y = g.normal(size=(B, M)).astype(np.float32)
    Y[3] = 0.0        # stops before its first pick
    caps = torch.from_numpy(g.integers(0, S + 1, B).astype(np.int32)).cuda()
    At, Yt = torch.from_numpy(A).cuda(), torch.from_numpy(Y).cuda()
    d = omp.Dictionary(At, "fp32")
    print(f"case gram panels M={M} N={N} B={B} S={S} ties={ties}", flush=True)

    def solve(lo, hi):
        r = omp.solve(At, Yt[lo:hi], S, dictionary=d, gram_domain=True, flag_near_ties=ties,
                      S_per_signal=caps[lo:hi].contiguous())
        return [t.cpu().numpy() for t in r]

    whole = solve(0, B)
    parts = [solve(lo, min(B, lo + 511)) for lo in range(0, B, 511)]
    for w, p in zip(whole, zip(*parts)):
        assert np.array_equal(w, np.concatenate(p))
