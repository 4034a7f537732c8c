"""Algorithm v0 with its state in memory (FP32, and FP64 beyond the register path): the pick's
correlation is read by every thread of the workgroup and overwritten by one of them."""
import numpy as np
import pytest

from tests import parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("form,M,N,B,S", [("fp64", 300, 600, 2000, 40), ("fp64", 100, 400, 900, 90), ("fp64", 200, 1100, 700, 24),
                                          ("v0", 256, 1024, 2000, 32), ("v0", 100, 300, 700, 90)])
def test_every_thread_updates_with_the_same_coefficient(orc, form, M, N, B, S):
    """Runs give the same bits each time, and the picks are the oracle's; in FP32 those past the
    true sparsity, on residuals near rounding, as far as FP32 resolves them."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2407_06434_amd import omp, workloads
    w = workloads.custom(M, N, B, S, seed=M + S, k_true=S // 2)
    prec, kw = ("fp64", {}) if form == "fp64" else ("fp32", {"v0": True})
    A, Y = torch.from_numpy(w.A).cuda(), torch.from_numpy(w.Y).cuda()
    d = omp.Dictionary(A, prec)
    print(f"case v0 picks {form} M={M} N={N} B={B} S={S}", flush=True)
    runs = [omp.solve(A, Y, S, precision=prec, dictionary=d, **kw) for _ in range(4)]
    for k in ("support", "coef", "status", "rnorm"):
        for r in runs[1:]:
            assert torch.equal(getattr(runs[0], k), getattr(r, k)), k
    got = {k: getattr(runs[0], k).cpu().numpy() for k in ("support", "coef", "status", "rnorm", "X")}
    rep = parity.check(w, got, orc, idx=np.random.default_rng(S).choice(B, 150, replace=False),
                       residual_rounding=form == "v0")
    assert rep["passed"] + rep["unresolved_fp32"] == 150
