"""Proposal and least-squares check at the edges of their unrolled factor lengths (16, 32,
64), with tied scores and signals that are no whole number of 16-byte chunks."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _torch():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.mark.parametrize("S,M,N", [(1, 64, 256), (7, 66, 256), (16, 255, 256), (17, 300, 512), (32, 256, 1024),
                                   (33, 301, 512), (64, 520, 2048)])
def test_proposal_and_check_at_the_edges(S, M, N):
    """Every signal gets the same proposal: S - 2 marked atoms with tied scores, then the
    lowest of the unmarked ones, which are tied too. Accepted signals carry the FP64
    least-squares coefficients to the suite's 1e-4 of each coefficient."""
    torch = _torch()
    from oracle import learned_oracle as lo
    from paper_2407_06434_amd import omp, workloads
    B = 67
    g = np.random.default_rng(S + M)
    A = (g.normal(size=(N, M)) / np.sqrt(M)).astype(np.float32)
    p = workloads.mlp_init_params(N, 256, N)
    p["W3"][:] = 0.0
    p["b3"][:] = 0.0
    p["b3"][np.sort(g.choice(N, max(S - 2, 1), replace=False))] = 1.0
    P = lo.top_s(np.tile(p["b3"].astype(np.float64), (B, 1)), S)
    x = g.choice([-1, 1], size=(B, S)) * (1 + np.abs(g.normal(size=(B, S))))
    Y = (x @ A[P[0]].astype(np.float64) + 0.01 * g.normal(size=(B, M)) / np.sqrt(M)).astype(np.float32)
    Y[B // 2:] += g.normal(size=(B - B // 2, M)).astype(np.float32)  # not on the proposal: plain OMP's
    eps = np.full(B, 0.1, np.float32)
    dev = torch.device("cuda:0")
    Yb = torch.full((B, M + 3), float("nan"), device=dev)  # rows at every alignment
    Yb[:, :M] = torch.from_numpy(Y).to(dev)
    At = torch.from_numpy(A).to(dev)
    d = omp.Dictionary(At, "bf16")
    print(f"case proposal edges S={S} M={M} N={N}", flush=True)
    out, nacc = omp.learned_solve(d, omp.MLP(p), Yb[:, :M], S, eps_per_signal=torch.from_numpy(eps).to(dev))
    X, rn, ok = lo.ls_check(A, Y, P, eps)
    acc = (out.status.cpu().numpy() & omp.SIG_LEARNED) != 0
    assert np.array_equal(acc, ok) and nacc == int(ok.sum()) == B // 2
    assert np.array_equal(out.support.cpu().numpy()[acc], P[acc])
    scale = np.maximum(np.abs(X[acc]), 1e-2 * np.abs(X[acc]).max(axis=1, keepdims=True))
    assert np.all(np.abs(out.coef.cpu().numpy()[acc] - X[acc]) <= 1e-4 * scale)
    assert np.allclose(out.rnorm.cpu().numpy()[acc], rn[acc], rtol=1e-4, atol=1e-6)


@pytest.mark.parametrize("ni,nh,no,B", [(256, 512, 768, 1), (512, 256, 256, 700), (256, 256, 512, 1281),
                                        (768, 256, 256, 2300)])
def test_gradients_at_ragged_batches(ni, nh, no, B):
    """Loss and gradients where the layers differ in size and the batch fills its row groups
    and batch slices unevenly. Tolerances of the suite's gradient test: the same BF16 rounding
    points on both sides, one flipped rounding moves an entry by 2^-8 of its largest term."""
    torch = _torch()
    from oracle import learned_oracle as lo
    from paper_2407_06434_amd import omp, workloads
    g = np.random.default_rng(ni + B)
    p = workloads.mlp_init_params(ni, nh, no, seed=B)
    F = lo.bf16_round(np.abs(g.normal(size=(B, ni))))
    sup = np.argsort(g.random((B, no)), axis=1)[:, :9].astype(np.int32)
    sup[0, 4:] = -1
    dev = torch.device("cuda:0")
    bits = (F.astype(np.float32).view(np.uint32) >> 16).astype(np.uint16).view(np.int16)
    net = omp.MLP(p)
    print(f"case gradients ni={ni} nh={nh} no={no} B={B}", flush=True)
    loss, got = net.grad(torch.from_numpy(bits).to(dev), torch.from_numpy(sup).to(dev))
    want_loss, want = lo.backward({k: v.astype(np.float64) for k, v in p.items()}, F, lo.multi_hot(sup, no),
                                  lo.bf16_round)
    assert abs(float(loss) - want_loss) <= 1e-3 * abs(want_loss)
    for k in want:
        e = got[k].cpu().numpy().astype(np.float64) - want[k]
        assert np.abs(e).max() <= 1e-2 * np.abs(want[k]).max(), k
        assert np.linalg.norm(e) <= 2e-3 * np.linalg.norm(want[k]), k


@pytest.mark.parametrize("value", [float("inf"), float("nan"), 3e38])
@pytest.mark.parametrize("S", [1, 5, 6, 17, 35])
def test_check_reads_the_proposed_atoms_only(S, value):
    """Atom 0 is not finite (or overflows FP32 in a product) and not proposed: whether a
    proposal explains its signal does not depend on it, however S divides into the rounds
    that the check reads atoms in. Every signal is its proposal's combination."""
    torch = _torch()
    from paper_2407_06434_amd import omp, workloads
    M, N, B = 130, 256, 21
    g = np.random.default_rng(S)
    A = (g.normal(size=(N, M)) / np.sqrt(M)).astype(np.float32)
    A[0] = value
    P = np.sort(1 + g.choice(N - 1, S, replace=False))
    p = workloads.mlp_init_params(N, 256, N)
    for k in ("W1", "W2", "W3", "b1", "b2", "b3"):
        p[k][:] = 0.0
    p["b3"][P] = 1.0  # the network proposes these atoms whatever the signal
    Y = (1 + np.abs(g.normal(size=(B, S)))).astype(np.float32) @ A[P]
    dev = torch.device("cuda:0")
    d = omp.Dictionary(torch.from_numpy(A).to(dev), "bf16")
    print(f"case proposed atoms only S={S} value={value}", flush=True)
    out, nacc = omp.learned_solve(d, omp.MLP(p), torch.from_numpy(Y).to(dev), S, 1e-2)
    assert nacc == B
    assert np.array_equal(out.support.cpu().numpy(), np.tile(P, (B, 1)))
