"""The work whose speed this framework is measured on: complete calls of its
public entry points, over the sizes and options its users run.

Four kinds of call:
  solve    batched OMP of one batch over one dictionary (`omp.solve`), in the
           precisions and forms a caller can choose
  multi    uneven batches over several dictionaries in one call (`omp.solve_multi`)
  learned  network proposal, least-squares check and OMP fallback (`omp.learned_solve`)
  grad     forward and backward pass of the proposal network (`omp.MLP.grad`)

Inputs are drawn on the GPU from the seed alone: Gaussian N(0, 1/M) dictionaries
(optionally with atom norms from U[0.5, 2]) and signals with +-(1 + |N(0,1)|)
coefficients on a random support, white noise at a given SNR, the distributions of
the package's own workloads.
"""
from __future__ import annotations

import math

import torch

from paper_2407_06434_amd import omp, workloads

DEVICE = "cuda"


def _solve(name, M, N, B, S, precision, **kw):
    case = {"kind": "solve", "name": name, "M": M, "N": N, "B": B, "S": S, "precision": precision,
            "gram_auto": False, "prepared": True, "dense": True, "snr_db": 30.0, "eps_rel": 0.0, "norms": False}
    case.update(kw)
    return case


def listed():
    return [
        # The smallest everyday call: a batch of 100 short signals (the paper's smallest
        # dictionary), where launches and latency are the whole cost.
        _solve("plain_64x256_B100", 64, 256, 100, 8, "fp32"),
        # A one-off call with ragged sizes and a tolerance: no prepared dictionary, so the
        # norms and the Gram matrix are part of the call.
        _solve("oneoff_100x300_B37", 100, 300, 37, 12, "fp32", prepared=False, eps_rel=0.1),
        # Image patches (Section 4.2 of the paper: 256 x 1024, S = 32) in the default
        # precision, the form left to the library.
        _solve("patches_256x1024_B5000", 256, 1024, 5000, 32, "fp32", gram_auto=True, norms=True),
        # The batched workload with compact outputs in BF16.
        _solve("batched_256x1024_B10000", 256, 1024, 10000, 32, "bf16", dense=False, norms=True),
        # The benchmark workload in the BF16 form.
        _solve("bench_1024x4096_B4096", 1024, 4096, 4096, 64, "bf16"),
        # The same batch in plain FP32, the precision a caller gets by default.
        _solve("fp32_1024x4096_B4096", 1024, 4096, 4096, 64, "fp32"),
        # Face recognition (Section 4.2: 8064 pixels, 1207 training faces): a tall
        # dictionary, FP32 with the form left to the library.
        _solve("faces_8064x1207_B1200", 8064, 1207, 1200, 30, "fp32", gram_auto=True),
        # Audio frames (Section 4.2: 512 x 2048, S = 64) in half-precision storage, stopping
        # on a tolerance.
        _solve("audio_512x2048_B5000", 512, 2048, 5000, 64, "fp16", eps_rel=0.05),
        # The accurate mode: every quantity in FP64.
        _solve("fp64_256x1024_B2000", 256, 1024, 2000, 32, "fp64"),
        # Uneven batches: two dictionaries in one call, every signal with its own sparsity
        # cap and tolerance.
        {"kind": "multi", "name": "uneven_128x512_512x2048", "precision": "bf16", "snr_db": 60.0, "S": 64,
         "M0": 128, "N0": 512, "B0": 10000, "M1": 512, "N1": 2048, "B1": 10000},
        # The learned proposal at inference, with OMP as its judge and fallback.
        {"kind": "learned", "name": "learned_256x1024_B16384", "M": 256, "N": 1024, "H": 1024, "B": 16384, "S": 32,
         "snr_db": 20.0},
        # One training batch of the proposal network: loss and every gradient.
        {"kind": "grad", "name": "grad_1024_B1024", "M": 256, "N": 1024, "H": 1024, "B": 1024, "S": 32,
         "snr_db": 20.0},
    ]


# ---- drawn cases -------------------------------------------------------------

def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# Cost of a solve in multiply-adds, and the bound the largest listed case sets.
def _cost(M, N, B, S):
    return M * N * B * S


_MAX_COST = _cost(1024, 4096, 4096, 64)


def _draw_solve(rng):
    precision = rng.choice(("fp32", "fp32", "bf16", "fp16", "fp64"))
    while True:
        M = _log_int(rng, 16, 2048)
        N = max(32, min(4096, _log_int(rng, max(16, M // 2), 8 * M)))
        B = _log_int(rng, 1, 10000)
        S = max(1, min(64, _log_int(rng, 2, max(3, min(M, N) // 5))))
        # the FP64 form works on 16 N S^2 bytes per signal instead of on the product
        if _cost(M, N, B, S) <= _MAX_COST and (precision != "fp64" or B * N * S * S < (1 << 32)):
            break
    return _solve("", M, N, B, S, precision, gram_auto=precision == "fp32" and rng.random() < 0.4,
                  prepared=rng.random() < 0.8, dense=rng.random() < 0.7, snr_db=float(rng.choice((20, 30, 40))),
                  eps_rel=rng.choice((0.0, 0.0, 0.1, 0.3)), norms=rng.random() < 0.5)


def _draw_multi(rng):
    case = {"kind": "multi", "precision": rng.choice(("bf16", "fp32")), "snr_db": 60.0, "S": rng.choice((16, 32, 64))}
    for i in range(2):
        M = _log_int(rng, 5 * case["S"], 512)
        case.update({f"M{i}": M, f"N{i}": _log_int(rng, 2 * M, 4 * M), f"B{i}": _log_int(rng, 50, 10000)})
    return case


def draw(rng):
    u = rng.random()
    if u < 0.65:
        case = _draw_solve(rng)
        del case["name"]
        return case
    if u < 0.75:
        return _draw_multi(rng)
    N, H = rng.choice((256, 512, 1024)), rng.choice((256, 512, 1024))
    net = {"M": N // 4, "N": N, "H": H, "S": N // 32, "snr_db": 20.0}
    if u < 0.85:
        return {"kind": "learned", "B": _log_int(rng, 64, 16384), **net}
    return {"kind": "grad", "B": _log_int(rng, 64, 4096), **net}


# ---- inputs ------------------------------------------------------------------

def _generator(seed, *salt):
    g = torch.Generator(device=DEVICE)
    for s in salt:
        seed = (seed * 1000003 + s + 1) % (1 << 62)
    g.manual_seed(seed)
    return g


def _dictionary(M, N, g, norms=False):
    A = torch.randn((N, M), generator=g, device=DEVICE, dtype=torch.float64) / math.sqrt(M)
    if norms:
        A /= A.norm(dim=1, keepdim=True)
        A *= 0.5 + 1.5 * torch.rand((N, 1), generator=g, device=DEVICE, dtype=torch.float64)
    return A.float()


def _signals(A, B, S, snr_db, g, caps=None):
    """(Y (B, M) float32, true support (B, S) int32 padded with -1 past caps[b], noise std (B,))."""
    N, M = A.shape
    sup = torch.rand((B, N), generator=g, device=DEVICE).topk(S, dim=1).indices
    v = torch.randn((B, S), generator=g, device=DEVICE, dtype=torch.float64)
    v = torch.sign(v) * (1.0 + v.abs())
    if caps is not None:
        dead = torch.arange(S, device=DEVICE)[None, :] >= caps[:, None]
        v.masked_fill_(dead, 0.0)
    X = torch.zeros((B, N), device=DEVICE, dtype=torch.float64).scatter_(1, sup, v)
    clean = X @ A.double()
    sigma = clean.norm(dim=1) / math.sqrt(M * 10.0 ** (snr_db / 10.0))
    Y = clean + sigma[:, None] * torch.randn((B, M), generator=g, device=DEVICE, dtype=torch.float64)
    sup = sup.int()
    if caps is not None:
        sup.masked_fill_(dead, -1)
    return Y.float(), sup, sigma


def _solve_inputs(case, seed):
    g = _generator(seed, 1)
    A = _dictionary(case["M"], case["N"], g, case["norms"])
    Y, _, _ = _signals(A, case["B"], case["S"], case["snr_db"], g)
    eps = (case["eps_rel"] * Y.double().norm(dim=1)).float() if case["eps_rel"] > 0 else None
    return A, Y, eps


def _multi_inputs(case, seed):
    out = []
    for i in range(2):
        g = _generator(seed, 2, i)
        A = _dictionary(case[f"M{i}"], case[f"N{i}"], g)
        B = case[f"B{i}"]
        caps = torch.randint(4, case["S"] + 1, (B,), generator=g, device=DEVICE, dtype=torch.int32)
        Y, _, _ = _signals(A, B, case["S"], case["snr_db"], g, caps)
        out.append((A, Y, caps, (1e-2 * Y.double().norm(dim=1)).float()))
    return out


def _net_inputs(case, seed):
    g = _generator(seed, 3)
    A = _dictionary(case["M"], case["N"], g)
    Y, sup, sigma = _signals(A, case["B"], case["S"], case["snr_db"], g)
    params = workloads.mlp_init_params(case["N"], case["H"], case["N"], seed=seed % (1 << 31))
    return A, Y, sup, (sigma * math.sqrt(case["M"])).float(), params


def _features(A, Y):
    """sqrt(M) |a_n^T y| / (||a_n|| ||y||), rounded to BF16."""
    Ad, Yd = A.double(), Y.double()
    f = (Yd @ Ad.T).abs() / (Ad.norm(dim=1)[None, :] * Yd.norm(dim=1, keepdim=True)) * math.sqrt(A.shape[1])
    return f.float().bfloat16()


def prepare(case, seed):
    kind = case["kind"]
    if kind == "solve":
        A, Y, eps = _solve_inputs(case, seed)
        d = omp.Dictionary(A, case["precision"]) if case["prepared"] else None
        return {"kind": kind, "A": A, "Y": Y, "eps": eps, "d": d, "S": case["S"], "precision": case["precision"],
                "gram": "auto" if case["gram_auto"] else False, "dense": case["dense"]}
    if kind == "multi":
        problems = [omp.Problem(omp.Dictionary(A, case["precision"]), Y, case["S"], S_per_signal=caps,
                                eps_per_signal=eps) for A, Y, caps, eps in _multi_inputs(case, seed)]
        return {"kind": kind, "problems": problems, "precision": case["precision"]}
    A, Y, sup, eps, params = _net_inputs(case, seed)
    mlp = omp.MLP(params, device=torch.device(DEVICE, torch.cuda.current_device()))
    if kind == "learned":
        return {"kind": kind, "d": omp.Dictionary(A, "bf16"), "mlp": mlp, "Y": Y, "S": case["S"], "eps": eps}
    return {"kind": kind, "mlp": mlp, "F": _features(A, Y).view(torch.int16), "sup": sup}


def run(state):
    kind = state["kind"]
    if kind == "solve":
        r = omp.solve(state["A"], state["Y"], state["S"], precision=state["precision"], dictionary=state["d"],
                      eps_per_signal=state["eps"], dense=state["dense"], gram_domain=state["gram"])
        return [t for t in r if t is not None]
    if kind == "multi":
        return [list(r[1:]) for r in omp.solve_multi(state["problems"], state["precision"])]
    if kind == "learned":
        r, accepted = omp.learned_solve(state["d"], state["mlp"], state["Y"], state["S"], eps_per_signal=state["eps"])
        return [*r[1:], accepted]
    loss, g = state["mlp"].grad(state["F"], state["sup"])
    return {"loss": loss, **g}


# ---- what a pass cannot do without -------------------------------------------

def _solve_work(M, N, B, S, precision, gram, outputs):
    el = 8 if precision == "fp64" else 4
    nbytes = 4 * (M * N + B * M) + outputs
    if precision == "fp64":
        # A^T y, then per step the columns of the support's atoms over all atoms
        flops = 2 * M * N * B + B * N * S * S
    elif gram:
        flops = 2 * M * N * B + B * N * S * S
        nbytes += el * N * N
    else:
        # the correlations of every step's residual, and the residual itself
        flops = S * 2 * M * N * B + B * M * S * S
    return nbytes, flops


def work(case):
    kind = case["kind"]
    if kind == "solve":
        M, N, B, S = case["M"], case["N"], case["B"], case["S"]
        gram = case["gram_auto"] and 4 * M >= N and (B <= 4096 or 4 * M * N >= 1 << 20)
        nbytes, flops = _solve_work(M, N, B, S, case["precision"], gram,
                                    (4 * B * N if case["dense"] else 0) + 8 * B * S + 8 * B)
        if not case["prepared"]:
            flops += M * N * (N + 1)
        return {"bytes": nbytes, "flops": flops}
    if kind == "multi":
        nbytes = flops = 0
        for i in range(2):
            # per-signal caps are uniform in 4 .. S: the mean support size counts
            M, N, B, k = case[f"M{i}"], case[f"N{i}"], case[f"B{i}"], (4 + case["S"]) / 2
            nb, fl = _solve_work(M, N, B, k, case["precision"], False, 8 * B * case["S"] + 16 * B)
            nbytes, flops = nbytes + nb, flops + fl
        return {"bytes": int(nbytes), "flops": int(flops)}
    N, H, B, S = case["N"], case["H"], case["B"], case["S"]
    weights = 2 * N * H + H * H
    if kind == "learned":
        M = case["M"]
        nb, fl = _solve_work(M, N, B, S, "bf16", False, 8 * B * S + 8 * B)
        return {"bytes": nb + 2 * weights, "flops": fl + 2 * B * (M * N + weights)}
    return {"bytes": 2 * B * N + 4 * B * S + (2 + 4) * weights, "flops": 2 * B * (weights + weights + N * H + H * H)}


# ---- the same in 64 bits, in plain torch -------------------------------------

def _omp64(A, Y, S, caps=None, eps=None):
    """OMP in FP64 by Gram-Schmidt: (support (B, S), coef (B, S), ||r|| (B,))."""
    A, Y = A.double(), Y.double()
    B, M = Y.shape
    inv = 1.0 / A.norm(dim=1)
    Q = torch.zeros((B, S, M), device=DEVICE, dtype=torch.float64)
    R = torch.eye(S, device=DEVICE, dtype=torch.float64).repeat(B, 1, 1)
    sup = torch.zeros((B, S), device=DEVICE, dtype=torch.int64)
    size = torch.zeros(B, device=DEVICE, dtype=torch.int64)
    live = torch.ones(B, device=DEVICE, dtype=torch.bool)
    taken = torch.zeros((B, A.shape[0]), device=DEVICE, dtype=torch.bool)
    r, rows = Y.clone(), torch.arange(B, device=DEVICE)
    for k in range(S):
        if eps is not None:
            live &= r.norm(dim=1) > eps.double()
        if caps is not None:
            live &= caps > k
        score = ((r @ A.T).abs() * inv[None, :]).masked_fill_(taken, -1.0)
        n = score.argmax(dim=1)
        del score
        q = A[n]
        for _ in range(2):  # the second pass restores orthogonality
            if k:
                c = torch.bmm(Q[:, :k], q.unsqueeze(2))
                q = q - torch.bmm(c.transpose(1, 2), Q[:, :k]).squeeze(1)
                R[:, :k, k] += torch.where(live[:, None], c.squeeze(2), 0.0)
        d = q.norm(dim=1)
        q = torch.where(live[:, None], q / d[:, None], 0.0)
        R[:, k, k] = torch.where(live, d, 1.0)
        Q[:, k] = q
        r = r - (q * r).sum(dim=1, keepdim=True) * q
        sup[:, k] = n
        taken[rows[live], n[live]] = True
        size += live
    u = torch.bmm(Q, Y.unsqueeze(2))
    x = torch.linalg.solve_triangular(R, u, upper=True).squeeze(2)
    past = torch.arange(S, device=DEVICE)[None, :] >= size[:, None]
    return sup.masked_fill_(past, -1), x.masked_fill_(past, 0.0), r.norm(dim=1)


def exact(case, seed):
    kind = case["kind"]
    if kind == "solve":
        A, Y, eps = _solve_inputs(case, seed)
        sup, x, rn = _omp64(A, Y, case["S"], eps=eps)
        out = [None, x, None, rn]
        if case["dense"]:
            X = torch.zeros((case["B"], case["N"]), device=DEVICE, dtype=torch.float64)
            out.insert(0, X.scatter_add_(1, sup.clamp(min=0), x))
        return out
    if kind == "multi":
        out = []
        for A, Y, caps, eps in _multi_inputs(case, seed):
            _, x, rn = _omp64(A, Y, case["S"], caps, eps)
            out.append([None, x, None, rn])
        return out
    A, Y, sup, eps, params = _net_inputs(case, seed)
    if kind == "learned":
        _, x, rn = _omp64(A, Y, case["S"], eps=eps)
        return [None, x, None, rn, None]
    p = {k: torch.from_numpy(v).to(DEVICE).double() for k, v in params.items()}
    f = _features(A, Y).double()
    t = torch.zeros((case["B"], case["N"]), device=DEVICE, dtype=torch.float64).scatter_(1, sup.long(), 1.0)
    a1 = f @ p["W1"].T + p["b1"]
    h1 = a1.clamp(min=0)
    a2 = h1 @ p["W2"].T + p["b2"]
    h2 = a2.clamp(min=0)
    z = h2 @ p["W3"].T + p["b3"]
    loss = torch.nn.functional.binary_cross_entropy_with_logits(z, t, reduction="sum") / case["B"]
    dz = (torch.sigmoid(z) - t) / case["B"]
    d2 = (dz @ p["W3"]) * (a2 > 0)
    d1 = (d2 @ p["W2"]) * (a1 > 0)
    return {"loss": loss.reshape(1), "W1": d1.T @ f, "b1": d1.sum(0), "W2": d2.T @ h1, "b2": d2.sum(0),
            "W3": dz.T @ h2, "b3": dz.sum(0)}
