"""The work that a program has this library do, as timing cases.

A case is one call sequence through the package's public entry points on inputs resident in
device memory:

    forward   wf.forward: the table, the score and the checkpoint grid, or the score alone
    step      the differentiable sweep of one matrix: score, then its gradient (wf.sweep)
    train     the benchmark's step: forward with table and checkpoint grid, adjoint of the score
    table     the differentiable sweep with a loss on the whole table (an upstream gradient)
    batch     a ragged batch's scores through a plan (wf.Plan)
    bstep     the differentiable sweep of a batch of equal matrices
    soft      the soft-min sweep and its gradient
    tri       the tridiagonal partition solver through a plan

listed() names the sizes of the repository's own benchmark, tests and sweeps beside odd ones;
draw() takes others of the same ranges.  exact() evaluates the same quantities by plain torch
in 64 bits, one anti-diagonal at a time.
"""
import math
import random

import torch

import paper_2510_27351_amd as wf
from paper_2510_27351_amd import tri

F32, F64, I32 = "float32", "float64", "int32"
DT = {F32: torch.float32, F64: torch.float64, I32: torch.int32}
INF = math.inf


def listed():
    return [
        # two short sequences compared: the smallest call, launch and latency
        {"name": "pair-200x300", "op": "forward", "dtype": F32, "m": 200, "n": 300, "values": "uniform",
         "table": True, "ckpt_k": 0},
        # integer costs, only the score wanted, an odd wide shape
        {"name": "score-i32-1500x4001", "op": "forward", "dtype": I32, "m": 1500, "n": 4001, "values": "integers",
         "table": False, "ckpt_k": 0},
        # a training step on the score of one ordinary matrix
        {"name": "step-4096", "op": "step", "dtype": F32, "m": 4096, "n": 4096, "values": "uniform", "ckpt_k": 64},
        # the repository's benchmark: the largest single matrix
        {"name": "train-16384", "op": "train", "dtype": F32, "m": 16384, "n": 16384, "values": "normal",
         "ckpt_k": 64},
        # a loss that reads the whole table: the adjoint with an upstream gradient
        {"name": "table-3000x2500", "op": "table", "dtype": F32, "m": 3000, "n": 2500, "values": "uniform"},
        # the same in double, as gradient checks and small double programs run it
        {"name": "table-f64-1023x1300", "op": "table", "dtype": F64, "m": 1023, "n": 1300, "values": "uniform"},
        # the benchmark's ragged batch: 512 pairs of 64 to 2048
        {"name": "batch-512", "op": "batch", "dtype": F32, "batch": 512, "lo": 64, "hi": 2048, "shapes": 3,
         "table": False},
        # the benchmark's batched differentiable sweep
        {"name": "bstep-64x2048", "op": "bstep", "dtype": F32, "batch": 64, "m": 2048, "n": 2048, "ckpt_k": 64},
        # the smooth recurrence as a training loss
        {"name": "soft-4096", "op": "soft", "dtype": F32, "m": 4096, "n": 4096, "values": "uniform", "gamma": 1.0},
        # the same in double, ragged, sharper
        {"name": "soft-f64-500x700", "op": "soft", "dtype": F64, "m": 500, "n": 700, "values": "uniform",
         "gamma": 0.1},
        # the partition solver on the paper's largest system
        {"name": "tri-1e8", "op": "tri", "dtype": F64, "batch": 1, "N": 100_000_000},
        # and on an ordinary one, where its levels and launches count
        {"name": "tri-1e5", "op": "tri", "dtype": F64, "batch": 1, "N": 100_000},
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng: random.Random):
    op = rng.choice(["forward", "step", "table", "batch", "bstep", "soft", "tri"])
    if op == "forward":
        dtype = rng.choice([F32, F32, F64, I32])
        top = 16384 if dtype != F64 else 8192
        table = rng.random() < 0.6
        return {"op": op, "dtype": dtype, "m": _log(rng, 64, top), "n": _log(rng, 64, top),
                "values": "integers" if dtype == I32 else rng.choice(["uniform", "normal"]), "table": table,
                "ckpt_k": 64 if rng.random() < 0.3 else 0}
    if op in ("step", "table"):
        dtype = rng.choice([F32, F32, F64])
        top = 8192 if dtype == F32 else 4096
        c = {"op": op, "dtype": dtype, "m": _log(rng, 64, top), "n": _log(rng, 64, top),
             "values": rng.choice(["uniform", "normal"])}
        return {**c, "ckpt_k": rng.choice([64, 64, 100])} if op == "step" else c
    if op == "batch":
        lo = _log(rng, 16, 256)
        return {"op": op, "dtype": rng.choice([F32, F32, I32, F64]), "batch": _log(rng, 4, 512), "lo": lo,
                "hi": _log(rng, 2 * lo, 2048), "shapes": rng.randrange(1 << 20), "table": rng.random() < 0.3}
    if op == "bstep":
        return {"op": op, "dtype": rng.choice([F32, F32, F64]), "batch": _log(rng, 2, 48), "m": _log(rng, 64, 2048),
                "n": _log(rng, 64, 2048), "ckpt_k": 64}
    if op == "soft":
        dtype = rng.choice([F32, F32, F64])
        top = 4096 if dtype == F32 else 2048
        return {"op": op, "dtype": dtype, "m": _log(rng, 64, top), "n": _log(rng, 64, top), "values": "uniform",
                "gamma": rng.choice([0.1, 0.5, 1.0])}
    batch = rng.choice([1, 1, 1, _log(rng, 2, 256)])
    return {"op": op, "dtype": rng.choice([F64, F64, F32]), "batch": batch,
            "N": _log(rng, 100, 100_000_000 if batch == 1 else 20_000_000 // batch)}


# --- inputs ---------------------------------------------------------------------------------

def _dev():
    return torch.device("cuda", torch.cuda.current_device())


def _values(kind, shape, dtype, g):
    if kind == "integers":
        return torch.randint(0, 1001, shape, dtype=dtype, device=_dev(), generator=g)
    if kind == "normal":
        return torch.randn(shape, dtype=dtype, device=_dev(), generator=g).clamp_(-4.0, 4.0)
    return torch.rand(shape, dtype=dtype, device=_dev(), generator=g)


def _shapes(c):
    r = random.Random(c["shapes"])
    pick = lambda: [r.randint(c["lo"], c["hi"]) for _ in range(c["batch"])]  # noqa: E731
    ms = pick()
    return ms, pick()


def _system(c, g):
    shape = (c["N"],) if c["batch"] == 1 else (c["batch"], c["N"])
    dt = DT[c["dtype"]]
    r = lambda: torch.rand(shape, dtype=dt, device=_dev(), generator=g)  # noqa: E731
    a, cc, d = r().mul_(2).sub_(1), r().mul_(2).sub_(1), r().mul_(2).sub_(1)
    a[..., 0] = 0
    cc[..., -1] = 0
    b = r().add_(1).add_(a.abs()).add_(cc.abs())  # diagonally dominant, both signs
    b = torch.where(r() < 0.5, -b, b)
    return a, b, cc, d


def _inputs(c, seed):
    g = torch.Generator(device=_dev()).manual_seed(seed)
    op, dt = c["op"], DT[c["dtype"]]
    s = {}
    if op == "tri":
        s["a"], s["b"], s["c"], s["d"] = _system(c, g)
    elif op == "batch":
        # instances packed in order at 256-byte aligned starts, as a plan lays them out
        s["ms"], s["ns"] = _shapes(c)
        unit = 256 // (8 if c["dtype"] == F64 else 4)
        s["off"], end = [], 0
        for m, n in zip(s["ms"], s["ns"]):
            s["off"].append(end)
            end += (m * n + unit - 1) // unit * unit
        s["C"] = _values("integers" if c["dtype"] == I32 else "uniform", (end,), dt, g)
    else:
        shape = (c["batch"], c["m"], c["n"]) if op == "bstep" else (c["m"], c["n"])
        s["C"] = _values(c.get("values", "uniform"), shape, dt, g)
        if op == "bstep":
            s["gs"] = torch.rand(c["batch"], dtype=dt, device=_dev(), generator=g).add_(0.5)
        elif op in ("step", "train", "soft", "table"):
            s["gs"] = torch.rand((), dtype=dt, device=_dev(), generator=g).add_(0.5)
        if op == "table":
            s["gD"] = torch.randn(shape, dtype=dt, device=_dev(), generator=g)
    return s


def prepare(case, seed):
    s = {"case": case, **_inputs(case, seed)}
    if case["op"] == "batch":
        s["plan"] = wf.Plan(s["ms"], s["ns"], dtype=DT[case["dtype"]])
        if s["plan"].offsets != s["off"]:
            raise RuntimeError("the plan packs its instances another way")
    elif case["op"] == "tri":
        s["plan"] = tri.Plan(case["batch"], case["N"], DT[case["dtype"]])
    elif case["op"] in ("step", "table", "bstep", "soft"):
        s["C"].requires_grad_()
    return s


def run(s):
    c = s["case"]
    op = c["op"]
    if op == "forward":
        D, score, ck = wf.forward(s["C"], table=c["table"], ckpt_k=c["ckpt_k"])
        return {"score": score, "D": D, "grid": ck}
    if op in ("step", "bstep"):
        score = wf.sweep(s["C"], ckpt_k=c["ckpt_k"])
        (gC,) = torch.autograd.grad(score, s["C"], s["gs"])
        return {"score": score, "gC": gC}
    if op == "train":
        D, score, ck = wf.forward(s["C"], table=True, ckpt_k=c["ckpt_k"])
        gC = wf.backward(s["C"], g_score=s["gs"], ckpt=ck, ckpt_k=c["ckpt_k"])
        return {"score": score, "D": D, "gC": gC}
    if op == "table":
        D, score = wf.sweep(s["C"], table=True)
        (gC,) = torch.autograd.grad((D, score), s["C"], (s["gD"], s["gs"]))
        return {"score": score, "D": D, "gC": gC}
    if op == "batch":
        scores, D = s["plan"].forward(s["C"], table=c["table"])
        return {"scores": scores, "D": _tables(D, s) if D is not None else None}
    if op == "soft":
        D, score = wf.soft_sweep(s["C"], c["gamma"])
        (gC,) = torch.autograd.grad(score, s["C"], s["gs"])
        return {"score": score, "D": D, "gC": gC}
    return {"x": s["plan"].solve(s["a"], s["b"], s["c"], s["d"])}


def _tables(D, s):
    """The first tables of the packed buffer (the gaps between instances hold nothing)."""
    p = s["plan"]
    return [D[o:o + m * n] for o, m, n in list(zip(p.offsets, p.ms, p.ns))[:32]]


def work(c):
    es = {F32: 4, F64: 8, I32: 4}[c["dtype"]]
    op = c["op"]
    if op == "tri":
        n = c["batch"] * c["N"]
        return {"bytes": 5 * n * es, "flops": 9 * n}
    if op == "batch":
        ms, ns = _shapes(c)
        cells = sum(m * n for m, n in zip(ms, ns))
        return {"bytes": cells * es * (2 if c["table"] else 1), "flops": 3 * cells}
    cells = c["m"] * c["n"] * c.get("batch", 1)
    grid = cells // 64 + cells // c["ckpt_k"] if c.get("ckpt_k") and op in ("forward", "train") else 0
    if op == "forward":
        return {"bytes": es * (cells * (2 if c["table"] else 1) + grid), "flops": 3 * cells}
    # C in and the gradient out; the table out (and its gradient in) where the call has them
    arrays = {"step": 2, "bstep": 2, "train": 3, "soft": 3, "table": 4}[op]
    return {"bytes": es * (cells * arrays + grid), "flops": (16 if op == "soft" else 6) * cells}


# --- the same by plain torch in 64 bits ------------------------------------------------------

def _skew(C, fill):
    """C (B, m, n) as S (m+n-1, B, m): S[d, b, i] = C[b, i, d-i], 'fill' outside the matrix."""
    B, m, n = C.shape
    P = torch.full((B, m, n + m), fill, dtype=C.dtype, device=C.device)
    P[:, :, :n] = C
    S = P.view(B, -1)[:, :m * (n + m - 1)].view(B, m, n + m - 1)
    return S.permute(2, 0, 1).contiguous()


def _unskew(S, n):
    """The inverse of _skew."""
    W, B, m = S.shape
    P = torch.empty((B, m * (W + 1)), dtype=S.dtype, device=S.device)
    P[:, :m * W].view(B, m, W).copy_(S.permute(1, 2, 0))
    return P.view(B, m, W + 1)[:, :, :n].contiguous()


def _sweep64(C, dtype, soft=0.0, keep=True, ends=None):
    """Anti-diagonal sweep of C (B, m, n) in 'dtype': the skewed table (m+n-1, B, m+1) whose
    column 0 is the virtual row above (keep), or the values at 'ends' [(diagonal, b, row)]."""
    S = _skew(C, INF)
    W, B, m = S.shape
    full = lambda: torch.full((B, m + 1), INF, dtype=dtype, device=C.device)  # noqa: E731
    D = torch.full((W, B, m + 1), INF, dtype=dtype, device=C.device) if keep else None
    at = {}
    for d, b, i in ends or []:
        at.setdefault(d, []).append((b, i))
    got = {}
    p1, p2 = full(), full()
    for d in range(W):
        cur = D[d] if keep else full()
        if d == 0:
            cur[:, 1] = S[0, :, 0].to(dtype)
        else:
            nw, no, we = p2[:, :-1], p1[:, :-1], p1[:, 1:]
            if soft:
                mn = torch.minimum(torch.minimum(nw, no), we)
                z = torch.where(torch.isinf(mn), torch.zeros_like(mn), mn)
                t = torch.exp((z - nw) / soft) + torch.exp((z - no) / soft) + torch.exp((z - we) / soft)
                v = mn - soft * torch.log(torch.where(torch.isinf(mn), torch.ones_like(t), t))
            else:
                v = torch.minimum(torch.minimum(nw, no), we)
            torch.add(v, S[d].to(dtype), out=cur[:, 1:])
        for b, i in at.get(d, ()):
            got[b] = cur[b, i + 1].clone()
        p2, p1 = p1, cur
    return D if keep else torch.stack([got[b] for b in range(B)])


def _adjoint64(C, D, gD, gs, soft=0.0):
    """The adjoint of sum(gD * D) + gs * score in 64 bits over the skewed table D: routed by
    the table's own selections, or weighted by the soft minimum's derivatives."""
    B, m, n = C.shape
    S = _skew(C, INF)
    G = None if gD is None else _skew(gD.double(), 0.0)
    W = m + n - 1
    dev = C.device
    A = torch.zeros((W, B, m), dtype=torch.float64, device=dev)
    pad = torch.zeros((B, m + 1), dtype=torch.float64, device=dev)
    # what each cell routes to its three predecessors: (to NW, to N, to W), one diagonal at a time
    later = [(pad, pad, pad), (pad, pad, pad)]  # diagonals d+1, d+2
    infs = torch.full((B, m + 1), INF, dtype=D.dtype, device=dev)
    for d in range(W - 1, -1, -1):
        (nw1, n1, w1), (nw2, _, _) = later
        a = nw2[:, 1:] + n1[:, 1:] + w1[:, :-1]
        if G is not None:
            a = a + G[d]
        if d == W - 1:
            a[:, m - 1] += gs.double()
        a = torch.where(torch.isinf(S[d]), torch.zeros_like(a), a)
        A[d] = a
        p1 = D[d - 1] if d >= 1 else infs
        p2 = D[d - 2] if d >= 2 else infs
        nw, no, we = p2[:, :-1], p1[:, :-1], p1[:, 1:]
        to = torch.zeros((3, B, m + 1), dtype=torch.float64, device=dev)
        if soft:
            v = D[d][:, 1:] - S[d]
            for k, x in enumerate((nw, no, we)):
                w = torch.where(torch.isinf(x) | torch.isinf(S[d]), torch.zeros_like(a), torch.exp((v - x) / soft))
                to[k, :, :-1] = w * a
        else:
            north = no < nw
            west = we < torch.minimum(nw, no)
            to[2, :, :-1] = a * west
            to[1, :, :-1] = a * (north & ~west)
            to[0, :, :-1] = a * (~north & ~west)
        later = [tuple(to), later[0]]
    return _unskew(A, n)


def _grid(D, k):
    """The checkpoint grid of one table: band rows 63, 127, ..., then block columns."""
    m, n = D.shape
    rows = [D[r] for r in range(63, m - 1, 64)]
    cols = [D[:, q * k - 1] for q in range(1, (n + k - 1) // k)]
    return torch.cat(rows + cols) if rows or cols else D.new_empty(0)


def _tridiagonal64(a, b, c, d):
    """Parallel cyclic reduction in 64 bits."""
    a, b, c, d = (v.double().reshape(-1, v.shape[-1]) for v in (a, b, c, d))
    a, c = a / b, c / b
    d = d / b
    N = a.shape[1]
    k = 1
    while k < N:
        up = lambda v: torch.nn.functional.pad(v[:, :-k], (k, 0))  # noqa: E731
        dn = lambda v: torch.nn.functional.pad(v[:, k:], (0, k))  # noqa: E731
        r = 1.0 / (1.0 - a * up(c) - c * dn(a))
        a, c, d = -r * a * up(a), -r * c * dn(c), r * (d - a * up(d) - c * dn(d))
        k *= 2
        if not (a.abs().max() > 1e-300) and not (c.abs().max() > 1e-300):
            break
    return d


def exact(case, seed):
    c, s = case, _inputs(case, seed)
    op = c["op"]
    if op == "tri":
        x = _tridiagonal64(s["a"], s["b"], s["c"], s["d"])
        return {"x": x.reshape(s["a"].shape)}
    if op == "batch":
        C = torch.zeros((c["batch"], max(s["ms"]), max(s["ns"])), dtype=torch.float64 if c["dtype"] == F64 else
                        torch.float32, device=_dev())  # integers below 1001 are exact in float32
        for b, (o, m, n) in enumerate(zip(s["off"], s["ms"], s["ns"])):
            C[b, :m, :n] = s["C"][o:o + m * n].view(m, n)
        ends = [(m + n - 2, b, m - 1) for b, (m, n) in enumerate(zip(s["ms"], s["ns"]))]
        scores = _sweep64(C, torch.float64, keep=False, ends=ends)
        return {"scores": scores, "D": [None] * min(32, c["batch"]) if c["table"] else None}
    C = s["C"]
    n = c["n"]
    C3 = C if C.dim() == 3 else C[None]
    if c["dtype"] == I32:
        C3 = C3.double()
    soft = c.get("gamma", 0.0)
    D = _sweep64(C3.double(), torch.float64, soft=soft)
    score = D[-1, :, -1].clone()
    if op == "forward":
        T = _unskew(D[:, :, 1:], n)[0]
        return {"score": score.reshape(()), "D": T if c["table"] else None,
                "grid": _grid(T, c["ckpt_k"]) if c["ckpt_k"] else None}
    if op == "soft":
        gC = _adjoint64(C3.double(), D, None, s["gs"], soft=soft)
        return {"score": score.reshape(()), "D": _unskew(D[:, :, 1:], n)[0], "gC": gC[0]}
    T = _unskew(D[:, :, 1:], n)[0] if op in ("train", "table") else None
    # the gradient follows the selections of the sweep in its own type: at a near tie the
    # double table may select another predecessor, which is another (as valid) subgradient
    if c["dtype"] == F32:
        del D
        D = _sweep64(C3, torch.float32)
    gC = _adjoint64(C3, D, s["gD"][None] if op == "table" else None, s["gs"])
    if op == "bstep":
        return {"score": score, "gC": gC}
    out = {"score": score.reshape(()), "gC": gC[0]}
    return {**out, "D": T} if T is not None else out
