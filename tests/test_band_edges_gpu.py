"""Edges of the band pipelines on the GPU: the forward sweep with one, two and four rows per
lane, autotuned batches, the soft-min adjoint, the reverse sweep.

Which of them a shape takes depends on m / n; the shapes here lie on both sides of the rule's
lines and of the band edges (64, 128 and 256 rows), with matrices narrower than one handoff
unit, one column wide and with padded rows.  Tables, scores and checkpoint grids are bitwise
equal to the float32 / float64 / int64 oracle's (one add per cell in every schedule).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2510_27351_amd as wf
from paper_2510_27351_amd import inputs

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SHAPES = [(65, 600), (64, 64), (65, 64), (127, 63), (128, 128), (129, 130), (300, 300), (255, 33), (256, 40),
          (257, 60), (512, 100), (513, 7), (700, 1), (1025, 200), (1300, 31), (2049, 257)]


def matrix(dtype, m, n, seed):
    if dtype == torch.int32:
        return inputs.integers(m, n, seed, lo=-100, hi=1000), "i64"
    return inputs.normal_clipped(m, n, seed, dtype), "f32" if dtype == torch.float32 else "f64"


def grid_of(D, k):
    m, n = D.shape
    parts = [D[r] for r in range(63, m - 1, 64)] + [D[:, q * k - 1] for q in range(1, (n + k - 1) // k)]
    return torch.cat(parts) if parts else D.new_empty(0)


@pytest.mark.parametrize("dtype", [torch.float32, torch.int32, torch.float64])
@pytest.mark.parametrize("m,n", SHAPES)
def test_rows_per_lane_bitwise(dtype, m, n):
    C, prec = matrix(dtype, m, n, 7 * m + n)
    ref, _ = oracle.forward(C.numpy(), prec, want_sel=False)
    pad = torch.full((m, n + 5), 3, dtype=dtype, device=DEV)
    pad[:, :n] = C.to(DEV)
    out = torch.full((m, n + 3), -7, dtype=dtype, device=DEV)
    for tile in (0, 16, 64):
        wf.set_tile(tile)
        try:
            D, score, ck = wf.forward(pad[:, :n], D=out[:, :n], ckpt_k=5)
            _, alone, _ = wf.forward(C.to(DEV), table=False)
            wf.last_async_error()
        finally:
            wf.set_tile(0)
        got = D.cpu().numpy().astype(ref.dtype)
        assert np.array_equal(got, ref), f"{m}x{n} tile {tile}: {(got != ref).sum()} cells differ"
        assert score.item() == ref[-1, -1] and alone.item() == ref[-1, -1]
        assert torch.equal(ck.cpu(), grid_of(D, 5).cpu())
        assert bool((out[:, n:] == -7).all())


@pytest.mark.parametrize("table", [False, True])
@pytest.mark.parametrize("count", [3, 40, 1600])
def test_autotuned_batch_bitwise(count, table):
    """Small and large batches with the library's own configurations (runs with and without
    tables may take different ones), one plan used for both in turn."""
    g = torch.Generator().manual_seed(count)
    ms = torch.randint(1, 140, (count,), generator=g).tolist()
    ns = torch.randint(1, 90, (count,), generator=g).tolist()
    mats = [torch.randn(m, n, generator=g) for m, n in zip(ms, ns)]
    plan = wf.Plan(ms, ns)
    C = plan.pack([x.to(DEV) for x in mats])
    for t in (table, not table, table):
        scores, D = plan.forward(C, table=t)
        wf.last_async_error()
        got = scores.cpu().numpy()
        tabs = [d.cpu().numpy() for d in plan.unpack(D)] if t else None
        for i, x in enumerate(mats):
            ref, _ = oracle.forward(x.numpy(), "f32", want_sel=False)
            assert got[i] == ref[-1, -1], f"instance {i} {ms[i]}x{ns[i]}"
            if t:
                assert np.array_equal(tabs[i], ref), f"instance {i} {ms[i]}x{ns[i]}"


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("m,n", [(1, 1), (1, 40), (40, 1), (63, 64), (64, 65), (65, 31), (129, 33), (200, 47), (321, 200)])
def test_soft_adjoint_edges(dtype, m, n):
    """The soft-min adjoint at its tile edges (units of 16 columns, sub-chunks of 16 and 32,
    bands of 64 rows), with padded rows, with and without gD, and with the gradient written
    over D, over C and over gD.  Bounds: the float64 result against the oracle on the same
    table, 1e-10; float32 against it by the path-length law 12 sqrt(m+n-1) u max|D| / gamma
    (at least 1e-4), as in the soft-min tests."""
    gamma = 0.5
    C = inputs.uniform(m, n, 31 * m + n).to(dtype)
    gD = inputs.normal_clipped(m, n, 17 * m + n).to(dtype)
    D, _ = wf.soft_forward(C.to(DEV), gamma)
    gs = torch.tensor(0.75, dtype=dtype, device=DEV)
    u = np.finfo(np.float32 if dtype == torch.float32 else np.float64).eps / 2
    law = 12 * (m + n - 1) ** 0.5 * u * max(1.0, float(D.abs().max())) / gamma
    tol = max(1e-4 if dtype == torch.float32 else 1e-10, law)
    for g in (None, gD):
        ref = oracle.soft_backward(C.double().numpy(), D.double().cpu().numpy(), gamma,
                                   None if g is None else g.double().numpy(), 0.75)
        gdev = None if g is None else g.to(DEV)
        pad = torch.full((m, n + 3), -9, dtype=dtype, device=DEV)
        out = wf.soft_backward(C.to(DEV), D, gamma, g_score=gs, g_D=gdev, g_C=pad[:, :n])
        wf.last_async_error()
        got = out.double().cpu().numpy()
        assert np.max(np.abs(got - ref)) <= tol * max(1.0, np.max(np.abs(ref)))
        assert bool((pad[:, n:] == -9).all())
        over_D, over_C = D.clone(), C.to(DEV)
        wf.soft_backward(C.to(DEV), over_D, gamma, g_score=gs, g_D=gdev, g_C=over_D)
        wf.soft_backward(over_C, D, gamma, g_score=gs, g_D=gdev, g_C=over_C)
        assert torch.equal(over_D, out) and torch.equal(over_C, out)
        if g is not None:
            wf.soft_backward(C.to(DEV), D, gamma, g_score=gs, g_D=gdev, g_C=gdev)
            assert torch.equal(gdev, out)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("m,n", [(1, 65), (2, 63), (31, 130), (33, 64), (65, 257), (95, 128), (97, 1), (120, 700), (191, 62)])
def test_adjoint_ragged_rows_padded(dtype, m, n):
    """The reverse sweep where the last band holds a part of its rows (either half of them, with
    whole and partial column edges), gD and gC with a leading dimension beyond n, gC also written
    over gD: bitwise equal to the oracle, nothing written beside the matrix."""
    prec = "f32" if dtype == torch.float32 else "f64"
    C = inputs.normal_clipped(m, n, 5 * m + n, dtype)
    gD = inputs.normal_clipped(m, n, 3 * m + n, dtype)
    D, sel = oracle.forward(C.numpy(), prec, want_sel=True)
    ref = torch.from_numpy(oracle.backward(sel, gD.numpy(), 0.75, prec))
    gs = torch.tensor(0.75, dtype=dtype, device=DEV)
    Dd = torch.from_numpy(D).to(DEV)
    for pad in (0, 3):
        g_in = torch.full((m, n + pad), 1e30, dtype=dtype, device=DEV)
        g_in[:, :n] = gD.to(DEV)
        out = torch.full((m + 2, n + pad), -9, dtype=dtype, device=DEV)
        wf.backward(C.to(DEV), g_score=gs, g_D=g_in[:, :n], D=Dd, g_C=out[1:m + 1, :n])
        wf.backward(C.to(DEV), g_score=gs, g_D=g_in[:, :n], D=Dd, g_C=g_in[:, :n])
        wf.last_async_error()
        assert torch.equal(out[1:m + 1, :n].cpu(), ref) and torch.equal(g_in[:, :n].cpu(), ref)
        assert bool((out[0] == -9).all()) and bool((out[m + 1] == -9).all()) and bool((out[:, n:] == -9).all())
        assert bool((g_in[:, n:] == g_in.new_tensor(1e30)).all())


@pytest.mark.parametrize("gamma", [1e-3, 0.02, 1.0, 50.0])
@pytest.mark.parametrize("m,n", [(1, 1), (3, 70), (70, 3), (130, 77), (64, 129)])
def test_soft_forward_f64_weights(m, n, gamma):
    """The float64 soft minimum from terms that vanish (small gamma: exponents far below -64) to
    three nearly equal ones (large gamma, and one matrix of equal values), against the oracle.
    Bound: a cell rounds its scaled sum, its minimum's difference and C's scaling once each and
    takes two exponentials and a logarithm of two units in the last place at most, about 8 u of
    the largest scaled value per cell of a path."""
    u = 2.0 ** -53
    for C in (inputs.uniform(m, n, 3 * m + n, torch.float64, lo=-2.0, hi=3.0), torch.full((m, n), 0.25, dtype=torch.float64)):
        D, score = wf.soft_forward(C.to(DEV), gamma)
        wf.last_async_error()
        ref = oracle.soft_forward(C.numpy(), gamma)
        tol = 8 * (m + n - 1) * u * max(float(np.max(np.abs(ref))), 2 * gamma)
        assert np.max(np.abs(D.cpu().numpy() - ref)) <= tol
        assert float(score) == float(D[-1, -1])


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("m,n", [(1, 700), (2, 64), (3, 1000), (64, 3000), (65, 4097), (130, 1500), (700, 1), (200, 5)])
def test_path_walk_long_runs(dtype, m, n):
    """The score's gradient where the path has runs of W selections through several 64-slot
    sub-chunks, ending on, before and after their edges: random matrices much wider than high,
    and matrices whose path turns at given columns; bitwise equal to the oracle."""
    prec = "f32" if dtype == torch.float32 else "f64"
    mats = [inputs.uniform(m, n, 7 * m + n, dtype)]
    for turn in (0, 63, 64, 65, 127, 512):  # one cheap row until 'turn', another from there on
        if m > 1 and turn < n:
            C = torch.full((m, n), 100.0, dtype=dtype)
            C[0, :turn + 1] = 1.0
            C[:, turn] = 1.0
            C[m - 1, turn:] = 1.0
            mats.append(C)
    gs = torch.tensor(1.5, dtype=dtype, device=DEV)
    for C in mats:
        D, sel = oracle.forward(C.numpy(), prec, want_sel=True)
        ref = torch.from_numpy(oracle.backward(sel, None, 1.5, prec))
        got = wf.backward(C.to(DEV), g_score=gs, D=torch.from_numpy(D).to(DEV))
        wf.last_async_error()
        assert torch.equal(got.cpu(), ref)
