"""Partition solver: plans whose deep levels fill the last launch's LDS to just below, exactly
at and just above its limit, and its direct solve there (GPU).

The last launch takes a level and every deeper one if 4 (rows of the deepest system + padded
rows of the levels above it) + 16 elements fit in 144 KiB, or in 36 KiB for more than 256
systems; a level of P sub-systems of m rows takes P times the odd number from m + 1 on.  The operations are those
of the staged kernels in the same order, so every solution is bitwise equal to the oracle's
partition method.
"""
import numpy as np
import pytest
import torch

from oracle import tridiag
from paper_2510_27351_amd import inputs
from paper_2510_27351_amd import tri

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
SIZE = {torch.float64: 8, torch.float32: 4}
PREC = {torch.float64: "f64", torch.float32: "f32"}


def limit(dtype, batch):
    """Rows (deepest and padded) that fit."""
    return ((144 if batch <= 256 else 36) * 1024 // SIZE[dtype] - 16) // 4


def pitch(m):
    return m + 1 if m % 2 == 0 else m + 2


def cases(dtype, batch):
    """(N, [m, ..], rows of the levels the limit is about) around the limit."""
    e = limit(dtype, batch)
    out = []
    for d in (-2, 0, 2):  # the deepest system alone
        out.append((4 * ((e + d) // 2), [4], 2 * ((e + d) // 2)))
    for m in (2, 3, 16, 31):  # and one level above it
        per = 2 + pitch(m)
        for P in (e // per, e // per + 1):
            out.append((P * m, [m], P * per))
            out.append((P * m + 1, [m], P * per))  # the last sub-system takes a row more
    # one level, filled to the last row
    per = next(q for q in range(5, e, 2) if e % q == 0)
    m = per - 3
    out += [(e // per * m, [m], e), (e // per * m + 1, [m], e)]
    # several levels: the largest system that fits whole and the next larger one that does not
    for ms in ([7, 5], [4, 3, 6]):
        N = 2
        while rows_of(N + 1, ms) <= e:
            N += 1
        out += [(N, ms, rows_of(N, ms)), (N + 1, ms, rows_of(N + 1, ms))]
    return out


def rows_of(N, ms):
    """Rows of the deepest system and padded rows of every level above it."""
    rows = 0
    for m in ms:
        P = tri.subsystems(N, m)
        rows += P * pitch(m)
        N = 2 * P
    return rows + N


CASES = [(dt, b, c) for dt in SIZE for b in (1, 256, 257) for c in cases(dt, b)]


def test_cases_straddle_the_limit():
    for dt in SIZE:
        for b in (1, 257):
            e = limit(dt, b)
            rows = [r for _, _, r in cases(dt, b)]
            assert e in rows and any(e - 40 < r < e for r in rows) and any(e < r < e + 40 for r in rows)


@pytest.mark.parametrize("dtype,batch,case", CASES, ids=lambda v: str(v).replace("torch.", ""))
def test_bitwise_at_the_limit(dtype, batch, case):
    N, ms, _ = case
    kinds = min(batch, 2)  # distinct systems, repeated over the batch
    base = [tuple(v.to(dtype) for v in inputs.tridiagonal_dd(N, 7 * N + k)) for k in range(kinds)]
    order = [k % kinds for k in range(batch)]
    args = [torch.stack([base[k][q] for k in order]).to(DEV) for q in range(4)]
    plan = tri.Plan(batch, N, dtype, m=ms[0], R=len(ms) - 1, ms=ms[1:])
    x = plan.solve(*args).cpu().numpy()
    want = [tridiag.c_partition_solve(*(v.numpy() for v in base[k]), ms, PREC[dtype]) for k in range(kinds)]
    for i, k in enumerate(order):
        assert np.array_equal(x[i], want[k]), (i, k)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("batch,N,ms", [
    (2048, 20, [4]), (2049, 2, [2]), (2049, 20, [4]), (2049, 100, [16]), (2049, 131, [16]), (2500, 170, [9]),
    (2500, 260, [16]), (2500, 300, [16]), (2500, 420, [16, 4]), (2500, 560, [8, 6]), (2500, 1000, [16])])
def test_many_systems_bitwise(batch, N, ms, dtype):
    """One, two and four waves per system, on both sides of eight systems per compute unit."""
    base = [tuple(v.to(dtype) for v in inputs.tridiagonal_dd(N, 5 * N + k)) for k in range(3)]
    args = [torch.stack([base[k % 3][q] for k in range(batch)]).to(DEV) for q in range(4)]
    plan = tri.Plan(batch, N, dtype, m=ms[0], R=len(ms) - 1, ms=ms[1:])
    x = plan.solve(*args).cpu()
    for k in range(3):
        want = torch.from_numpy(tridiag.c_partition_solve(*(v.numpy() for v in base[k]), ms, PREC[dtype]))
        assert torch.equal(x[k::3], want.expand_as(x[k::3])), k
