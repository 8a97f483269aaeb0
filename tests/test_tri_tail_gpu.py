"""The deep levels of a tridiagonal plan in one workgroup (GPU): sizes on both sides of what its
LDS holds, from the whole plan in it to the direct solve alone.

The kernel takes the operations of the staged kernels in the same order, so every solution is
bitwise equal to the oracle's partition method, in float32 and in float64.
"""
import numpy as np
import pytest
import torch

from oracle import tridiag
from paper_2510_27351_amd import inputs
from paper_2510_27351_amd import tri

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
PREC = {torch.float64: "f64", torch.float32: "f32"}

# (batch, N, [m, m_1, ..] or None for the predicted plan).  One workgroup holds about 4600
# float64 rows (padded, all levels), 9200 float32 ones, and a quarter of that from 257 systems on.
CASES = [
    (1, 2, None), (1, 3, [2]), (1, 7, [2, 2]), (1, 9, []), (1, 17, []), (1, 18, [3]),
    (1, 3500, [16]), (1, 3700, [16]), (1, 4000, [16, 8]), (1, 4600, []), (1, 4610, []),
    (1, 7600, [16]), (1, 8300, [16]), (1, 9214, []), (1, 9300, []), (1, 9000, [4, 2, 2, 2, 2, 2, 2]),
    (2, 40001, [8, 5]), (2, 30000, [37, 100]), (3, 9001, [900]), (257, 900, [16]), (257, 1020, [16]),
    (256, 1150, []), (257, 1150, []), (257, 1151, [64, 4]), (300, 2310, []), (300, 5000, [12, 8]),
]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("batch,N,ms", CASES)
def test_tail_bitwise(batch, N, ms, dtype):
    kinds = min(batch, 3)  # distinct systems, repeated over the batch
    base = [tuple(v.to(dtype) for v in inputs.tridiagonal_dd(N, 31 * N + k)) for k in range(kinds)]
    order = [k % kinds for k in range(batch)]
    args = [torch.stack([base[k][q] for k in order]).to(DEV) for q in range(4)]
    if ms is None:
        plan = tri.Plan(batch, N, dtype)
        sizes = [plan.m] + plan.ms
    elif not ms:  # the direct solve alone: through its own entry point
        plan, sizes = None, []
    else:
        plan = tri.Plan(batch, N, dtype, m=ms[0], R=len(ms) - 1, ms=ms[1:])
        sizes = ms
    x = (plan.solve(*args) if plan else tri.thomas(*args)).cpu().numpy()
    want = [tridiag.c_partition_solve(*(v.numpy() for v in base[k]), sizes, PREC[dtype]) for k in range(kinds)]
    for i, k in enumerate(order):
        assert np.array_equal(x[i], want[k]), (i, k)
