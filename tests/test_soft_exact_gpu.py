"""Soft-min forward where its result has to be exact, or nearly: cells with one live
predecessor, and values far below the temperature.

With one predecessor whose weight is not zero (the first row and column, and any cell whose
other neighbours lie far above it) the soft minimum is that predecessor, so the table is a
plain running sum: zeros stay zero, and positive terms of any size keep their relative
accuracy.  The sum of L scaled terms carries L products and L - 1 sums of one rounding each, the
two scale factors' roundings and the last product's: at most (L + 4) u relative, u = 2^-53,
on the device and, with fewer of them, in the oracle: the two differ by at most twice that.
"""
import numpy as np
import pytest
import torch

import paper_2510_27351_amd as wf
from paper_2510_27351_amd import inputs

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
U = 2.0 ** -53


@pytest.mark.parametrize("gamma", [0.01, 1.0, 10.0])
@pytest.mark.parametrize("c", [0.0, 1e-16, 1e-9, 1e-5])
def test_first_row_and_column_f64(c, gamma, oracle_mod):
    m, n = 200, 1000
    C = torch.full((m, n), c, dtype=torch.float64)
    D, _ = wf.soft_forward(C.to(DEV), gamma)
    D, want = D.cpu().numpy(), oracle_mod.soft_forward(C.numpy(), gamma)
    for got, ref in ((D[0], want[0]), (D[:, 0], want[:, 0])):
        bar = (np.arange(1, len(ref) + 1) + 4) * U * np.abs(ref)
        assert np.all(np.abs(got - ref) <= 2 * bar), float(np.max(np.abs(got - ref) / np.maximum(np.abs(ref), 1e-300)))


@pytest.mark.parametrize("gamma", [0.01, 1.0, 10.0])
@pytest.mark.parametrize("gap", [70.0, 700.0, 1000.0, 1e6])
def test_corridor_f64(gap, gamma, oracle_mod):
    """A corridor of small costs along the first row, down one column and along the last row,
    through cells that lie 'gap' times gamma above it.  A neighbour off the corridor weighs at
    most 3 exp(-gap) (the corridor's whole cost is far below gamma) in the table and in the
    oracle alike, so that what the two make of a cell's two such neighbours differs by less than
    2 gamma exp(1 - gap), and L of these add up; beyond 700 that is nothing."""
    m, n, col = 150, 400, 263
    C = torch.full((m, n), gap * gamma, dtype=torch.float64)
    c = 1e-9 * gamma
    C[0, :col + 1] = c
    C[:, col] = c
    C[m - 1, col:] = c
    D, score = wf.soft_forward(C.to(DEV), gamma)
    D, want = D.cpu().numpy(), oracle_mod.soft_forward(C.numpy(), gamma)
    got = np.concatenate([D[0, :col + 1], D[1:, col], D[m - 1, col + 1:]])
    ref = np.concatenate([want[0, :col + 1], want[1:, col], want[m - 1, col + 1:]])
    steps = np.arange(1, len(ref) + 1)
    bar = 2 * (steps + 4) * U * np.abs(ref) + steps * 2 * gamma * np.exp(1 - gap)
    assert np.all(np.abs(got - ref) <= bar), float(np.max(np.abs(got - ref) / ref))
    assert float(score) == D[-1, -1]


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("cell", [(0, 0), (0, 70), (64, 0), (37, 130), (99, 149)])
def test_nan_in_the_input_shows_at_its_cell(cell, dtype):
    """The library asks for finite inputs; a NaN among them is not hidden at its own cell, and
    cells that no path through it reaches are as without it."""
    C = inputs.uniform(100, 150, seed=5, dtype=dtype).to(DEV)
    ref, _ = wf.soft_forward(C, 0.5)
    C[cell] = float("nan")
    D, _ = wf.soft_forward(C, 0.5)
    i, j = cell
    assert torch.isnan(D[i, j])
    assert torch.equal(D[:i], ref[:i]) and torch.equal(D[:, :j], ref[:, :j])
