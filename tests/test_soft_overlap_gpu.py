"""Soft-min adjoint whose gradient lies in one buffer with its inputs (GPU): side by side, where
nothing is shared and no copy is needed, so that a call may be captured like any other; and
over an input, shifted by rows or columns."""
import pytest
import torch

import paper_2510_27351_amd as wf
from paper_2510_27351_amd import inputs

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
M, N = 150, 90


def case(dtype):
    C = inputs.uniform(M, N, seed=11, dtype=dtype).to(DEV)
    D, _ = wf.soft_forward(C, 0.7)
    gs = torch.ones((), dtype=dtype, device=DEV)
    return C, D, gs, wf.soft_backward(C, D, 0.7, g_score=gs)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("side", ["right of C", "left of C", "between C and D"])
def test_side_by_side_is_captured(side, dtype):
    C, D, gs, want = case(dtype)
    order = {"right of C": (0, 2, 1), "left of C": (1, 2, 0), "between C and D": (0, 2, 1)}[side]
    big = torch.zeros((M, 3 * N + 5), dtype=dtype, device=DEV)
    c, d, g = (big[:, k * N:(k + 1) * N] for k in order)
    c.copy_(C)
    d.copy_(D)
    if side != "between C and D":
        d = D  # contiguous, another stride
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        wf.soft_backward(C, D, 0.7, g_score=gs, g_C=torch.empty_like(C))  # sizes the stream's workspace
    stream.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        wf.soft_backward(c, d, 0.7, g_score=gs, g_C=g)
    for _ in range(3):
        g.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(g, want) and torch.equal(c, C) and torch.equal(d, D)
    wf.last_async_error()


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("rows,cols", [(0, 0), (1, 0), (-1, 0), (0, 1), (0, -1), (3, -89), (-2, 89), (64, 0), (149, 0)])
def test_over_an_input(rows, cols, dtype):
    """The gradient's buffer is C's, moved by rows and columns of the same stride: every cell that the
    two share is read before it counts as written."""
    C, D, gs, want = case(dtype)
    big = torch.zeros((3 * M, 3 * N), dtype=dtype, device=DEV)
    c = big[M:2 * M, N:2 * N]
    g = big[M + rows:2 * M + rows, N + cols:2 * N + cols]
    c.copy_(C)
    wf.soft_backward(c, D, 0.7, g_score=gs, g_C=g)
    wf.last_async_error()
    assert torch.equal(g, want)
