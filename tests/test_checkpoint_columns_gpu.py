"""The checkpoint grid holds the table's own values, for spacings around the storers' sub-chunks
(32 and 64 slots), one to a few columns and wider than the matrix, with one, two and four rows
per lane (GPU)."""
import pytest
import torch

import paper_2510_27351_amd as wf
from paper_2510_27351_amd import inputs

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64, torch.int32])
@pytest.mark.parametrize("m,n", [(70, 1000), (1, 200), (300, 301), (1000, 130), (700, 2)])
@pytest.mark.parametrize("k", [1, 2, 3, 31, 32, 33, 63, 64, 65, 129, 4096])
def test_grid_is_the_tables(m, n, k, dtype):
    if dtype == torch.int32:
        C = torch.randint(-1000, 1000, (m, n), dtype=dtype, generator=torch.Generator().manual_seed(m + n))
    else:
        C = inputs.uniform(m, n, seed=m + n, dtype=dtype)
    D, _, ck = wf.forward(C.to(DEV), ckpt_k=k)
    wf.last_async_error()
    rows = D[63:m - 1:64, :].reshape(-1)
    cols = D[:, k - 1:n - 1:k].T.reshape(-1)
    assert torch.equal(ck, torch.cat([rows, cols]))
