"""Rows per lane of an autotuned plan's runs that write tables (GPU): one row per lane where the
batch is bound by its memory traffic, else the rows tuned for scores, and the tables are the
instances' own either way."""
import pytest
import torch

import paper_2510_27351_amd as wf

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.mark.parametrize("dtype", [torch.float32, torch.int32])
@pytest.mark.parametrize("count,m,n,rows", [
    (64, 2048, 2048, 1),   # traffic is twice the bands' time
    (100, 4500, 60, 2),    # 27 bands of 64 rows per compute unit, but short ones
    (600, 180, 180, 2), (4, 300, 300, 2)])
def test_rows_of_runs_with_tables(count, m, n, rows, dtype):
    plan = wf.Plan([m] * count, [n] * count, dtype=dtype)
    # (the tuner times runs for scores, where two rows win but for the smallest batch, a near tie)
    assert plan.rows == 2 or count == 4
    assert plan.table_rows == min(rows, plan.rows)
    gen = torch.Generator(device=DEV).manual_seed(count)
    C = torch.randint(0, 1000, (plan.elems,), dtype=dtype, device=DEV, generator=gen) if dtype == torch.int32 else \
        torch.rand(plan.elems, dtype=dtype, device=DEV, generator=gen)
    scores, D = plan.forward(C, table=True)
    alone, _ = plan.forward(C)
    wf.last_async_error()
    assert torch.equal(scores, alone)
    for i in (0, count // 2, count - 1):
        ref, score, _ = wf.forward(plan.unpack(C)[i])
        assert torch.equal(plan.unpack(D)[i], ref) and scores[i] == score
    plan.close()
