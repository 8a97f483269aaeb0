"""wf_forward_config: what wf_forward would run, without a device (CPU)."""
import ctypes

import pytest
import torch

import paper_2510_27351_amd as wf
from paper_2510_27351_amd import _lib

SHAPES = [(1, 1), (64, 64), (300, 200), (1500, 4001), (4096, 4096), (16384, 1024), (16384, 16384), (64, 1 << 20)]


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64, torch.int32])
@pytest.mark.parametrize("m,n", SHAPES)
def test_within_the_prediction_and_its_bounds(m, n, dtype):
    tile, rows = wf.forward_config(m, n, dtype)
    assert rows in ((1, 2) if dtype == torch.float64 else (1, 2, 4))
    cap = 64 if rows == 1 else 32 if rows == 2 and dtype != torch.float64 else 16
    assert tile == min(wf.predict_tile(m, n, dtype=dtype), cap)
    assert wf.forward_config(m, n, dtype, table=False) == (tile, rows)


def test_the_benchmarks_size():
    assert wf.predict_tile(16384, 16384) == 64
    assert wf.forward_config(16384, 16384) == (32, 2)  # not the prediction


def test_forced_tile():
    try:
        wf.set_tile(64)
        assert wf.forward_config(16384, 1024) == (64, 4)
    finally:
        wf.set_tile(0)
    assert wf.forward_config(16384, 1024) == (16, 4)


def test_leading_dimension_bounds_the_rows():
    lib = _lib.load()
    t, r = ctypes.c_int32(), ctypes.c_int32()
    got = []
    for ld in (64, (1 << 31) // 256 // 4 - 4, (1 << 31) // 256 // 4, (1 << 31) // 128 // 4 - 4):
        assert lib.wf_forward_config(0, 16384, 64, ld, 0, ctypes.byref(t), ctypes.byref(r)) == 0
        got.append(r.value)
    assert got == [4, 4, 2, 2]
    assert lib.wf_forward_config(0, 16384, 64, (1 << 31) // 128 // 4, 0, None, None) == _lib.WF_E_UNSUPPORTED


@pytest.mark.parametrize("args", [(7, 8, 8, 8, 8), (0, 0, 8, 8, 8), (0, 8, 0, 8, 8), (0, 8, 8, 7, 8), (0, 8, 8, 8, 7),
                                  (0, 8, 8, 8, -1), (0, 1 << 40, 1 << 31, 1 << 31, 0)])
def test_refused(args):
    assert _lib.load().wf_forward_config(*args, None, None) == _lib.WF_E_ARG
