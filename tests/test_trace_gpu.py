"""wf_trace_fetch writes 24 words per band and no more, whatever rows per lane the sweep took (GPU)."""
import ctypes

import pytest
import torch

import paper_2510_27351_amd as wf
from paper_2510_27351_amd import _lib, inputs

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
WORDS = 24


@pytest.mark.parametrize("m,n", [(70, 500), (300, 300), (1000, 100)])  # one, two and four rows per lane
def test_records_fill_their_words(m, n):
    lib = _lib.load()
    bands = -(-m // (64 * wf.forward_config(m, n)[1]))
    C = inputs.uniform(m, n, seed=3).to(DEV)
    ref, _, _ = wf.forward(C)
    guard = 0x5A5A5A5A5A5A5A5A
    buf = (ctypes.c_uint64 * (WORDS * bands + 8))(*([guard] * (WORDS * bands + 8)))
    try:
        assert lib.wf_trace_enable(bands) == 0
        D, _, _ = wf.forward(C)
        assert lib.wf_trace_fetch(buf, bands) == bands
    finally:
        lib.wf_trace_enable(0)
    assert torch.equal(D, ref)
    assert list(buf[WORDS * bands:]) == [guard] * 8
    for b in range(bands):
        claimed, ready, computed, stored = buf[WORDS * b:WORDS * b + 4]
        assert 0 < claimed <= ready < computed and claimed < stored
        assert buf[WORDS * b + 23] != guard
