"""Launches of many (sequence, head, chunk) units, whose blocks are numbered by
workspace slot: batches around the 64 sequences one wave compares at once,
with empty sequences, one-chunk sequences and intervals that are no multiple
of the chunk, against the oracle."""
import numpy as np
import pytest
import torch

from paper_2609_15030_amd import api
from paper_2609_15030_amd import linattn as la
from paper_2609_15030_amd import workloads as wl
from parity import TOL, compare, oracle_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,C,io", [(63, 256, wl.BF16), (64, 100, wl.BF16), (65, 256, wl.BF16), (150, 48, wl.BF16),
                                    (300, 64, wl.BF16), (129, 100, wl.F32)])
def test_many_short_sequences(n, C, io):
    rng = np.random.default_rng(n + C)
    lens = [int(v) for v in rng.integers(0, 90, n)]
    lens[0] = lens[n // 2] = lens[-1] = 0
    lens[3] = 400                                   # the longest: many chunk numbers that others lack
    H, d = 8, 64
    assert n * H * (-(-400 // 64)) > 2048           # numbered by slot
    x = wl.random_inputs(n, lens, H, d, d, io, gate_scale=0.1)
    res = api.prefill(api.to_device(x), C)
    torch.cuda.synchronize()
    compare(res, oracle_run(x, interval=C), x.cu_seqlens, TOL[la.LA_BF16 if io == wl.BF16 else la.LA_F32],
            f"{n} sequences, C={C}")
