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


def test_fp32_output_kernel_by_slot():
    """fp32 at dk = 128 launches the split output kernel over the same units."""
    n, C, H = 65, 100, 8
    rng = np.random.default_rng(n)
    lens = [int(v) for v in rng.integers(0, 260, n)]
    lens[0] = lens[31] = lens[-1] = 0
    assert n * H * 2 * -(-max(lens) // C) > 2048
    for dv in (64, 128):
        x = wl.random_inputs(400 + dv, lens, H, 128, dv, wl.F32, gate_scale=0.05)
        shape = la.make_shape(n, H, 128, dv, C, la.LA_F32)
        assert la.la_prefill_form(shape) == la.LA_FORM_SPLIT_DK_SCAN
        res = api.prefill(api.to_device(x), C)
        torch.cuda.synchronize()
        compare(res, oracle_run(x, interval=C), x.cu_seqlens, TOL[la.LA_F32], f"fp32 dk=128 dv={dv} by slot")


@pytest.mark.parametrize("io", [wl.BF16, wl.F32])
def test_one_long_sequence_by_slot(io):
    """One sequence needs no lookup; its slots still run past its chunks (C = 100)."""
    N, C, H = 13050, 100, 8
    assert H * (N // C * 2 + 1) > 2048
    x = wl.random_inputs(500, [N], H, 64, 64, io, gate_scale=0.02)
    res = api.prefill(api.to_device(x), C)
    torch.cuda.synchronize()
    compare(res, oracle_run(x, interval=C), x.cu_seqlens, TOL[la.LA_BF16 if io == wl.BF16 else la.LA_F32],
            f"one sequence of {N} by slot")
