"""The fused scan's chunk pipeline at its edges (bf16).

The scan, output and loader waves of a workgroup work on different chunks
between two barriers, so runs of one to a few chunks exercise the
pipeline's fill and drain, odd and even counts its two register sets, and
ragged tails its masked rows.  Every width is compared with the oracle, and
with the same sequence inside a batch of 512 chains (128 columns at
dk = dv = 128), whose bits must be equal with gates that keep the state
alive as well as with ones that do not.
"""
import numpy as np
import pytest
import torch

from paper_2609_15030_amd import api
from paper_2609_15030_amd import linattn as la
from paper_2609_15030_amd import workloads as wl
from parity import TOL, compare, oracle_run

pytestmark = pytest.mark.gpu


def _batch(xs):
    cat = lambda f: np.concatenate([getattr(x, f) for x in xs])
    lens = np.concatenate([np.diff(x.cu_seqlens) for x in xs])
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    return wl.Inputs(cat("q"), cat("k"), cat("v"), cat("g"), cat("beta"), cu, xs[0].io_dtype)


def _run(x, C, variant=0):
    res = api.prefill(api.to_device(x), C, variant)
    torch.cuda.synchronize()
    return res


@pytest.mark.parametrize("dk,dv", [(128, 128), (64, 128), (128, 64), (64, 64)])
@pytest.mark.parametrize("C", [64, 100, 256])
def test_short_runs_against_the_oracle(dk, dv, C):
    lens = [0, 1, 15, 16, 17, 63, 64, 65, 128, 129, 191, 193, 256, 300, 330]
    x = wl.random_inputs(900 + dk + dv + C, lens, 3, dk, dv, wl.BF16, gate_scale=0.05)
    compare(_run(x, C, 1), oracle_run(x, interval=C, variant=1), x.cu_seqlens, TOL[la.LA_BF16],
            f"pipeline edges dk={dk} dv={dv} C={C}")


@pytest.mark.parametrize("gate_scale", [1.0, 0.01])
@pytest.mark.parametrize("length", [65, 300, 1500])
def test_widths_agree_bit_for_bit(length, gate_scale):
    H, C = 8, 256
    x = wl.random_inputs(950 + length, [length], H, 128, 128, wl.BF16, gate_scale=gate_scale)
    fill = wl.random_inputs(951, [40] * 63, H, 128, 128, wl.BF16, gate_scale=gate_scale)
    even = wl.random_inputs(952, [length] * 31, H, 128, 128, wl.BF16, gate_scale=gate_scale)
    alone = _run(x, C)
    for batch, width in ((_batch([fill, x]), 128), (_batch([even, x]), 64)):
        shape = la.make_shape(batch.n_seqs, H, 128, 128, C, la.LA_BF16)
        assert la.la_prefill_scan_columns(shape, batch.cu_seqlens)[0] == width
        res = _run(batch, C)
        assert torch.equal(res.o[-length:], alone.o) and torch.equal(res.final_state[-1], alone.final_state[0]), width
        if alone.n_ckpt_rows:
            assert torch.equal(res.ckpt[-alone.n_ckpt_rows:], alone.ckpt), width
