"""fp32 prefill over the row tiles a chunk can have: the interval bounds a
chunk's rows, so C = 1 .. 16, 17 .. 32, 33 .. 48 and above run kernels of one
to four 16-row tiles.  Cold and resumed runs against the oracle at the
edges of those ranges, for every head size and both rules."""
import numpy as np
import pytest
import torch

from paper_2609_15030_amd import api
from paper_2609_15030_amd import linattn as la
from paper_2609_15030_amd import workloads as wl
from parity import TOL, compare, oracle_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dk,dv", [(64, 64), (64, 128), (128, 64), (128, 128)])
@pytest.mark.parametrize("C", [1, 15, 16, 17, 32, 33, 48, 49, 64, 80])
def test_row_tiles_against_the_oracle(dk, dv, C):
    H, lens = 2, [0, 1, 16, 17, 47, 64, 97, 130]
    x = wl.random_inputs(1000 + C + dk + 2 * dv, lens, H, dk, dv, wl.F32, gate_scale=0.05)
    variant = C % 2
    res = api.prefill(api.to_device(x), C, variant)
    torch.cuda.synchronize()
    compare(res, oracle_run(x, interval=C, variant=variant), x.cu_seqlens, TOL[la.LA_F32],
            f"fp32 tiles dk={dk} dv={dv} C={C}")
    # the last sequence resumed from one of its checkpoints: the cold run's bits
    B = 130 // (2 * C) * C
    if B:
        seq = x.seq(len(lens) - 1)
        row = int(res.ckpt_offsets[-1]) + B // C - 1
        r2 = api.prefill_resume(api.to_device(seq.tokens(B, 130)), [B], res.ckpt[row:row + 1].clone(), C, variant)
        torch.cuda.synchronize()
        assert torch.equal(r2.o, res.o[-(130 - B):]) and torch.equal(r2.final_state[0], res.final_state[-1])
