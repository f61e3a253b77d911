"""Column widths of the fused scan: the narrow count of its mixed launch,
against a schedule of whole workgroups (in dispatch order, each to the compute
unit of its XCD that is free first, one workgroup per unit: two do not fit its
LDS), and the widths of the two-level passes."""
import heapq

import numpy as np
import pytest

from paper_2609_15030_amd import linattn as la

XCDS, XCD_CUS = 8, 32
STEP = {32: 0.76, 64: 1.0}       # a chunk's time at either width


def chunks(n, C):
    return n // C * -(-C // 64) + -(-(n % C) // 64)


def span(chains, narrow):
    """chains: chunk counts, longest first; the first `narrow` at 32 columns."""
    free = [[0.0] * XCD_CUS for _ in range(XCDS)]
    for rank, n in enumerate(chains):
        width = 32 if rank < narrow else 64
        for _ in range(128 // width):
            heap = free[rank % XCDS]
            heapq.heapreplace(heap, heap[0] + STEP[width] * n)
    return max(max(h) for h in free)


def choice(lens, H, C):
    """(narrow chains chosen, chunk counts longest first)"""
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    width, narrow = la.la_prefill_scan_columns(la.make_shape(len(lens), H, 128, 128, C, la.LA_BF16), cu)
    assert width in (32, 64)
    return narrow, sorted((chunks(n, C) for n in lens for _ in range(H)), reverse=True)


@pytest.mark.parametrize("n", [8, 9, 10, 12, 16])
def test_even_batches_take_no_second_round(n):
    """Up to 128 equal chains fit the chip at once at 64 columns: a mix with more
    workgroups than compute units would take a second whole chain."""
    narrow, chains = choice([4096] * n, 8, 256)
    assert 4 * narrow + 2 * (len(chains) - narrow) <= XCDS * XCD_CUS
    assert n > 8 or narrow == 64


def test_chosen_count_is_near_the_best_schedule():
    rng = np.random.default_rng(12)
    for _ in range(150):
        n, H, C = int(rng.integers(1, 45)), int(rng.choice([1, 3, 8])), int(rng.choice([64, 128, 256]))
        if n * H >= 512:
            continue
        w = rng.random(n) ** rng.integers(0, 4) + 0.02
        lens = np.maximum(1, np.exp(rng.uniform(np.log(1000), np.log(60000))) * w / w.sum()).astype(int)
        narrow, chains = choice(lens, H, C)
        counts = [0, len(chains)] + (list(range(8, len(chains), 8)) if n > 1 else [])
        best = min(span(chains, k) for k in counts)
        assert span(chains, narrow) <= 1.03 * best, (lens.tolist(), H, C, narrow)


@pytest.mark.parametrize("segments,width", [(1, 64), (16, 64), (17, 128), (32, 128), (34, 64), (48, 64), (50, 128),
                                            (64, 128), (72, 64), (82, 128)])
def test_replay_width_follows_the_rounds(segments, width):
    """The two-level replay (one workgroup per compute unit at 64 and at 128
    columns): the width whose rounds over 8 heads x segments are shorter."""
    shape = la.make_shape(1, 8, 128, 128, 1024, la.LA_BF16)
    assert la.la_prefill_scan_columns(shape, np.array([0, 1024 * segments], np.int32)) == (width, 0)


@pytest.mark.gpu
def test_two_level_widths_give_the_same_bits():
    """8,704 tokens of 8 heads at C = 512 (136 units: maps and replay at 128
    columns) against the oracle, and resumed at 4,608 (64 units: both at 64) and
    at 4,096 (72: maps at 128, replay at 64) with the cold run's bits."""
    import torch

    from paper_2609_15030_amd import api
    from paper_2609_15030_amd import workloads as wl
    from parity import TOL, compare, oracle_run
    N, C = 8704, 512
    x = wl.random_inputs(77, [N], 8, 128, 128, wl.BF16, gate_scale=0.02)
    res = api.prefill(api.to_device(x), C)
    torch.cuda.synchronize()
    compare(res, oracle_run(x, interval=C), x.cu_seqlens, TOL[la.LA_BF16], "two-level widths")
    for B in (4608, 4096):
        row = B // C - 1
        r2 = api.prefill_resume(api.to_device(x.tokens(B, N)), [B], res.ckpt[row:row + 1].clone(), C)
        torch.cuda.synchronize()
        assert torch.equal(r2.o, res.o[B:]) and torch.equal(r2.final_state, res.final_state)
        assert torch.equal(r2.ckpt, res.ckpt[row + 1:])
