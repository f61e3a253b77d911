"""The narrow count of the fused scan's mixed launch, against a schedule of
whole workgroups: in dispatch order, each to the compute unit of its XCD that is
free first, one workgroup per unit (two do not fit its LDS)."""
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
