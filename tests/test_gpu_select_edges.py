"""Selection on an MI355X at the edges of its register slots, against the
oracle bit for bit: candidate counts around two slots, the groups of eight
slots and all 32 slots of a block (256 threads per head, 1024 for head sums),
with windows that shift the candidates, ties, infinities and NaN.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_06029_amd import lethe as L

from test_gpu_shrink import DEV, make_cache, masks_of, note

pytestmark = pytest.mark.gpu


def edges(threads):
    return [k * threads + d for k in (1, 2, 8, 9, 16, 24, 32) for d in (-1, 0, 1)]


@pytest.mark.parametrize("kind", ["zipf", "ties", "special"])
def test_per_head_slots(kind):
    """Candidates are n - recent - sink rows: 68 more rows put them on the edge."""
    note("select edges per head, %s" % kind)
    lengths = edges(256) + [n + 68 for n in edges(256)]
    c, s = make_cache(lengths, 1, 2, 5, kind)
    budget = np.array([[max(1, int(n * (0.9 if b % 2 else 0.3)))] for b, n in enumerate(lengths)], np.int32)
    keep = torch.full((1, c.rows_per_layer), 7, dtype=torch.uint8, device=DEV)
    L.rasr_select(c, torch.from_numpy(budget).to(DEV), 64, 4, keep)
    torch.cuda.synchronize()
    got = masks_of(c, keep, lengths, 1, 2)
    for b, n in enumerate(lengths):
        for h in range(2):
            want = oracle.rasr_select(s[0, b, h], budget[b, 0], 64, 4)
            np.testing.assert_array_equal(got[0, b, h], want, err_msg="n=%d h%d" % (n, h))
    assert int(c.dev_status[0]) == 0


# Every number of heads in the group of the head sums, and a second group short of a head.
@pytest.mark.parametrize("HK,kind", [(1, "zipf"), (2, "special"), (3, "zipf"), (4, "ties"), (5, "zipf"), (6, "zipf"),
                                     (8, "zipf")])
def test_head_sum_slots(HK, kind):
    note("select edges head sums, HK=%d %s" % (HK, kind))
    lengths = edges(1024)
    c, s = make_cache(lengths, 1, HK, 7 + HK, kind)
    sums = [oracle.head_sum_f32(np.stack([s[0, b, h] for h in range(HK)])) for b in range(len(lengths))]
    budget = np.array([[int(n * (0.9 if b % 2 else 0.3))] for b, n in enumerate(lengths)], np.int32)
    keep = torch.full((1, c.rows_per_layer), 7, dtype=torch.uint8, device=DEV)
    L.rasr_select_shared(c, torch.from_numpy(budget).to(DEV), 0, 0, keep)
    torch.cuda.synchronize()
    got = masks_of(c, keep, lengths, 1, HK)
    for b, n in enumerate(lengths):
        want = oracle.rasr_select_shared(np.stack([s[0, b, h] for h in range(HK)]), budget[b, 0], 0, 0)
        for h in range(HK):
            np.testing.assert_array_equal(got[0, b, h], want, err_msg="shared n=%d h%d" % (n, h))
    ev = torch.full((1, len(lengths)), 100, dtype=torch.int32, device=DEV)
    bp = torch.zeros((1, len(lengths)), dtype=torch.int32, device=DEV)
    L.segmented_shrink(c, 10, 20.0, 16, 2, ev, bp, keep)
    torch.cuda.synchronize()
    got = masks_of(c, keep, lengths, 1, HK)
    for b, n in enumerate(lengths):
        want, wbp, wlev = oracle.segmented_shrink(sums[b], 10, 20.0, 16, 2, 100)
        assert (int(bp[0, b]), int(ev[0, b])) == (wbp, wlev), n
        for h in range(HK):
            np.testing.assert_array_equal(got[0, b, h], want, err_msg="shrink n=%d h%d" % (n, h))
    assert int(c.dev_status[0]) == 0
