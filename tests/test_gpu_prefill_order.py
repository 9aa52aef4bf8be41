"""GPU parity of the prefill kernels where their tiling changes (run on an
MI355X): units of one block that lie in different query tiles, steps of 64
keys, key blocks of 64 and 128 rows with several item groups, and batches of
different lengths whose blocks are ordered over all sequences.  Outputs and
scores against the oracle, within the tolerance of test_gpu_prefill.py.
"""
import numpy as np
import pytest
import torch

from test_gpu_prefill import Case, f32, note

pytestmark = pytest.mark.gpu

# Around the 32-query tiles, the 64-key steps and the 64- and 128-row key blocks.
EDGES = [63, 64, 65, 127, 128, 129, 191, 193]


@pytest.mark.parametrize("D,G,HK", [(128, 4, 1), (128, 1, 2), (64, 3, 2), (128, 7, 1), (64, 8, 1), (128, 6, 1)])
def test_tile_edges(D, G, HK):
    note("prefill edges D=%d G=%d HK=%d" % (D, G, HK))
    qlens = [min(q, n) for q, n in zip([63, 1, 33, 127, 96, 129, 31, 64], EDGES)]
    cs = Case(D, G, HK, EDGES, qlens, seed=7 * D + G, s_init=True)
    cs.run()
    cs.check()


# Grids past the 512 resident blocks: 48 or 40 segments of up to 700 rows.
@pytest.mark.parametrize("G,HK,lengths,qlens", [
    (4, 8, [700, 33, 257, 1, 512, 64], None),
    (3, 8, [90, 700, 300, 31, 650, 128], [90, 650, 1, 0, 100, 128]),
    (7, 8, [700, 40, 444, 95, 330], [300, 40, 299, 17, 330]),
    (4, 8, [640] * 6, None),
])
def test_blocks_over_all_sequences(G, HK, lengths, qlens):
    note("prefill order G=%d lengths=%s" % (G, lengths))
    cs = Case(128, G, HK, lengths, qlens or lengths, seed=G + len(lengths))
    cs.run()
    assert np.all(np.isfinite(f32(cs.out)))  # every row written
    cs.check(heads=[0, HK - 1])


# One lane a sequence: 64 are ordered, 65 keep unit order (1280 and more blocks).
@pytest.mark.parametrize("D,G,nseq", [(64, 2, 64), (64, 2, 65), (128, 3, 64)])
def test_most_sequences_of_an_ordered_batch(D, G, nseq):
    note("prefill order, %d sequences, D=%d" % (nseq, D))
    lengths = [1 + (53 * b) % 300 for b in range(nseq)]
    lengths[7] = 301
    qlens = [n if b % 3 else max(0, n - 40) for b, n in enumerate(lengths)]
    cs = Case(D, G, 4, lengths, qlens, seed=nseq + D)
    cs.run()
    assert np.all(np.isfinite(f32(cs.out)))
    cs.check(seqs=[0, 1, 6, 7, 31, 62, nseq - 1], heads=[0, 3])


def test_flagged_sequences_in_an_ordered_batch():
    lengths, qlens = [700, 64, 300, 512, 33, 200], [700, 64, 300, 512, 33, 200]
    note("prefill order, flagged")
    cs = Case(128, 4, 8, lengths, qlens, seed=3)
    cs.q_len[1] = 65   # more queries than rows
    cs.q_len[4] = 0    # no queries, and a length past its capacity
    cs.c.len[cs.layer, 4] = 99
    cs.run(max_q=700, max_kv=700)
    from paper_2511_06029_amd import lethe as L
    assert int(cs.c.dev_status[0]) == L.DEV_BAD_LAYOUT
    cs.c.dev_status.zero_()
    out = f32(cs.out)
    for b in (1, 4):
        r = int(cs.starts[b])
        assert np.all(np.isnan(out[r:r + qlens[b]])), "a flagged sequence's rows were written"
    cs.check(seqs=[0, 2, 3, 5], heads=[0, 7])


@pytest.mark.parametrize("G", [3, 4, 7])
def test_infinite_value_row_reaches_later_queries_only(G):
    """A value row with an infinity may reach the queries of its own 32-query
    tile (their weight-0 products) and later ones, never an earlier tile's,
    also where both tiles' units share a block."""
    note("prefill inf G=%d" % G)
    cs = Case(128, G, 1, [96], [96], seed=G)
    r0, _ = cs.c.seg_rows(0, 0)
    cs.c.v[cs.layer, r0 + 40, 5] = float("inf")
    cs.run()
    out = f32(cs.out)
    assert np.all(np.isfinite(out[:32]))
    assert not np.isfinite(out[40:, :, 5]).any()
    assert np.all(np.isfinite(np.delete(out, 5, axis=2)))
