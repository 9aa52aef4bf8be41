"""Decode tiling on an MI355X at the edges of its rules, against the oracle:
segments whose first round of steps covers every row (and the appended one),
one row or one step more, in both storage types; and batches whose chunks
rounded up pass the resident blocks, so that the chunks are lengthened.
"""
import numpy as np
import pytest

from workloads import synth

from test_gpu_parity import Harness, close
from test_gpu_tiling import note, ragged, step

pytestmark = pytest.mark.gpu


# A chunk's four waves take 4 steps of 32 rows (fp32: of 16 or 8 rows).
@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("bf16", 64), ("f32", 64), ("f32", 128)])
def test_one_round_edges(dtype, D):
    lengths = [0, 1, 23, 24, 25, 47, 48, 49, 95, 96, 97, 127, 128, 129, 255, 256, 257, 1151, 1152, 1153]
    note("one round %s D=%d" % (dtype, D))
    rng = np.random.default_rng(D)
    HK, G = 1, 4
    H = Harness(1, [n + 8 for n in lengths], G * HK, HK, D, dtype)
    for b, n in enumerate(lengths):
        H.fill(0, b, 0, rng.standard_normal((n, D)).astype(np.float32), rng.standard_normal((n, D)).astype(np.float32),
               synth.score_vector(rng, n, "zipf"))
        H.set_len(0, b, n)
    H.c.flush()
    for t in range(3):
        out, ref = step(H, rng)
        close(out, ref, "step %d" % t)
    H.check_scores(0)
    assert int(H.c.dev_status[0]) == 0


@pytest.mark.parametrize("lengths,HK", [([2300, 2411, 2527, 2650, 2777, 2911, 3040, 3100], 8),
                                        ([1000] * 15 + [30000], 4),
                                        ([513] * 31 + [4097], 8),
                                        ([700 + 37 * b for b in range(70)], 3)])
def test_chunks_fit_the_resident_blocks(lengths, HK):
    note("fit %d sequences, %d heads" % (len(lengths), HK))
    rng = np.random.default_rng(len(lengths))
    H = ragged(rng, lengths=lengths, HK=HK, G=2, D=64)
    H.c.flush()
    for t in range(2):
        out, ref = step(H, rng)
        close(out, ref, "step %d" % t)
    H.check_scores(0)
    assert int(H.c.dev_status[0]) == 0
