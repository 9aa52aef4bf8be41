"""Rounding of the prefill outputs on an MI355X.  The weights enter the P V
product in two bf16 halves (17 bits), and an output is divided by the sum of
the halves.  With V = 1 every output is therefore 1 up to the fp32 roundings
of two sums over the same values.
"""
import numpy as np
import pytest
import torch

from test_gpu_prefill import Case, f32, note

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,G", [(128, 4), (64, 3), (128, 7)])
@pytest.mark.parametrize("lengths", [[3, 17, 32, 33, 64], [5, 29, 41, 50, 63]])
def test_weights_of_one_step_sum_to_one(D, G, lengths):
    """Rows of one 64-key step: two sums of up to 128 terms of one sign and of
    at most 1, each term rounded once at 2^-24 of the running sum.  As a random
    walk that is sqrt(128) 2^-24 / sqrt(3) = 3.9e-7 of the sum at the most, and
    a quarter of it where a few keys hold the weight; divided by the sum of the
    unsplit weights instead, the halves' missing 2^-18 shows (5e-7)."""
    note("prefill rounding D=%d G=%d %s" % (D, G, lengths))
    cs = Case(D, G, 2, lengths, lengths, seed=D + G)
    cs.c.v[cs.layer].fill_(1.0)
    cs.run()
    err = f32(cs.out).astype(np.float64) - 1.0
    rms = float(np.sqrt(np.mean(err**2)))
    note("rms %.3e" % rms)
    assert rms < 3e-7
    assert int(cs.c.dev_status[0]) == 0
    torch.cuda.synchronize()
