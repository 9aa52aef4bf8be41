"""GPU test of the prefill call's host bounds (run on an MI355X): max_q_len and
max_kv_len are upper bounds that may be loose, up to INT32_MAX.  The outputs
and scores are those of the tight bounds, bit for bit, and a sequence whose
sizes do not fit is still flagged.
"""
import numpy as np
import pytest
import torch

from paper_2511_06029_amd import lethe as L

from test_gpu_prefill import Case, close, f32, note

pytestmark = pytest.mark.gpu

INT32_MAX = 2**31 - 1


def results(cs, **bounds):
    cs.out.fill_(float("nan"))
    cs.c.score.zero_()
    cs.run(**bounds)
    return f32(cs.out), f32(cs.c.score)


@pytest.mark.parametrize("max_q,max_kv", [(None, 1 << 20), (1 << 20, INT32_MAX), (INT32_MAX, INT32_MAX)])
@pytest.mark.parametrize("B,HK", [(3, 2), (128, 8)])  # 64- and 128-row key blocks at the loose bound
def test_loose_bounds(B, HK, max_q, max_kv):
    """1024 segments and a bound of 2^20 rows make more than 2^32 threads of
    key blocks, nearly all of them empty."""
    note("prefill bounds B=%d HK=%d max_q=%s max_kv=%s" % (B, HK, max_q, max_kv))
    lengths = [1 + (11 * b) % 41 for b in range(B)]
    cs = Case(64, 2, HK, lengths, [(n + 1) // 2 for n in lengths], seed=B)
    out, score = results(cs)
    assert np.all(np.isfinite(out))
    loose_out, loose_score = results(cs, max_q=max_q, max_kv=max_kv)
    np.testing.assert_array_equal(loose_out, out)
    np.testing.assert_array_equal(loose_score, score)
    assert int(cs.c.dev_status[0]) == 0


def test_more_queries_than_rows_is_flagged_at_any_bound():
    note("prefill bounds, flagged")
    cs = Case(64, 2, 2, [40, 50], [20, 30], seed=1)
    cs.q_len[1] = 51
    cs.run(max_q=INT32_MAX, max_kv=INT32_MAX)
    assert int(cs.c.dev_status[0]) == L.DEV_BAD_LAYOUT
    out = f32(cs.out)
    assert np.all(np.isfinite(out[:20])) and np.all(np.isnan(out[20:]))
    torch.cuda.synchronize()


def test_keys_past_the_grids_second_dimension():
    """32768 blocks of 128 keys fill the second grid dimension; the rows after
    them lie in the third.  One query over them against float64.  A weight's sum is
    65536 dependent fp32 additions of a lane, whose roundings of 2^-24 grow as
    their square root (1.5e-5 relative); an output is 524288 of them, at worst
    2^-24 each in one direction (3e-2), so the suite's tolerance is what it is
    held to."""
    n = 32768 * 128 + 70
    note("prefill bounds, %d keys" % n)
    c = L.LetheCache(1, [n], 1, 1, 64, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(5)
    c.k[0].normal_(generator=g)
    c.v[0].normal_(generator=g)
    c.len.fill_(n)
    q = torch.randn((1, 1, 64), generator=g, device="cuda").to(torch.bfloat16)
    out = torch.zeros((1, 1, 64), device="cuda")
    one = torch.ones(1, dtype=torch.int32, device="cuda")
    L.prefill_attn_score(c, 0, q, torch.zeros(1, dtype=torch.int64, device="cuda"), one, 1, INT32_MAX, 0.0, out,
                         c.prefill_workspace(1))
    torch.cuda.synchronize()
    p = torch.softmax(torch.mv(c.k[0].double(), q[0, 0].double()) / 8.0, dim=0)
    ref = torch.mv(c.v[0].double().t().contiguous(), p)
    assert float(((c.score[0].double() - p).abs() / p).max()) < 2e-5
    close(f32(out[0, 0]), ref.cpu().numpy(), "out")
    assert int(c.dev_status[0]) == 0
