"""Decode tiling on an MI355X at the edges of its rules, against the oracle:
segments whose first round of steps covers every row (and the appended one),
one row or one step more, in both storage types; and batches whose chunks
rounded up pass two blocks a CU, so that the chunks may be lengthened; and how
many blocks the split then keeps.
"""
import numpy as np
import pytest
import torch

from paper_2511_06029_amd import lethe as L
from workloads import synth

from test_gpu_parity import DEV, Harness, close
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


def multi_chunk_blocks(lengths, HK, G=2, D=64, spare=40):
    """Blocks a decode call's split gives segments of more than one chunk: each
    writes one partial, and no other block writes to the workspace."""
    c = L.LetheCache(1, [n + spare for n in lengths], G * HK, HK, D, device=DEV)
    c.k.normal_()
    c.v.normal_()
    c.len.copy_(torch.tensor([lengths], dtype=torch.int32))
    c.flush()
    q = torch.randn((len(lengths), G * HK, D), device=DEV).to(torch.bfloat16)
    kn = torch.randn((len(lengths), HK, D), device=DEV).to(torch.bfloat16)
    ws = c.workspace(L.OP_DECODE)
    ws.fill_(0xA5)
    out = torch.zeros(q.shape, device=DEV)
    L.decode_attn_score(c, 0, q, kn, kn, 0.9, 0.0, out, ws)
    torch.cuda.synchronize()
    stride = (4 * G * (D + 2) + 127) // 128 * 128
    parts = ws[:ws.numel() // stride * stride].view(-1, stride)
    assert int(c.dev_status[0]) == 0 and bool(torch.isfinite(out).all())
    return int((parts != 0xA5).any(dim=1).sum())


# Lengths and the blocks of their split.  Lengthening would leave 352, 528,
# 384, 312 and 576 of the first five; the last three pass.
@pytest.mark.parametrize("lengths,HK,blocks", [([2000] * 22, 8, 528), ([3300] * 22, 8, 704), ([1300] * 48, 4, 576),
                                               ([513] * 31 + [4097], 8, 592), ([3300] * 24, 8, 768),
                                               ([2000] * 13, 8, 416), ([2000] * 17, 8, 408), ([5000] * 32, 4, 512)])
def test_chunks_are_lengthened_only_where_most_blocks_stay(lengths, HK, blocks):
    note("fit %d sequences of %d to %d rows" % (len(lengths), min(lengths), max(lengths)))
    assert multi_chunk_blocks(lengths, HK) == blocks


# Steps of 32 rows: 63 a segment.  The default split has 32, 64 and 416 blocks.
@pytest.mark.parametrize("env,lengths,HK,blocks", [
    ({"LETHE_DECODE_STEPS_PER_CHUNK": "1"}, [2000], 2, 126),   # one step a chunk
    ({"LETHE_DECODE_MIN_CHUNKS": "512"}, [2000], 2, 126),
    ({"LETHE_DECODE_STEPS_PER_CHUNK": "2", "LETHE_DECODE_MIN_CHUNKS": "1"}, [2000] * 2, 2, 128),  # two
    ({"LETHE_DECODE_BLOCKS": "512"}, [2000] * 13, 8, 520),     # 512, and one more for some segments
])
def test_settings_of_the_environment_are_taken_as_they_are(env, lengths, HK, blocks, monkeypatch):
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    note("split by %s" % env)
    assert multi_chunk_blocks(lengths, HK) == blocks


@pytest.mark.parametrize("lengths,HK,blocks", [([2000], 2, 32), ([2000] * 2, 2, 64), ([130], 1, 2)])
def test_default_chunks_have_four_steps(lengths, HK, blocks):
    note("default split of %s" % lengths)
    assert multi_chunk_blocks(lengths, HK) == blocks


@pytest.mark.parametrize("lengths,HK,frac,blocks", [([2000], 2, 0.4, 32), ([2000], 2, 1.0, 32), ([1300] * 2, 3, 0.1, 66)])
def test_compacting_call_is_split_by_the_rows_it_reads(lengths, HK, frac, blocks):
    """Four 32-row steps a chunk (63 and 41 steps and the spare one), whatever
    the plan keeps; a segment's row count after the call is what it keeps."""
    note("compacting call, %.0f%% of %s" % (100 * frac, lengths))
    D, G = 64, 2
    c = L.LetheCache(1, [n + 40 for n in lengths], G * HK, HK, D, device=DEV)
    c.k.normal_()
    c.v.normal_()
    c.len.copy_(torch.tensor([lengths], dtype=torch.int32))
    c.flush()
    keep = torch.zeros((1, c.rows_per_layer), dtype=torch.uint8, device=DEV)
    kept = [int(frac * n) for n in lengths]
    for b, n in enumerate(lengths):
        for h in range(HK):
            r0, _ = c.seg_rows(b, h)
            keep[0, r0 + n - kept[b]:r0 + n] = 1
    plan, ws = c.workspace(L.OP_COMPACT_PLAN), c.workspace(L.OP_DECODE)
    L.kv_compact_plan(c, keep, plan)
    ws.fill_(0xA5)
    q = torch.randn((len(lengths), G * HK, D), device=DEV).to(torch.bfloat16)
    kn = torch.randn((len(lengths), HK, D), device=DEV).to(torch.bfloat16)
    out = torch.zeros(q.shape, device=DEV)
    L.decode_attn_score_compact(c, 0, q, kn, kn, 0.9, 0.0, out, plan, ws)
    torch.cuda.synchronize()
    stride = (4 * G * (D + 2) + 127) // 128 * 128
    parts = ws[:ws.numel() // stride * stride].view(-1, stride)
    assert int(c.dev_status[0]) == 0 and bool(torch.isfinite(out).all())
    assert c.len[0].tolist() == [k + 1 for k in kept]
    assert int((parts != 0xA5).any(dim=1).sum()) == blocks
