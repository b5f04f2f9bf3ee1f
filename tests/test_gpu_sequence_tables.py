"""A call on whole sequences has them, instead of its tiles, in the launch arguments where they fit (12 bytes of each and 2 of each of their
blocks, 3584 bytes in all) and the launch is short. O, LSE and dQ are the same bits as with a table in memory, dK and dV those of the
same kernel: both sides of the limits, remainders of blocks, equal lengths, empty and flagged sequences, more heads than XCDs."""
import numpy as np
import pytest
import torch

from paper_2509_21841_amd import binding as B
from paper_2509_21841_amd import synth
from test_gpu_tile_tables import bits, run

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TABLE = [1] * 300   # behind a batch: no longer fits


def uploads(lengths, Hq, Hkv, q, k, v, do, n):
    """Whether the forward's and the backward's table go through the workspace: the counters in front of it are written with it."""
    cu, d = synth.cu_seqlens(lengths), q.shape[2]
    q, k, v, do = q[:n], k[:n], v[:n], do[:n]
    sh = B.make_shape(n, len(lengths), Hq, Hkv, d)
    ws = [torch.full((B.workspace_bytes(fn, sh, cu),), 0xA5, dtype=torch.uint8, device=DEV) for fn in (B.FN_FWD, B.FN_BWD)]
    o, lse = B.varlen_attn_fwd(q, k, v, cu, ws=ws[0])
    B.varlen_attn_bwd(do, q, k, v, o, lse, cu, ws=ws[1])
    return tuple(not bool((w[:64] == 0xA5).all()) for w in ws)


# Launches whose tiles do not fit the arguments (over 112, 1024 items and more), and whether their tables are uploaded. The first five fill
# 3584 bytes exactly, exactly with more blocks, by four bytes less, and by 4 and 16 too many; the seventh and eighth have 18 and 16 KV
# heads; the tenth and eleventh are on the two sides of the backward's limit on a launch's work, the last one is beyond the forward's
@pytest.mark.parametrize("lengths,Hq,Hkv,dims,table", [
    ([100] * 256, 2, 1, (64, 128), (False, False)), ([128] * 248 + [129] * 7, 2, 2, (64, 128), (False, False)),
    ([128] * 250 + [129] * 5, 2, 1, (64, 128), (False, False)), ([128] * 255 + [129, 0], 2, 2, (64, 128), (True, True)),
    ([1] * 257, 2, 1, (64, 128), (True, True)), ([127, 128, 129, 0, 257, 1] * 20, 4, 2, (64, 128), (False, False)),
    ([300, 0, 257] * 20, 18, 18, (64, 128), (False, False)), ([2049, 2049, 640, 1], 32, 16, (64,), (False, False)),
    ([130, 390, 130] * 30, 3, 3, (64, 128), (False, False)), ([700, 129, 1] * 24, 8, 2, (128,), (False, False)),
    ([700, 129, 1] * 24, 16, 4, (128,), (False, True)),
    ([900] * 48, 16, 16, (128,), (True, True))])
def test_sequences_in_the_arguments_equal_a_table(lengths, Hq, Hkv, dims, table):
    blocks = sum(-(-x // 128) for x in lengths)
    assert blocks > 112 or blocks * Hq >= 1024
    for d in dims:
        check(lengths, Hq, Hkv, d, table)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lengths,Hq,Hkv", [([2049, 2049, 640, 1], 16, 8), ([33, 4000], 18, 18)])
def test_tiles_in_the_arguments_equal_a_table(lengths, Hq, Hkv, d):
    check(lengths, Hq, Hkv, d, (False, False))


def check(lengths, Hq, Hkv, d, table):
    n = sum(lengths)
    q, k, v, do = synth.make_qkv(n + len(TABLE), Hq, Hkv, d, 201, DEV, with_dout=True)
    assert uploads(lengths, Hq, Hkv, q, k, v, do, n) == table
    assert uploads(lengths + TABLE, Hq, Hkv, q, k, v, do, n + len(TABLE)) == (True, True)
    got, want = run(lengths, q, k, v, do, n), run(lengths + TABLE, q, k, v, do, n + len(TABLE))
    for a, b in zip(got[:3], want[:3]):
        assert torch.equal(bits(a), bits(b[:n]))
    for a, b in zip(got[3:], want[3:]):  # (the bound of test_gpu_tile_tables.py: two orders of the float sums)
        a, b = a.float(), b[:n].float()
        assert bool(((a - b).abs() <= 2.0 ** -7 * torch.maximum(a.abs(), b.abs()) + 1e-4).all())


def test_flagged_sequences():
    lengths, Hq, Hkv, d = [300, 0, 129, 700, 1, 300] * 12, 8, 2, 128
    skip = np.asarray([i % 3 == 0 for i in range(len(lengths))], np.uint8)
    cu = synth.cu_seqlens(lengths)
    q, k, v = synth.make_qkv(sum(lengths), Hq, Hkv, d, 203, DEV)
    o, lse = B.varlen_attn_fwd(q, k, v, cu)
    rows = torch.from_numpy(np.repeat(skip, lengths).astype(bool)).to(DEV)
    for call in (B.varlen_attn_fwd, B.varlen_attn_fwd_noalloc):
        o2, lse2 = torch.full_like(o, 3.0), torch.full_like(lse, 3.0)
        call(q, k, v, cu, o=o2, lse=lse2, seq_skip=skip)
        assert bool((o2[rows] == 3.0).all()) and bool((lse2[:, rows] == 3.0).all())
        assert torch.equal(bits(o2[~rows]), bits(o[~rows])) and torch.equal(bits(lse2[:, ~rows]), bits(lse[:, ~rows]))


def test_uploaded_and_argument_tables_in_one_graph():
    """Replays read their own copy of either kind, whatever calls run in between."""
    Hq, Hkv, d = 8, 2, 128
    batches = [[130] * 64, [130] * 64 + TABLE]
    T = sum(batches[1])
    q, k, v, do = synth.make_qkv(T, Hq, Hkv, d, 205, DEV, with_dout=True)
    outs = [[torch.empty_like(x[:sum(l)]) for x in (q, q, k, v)] + [torch.empty((Hq, sum(l)), device=DEV)] for l in batches]

    def call():
        for l, (o, dq, dk, dv, lse) in zip(batches, outs):
            n, cu = sum(l), synth.cu_seqlens(l)
            B.varlen_attn_fwd(q[:n], k[:n], v[:n], cu, o=o, lse=lse)
            B.varlen_attn_bwd(do[:n], q[:n], k[:n], v[:n], o, lse, cu, dq=dq, dk=dk, dv=dv)

    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for seed in (207, 209, 211):
        q.copy_(synth.make_qkv(T, Hq, Hkv, d, seed, DEV)[0])
        graph.replay()
        torch.cuda.synchronize()
        got = [x.clone() for out in outs for x in out]
        call()
        torch.cuda.synchronize()
        for a, b in zip(got, [x for out in outs for x in out]):
            assert torch.equal(bits(a), bits(b))
