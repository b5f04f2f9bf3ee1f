"""Where a call's tile table travels: in the launch arguments (up to 112 tiles and under 1024 work items) or through the
workspace. O, LSE and dQ of a sequence are the same bits whichever way its table took and whatever else is in the batch
(dK and dV up to the order of their float sums, which depends on how full the launch is); the table's length and the
number of items are taken to both sides of their limits. Calls that upload a table are also recorded into a HIP
graph and replayed between other calls that use the staging buffers."""
import numpy as np
import pytest
import torch

from paper_2509_21841_amd import binding as B
from paper_2509_21841_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# behind a batch: more sequences than the launch arguments hold (298), so that its tables are in memory
MANY = [1] * 300


def bits(t):
    return t.contiguous().view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32)


def run(lengths, q, k, v, do, n):
    """Forward and backward of the first n tokens, cut into `lengths`."""
    cu = synth.cu_seqlens(lengths)
    q, k, v, do = q[:n], k[:n], v[:n], do[:n]
    o, lse = B.varlen_attn_fwd(q, k, v, cu)
    o2, lse2 = torch.zeros_like(o), torch.zeros_like(lse)
    B.varlen_attn_fwd_noalloc(q, k, v, cu, o2, lse2)
    assert torch.equal(bits(o), bits(o2)) and torch.equal(bits(lse), bits(lse2))
    return (o, lse.t()) + tuple(B.varlen_attn_bwd(do, q, k, v, o, lse, cu))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("tiles,Hq,Hkv", [(1, 1, 1), (55, 2, 1), (56, 2, 2), (57, 2, 1), (111, 4, 2), (112, 1, 1), (112, 2, 2),
                                          (113, 1, 1), (50, 20, 4), (52, 20, 4), (31, 33, 11)])
def test_short_tables_equal_long_ones(tiles, Hq, Hkv, d):
    # forward: `tiles` tiles; backward: twice that in one table (56 is its limit)
    lengths = [129 + i % 100 for i in range(tiles // 2)] + ([40] if tiles % 2 else [])
    extra = [1000] * 15   # 120 more tiles: the other route
    n = sum(lengths)
    q, k, v, do = synth.make_qkv(n + sum(extra), Hq, Hkv, d, 83, DEV, with_dout=True)
    got = run(lengths, q, k, v, do, n)
    want = run(lengths + extra, q, k, v, do, n + sum(extra))
    for a, b in zip(got[:3], want[:3]):
        assert torch.equal(bits(a), bits(b[:n]))
    for a, b in zip(got[3:], want[3:]):
        # the same products added up in float in two orders (under 1e-5 apart: a thousand terms of order one at 2^-24 each),
        # then rounded to bfloat16: neighbouring values at most, 2^-7 of the larger one
        a, b = a.float(), b[:n].float()
        assert bool(((a - b).abs() <= 2.0 ** -7 * torch.maximum(a.abs(), b.abs()) + 1e-4).all())


def test_uploaded_tables_in_a_captured_graph():
    """Replays of a graph that uploads tables, between other calls that use the staging buffers."""
    lengths = [130] * 64 + MANY
    Hq, Hkv, d, T = 8, 2, 128, sum(lengths)
    cu = synth.cu_seqlens(lengths)
    q, k, v, do = synth.make_qkv(T, Hq, Hkv, d, 91, DEV, with_dout=True)
    o, lse = B.varlen_attn_fwd(q, k, v, cu)
    grads = [torch.empty_like(x) for x in (q, k, v)]
    call = lambda: (B.varlen_attn_fwd(q, k, v, cu, o=o, lse=lse),
                    B.varlen_attn_bwd(do, q, k, v, o, lse, cu, dq=grads[0], dk=grads[1], dv=grads[2]))
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        for _ in range(4):
            call()                               # the workspaces of the capture stream
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        call()
    other = [300, 1, 77] * 40
    oq, ok, ov = synth.make_qkv(sum(other), Hq, Hkv, d, 92, DEV)
    for rep in range(4):
        fresh = synth.make_qkv(T, Hq, Hkv, d, 930 + rep, DEV, with_dout=True)
        for dst, src in zip((q, k, v, do), fresh):
            dst.copy_(src)
        B.varlen_attn_fwd(oq, ok, ov, synth.cu_seqlens(other))       # takes free staging buffers in between
        wo, wl = B.varlen_attn_fwd(q, k, v, cu)
        want = [wo, wl] + list(B.varlen_attn_bwd(do, q, k, v, wo, wl, cu))
        for t in (o, lse, *grads):
            t.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for a, b in zip((o, lse, *grads), want):
            assert torch.equal(bits(a), bits(b)), f"replay {rep}"


def test_noalloc_with_a_long_table_replays_from_a_captured_graph():
    lengths = [900, 129, 0, 1, 2049] * 8 + MANY
    Hq, Hkv, d, T = 8, 2, 128, sum(lengths)
    cu = synth.cu_seqlens(lengths)
    q, k, v = synth.make_qkv(T, Hq, Hkv, d, 95, DEV)
    o, lse = torch.zeros_like(q), torch.zeros((Hq, T), dtype=torch.float32, device=DEV)
    B.varlen_attn_fwd_noalloc(q, k, v, cu, o, lse)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.varlen_attn_fwd_noalloc(q, k, v, cu, o, lse)
    for rep in range(3):
        for dst, src in zip((q, k, v), synth.make_qkv(T, Hq, Hkv, d, 960 + rep, DEV)):
            dst.copy_(src)
        wo, wl = B.varlen_attn_fwd(q, k, v, cu)
        o.zero_(); lse.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(bits(o), bits(wo)) and torch.equal(bits(lse), bits(wl)), f"replay {rep}"


def uploading_calls(lengths, Hq, Hkv, d, seed):
    """Inputs, outputs and a call (inputs, outputs) that uploads long tables: forward, chunk pairs and merge of a first
    sequence over 4000 tokens, backward, all with one workspace of their own."""
    T, cu = sum(lengths), synth.cu_seqlens(lengths)
    x = synth.make_qkv(T, Hq, Hkv, d, seed, DEV, with_dout=True)
    outs = [torch.zeros_like(x[0]), torch.zeros((Hq, T), dtype=torch.float32, device=DEV)] + [torch.zeros_like(t) for t in x[:3]]
    pairs, merges, rows = B.chunk_pairs(0, lengths[0], 4) if lengths[0] > 4000 else (None, None, 0)
    parts = (torch.empty((rows, Hq, d), dtype=torch.float32, device=DEV), torch.empty((Hq, rows), dtype=torch.float32, device=DEV))
    sh = B.make_shape(T, len(lengths), Hq, Hkv, d)
    ws = torch.empty(max(B.workspace_bytes(B.FN_FWD, sh, cu), B.workspace_bytes(B.FN_BWD, sh, cu), B.workspace_bytes(B.FN_PARTIAL, sh, None, 10),
                         B.workspace_bytes(B.FN_MERGE, sh, None, 4)), dtype=torch.uint8, device=DEV)
    skip = np.asarray([rows > 0] + [False] * (len(lengths) - 1), np.uint8)

    def call(x, outs):
        q, k, v, do = x
        o, lse, dq, dk, dv = outs
        B.varlen_attn_fwd(q, k, v, cu, o=o, lse=lse, seq_skip=skip, ws=ws)
        if rows:
            B.chunk_attn_partial(q, k, v, pairs, rows, o_part=parts[0], lse_part=parts[1], ws=ws)
            B.lse_merge(*parts, merges, o, lse, ws=ws)
        B.varlen_attn_bwd(do, q, k, v, o, lse, cu, dq=dq, dk=dk, dv=dv, ws=ws)
    return x, outs, call


def test_captures_need_no_staging_buffers():
    """Two graphs with more uploading calls each than the process has ever had under way at once, captured without a call
    before them on their stream: the tables of a captured call belong to its graph (there is nothing to allocate for them
    while the stream is capturing, and nothing to give back)."""
    Hq, Hkv, d = 8, 2, 128
    side = torch.cuda.Stream()
    graphs = []
    for seed, lengths in ((97, [130] * 64 + MANY), (98, [8192, 40, 1, 3000])):
        x, outs, call = uploading_calls(lengths, Hq, Hkv, d, seed)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            for _ in range(30):
                call(x, outs)
        graphs.append((graph, x, outs, call))
    for rep in range(3):
        for n, (graph, x, outs, call) in enumerate(graphs):
            for dst, src in zip(x, synth.make_qkv(x[0].shape[0], Hq, Hkv, d, 980 + 2 * rep + n, DEV, with_dout=True)):
                dst.copy_(src)
            want = [torch.zeros_like(t) for t in outs]
            call(x, want)
            for t in outs:
                t.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            for a, b in zip(outs, want):
                assert torch.equal(bits(a), bits(b)), (rep, n)


def test_a_graph_outlives_the_scratch_of_its_stream():
    """Calls captured without a workspace of the caller's, then a larger eager call on the capture stream (which replaces
    that stream's cached scratch) and new tensors: replays give the right results and write to nobody else's memory."""
    Hq, Hkv, d = 8, 2, 128
    side = torch.cuda.Stream()
    small, large = [130] * 64 + MANY, [700] * 64 + MANY

    def call(x, outs, cu):
        q, k, v, do = x
        o, lse, dq, dk, dv = outs
        B.varlen_attn_fwd(q, k, v, cu, o=o, lse=lse)
        B.varlen_attn_bwd(do, q, k, v, o, lse, cu, dq=dq, dk=dk, dv=dv)

    def buffers(lengths, seed):
        x = synth.make_qkv(sum(lengths), Hq, Hkv, d, seed, DEV, with_dout=True)
        return x, [torch.zeros_like(x[0]), torch.zeros((Hq, sum(lengths)), dtype=torch.float32, device=DEV)] + [torch.zeros_like(t) for t in x[:3]]

    x, outs = buffers(small, 99)
    bx, bouts = buffers(large, 100)
    graphs = []
    for _ in range(2):
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            call(x, outs, synth.cu_seqlens(small))
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            call(x, outs, synth.cu_seqlens(small))
        with torch.cuda.stream(side):
            call(bx, bouts, synth.cu_seqlens(large))
        torch.cuda.synchronize()
        graphs.append(graph)
    need = B.workspace_bytes(B.FN_BWD, B.make_shape(sum(small), len(small), Hq, Hkv, d), synth.cu_seqlens(small))
    others = [torch.full((n,), 0x5A, dtype=torch.uint8, device=DEV) for n in (4096, 4096, need, need, need)]
    for rep in range(3):
        for dst, src in zip(x, synth.make_qkv(sum(small), Hq, Hkv, d, 990 + rep, DEV, with_dout=True)):
            dst.copy_(src)
        want = [torch.zeros_like(t) for t in outs]
        call(x, want, synth.cu_seqlens(small))
        for graph in graphs:
            for t in outs:
                t.zero_()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            for a, b in zip(outs, want):
                assert torch.equal(bits(a), bits(b)), rep
    for t in others:
        assert bool((t == 0x5A).all())


def test_scratch_of_a_given_stream_is_allocated_for_it():
    """stream= other than the current one: the cached scratch belongs to that stream for the allocator too, so that one which
    is outgrown is handed out again only behind the calls that still use it."""
    side = torch.cuda.Stream()
    lengths = [130] * 64 + MANY
    q, k, v = synth.make_qkv(sum(lengths), 4, 2, 64, 111, DEV)
    want = B.varlen_attn_fwd(q, k, v, synth.cu_seqlens(lengths))
    side.wait_stream(torch.cuda.current_stream())
    got = B.varlen_attn_fwd(q, k, v, synth.cu_seqlens(lengths), stream=side)
    torch.cuda.synchronize()
    assert torch.equal(bits(got[0]), bits(want[0])) and torch.equal(bits(got[1]), bits(want[1]))
    at = B.workspace(1, q.device, "fwd", side).data_ptr()
    owner = [s["stream"] for s in torch.cuda.memory_snapshot() if s["address"] <= at < s["address"] + s["total_size"]]
    assert owner == [side.cuda_stream]
