"""dK/dV of launches whose longest chain of iterations is long beside what a CU has to do: the blocks of long sequences are cut into shares,
a workgroup each, and the last one to end adds up their sums. One long sequence among many short ones (whose tile table does not
fit the launch arguments): block and tile edges, four to eight heads per KV head, skipped sequences, strided inputs, against the fp64
oracle; the same bits on every call, whatever the workspace held."""
import pytest
import torch

import oracle
from paper_2509_21841_amd import binding as B
from paper_2509_21841_amd import synth
from test_gpu_dkdv_split import MAXABS, RELL2
from util import Checks, widen

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def profiled(call):
    B.profile_enable(True)
    out = call()
    torch.cuda.synchronize()
    names = [name for name, _ in B.profile_records()]
    B.profile_enable(False)
    return out, names


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("long,Hq,Hkv", [(2944, 4, 1), (3001, 8, 1), (4097, 6, 1), (2049, 8, 2)])
def test_long_sequence_among_short_ones(long, Hq, Hkv, d):
    lengths = [1] * 20 + [long] + [17, 0, 33] * 15 + [1] * 20
    T, at = sum(lengths), 20
    qkv = torch.cat(synth.make_qkv(T, Hq, Hkv, d, 181, DEV), 1)
    do = synth.make_qkv(T, Hq, Hkv, d, 183, DEV)[0]
    q, k, v = qkv[:, :Hq], qkv[:, Hq:Hq + Hkv], qkv[:, Hq + Hkv:]
    cu = synth.cu_seqlens(lengths)
    o, lse = B.varlen_attn_fwd(q, k, v, cu)
    ws = torch.full((B.workspace_bytes(B.FN_BWD, B.make_shape(T, len(lengths), Hq, Hkv, d), cu),), 255, dtype=torch.uint8, device=DEV)
    call = lambda **kw: B.varlen_attn_bwd(do, q, k, v, o, lse, cu, ws=ws, **kw)
    got, names = profiled(call)
    assert names[-1] == "attn_bwd_dkdv_shares"
    c = lambda x: widen(x.contiguous())
    ref = oracle.varlen_attn_bwd(c(do), c(q), c(k), c(v), cu)
    # the short sequences have little to average over: the bound of test_gpu_dkdv_split.py
    checks = Checks()
    one = slice(at, at + long)
    for name, a, b in zip(("dQ", "dK", "dV"), got, ref):
        checks.close(name, widen(a), b, maxabs=MAXABS, rell2=3 * RELL2)
        checks.close(name + " long", widen(a[one]), b[one], maxabs=MAXABS, rell2=RELL2)
    checks.finish()
    for fill in (0, 127):
        ws.fill_(fill)
        for a, b in zip(got, call()):
            assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    # a workspace without room for sums does as well
    small = ws[:4096 + 64 * sum(-(-n // 128) for n in lengths) + 2 * (4 * Hq * T + 256)]
    other, names = profiled(lambda: B.varlen_attn_bwd(do, q, k, v, o, lse, cu, ws=small))
    assert names[-1] != "attn_bwd_dkdv_shares"
    for a, b in zip(other, got):
        assert float((a[one].float() - b[one].float()).norm() / b[one].float().norm()) < 2 ** -8
    # flagged: the long sequence's rows stay as they are, in the same workspace; the others only: their gradients do not change
    skip = torch.zeros(len(lengths), dtype=torch.uint8).numpy()
    skip[at] = 1
    kept = [torch.full_like(x, 3.0) for x in got]
    call(seq_skip=skip, dq=kept[0], dk=kept[1], dv=kept[2])
    for a in kept:
        assert bool((a[one] == 3.0).all())
    skip = 1 - skip
    kept = [torch.full_like(x, 3.0) for x in got]
    call(seq_skip=skip, dq=kept[0], dk=kept[1], dv=kept[2])
    for a, b in zip(kept, got):
        assert bool((a[:at] == 3.0).all()) and bool((a[at + long:] == 3.0).all())
        # (by itself it may take another kernel: the order of the float sums, bf16 outputs)
        assert float((a[one].float() - b[one].float()).norm() / b[one].float().norm()) < 2 ** -8


def test_shares_in_a_graph():
    """Every replay counts the shares that are done from zero."""
    lengths, Hq, Hkv, d = [3001] + [1] * 40, 8, 2, 128
    q, k, v, do = synth.make_qkv(sum(lengths), Hq, Hkv, d, 185, DEV, with_dout=True)
    cu = synth.cu_seqlens(lengths)
    o, lse = B.varlen_attn_fwd(q, k, v, cu)
    grads = [torch.empty_like(x) for x in (q, k, v)]
    call = lambda: B.varlen_attn_bwd(do, q, k, v, o, lse, cu, dq=grads[0], dk=grads[1], dv=grads[2])
    assert profiled(call)[1][-1] == "attn_bwd_dkdv_shares"
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for seed in (187, 189, 191):
        do.copy_(synth.make_qkv(sum(lengths), Hq, Hkv, d, seed, DEV)[0])
        graph.replay()
        torch.cuda.synchronize()
        got = [x.clone() for x in grads]
        call()
        torch.cuda.synchronize()
        for a, b in zip(got, grads):
            assert torch.equal(a.view(torch.int16), b.view(torch.int16))
