"""Backwards of a few workgroups do dQ and dK/dV in one launch, behind a small one for the row terms. In front of enough other sequences
the same ones take launches of their own, and the results are the same bits: edges of 16-row sub-blocks, 32-row key blocks and 64-row
tiles, one to eight heads per KV head, empty sequences, strided inputs, written and accumulated, more workgroups than CUs."""
import pytest
import torch

from paper_2509_21841_amd import binding as B
from paper_2509_21841_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# and how many sequences of how many tokens are the others. The last one: 34 tiles of 64 rows x 8 heads and 66 key parts x 2 heads, more than
# 256 workgroups behind a chain of 33 key tiles
BATCHES = [([33, 1], 1, 1, 49, 110), ([15, 16, 17, 0, 31, 32, 33], 2, 1, 25, 180), ([63, 64, 65], 3, 3, 10, 230), ([127, 128, 129, 1], 4, 2, 15, 250),
           ([255, 257], 8, 1, 14, 330), ([700], 6, 3, 16, 260), ([2063, 14], 8, 2, 16, 230)]


def bits(t):
    return t.contiguous().view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32)


def check(call):
    """call(alone) -> the results for the batch's rows."""
    plain = call(True)
    B.profile_enable(True)
    alone = call(True)
    torch.cuda.synchronize()
    names = [name for name, _ in B.profile_records()]
    B.profile_enable(True)
    apart = call(False)
    torch.cuda.synchronize()
    others = [name for name, _ in B.profile_records()]
    B.profile_enable(False)
    assert names == ["attn_bwd_both"]
    assert others[0].startswith("attn_bwd_dq") and others[1:] == ["attn_bwd_dkdv_split"]
    for a, b, c in zip(plain, alone, apart):
        assert torch.equal(bits(a), bits(b)) and torch.equal(bits(a), bits(c))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lengths,Hq,Hkv,n,each", BATCHES)
def test_one_launch_is_the_same_bits(lengths, Hq, Hkv, n, each, d):
    rows, T = sum(lengths), sum(lengths) + n * each
    qkv = torch.cat(synth.make_qkv(T, Hq, Hkv, d, 161, DEV), 1)
    do = synth.make_qkv(T, Hq, Hkv, d, 163, DEV)[0]
    q, k, v = qkv[:, :Hq], qkv[:, Hq:Hq + Hkv], qkv[:, Hq + Hkv:]
    o, lse = B.varlen_attn_fwd(q, k, v, synth.cu_seqlens(lengths + [each] * n), scale=0.13)

    def written(alone):
        cut, own = (slice(rows), lengths) if alone else (slice(T), lengths + [each] * n)
        grads = B.varlen_attn_bwd(do[cut], q[cut], k[cut], v[cut], o[cut], lse[:, cut].contiguous(), synth.cu_seqlens(own), scale=0.13)
        return [x[:rows] for x in grads]

    check(written)
    q, k, v = q.contiguous(), k.contiguous(), v.contiguous()

    def accumulated(alone):
        own = lengths if alone else lengths + [each] * n
        cu = synth.cu_seqlens(own)
        pairs = [dict(q_tok0=int(cu[i]), q_len=x, k_tok0=int(cu[i]), k_len=x, q_pos0=0, k_pos0=0, out_row0=0) for i, x in enumerate(own) if x]
        acc = [torch.ones((T, h, d), dtype=torch.float32, device=DEV) for h in (Hq, Hkv, Hkv)]
        B.chunk_attn_partial_bwd(do, q, k, v, o, lse, pairs, *acc, scale=0.13)
        return [x[:rows] for x in acc]

    check(accumulated)


def test_one_launch_in_a_graph():
    """The row terms are written anew by every replay."""
    lengths, Hq, Hkv, d = [329, 64, 1, 100], 4, 2, 128
    q, k, v, do = synth.make_qkv(sum(lengths), Hq, Hkv, d, 165, DEV, with_dout=True)
    cu = synth.cu_seqlens(lengths)
    o, lse = B.varlen_attn_fwd(q, k, v, cu)
    grads = [torch.empty_like(x) for x in (q, k, v)]
    call = lambda: B.varlen_attn_bwd(do, q, k, v, o, lse, cu, dq=grads[0], dk=grads[1], dv=grads[2])
    call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call()
    for seed in (167, 169, 171):
        do.copy_(synth.make_qkv(sum(lengths), Hq, Hkv, d, seed, DEV)[0])
        graph.replay()
        torch.cuda.synchronize()
        got = [x.clone() for x in grads]
        call()
        torch.cuda.synchronize()
        for a, b in zip(got, grads):
            assert torch.equal(bits(a), bits(b))
