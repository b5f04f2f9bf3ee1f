"""Backwards of a few workgroups do dQ and dK/dV in one launch, behind a small one for the row terms; while the profile is on they are
launches of their own. The results are the same bits either way: edges of 16-row sub-blocks, 32-row key blocks and 64-row tiles,
one to eight heads per KV head, empty sequences, strided inputs, written and accumulated, more workgroups than CUs."""
import pytest
import torch

from paper_2509_21841_amd import binding as B
from paper_2509_21841_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# the last one: 34 tiles of 64 rows x 8 heads and 66 key parts x 2 heads, more than 256 workgroups behind a chain of 33 key tiles
BATCHES = [([33, 1], 1, 1), ([15, 16, 17, 0, 31, 32, 33], 2, 1), ([63, 64, 65], 3, 3), ([127, 128, 129, 1], 4, 2), ([255, 257], 8, 1), ([700], 6, 3),
           ([2063, 14], 8, 2)]


def bits(t):
    return t.contiguous().view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32)


def twice(call):
    """The results without and with the profile, and its labels."""
    plain = [x.clone() for x in call()]
    B.profile_enable(True)
    out = call()
    torch.cuda.synchronize()
    names = [name for name, _ in B.profile_records()]
    B.profile_enable(False)
    return plain, out, names


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lengths,Hq,Hkv", BATCHES)
def test_one_launch_is_the_same_bits(lengths, Hq, Hkv, d):
    T = sum(lengths)
    qkv = torch.cat(synth.make_qkv(T, Hq, Hkv, d, 161, DEV), 1)
    do = synth.make_qkv(T, Hq, Hkv, d, 163, DEV)[0]
    q, k, v = qkv[:, :Hq], qkv[:, Hq:Hq + Hkv], qkv[:, Hq + Hkv:]
    cu = synth.cu_seqlens(lengths)
    o, lse = B.varlen_attn_fwd(q, k, v, cu, scale=0.13)
    plain, apart, names = twice(lambda: B.varlen_attn_bwd(do, q, k, v, o, lse, cu, scale=0.13))
    assert names == ["attn_bwd_dq_pair", "attn_bwd_dkdv_split"]
    for a, b in zip(plain, apart):
        assert torch.equal(bits(a), bits(b))
    pairs = [dict(q_tok0=int(cu[i]), q_len=n, k_tok0=int(cu[i]), k_len=n, q_pos0=0, k_pos0=0, out_row0=0) for i, n in enumerate(lengths) if n]

    def accumulate():
        acc = [torch.ones((T, h, d), dtype=torch.float32, device=DEV) for h in (Hq, Hkv, Hkv)]
        B.chunk_attn_partial_bwd(do, q.contiguous(), k.contiguous(), v.contiguous(), o, lse, pairs, *acc, scale=0.13)
        return acc

    plain, apart, names = twice(accumulate)
    assert names == ["attn_bwd_dq_pair", "attn_bwd_dkdv_split"]
    for a, b in zip(plain, apart):
        assert torch.equal(bits(a), bits(b))


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
