"""The forward at head dimension 128 has two forms of its main kernel, by how a CU's share of the launch compares with the longest
item. A row's results are the same bits in both: edges of 16-row sub-blocks, 64-key tiles (one to seven of them, so that every
rotation of the three buffers ends somewhere) and 128-row blocks, references that move, chunk pairs that see no key, updates."""
import pytest
import torch

from paper_2509_21841_amd import binding as B
from paper_2509_21841_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
D, HQ, HKV = 128, 4, 2
EDGES = [1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 257, 320, 385, 448, 449, 1000]


def bits(t):
    return t.contiguous().view(torch.int16 if t.dtype == torch.bfloat16 else torch.int32)


def labelled(call, label):
    """The results of a call whose one launch has this profile label."""
    B.profile_enable(True)
    out = call()
    torch.cuda.synchronize()
    names = [name for name, _ in B.profile_records()]
    B.profile_enable(False)
    assert names == [label]
    return out


@pytest.mark.parametrize("steep", [False, True])
def test_both_forms_are_the_same_bits(steep):
    many, one = EDGES + [700] * 180, EDGES + [15000]
    n, T = sum(EDGES), max(sum(many), sum(one))
    q, k, v = synth.make_qkv(T, HQ, HKV, D, 151, DEV)
    if steep:   # scores that rise along the sequence: references move in later tiles
        k += (torch.arange(T, device=DEV) % 997 * 0.02)[:, None, None].to(torch.bfloat16)
        q += 0.5
    got = [labelled(lambda: B.varlen_attn_fwd(q[:sum(x)], k[:sum(x)], v[:sum(x)], synth.cu_seqlens(x), scale=0.13), label)
           for x, label in ((many, "attn_fwd_turns"), (one, "attn_fwd"))]
    assert torch.equal(bits(got[0][0][:n]), bits(got[1][0][:n])) and torch.equal(bits(got[0][1][:, :n]), bits(got[1][1][:, :n]))


def test_chunk_pairs_of_both_forms_are_the_same_bits():
    shapes = [(0, 0, 128, 128), (40, 70, 128, 130), (0, 100, 200, 90), (64, 1, 17, 127), (0, 127, 128, 1), (0, 128, 128, 64), (300, 0, 65, 299),
              (33, 0, 15, 512), (900, 0, 129, 449)]   # q_pos0, k_pos0, q_len, k_len
    pairs, row = [], 0
    for i, (qp, kp, ql, kl) in enumerate(shapes):
        pairs.append(dict(q_tok0=row, q_len=ql, k_tok0=2000 + 7 * i, k_len=kl, q_pos0=qp, k_pos0=kp, out_row0=row))
        row += ql
    whole = lambda at, n: dict(q_tok0=at, q_len=n, k_tok0=at, k_len=n, q_pos0=0, k_pos0=0, out_row0=at)
    many, one = [whole(3000 + 700 * i, 700) for i in range(180)], [whole(3000, 15000)]
    T = 3000 + 700 * 180
    q, k, v = synth.make_qkv(T, HQ, HKV, D, 153, DEV)
    forms = ((many, "attn_fwd_partial_turns"), (one, "attn_fwd_partial"))
    part = [labelled(lambda: B.chunk_attn_partial(q, k, v, pairs + x, T), label) for x, label in forms]
    assert torch.equal(bits(part[0][0][:row]), bits(part[1][0][:row])) and torch.equal(bits(part[0][1][:, :row]), bits(part[1][1][:, :row]))
    runs = []
    for x, label in forms:   # folded into rows that have seen keys already, and into rows that have not
        o_run, lse_run = torch.full((T, HQ, D), 7.0, device=DEV), torch.full((HQ, T), float("-inf"), device=DEV)
        B.chunk_attn_update(q, k, v, [dict(q_tok0=0, q_len=row // 2, k_tok0=100, k_len=77, q_pos0=500, k_pos0=0, out_row0=0)], o_run, lse_run)
        labelled(lambda: B.chunk_attn_update(q, k, v, pairs + x, o_run, lse_run), label)
        runs.append((o_run[:row], lse_run[:, :row]))
    assert torch.equal(bits(runs[0][0]), bits(runs[1][0])) and torch.equal(bits(runs[0][1]), bits(runs[1][1]))
