"""Scratch memory of the backward: a call that would share key blocks among workgroups needs room for their sums, and does without
sharing in a smaller workspace. The binding's cached scratch must therefore never decide: it asks for the size wherever there may be sums."""
import random

import pytest
import torch

from paper_2509_21841_amd import binding as B
from paper_2509_21841_amd import synth

DEV = "cuda:0"
HEADS = [(4, 1), (8, 2), (8, 8), (16, 1), (32, 1), (32, 8), (48, 1), (64, 1), (64, 2), (64, 8), (18, 6), (33, 11)]


def scratch(lengths, Hq, Hkv, d):
    return B.workspace_bytes(B.FN_BWD, B.make_shape(sum(lengths), len(lengths), Hq, Hkv, d), synth.cu_seqlens(lengths))


def without_sums(lengths, Hq):
    """A tile table, two values per row and head, and a few kilobytes of counters and padding."""
    return 64 * sum(-(-n // 128) for n in lengths) + 2 * 4 * Hq * sum(lengths) + 8192


def test_the_binding_asks_wherever_there_may_be_sums():
    """One sequence of 1900 tokens, 64/1 heads, is 15 blocks, whose units are padded to 16 before they count as 1024 work items."""
    rng = random.Random(3)
    batches = [([1900], 64, 1, 128), ([1900], 64, 2, 64), ([2500], 48, 1, 128), ([3900], 32, 1, 64)]
    for _ in range(2000):
        lengths = [int(20 * 300 ** rng.random()) for _ in range(rng.choice([1, 1, 2, 3, 8, 40]))]
        batches.append((lengths, *rng.choice(HEADS), rng.choice([64, 128])))
    some = 0
    for lengths, Hq, Hkv, d in batches:
        if scratch(lengths, Hq, Hkv, d) > without_sums(lengths, Hq):
            assert B._bwd_may_share(sum(lengths), len(lengths), Hq, Hkv), (lengths, Hq, Hkv, d)
            some += 1
    assert some > 100
    assert B._bwd_may_share(100, 1, 4, 0)   # (not this function's to refuse: the library does)


# Launches that are not shared (an even load, or a chain that other kernels go through faster) and launches that are
WHOLE = [([1, 0, 3000, 900, 2500, 120, 700, 780], 32, 8, 128), ([1000] * 28, 8, 1, 128), ([7400], 8, 2, 128), ([544] * 12, 16, 1, 128),
         ([2000, 7000, 6000, 1000] * 6, 8, 8, 64), ([1660] * 5, 32, 8, 64)]
# (also one sequence by itself, and equal ones)
SHARED = [([1000] * 17, 8, 1, 128), ([9000], 8, 2, 128), ([3000] * 3, 16, 2, 128), ([8000], 16, 2, 64), ([1900], 64, 2, 64), ([3001] + [1] * 40, 8, 2, 128), ([1900], 64, 1, 128), ([24001 - 11048, 11048], 8, 2, 128), ([3802, 900, 3100, 40, 2500, 3300], 16, 4, 64)]


def test_room_for_sums_only_where_there_are_any():
    for batch in WHOLE:
        assert without_sums(batch[0], batch[1]) - 8192 <= scratch(*batch) <= without_sums(batch[0], batch[1]), batch
    for lengths, Hq, Hkv, d in SHARED:   # (dK and dV of 128 keys each in float, of two shares and more)
        assert scratch(lengths, Hq, Hkv, d) > without_sums(lengths, Hq) + 2 * 2 * 128 * 4 * d * Hkv


def last_label(call):
    B.profile_enable(True)
    call()
    torch.cuda.synchronize()
    name = B.profile_records()[-1][0]
    B.profile_enable(False)
    return name


@pytest.mark.gpu
@pytest.mark.parametrize("batch", WHOLE + SHARED)
def test_exactly_the_stated_size_decides(batch):
    """Shares where the size has room for them and only there, in a workspace of that size as in a larger one."""
    lengths, Hq, Hkv, d = batch
    q, k, v, do = synth.make_qkv(sum(lengths), Hq, Hkv, d, 233, DEV, with_dout=True)
    cu = synth.cu_seqlens(lengths)
    o, lse = B.varlen_attn_fwd(q, k, v, cu)
    ws = torch.empty(scratch(*batch), dtype=torch.uint8, device=DEV)
    large = torch.empty(ws.numel() + (256 << 20), dtype=torch.uint8, device=DEV)
    shares = {w: last_label(lambda: B.varlen_attn_bwd(do, q, k, v, o, lse, cu, ws=w)) == "attn_bwd_dkdv_shares" for w in (ws, large)}
    assert set(shares.values()) == {batch in SHARED}


def forget_scratch():
    for key in [key for key in B._ws_cache if key[1] == "bwd"]:
        del B._ws_cache[key]


@pytest.mark.gpu
@pytest.mark.parametrize("rest,Hq,Hkv,d", [([3001] + [1] * 40, 8, 2, 128), ([3802, 900, 3100, 40, 2500, 3300], 16, 4, 64)])
def test_what_is_left_of_a_flagged_batch_is_shared(rest, Hq, Hkv, d):
    """Eight flagged sequences of 9000 tokens, with which the batch would not be shared: the others are, whatever scratch there is, and
    give the bits that they give by themselves."""
    lengths, skip = [9000] * 4 + rest + [9000] * 4, [1] * 4 + [0] * len(rest) + [1] * 4
    assert scratch(lengths, Hq, Hkv, d) <= without_sums(lengths, Hq)
    own = slice(36000, 36000 + sum(rest))
    q, k, v, do = synth.make_qkv(sum(lengths), Hq, Hkv, d, 235, DEV, with_dout=True)
    cut = [x[own] for x in (do, q, k, v)]
    o, lse = torch.zeros_like(q), torch.zeros((Hq, len(q)), device=DEV)
    o[own], lse[:, own] = B.varlen_attn_fwd(*cut[1:], synth.cu_seqlens(rest))
    want = B.varlen_attn_bwd(*cut, o[own], lse[:, own].contiguous(), synth.cu_seqlens(rest))
    for room in (4096, 8 << 20, 512 << 20):
        forget_scratch()
        B.workspace(room, torch.device(DEV), "bwd")
        got = []
        call = lambda: got.append(B.varlen_attn_bwd(do, q, k, v, o, lse, synth.cu_seqlens(lengths), seq_skip=skip))
        assert last_label(call) == "attn_bwd_dkdv_shares"
        for x, y in zip(got[0], want):
            assert torch.equal(x[own].view(torch.int16), y.view(torch.int16))
    forget_scratch()


@pytest.mark.gpu
@pytest.mark.parametrize("length,Hq,Hkv,d", [(1900, 64, 1, 128), (2500, 48, 1, 128), (1900, 64, 2, 64)])
def test_the_same_bits_after_a_smaller_call(length, Hq, Hkv, d):
    def backward(n):
        q, k, v, do = synth.make_qkv(n, Hq, Hkv, d, 231, DEV, with_dout=True)
        cu = synth.cu_seqlens([n])
        o, lse = B.varlen_attn_fwd(q, k, v, cu)
        return B.varlen_attn_bwd(do, q, k, v, o, lse, cu)

    forget_scratch()
    B.workspace(2 << 20, torch.device(DEV), "bwd")   # room for everything but sums
    backward(300)
    after = backward(length)
    forget_scratch()
    for a, b in zip(after, backward(length)):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
