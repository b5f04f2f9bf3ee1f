"""The forward's running softmax reference: probabilities are taken against the reference a row already has, which moves
only when their sum grows out of range. Rows whose scores rise by large steps from tile to tile, fall, or start after
tiles they see nothing of, against the fp64 oracle; d = 64 and 128, whole sequences, chunk pairs and running updates."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_21841_amd import binding as B
from paper_2509_21841_amd import synth
from util import assert_close, assert_lse_close, widen

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def inputs(L, Hq, Hkv, d, seed, profile):
    """q along one direction per head and keys whose component along it follows `profile` over the positions, so that
    the scores (natural units, before the softmax) are about the profile's values."""
    q, k, v = synth.make_qkv(L, Hq, Hkv, d, seed, DEV)
    u = torch.ones(d, device=DEV) / d ** 0.5
    p = torch.as_tensor(profile(np.arange(L)), dtype=torch.float32, device=DEV)
    q = (0.05 * q.float() + 2.0 * u).to(torch.bfloat16)
    k = (0.05 * k.float() + (p[:, None, None] * d ** 0.5 / 2.0) * u).to(torch.bfloat16)
    return q, k, v


PROFILES = {
    "rising": lambda i: 0.3 * i,                                    # the reference moves in every tile, by 19 per tile
    "steps": lambda i: 40.0 * (i // 32 % 3) - 60.0,                 # up and down by 40 within and between tiles
    "falling": lambda i: -0.3 * i,
    "one-peak": lambda i: np.where(i == 70, 80.0, -80.0),
    # a lane's 16 probabilities of every tile behind the first near the sum that moves the reference (16 e^5.545 = 4096):
    # the row's own level is 2.5 % of the score wide, so that all rows stay under it, or all pass it
    "just-under": lambda i: np.where(i < 64, 0.0, 5.0),
    "just-over": lambda i: np.where(i < 64, 0.0, 6.2),
}


def second_tile_sums(q, k):
    """[Hq, rows from 128 on, 4]: sums of a row's four lanes over their keys of the second tile (keys 4 l .. 4 l + 3 of every
    16), against the row's maximum over the first tile."""
    L, Hq, d = q.shape
    grp = Hq // k.shape[1]
    qq, kk = widen(q)[128:], widen(k)[:128]
    s = np.stack([qq[:, h] @ kk[:, h // grp].T for h in range(Hq)]) * d ** -0.5
    p = np.exp(s[:, :, 64:] - s[:, :, :64].max(-1, keepdims=True))
    return p.reshape(Hq, L - 128, 4, 4, 4).sum((2, 4))


@pytest.mark.parametrize("d", [64, 128])
def test_profiles_around_the_limit(d):
    for profile, inside in (("just-under", True), ("just-over", False)):
        q, k, _ = inputs(333, 4, 2, d, 71, PROFILES[profile])
        sums = second_tile_sums(q, k)
        assert (sums < 4050).all() and sums.max() > 3000 if inside else (sums > 4150).all() and sums.min() < 5500


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("profile", list(PROFILES))
def test_scores_that_move_the_reference(profile, d):
    L, Hq, Hkv = 333, 4, 2
    q, k, v = inputs(L, Hq, Hkv, d, 71, PROFILES[profile])
    cu = synth.cu_seqlens([L])
    ro, rl = oracle.varlen_attn_fwd(widen(q), widen(k), widen(v), cu)
    o, lse = B.varlen_attn_fwd(q, k, v, cu)
    assert_close("O", widen(o), ro)
    # the stated 1e-3 is for LSE of order 10; a float carries 2^-24 of the scores it is made of, which here reach 100
    assert np.abs(widen(lse) - rl).max() <= 1e-3 + 2.0 ** -21 * np.abs(rl).max()
    # chunk pairs: a query row of a later tile may have no reference yet when a wave's other rows have one
    pairs, merges, rows = B.chunk_pairs(0, L, 3)
    op, lp = B.chunk_attn_partial(q, k, v, pairs, rows)
    opairs, _, orows = oracle.causal_pairs(0, L, 3)
    rop, rlp = oracle.chunk_attn_partial(widen(q), widen(k), widen(v), opairs, orows)
    assert_close("O_part", widen(op), rop, bf16_out=False)
    assert np.array_equal(np.isneginf(widen(lp)), np.isneginf(rlp))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("q_pos0,k_pos0,q_len,k_len", [(0, 0, 128, 128), (40, 70, 128, 130), (0, 100, 200, 90), (64, 1, 17, 127),
                                                       (5, 64, 113, 65), (0, 127, 128, 1), (0, 128, 128, 64)])
def test_partials_on_every_side_of_the_diagonal(q_pos0, k_pos0, q_len, k_len, d):
    """Chunk pairs whose diagonal crosses the two 16-row sub-blocks of a wave at every place: rows that see nothing, rows
    that first see a key in their second tile, blocks shorter than a sub-block."""
    T, Hq, Hkv = 512, 2, 1
    q, k, v = synth.make_qkv(T, Hq, Hkv, d, 73, DEV)
    pair = dict(q_tok0=3, q_len=q_len, k_tok0=250, k_len=k_len, q_pos0=q_pos0, k_pos0=k_pos0, out_row0=0)
    op, lp = B.chunk_attn_partial(q, k, v, [pair], q_len)
    rop, rlp = oracle.chunk_attn_partial(widen(q), widen(k), widen(v), [pair], q_len)
    assert_close("O_part", widen(op), rop, bf16_out=False)
    assert_lse_close("LSE_part", widen(lp), rlp)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("c", [1, 72, 200, 300])
def test_rows_do_not_depend_on_later_tokens(c, d):
    """O and LSE of the first c tokens are the same bits whatever follows them: the rows behind, which share a wave with
    them, get queries and keys that move their own reference in every tile."""
    L, Hq, Hkv = 333, 4, 2
    q, k, v = synth.make_qkv(L, Hq, Hkv, d, 77, DEV)
    cu = synth.cu_seqlens([L])
    want = B.varlen_attn_fwd(q, k, v, cu)
    for scale in (0.0, 8.0, 64.0):
        q2, k2, v2 = (x.clone() for x in (q, k, v))
        for x in (q2, k2, v2):
            x[c:] *= scale
        got = B.varlen_attn_fwd(q2, k2, v2, cu)
        assert torch.equal(got[0][:c].view(torch.int16), want[0][:c].view(torch.int16)), scale
        assert torch.equal(got[1][:, :c].contiguous().view(torch.int32), want[1][:, :c].contiguous().view(torch.int32)), scale
