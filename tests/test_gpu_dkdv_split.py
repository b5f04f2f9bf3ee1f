"""dK/dV of launches that leave most of the chip idle (four groups of two waves share a 32-row key block's query tiles by
turns): block and tile edges, fewer iterations than waves, one to eight heads per KV head, both head dimensions, written
and accumulated, against the fp64 oracle, and the launches around which the other two kernels take over."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_21841_amd import binding as B
from paper_2509_21841_amd import synth
from util import Checks, assert_close, kernels_of, widen

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
# The first keys of a sequence have a handful of terms dS_ij q_i, the largest about 8, whose bf16 operand carries 2^-9 of it
# (1.6e-2): two of them and the output's half-spacing (7.8e-3 below 4) make 4e-2. The relative-L2 bound is the stated one;
# batches of sequences under 200 tokens have little to average over and get three times that (a wrong mask or index is of
# order one in both).
MAXABS, RELL2 = 4e-2, 5e-3


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lengths,Hq,Hkv", [([1], 1, 1), ([15, 16, 17, 31, 32, 33], 2, 1), ([127, 128, 129], 3, 1), ([65, 1, 0, 300], 8, 1),
                                            ([500], 4, 4), ([97, 161], 4, 2), ([1100], 5, 1)])
def test_small_batches(lengths, Hq, Hkv, d):
    T = sum(lengths)
    q, k, v, do = synth.make_qkv(T, Hq, Hkv, d, 101, DEV, with_dout=True)
    cu = synth.cu_seqlens(lengths)
    o, lse = B.varlen_attn_fwd(q, k, v, cu)
    got = B.varlen_attn_bwd(do, q, k, v, o, lse, cu)
    ref = oracle.varlen_attn_bwd(widen(do), widen(q), widen(k), widen(v), cu)
    checks = Checks()
    for name, a, b in zip(("dQ", "dK", "dV"), got, ref):
        checks.close(name, widen(a), b, maxabs=MAXABS, rell2=RELL2 if min(lengths) >= 200 else 3 * RELL2)
    checks.finish()
    again = B.varlen_attn_bwd(do, q, k, v, o, lse, cu)
    for a, b in zip(got, again):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    # accumulated in float, one pair per sequence: the written results are these, rounded once
    acc = [torch.zeros(x.shape, dtype=torch.float32, device=DEV) for x in (q, k, v)]
    pairs = [dict(q_tok0=int(cu[i]), q_len=n, k_tok0=int(cu[i]), k_len=n, q_pos0=0, k_pos0=0, out_row0=0) for i, n in enumerate(lengths) if n]
    B.chunk_attn_partial_bwd(do, q, k, v, o, lse, pairs, *acc)
    for a, b in zip(acc, got):
        assert torch.equal(a.to(torch.bfloat16).view(torch.int16), b.view(torch.int16))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("n", [1, 8, 24, 40, 48, 64, 96])
def test_both_sides_of_the_rule(n, d):
    """n sequences of 300 tokens under 2 KV heads: the first and the last one's gradients do not depend on which kernel the
    batch takes beyond the order of the float sums."""
    L, Hq, Hkv = 300, 4, 2
    q, k, v, do = synth.make_qkv(L * n, Hq, Hkv, d, 103, DEV, with_dout=True)
    cu = synth.cu_seqlens([L] * n)
    o, lse = B.varlen_attn_fwd(q, k, v, cu)
    got = B.varlen_attn_bwd(do, q, k, v, o, lse, cu)
    for sl in [slice(0, L)] + [slice(L * n - L, L * n)] * (n > 1):
        ref = oracle.varlen_attn_bwd(widen(do[sl]), widen(q[sl]), widen(k[sl]), widen(v[sl]), synth.cu_seqlens([L]))
        for name, a, b in zip(("dQ", "dK", "dV"), got, ref):
            assert_close(name, widen(a[sl]), b, maxabs=MAXABS, rell2=RELL2)
    if n <= 8 or n >= 40:
        assert (dkdv_labels(do, q, k, v, o, lse, cu) == {"attn_bwd_dkdv_split"}) == (n <= 8)


def dkdv_labels(*call):
    B.profile_enable(True)
    B.varlen_attn_bwd(*call)
    torch.cuda.synchronize()
    labels = {name for name in kernels_of(B.profile_records()) if name.startswith("attn_bwd_dkdv")}
    B.profile_enable(False)
    return labels


# Which of the kernels ("": one workgroup per key block) is the fastest was measured for each of these launches; the next
# one is 5 to 170 % behind, but for 32 sequences of 100 tokens (2 %). n sequences of L tokens. (Backward of the two that are
# shared: 295 us by two groups and 213, 425 split and 339.)
@pytest.mark.parametrize("d,Hq,Hkv,L,n,kernel", [
    (128, 4, 4, 300, 3, "_split"), (128, 4, 4, 300, 10, "_pair"), (128, 4, 4, 300, 19, "_pair"), (128, 4, 4, 300, 24, ""),
    (128, 4, 4, 1000, 7, "_pair"), (128, 8, 1, 1000, 6, "_split"), (128, 8, 1, 1000, 17, "_shares"), (128, 8, 1, 1000, 28, "_pair"),
    (128, 8, 1, 4000, 2, "_shares"), (128, 32, 8, 300, 10, "_pair"), (128, 32, 8, 1000, 2, "_split"), (128, 32, 8, 1000, 9, "_pair"),
    (128, 4, 4, 100, 32, ""), (128, 32, 32, 3037, 1, ""), (128, 16, 4, 885, 16, ""), (128, 32, 8, 1360, 6, "_pair"),
    (128, 16, 4, 2628, 10, "_pair"), (128, 16, 4, 2699, 5, "_pair"), (128, 64, 8, 1411, 6, ""), (128, 8, 8, 983, 15, ""),
    (64, 4, 4, 300, 3, "_split"), (64, 4, 4, 300, 16, ""), (64, 16, 4, 300, 10, "_split"), (64, 16, 4, 300, 19, "_split"),
    (64, 8, 1, 1000, 6, "_split"), (64, 4, 2, 100, 13, "_split"), (64, 4, 2, 300, 38, ""), (64, 32, 32, 40, 4, ""),
    (64, 16, 16, 39, 8, ""), (64, 16, 16, 1030, 8, "")])
def test_the_fastest_kernel_is_taken(d, Hq, Hkv, L, n, kernel):
    check_kernel(d, Hq, Hkv, [L] * n, kernel)


# Ragged sequences of up to 100 tokens leave many workgroups of the split without keys, and at d = 128 it is the fastest by far:
# 24.2 us one workgroup per key block, 19.8 two groups, 11.5 split; 33.0, 25.2 and 14.7. The third: 34.6 and 40.8 split.
@pytest.mark.parametrize("d,Hq,Hkv,lengths,kernel", [
    (128, 16, 4, [100, 97, 93, 90, 88, 61, 55, 50, 47, 45, 40, 33, 30, 28, 21, 20, 12, 9], "_split"),
    (128, 64, 8, [87, 80, 75, 60, 52, 33, 21, 15, 10, 4], "_split"),
    (64, 64, 8, [20 + i * 37 % 81 for i in range(56)], "")])
def test_short_ragged_sequences(d, Hq, Hkv, lengths, kernel):
    check_kernel(d, Hq, Hkv, lengths, kernel)


def check_kernel(d, Hq, Hkv, lengths, kernel):
    q, k, v, do = synth.make_qkv(sum(lengths), Hq, Hkv, d, 107, DEV, with_dout=True)
    cu = synth.cu_seqlens(lengths)
    o, lse = B.varlen_attn_fwd(q, k, v, cu)
    assert dkdv_labels(do, q, k, v, o, lse, cu) == {"attn_bwd_dkdv" + kernel}
