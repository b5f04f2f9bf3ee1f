"""Every attention kernel's profile label is one that bench.py credits, whichever kernel a launch takes."""
import os
import re
from types import SimpleNamespace

import bench

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
KERNELS = {"attn_fwd": 2 * 300, "attn_fwd_partial": 2 * 700, "attn_bwd_dq": 3 * 1000, "attn_bwd_dkdv": 4 * 1000,
           "attn_bwd_both": 7 * 1000}   # products x pairs


def source_labels():
    labels = set()
    for name in ("attn_fwd.hip", "attn_bwd.hip"):
        text = open(os.path.join(ROOT, "paper_2509_21841_amd", "csrc", name)).read()
        for call in re.findall(r"zp_prof_begin\((.*)\);", text):
            labels |= set(re.findall(r'"(attn_\w+)"', call))
    return labels


def test_every_attention_label_is_credited():
    labels = source_labels()
    assert {"attn_fwd", "attn_fwd_turns", "attn_fwd_partial_turns", "attn_fwd_pair", "attn_bwd_dq_pair", "attn_bwd_dkdv_split", "attn_bwd_dkdv_pair",
            "attn_bwd_both"} <= labels
    job = SimpleNamespace(w=dict(d=64, Hq=2), pairs_total=1000, pairs_long=700)
    for label in labels:
        kernel = bench.kernel_of(label)
        assert label.startswith(kernel) and bench.kernel_flops(job, kernel) == 2 * 64 * 2 * KERNELS[kernel], label


def test_times_of_all_kernels_count():
    """A step whose launches take the kernels for part of the chip: their times are in the table and in the rates."""
    recs = [("attn_fwd_pair", 1.0), ("attn_fwd_partial_pair", 2.0), ("attn_bwd_dq_pair", 3.0), ("attn_bwd_dkdv_pair", 4.0),
            ("attn_bwd_dkdv_split", 5.0), ("remap", 6.0)]
    kern = bench.kernel_table(recs, 1)
    assert set(kern) == {"attn_fwd", "attn_fwd_partial", "attn_bwd_dq", "attn_bwd_dkdv", "remap"}
    assert kern["attn_bwd_dkdv"]["ms_per_step"] == 9.0 and kern["attn_bwd_dkdv"]["launches_per_step"] == 2
    fwd, bwd = bench.fwd_bwd_rates(SimpleNamespace(flops_fwd=3e9, flops_bwd=12e9), kern)
    assert abs(fwd - 1.0) < 1e-9 and abs(bwd - 1.0) < 1e-9
