"""The calls a user of the engine makes, for timing and for comparing two versions of the code: packed-batch attention
forward and backward, the forward that allocates nothing, long sequences as chunk pairs with a merge, one whole node's
placement (ring rounds and both remaps) and the token remap by itself. Sizes, head counts and length mixes are those of
bench.py, the tests and the smoke check; `draw` covers the range between them.

A case is a dict of plain values:
  op     fwd | noalloc | bwd | train (forward and backward) | chunked (sequences of 16K and more as C chunks + merge)
         | node (partitioner's placement on P devices: remaps, local sequences, ring rounds, forward and backward)
         | remap (row gather / scatter)
  mix    how the T tokens are cut into sequences (`_lengths`), lseed seeds it
  Hq, Hkv, d, scale (0: 1/sqrt(d)), fused (q, k, v are slices of one [T, Hq + 2 Hkv, d] buffer)
"""
import numpy as np
import torch

from paper_2509_21841_amd import binding as B
from paper_2509_21841_amd import node, synth

DEV = "cuda:0"
LONG = 16384   # tokens from which a chunked call cuts a sequence


def _case(name=None, **kw):
    c = dict(op="fwd", mix="lognormal", T=4096, lseed=1, Hq=32, Hkv=8, d=128, scale=0.0, fused=False, C=4, P=8, mode=0)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest batches: a unit-test sized model, where the call itself is most of the time
        _case("fwd-tiny-mha4-d64", op="fwd", mix="tiny", T=2048, lseed=1001, Hq=4, Hkv=4, d=64),
        _case("train-tiny-gqa4x2", op="train", mix="tiny", T=2048, lseed=1001, Hq=4, Hkv=2),
        # a serving loop's forward: few short requests, no allocation and no upload in the call
        _case("noalloc-8k-gqa32x8", op="noalloc", mix="ragged", T=8000, lseed=7),
        # training on short documents, multi-head attention
        _case("fwd-lognormal-64k-mha32", op="fwd", mix="lognormal", T=65536, lseed=1002, Hkv=32),
        _case("bwd-lognormal-64k-mha32", op="bwd", mix="lognormal", T=65536, lseed=1002, Hkv=32),
        # a smaller model: head dimension 64, lengths of every remainder, q/k/v straight from a fused projection
        _case("train-ragged-24k-gqa16x4-d64", op="train", mix="ragged", T=24001, lseed=11, Hq=16, Hkv=4, d=64, scale=0.11, fused=True),
        # the long-tailed batch of the benchmark: one long document among short ones
        _case("chunked-longtail-128k-gqa32x8", op="chunked", mix="longtail", T=131072, lseed=1003),
        _case("bwd-longtail-128k-gqa32x8", op="bwd", mix="longtail", T=131072, lseed=1003),
        # the widest batch: 256K tokens of short documents, 64 query heads
        _case("fwd-lognormal-256k-gqa64x8", op="fwd", mix="lognormal", T=262144, lseed=1005, Hq=64),
        # a node of 8 devices on one GPU: remap in, local sequences and ring rounds both ways, remap out
        _case("node-p8-longtail-32k", op="node", mix="longtail", T=32768, lseed=1003),
        # the remapping layer by itself: Q rows of the large batch, K rows of a small one on the way back
        _case("remap-128k-q32", op="remap", mix="lognormal", T=131072, lseed=1005, Hq=32, mode=0),
        _case("remap-4k-kv8", op="remap", mix="ragged", T=4099, lseed=13, Hq=8, mode=1),
    ]


def draw(rng):
    op = rng.choice(["fwd", "noalloc", "bwd", "train", "chunked", "node", "remap"])
    Hq, Hkv = rng.choice([(4, 4), (4, 2), (8, 2), (8, 8), (16, 4), (32, 8), (32, 32), (64, 8)])
    lo, hi = {"chunked": (32768, 131072), "node": (32768, 65536), "remap": (1024, 262144)}.get(op, (512, 131072))
    T = int(lo * (hi / lo) ** rng.random())
    if rng.random() < 0.7:
        T = T | 1
    mixes = ["ragged", "lognormal"]
    if T >= 32768:
        mixes += ["longtail", "table2:arxiv", "table2:github", "table2:prolong64k"]
    mix = "longtail" if op == "node" else rng.choice(mixes[2:] if op == "chunked" else mixes)
    fused = op in ("fwd", "bwd", "train", "noalloc") and rng.random() < 0.4
    c = _case(op=op, mix=mix, T=T, lseed=rng.randrange(1, 10000), Hq=Hq, Hkv=Hkv, d=rng.choice([64, 128, 128]),
              scale=rng.choice([0.0, 0.0, 0.11]) if op != "remap" else 0.0, fused=fused, C=rng.choice([2, 4, 8]),
              P=rng.choice([4, 8]), mode=rng.randrange(2))
    if op == "node" and Hq > 32:
        c["Hq"], c["Hkv"] = 32, 8
    most = work(next(x for x in listed() if x["name"] == "bwd-longtail-128k-gqa32x8"))["flops"]
    while work(c)["flops"] > most and c["Hq"] > 4:   # no dearer than the largest listed case
        c["Hkv"] = max(1, c["Hkv"] // 2)
        c["Hq"] //= 2
    return c


def _lengths(case):
    T, mix, seed = case["T"], case["mix"], case["lseed"]
    if mix == "tiny":
        return synth.lengths_tiny(seed, budget=T)
    if mix == "lognormal":
        return synth.lengths_lognormal(T, seed)
    if mix == "longtail":
        return synth.lengths_longtail(T, seed)[0]
    if mix.startswith("table2:"):
        return synth.lengths_table2(T, seed, mix.split(":")[1])
    # ragged: every remainder, single tokens and empty sequences among them
    r = np.random.Generator(np.random.PCG64(seed))
    out, left = [1, 0], T - 1
    while left > 0:
        n = int(min(left, r.integers(1, 4096) if r.random() < 0.5 else r.integers(1, 400)))
        out.append(n)
        left -= n
    return out


def _pairs(lengths):
    return int(sum(n * (n + 1) // 2 for n in lengths))


def work(case):
    lengths = _lengths(case)
    T, Hq, Hkv, d = sum(lengths), case["Hq"], case["Hkv"], case["d"]
    qb, kvb, lb = 2 * T * Hq * d, 2 * T * Hkv * d, 4 * T * Hq
    if case["op"] == "remap":
        return {"bytes": 2 * qb + 4 * T, "flops": 0}
    fwd = 4 * d * Hq * _pairs(lengths)
    fwd_bytes = 2 * qb + 2 * kvb + lb                  # q, k, v in; o, lse out
    bwd_bytes = 4 * qb + 4 * kvb + lb                  # dO, q, o, k, v, lse in; dq, dk, dv out
    if case["op"] in ("fwd", "noalloc", "chunked"):
        return {"bytes": fwd_bytes, "flops": fwd}
    if case["op"] == "bwd":
        return {"bytes": bwd_bytes, "flops": 5 * fwd // 2}
    return {"bytes": 3 * qb + 4 * kvb + qb + lb, "flops": 7 * fwd // 2}   # train, node: q, k, v, dO in; o, lse, dq, dk, dv out


# Measured against `exact` over the listed cases and six drawn ones: O is 2.0e-3 to 2.1e-3 off, dQ and dK 2.5e-3, dV
# 2.3e-3 (bf16 operands of the second products, bf16 output grid), LSE under 1e-7; about four times that.
def tolerance(case):
    if case["op"] == "remap":
        return "exact"
    return {"rel": 8e-3} if case["op"] in ("fwd", "noalloc", "chunked") else {"rel": 1e-2}


def _normal(shape, gen):
    out = torch.empty(shape, dtype=torch.bfloat16, device=DEV)
    flat = out.view(-1)
    for a in range(0, flat.numel(), 1 << 28):
        b = min(flat.numel(), a + (1 << 28))
        flat[a:b] = torch.randn(b - a, generator=gen, device=DEV, dtype=torch.float32)
    return out


def _inputs(case, seed):
    """Lengths and q, k, v, dO from the seed alone: N(0, 1) values in bf16."""
    lengths = _lengths(case)
    T, Hq, Hkv, d = sum(lengths), case["Hq"], case["Hkv"], case["d"]
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)
    if case["op"] == "remap":
        return lengths, _normal((T, Hq, d), gen), None, None, None
    if case["fused"]:
        qkv = _normal((T, Hq + 2 * Hkv, d), gen)
        q, k, v = qkv[:, :Hq], qkv[:, Hq:Hq + Hkv], qkv[:, Hq + Hkv:]
    else:
        q, k, v = _normal((T, Hq, d), gen), _normal((T, Hkv, d), gen), _normal((T, Hkv, d), gen)
    do = _normal((T, Hq, d), gen) if case["op"] in ("bwd", "train", "node") else None
    return lengths, q, k, v, do


def _layout(case, lengths):
    return synth.balanced_attention_layout(lengths, R=8)[0]


def prepare(case, seed):
    lengths, q, k, v, do = _inputs(case, seed)
    T, Hq, d, op = sum(lengths), case["Hq"], case["d"], case["op"]
    s = dict(op=op, scale=case["scale"], q=q, k=k, v=v, do=do, cu=synth.cu_seqlens(lengths))
    if op == "remap":
        s["idx"] = torch.from_numpy(_layout(case, lengths)).to(DEV)
        s["mode"], s["dst"] = case["mode"], torch.empty_like(q)
        return s
    if op == "node":
        P = case["P"]
        # capacity per device: an even share plus a quarter, as the benchmark's nodes have
        s["plan"] = node.NodePlan(lengths, P, 1, (sum(lengths) + P - 1) // P * 5 // 4, b_intra=1, b_inter=8)
        s["job"] = node.NodeJob(s["plan"], Hq, case["Hkv"], d, DEV)
        s["job"].lse.zero_()   # rows of ring sequences stay as they are: their LSE is in lse_run
        like = lambda x: torch.empty_like(x)
        s["in"] = [like(x) for x in (q, k, v, do)]
        s["out"] = [like(x) for x in (q, q, k, v)]
        return s
    s["o"] = torch.empty((T, Hq, d), dtype=torch.bfloat16, device=DEV)
    s["lse"] = torch.empty((Hq, T), dtype=torch.float32, device=DEV)
    if op in ("bwd", "train"):
        s["grads"] = [torch.empty(x.shape, dtype=x.dtype, device=DEV) for x in (q, k, v)]
    if op == "bwd":
        B.varlen_attn_fwd(q, k, v, s["cu"], o=s["o"], lse=s["lse"], scale=s["scale"])
    if op == "chunked":
        pairs, merges, rows = [], [], 0
        s["skip"] = np.zeros(len(lengths), np.uint8)
        for i, n in enumerate(lengths):
            if n >= LONG:
                s["skip"][i] = 1
                p, m, r = B.chunk_pairs(int(s["cu"][i]), n, case["C"], row0=rows)
                pairs += list(p)
                merges += list(m)
                rows += r
        s["rows"] = rows
        if rows:
            s["pairs"], s["merges"] = (B.ZpPair * len(pairs))(*pairs), (B.ZpMerge * len(merges))(*merges)
            s["o_part"] = torch.empty((rows, Hq, d), dtype=torch.float32, device=DEV)
            s["lse_part"] = torch.empty((Hq, rows), dtype=torch.float32, device=DEV)
    return s


def run(s):
    op = s["op"]
    if op == "remap":
        return B.remap_tokens(s["q"], s["idx"], s["mode"], dst=s["dst"])
    q, k, v, cu, scale = s["q"], s["k"], s["v"], s["cu"], s["scale"]
    if op == "node":
        j = s["job"]
        qa, ka, va = (j.to_attention(x, y) for x, y in zip((q, k, v), s["in"]))
        o, lse = j.forward(qa, ka, va, scale=scale)
        outs = [j.to_balanced(o, s["out"][0])]
        da = j.to_attention(s["do"], s["in"][3])
        outs += [j.to_balanced(x, y) for x, y in zip(j.backward(da, qa, ka, va, scale=scale), s["out"][1:])]
        return outs + [lse] + ([j.lse_run] if s["plan"].ring_segments else [])
    if op == "noalloc":
        return B.varlen_attn_fwd_noalloc(q, k, v, cu, s["o"], s["lse"], scale=scale)
    if op == "chunked":
        B.varlen_attn_fwd(q, k, v, cu, o=s["o"], lse=s["lse"], scale=scale, seq_skip=s["skip"])
        if s["rows"]:
            B.chunk_attn_partial(q, k, v, s["pairs"], s["rows"], o_part=s["o_part"], lse_part=s["lse_part"], scale=scale)
            B.lse_merge(s["o_part"], s["lse_part"], s["merges"], s["o"], s["lse"])
        return s["o"], s["lse"]
    if op != "bwd":
        B.varlen_attn_fwd(q, k, v, cu, o=s["o"], lse=s["lse"], scale=scale)
        if op == "fwd":
            return s["o"], s["lse"]
    dq, dk, dv = s["grads"]
    grads = B.varlen_attn_bwd(s["do"], q, k, v, s["o"], s["lse"], cu, dq=dq, dk=dk, dv=dv, scale=scale)
    return grads if op == "bwd" else (s["o"], s["lse"], *grads)


def _attention64(lengths, q, k, v, do, scale):
    """Causal attention of every sequence (and its gradients, if dO is given) in 64 bits: o, lse[, dq, dk, dv]."""
    T, Hq, d = q.shape
    Hkv = k.shape[1]
    grp, scale = Hq // Hkv, scale or d ** -0.5
    new = lambda x: torch.zeros(x.shape, dtype=torch.float64, device=x.device)
    o, lse = new(q), torch.zeros((Hq, T), dtype=torch.float64, device=q.device)
    grads = (new(q), new(k), new(v)) if do is not None else None
    t0 = 0
    for n in lengths:
        step = max(1, min(n, (1 << 26) // max(1, grp * n)))
        for g in range(Hkv if n else 0):
            heads, seq = slice(g * grp, (g + 1) * grp), slice(t0, t0 + n)
            kk, vv = k[seq, g].double(), v[seq, g].double()
            kt, vt = kk.t().contiguous(), vv.t().contiguous()
            for a in range(0, n, step):
                b = min(n, a + step)
                rows = slice(t0 + a, t0 + b)
                flat = lambda x: x[rows, heads].double().transpose(0, 1).reshape(-1, d)   # head by head
                back = lambda x: x.view(grp, b - a, d).transpose(0, 1)
                qq = flat(q)
                s = (qq @ kt[:, :b].contiguous()).mul_(scale)
                hidden = torch.arange(b, device=q.device)[None, :] > torch.arange(a, b, device=q.device)[:, None]
                s.view(grp, b - a, b).masked_fill_(hidden, float("-inf"))
                l = torch.logsumexp(s, 1, keepdim=True)
                p = s.sub_(l).exp_()
                oo = p @ vv[:b]
                o[rows, heads], lse[heads, rows] = back(oo), l.view(grp, b - a)
                if grads:
                    dd = flat(do)
                    grads[2][t0:t0 + b, g] += p.t().contiguous() @ dd
                    ds = (dd @ vt[:, :b].contiguous()).sub_((dd * oo).sum(1, keepdim=True)).mul_(p).mul_(scale)
                    grads[0][rows, heads] = back(ds @ kk[:b])
                    grads[1][t0:t0 + b, g] += ds.t().contiguous() @ qq
        t0 += n
    return (o, lse) + (grads or ())


def exact(case, seed):
    lengths, q, k, v, do = _inputs(case, seed)
    op = case["op"]
    if op == "remap":
        idx, x = torch.from_numpy(_layout(case, lengths)).to(DEV).long(), q.double()
        return x[idx] if case["mode"] == 0 else torch.empty_like(x).index_copy_(0, idx, x)
    if op == "node":
        P = case["P"]
        plan = node.NodePlan(lengths, P, 1, (sum(lengths) + P - 1) // P * 5 // 4, b_intra=1, b_inter=8)
        # balanced position -> position in the batch as drawn, through the attention layout
        drawn = torch.from_numpy(plan.orig).to(DEV)
        at = drawn[torch.from_numpy(plan.idx).to(DEV).long()]
        seq = lambda x: torch.empty_like(x).index_copy_(0, at, x)
        o, lse, dq, dk, dv = _attention64(lengths, seq(q), seq(k), seq(v), seq(do), case["scale"])
        lse = lse[:, drawn]
        ring = torch.from_numpy(np.repeat(plan.skip, np.diff(plan.cu)).astype(bool)).to(DEV)
        outs = [o[at], dq[at], dk[at], dv[at], lse.masked_fill(ring, 0.0)]
        return outs + ([lse.masked_fill(~ring, float("-inf"))] if plan.ring_segments else [])
    out = _attention64(lengths, q, k, v, do, case["scale"])
    return out[2:] if op == "bwd" else out
