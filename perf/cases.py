"""The performance cases of this library: what its users have it do, through its public entry points.

A case is one rank's micro-batch and one thing done with it.  Its lengths are a log-normal mix of
whole sequences (``median``, ``sigma``, ``lo``, ``hi``, ``tokens``) drawn with ``length_seed``, after
``long_count`` long sequences of about ``long_len`` tokens (each next one a twelfth shorter), which are
whole on this rank (``cp`` = 1) or cut over ``cp`` ranks, this one being ``rank``, contiguously or in
two chunks.  What is done:

  ``fwd``    skrull_attn_fwd on a plan the program keeps (the plan serves every layer of a model)
  ``bwd``    skrull_attn_bwd on such a plan, given the forward's O and LSE
  ``train``  skrull_attention and its gradients through torch.autograd on such a plan
  ``step``   a new plan, forward and backward, the plan released: a micro-batch's first layer

Tensors are bf16, LSE fp32; values are N(0,1), as in the repository's tests and benchmark.
"""
import math

import numpy as np
import torch

from paper_2505_19609_amd import binding as B
from paper_2505_19609_amd import workloads as W
from paper_2505_19609_amd.autograd import skrull_attention


def _case(what, heads, median, sigma, lo, hi, tokens, length_seed, long_len=0, long_count=0, cp=1, rank=0,
          two_chunks=False, name=None):
    hq, hkv, d = heads
    c = {"what": what, "q_heads": hq, "kv_heads": hkv, "head_dim": d, "median": median, "sigma": sigma, "lo": lo,
         "hi": hi, "tokens": tokens, "length_seed": length_seed, "long_len": long_len, "long_count": long_count,
         "cp": cp, "rank": rank, "two_chunks": two_chunks}
    return {"name": name, **c} if name else c


QWEN_05B = (14, 2, 64)   # query heads, key / value heads, head_dim
QWEN_7B = (28, 4, 128)
LLAMA_8B = (32, 8, 128)
MHA_64 = (16, 16, 64)


def listed():
    return [
        # the smallest calls: a handful of short sequences (the repository's 4-head test model), where launches and latency count
        _case("train", (4, 4, 64), 200, 1.0, 16, 511, 932, 1, name="tiny_train"),
        # the benchmark's 16,384-token micro-batch of the 0.5B model, a new plan for it included
        _case("step", QWEN_05B, 600, 1.0, 16, 8192, 16384, 2, name="qwen05b_16k_step"),
        # a full bucket (26K tokens, the paper's setting) of the 0.5B model on a long-tail corpus: each layer's forward and backward
        _case("fwd", QWEN_05B, 300, 1.1, 16, 8192, 26624, 11, name="qwen05b_26k_fwd"),
        _case("bwd", QWEN_05B, 300, 1.1, 16, 8192, 26624, 11, name="qwen05b_26k_bwd"),
        # the 0.5B model on the bimodal corpus: long sequences cut in two chunks over 8 ranks beside short ones
        _case("train", QWEN_05B, 700, 1.0, 16, 8192, 6000, 12, 49152, 3, 8, 2, True, name="qwen05b_bimodal_train"),
        # a full bucket (13K tokens) of the 7B model on a long-tail corpus
        _case("train", QWEN_7B, 500, 1.1, 16, 8192, 13312, 13, name="qwen7b_13k_train"),
        # short instruction data packed to 32,768 tokens
        _case("fwd", LLAMA_8B, 250, 0.6, 32, 1024, 32768, 14, name="llama8b_short_fwd"),
        _case("bwd", LLAMA_8B, 250, 0.6, 32, 1024, 32768, 14, name="llama8b_short_bwd"),
        # the headline micro-batch: one 24,576-token sequence and 8,192 tokens of short ones
        _case("fwd", LLAMA_8B, 800, 0.8, 32, 4096, 8192, 3, 24576, 1, name="llama8b_32k_fwd"),
        _case("bwd", LLAMA_8B, 800, 0.8, 32, 4096, 8192, 3, 24576, 1, name="llama8b_32k_bwd"),
        # the largest: a rank's share of a 131,072-token sequence cut over 8 ranks, with 8,192 tokens of its own
        _case("train", LLAMA_8B, 1000, 0.8, 64, 4096, 8192, 4, 131072, 1, 8, 3, True, name="llama8b_shard_train"),
        # a model without grouped heads on ragged sequences of middling length
        _case("train", MHA_64, 2500, 0.9, 33, 12000, 23053, 15, name="mha64_ragged_train"),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    heads = rng.choice([(4, 4, 64), QWEN_05B, QWEN_05B, MHA_64, QWEN_7B, LLAMA_8B, LLAMA_8B])
    tokens = log_int(500, 32768)
    long_len, count, cp, rank, two = 0, 0, 1, 0, False
    if rng.random() < 0.5:
        long_len = log_int(2048, 32768)
        count = rng.randint(1, 2)
        cp = rng.choice([1, 1, 2, 4, 8])
        rank = rng.randrange(cp)
        two = cp > 1 and rng.random() < 0.7
        if cp > 1:
            long_len = min(65536, long_len * 3)
        tokens = max(500, tokens // 2)
    lo = rng.randint(1, 64)
    hi = rng.choice([511, 1024, 4096, 8192])
    return _case(rng.choice(["fwd", "bwd", "train", "step"]), heads, log_int(100, 3000), round(rng.uniform(0.4, 1.1), 2),
                 lo, hi, tokens, rng.randrange(1 << 30), long_len, count, cp, rank, two)


def _micro_batch(case):
    """(lengths, degrees, indices, cuts) of the case."""
    rng = np.random.Generator(np.random.PCG64(case["length_seed"]))
    short = W.lognormal_lengths(rng, case["median"], case["sigma"], case["lo"], case["hi"], case["tokens"])
    longs = [case["long_len"] - i * (case["long_len"] // 12) for i in range(case["long_count"])]
    S = longs + short
    cut = [int(case["two_chunks"])] * len(longs) + [0] * len(short)
    return S, [case["cp"]] * len(longs) + [1] * len(short), [case["rank"]] * len(longs) + [0] * len(short), cut


def _segments(case):
    """[(first q row, q rows, position of the first, first k row)] of the query segments, and the totals of q and k rows."""
    out, tq, tk = [], 0, 0
    for s, n, r, z in zip(*_micro_batch(case)):
        chunks = n * (2 if z else 1)
        end = 0
        for i in ([r, 2 * n - 1 - r] if z else [r]):
            b, end = i * s // chunks, (i + 1) * s // chunks
            out.append((tq, end - b, b, tk))
            tq += end - b
        tk += end
    return out, tq, tk


def _new_plan(case):
    S, N, R, Z = _micro_batch(case)
    return B.skrull_attn_plan(S, N, R, case["q_heads"], case["kv_heads"], case["head_dim"], case["head_dim"] ** -0.5,
                              shard_cut=Z)


def _workspace(plan):
    return torch.empty(max(int(plan.bwd_workspace_bytes), 16), dtype=torch.uint8, device="cuda")


def _inputs(case, seed):
    """Q, K, V, dO on the GPU."""
    _, tq, tk = _segments(case)
    hq, hkv, d = case["q_heads"], case["kv_heads"], case["head_dim"]
    gen = torch.Generator(device="cuda").manual_seed(int(seed))
    return [torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).bfloat16()
            for shape in ((tq, hq, d), (tk, hkv, d), (tk, hkv, d), (tq, hq, d))]


def prepare(case, seed):
    q, k, v, do = _inputs(case, seed)
    st = {"case": case, "what": case["what"], "q": q, "k": k, "v": v, "do": do}
    if case["what"] == "train":
        for t in (q, k, v):
            t.requires_grad_()
        st["plan"] = _new_plan(case)
        return st
    st["o"] = torch.empty_like(q)
    st["lse"] = torch.empty((case["q_heads"], q.shape[0]), dtype=torch.float32, device="cuda")
    if case["what"] != "fwd":
        st.update(dq=torch.empty_like(q), dk=torch.empty_like(k), dv=torch.empty_like(v))
    if case["what"] != "step":
        st["plan"] = _new_plan(case)
    if case["what"] == "bwd":
        B.skrull_attn_fwd(st["plan"], q, k, v, st["o"], st["lse"])
        st["ws"] = _workspace(st["plan"])
    if case["what"] == "step":
        st["batch"] = _micro_batch(case)
    return st


def run(st):
    what = st["what"]
    if what == "fwd":
        B.skrull_attn_fwd(st["plan"], st["q"], st["k"], st["v"], st["o"], st["lse"])
        return {"o": st["o"], "lse": st["lse"]}
    if what == "bwd":
        B.skrull_attn_bwd(st["plan"], st["q"], st["k"], st["v"], st["o"], st["lse"], st["do"], st["dq"], st["dk"],
                          st["dv"], st["ws"])
        return {"dq": st["dq"], "dk": st["dk"], "dv": st["dv"]}
    if what == "train":
        o = skrull_attention(st["q"], st["k"], st["v"], st["plan"])
        dq, dk, dv = torch.autograd.grad(o, (st["q"], st["k"], st["v"]), st["do"])
        return {"o": o.detach(), "dq": dq, "dk": dk, "dv": dv}
    case = st["case"]
    S, N, R, Z = st["batch"]
    plan = B.skrull_attn_plan(S, N, R, case["q_heads"], case["kv_heads"], case["head_dim"], case["head_dim"] ** -0.5,
                              shard_cut=Z)
    B.skrull_attn_fwd(plan, st["q"], st["k"], st["v"], st["o"], st["lse"])
    B.skrull_attn_bwd(plan, st["q"], st["k"], st["v"], st["o"], st["lse"], st["do"], st["dq"], st["dk"], st["dv"],
                      _workspace(plan))
    plan.destroy()
    return {"o": st["o"], "lse": st["lse"], "dq": st["dq"], "dk": st["dk"], "dv": st["dv"]}


def _pairs(case):
    return sum(((p + n) * (p + n + 1) - p * (p + 1)) // 2 for _, n, p, _ in _segments(case)[0])


def work(case):
    _, tq, tk = _segments(case)
    hq, hkv, d = case["q_heads"], case["kv_heads"], case["head_dim"]
    q_bytes, k_bytes, lse = 2 * tq * hq * d, 2 * tk * hkv * d, 4 * tq * hq
    unit = _pairs(case) * d * hq
    fwd = {"bytes": 2 * q_bytes + 2 * k_bytes + lse, "flops": 4 * unit}   # Q, K, V -> O, LSE
    bwd = {"bytes": 4 * q_bytes + 4 * k_bytes + lse, "flops": 10 * unit}  # Q, K, V, O, dO, LSE -> dQ, dK, dV
    if case["what"] == "fwd":
        return fwd
    if case["what"] == "bwd":
        return bwd
    return {n: fwd[n] + bwd[n] for n in fwd}


def tolerance(case):
    # bf16 operands and results, fp32 sums: rounding P and dS to bf16 and the results once.  Against
    # `exact` the largest relative error of an output was 2.6e-3 (1.2e-3 of it the last rounding); "max" is set by rows that see few
    # keys, where the errors do not average out.
    return {"rel": 1e-2, "max": 0.25}


def exact(case, seed):
    """What run() returns, from 64-bit sums over whole rows of scores."""
    segments, tq, tk = _segments(case)
    hq, hkv, d = case["q_heads"], case["kv_heads"], case["head_dim"]
    g, scale = hq // hkv, d ** -0.5
    if _pairs(case) * hq > 4e10:
        return None
    q, k, v, do = (t.double().transpose(0, 1).contiguous() for t in _inputs(case, seed))  # [heads, rows, d]
    o, lse = torch.empty_like(q), torch.empty((hq, tq), dtype=torch.float64, device="cuda")
    dq, dk, dv = torch.empty_like(q), torch.zeros_like(k), torch.zeros_like(v)
    for q0, rows, p0, k0 in segments:
        step = max(1, min(rows, int(6e7 / (g * (p0 + rows)))))
        for c in range(hkv):
            hs = slice(c * g, (c + 1) * g)
            for i in range(0, rows, step):
                n = min(step, rows - i)
                keys = p0 + i + n
                qi, gi = (t[hs, q0 + i:q0 + i + n].reshape(g * n, d) for t in (q, do))
                kj, vj = (t[c, k0:k0 + keys] for t in (k, v))
                s = (qi @ kj.t()).view(g, n, keys).mul_(scale)
                late = torch.arange(keys, device="cuda")[None, :] > torch.arange(p0 + i, p0 + i + n, device="cuda")[:, None]
                s.masked_fill_(late[None], -math.inf)
                l = torch.logsumexp(s, dim=-1)
                p = s.sub_(l[..., None]).exp_().view(g * n, keys)
                oi = p @ vj
                o[hs, q0 + i:q0 + i + n] = oi.view(g, n, d)
                lse[hs, q0 + i:q0 + i + n] = l
                if case["what"] == "fwd":
                    continue
                dv[c, k0:k0 + keys] += p.t() @ gi
                ds = (gi @ vj.t()).sub_((gi * oi).sum(-1, keepdim=True)).mul_(p)
                dq[hs, q0 + i:q0 + i + n] = (ds @ kj).mul_(scale).view(g, n, d)
                dk[c, k0:k0 + keys] += (ds.t() @ qi).mul_(scale)
    o, dq, dk, dv = (t.transpose(0, 1).contiguous() for t in (o, dq, dk, dv))
    if case["what"] == "fwd":
        return {"o": o, "lse": lse}
    if case["what"] == "bwd":
        return {"dq": dq, "dk": dk, "dv": dv}
    if case["what"] == "train":
        return {"o": o, "dq": dq, "dk": dk, "dv": dv}
    return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}
