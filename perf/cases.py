"""The work whose speed counts here, as cases: packed varlen attention (forward, and forward + backward) and
packed cross-entropy (training and evaluation), each through the public entry points, from one pack of 512
tokens to one of 131072.

``listed()`` names the cases, ``draw(rng)`` gives more of the same ranges, ``prepare`` makes what a training
program holds before the call (inputs on the GPU, the pack's plan, its buffers), ``run`` is one pass,
``work`` what a pass cannot do without, ``tolerance`` how far another correct implementation at the same
precision may be off and ``exact`` the same outputs in 64 bits.
"""
import math

import numpy as np
import torch

import paper_2503_07680_amd as hbp
from paper_2503_07680_amd.runner import PackedAttention

# ------------------------------------------------------------------------------------------ the cases


def _attn(name, tokens, heads, kv_heads, d_qk, d_v, median, spread, lo, hi, long_sample=0, sigma=1.0,
          backward=True, row_pad=0, length_seed=0):
    """Samples: `long_sample` tokens first (0: none), then lognormal(median, spread) clipped to [lo, hi]
    until the pack holds `tokens`."""
    return {"name": name, "kind": "attention", "tokens": tokens, "heads": heads, "kv_heads": kv_heads,
            "d_qk": d_qk, "d_v": d_v, "median": median, "spread": spread, "lo": lo, "hi": hi,
            "long_sample": long_sample, "sigma": sigma, "backward": backward, "row_pad": row_pad,
            "length_seed": length_seed}


def _ce(name, tokens, vocab, samples, normalizer, grad, masked=0.3):
    return {"name": name, "kind": "loss", "tokens": tokens, "vocab": vocab, "samples": samples,
            "normalizer": normalizer, "grad": grad, "masked": masked}


def listed():
    return [
        # The smallest pack: 1024 tokens in a few short samples, 4 heads of 64.  A step of a small model, or the
        # last, under-full pack of a group: launches, latency and an almost empty chip.
        _attn("tiny-1k-train", 1024, 4, 4, 64, 64, 200, 0.8, 16, 512),
        # Multi-head attention at head size 64, a ragged number of tokens: one group size for every head layout
        # without key/value sharing, at the size of a short pack.
        _attn("mha64-5k-train", 5497, 8, 8, 64, 64, 500, 1.2, 16, 4096),
        # A pack of short instruction samples, 8192 tokens, grouped-query heads 32/8 of 128: the most frequent
        # kind of pack of a hybrid data set.  Forward alone: evaluation, and the second forward of a layer whose
        # activations are checkpointed.
        _attn("short-8k-forward", 8192, 32, 8, 128, 128, 400, 1.0, 16, 4096, backward=False),
        # The same pack, a training step of one layer.
        _attn("short-8k-train", 8192, 32, 8, 128, 128, 400, 1.0, 16, 4096),
        # One 16384-token sample among short ones, 32768 tokens: the imbalanced pack that the scheduler is for.
        _attn("mixed-32k-train", 32768, 32, 8, 128, 128, 600, 1.2, 16, 4096, long_sample=16384),
        # One GPU's share of a layer whose heads are dealt out over several GPUs: 8 query heads on one kv head.
        _attn("mixed-32k-8on1-train", 32768, 8, 1, 128, 128, 600, 1.2, 16, 4096, long_sample=16384),
        # Latent-attention shape: 128 heads, query/key size 192, value size 128, no key/value sharing.
        _attn("mla-32k-train", 32768, 128, 128, 192, 128, 1000, 1.3, 32, 8192),
        # The largest: a long-context pack, 98304 + 32768 tokens, 64/8 heads.
        _attn("long-128k-train", 131072, 64, 8, 128, 128, 32768, 0.0, 32768, 32768, long_sample=98304, sigma=0.5),
        # The loss of a training step: 8192 tokens against a vocabulary of 128256, loss and gradient.
        _ce("loss-8k-128k-train", 8192, 128256, 12, "stable", True),
        # A small pack and a small vocabulary, loss and gradient.
        _ce("loss-1k-32k-train", 1000, 32000, 5, "token_mean", True),
        # Evaluation: per-token losses without a gradient, the largest vocabulary in use.
        _ce("loss-4k-152k-eval", 4096, 151936, 9, "sample_mean", False),
    ]


#: head layouts of the repository's workloads and tests: (query heads, kv heads, d_qk, d_v, most tokens)
_LAYOUTS = [(4, 4, 64, 64, 32768), (8, 8, 64, 64, 32768), (6, 2, 64, 64, 32768), (32, 8, 128, 128, 65536),
            (32, 8, 128, 128, 65536), (8, 1, 128, 128, 65536), (64, 8, 128, 128, 65536), (24, 24, 128, 128, 32768),
            (12, 3, 128, 128, 32768), (128, 128, 192, 128, 16384), (16, 16, 192, 128, 32768)]
_VOCABS = [4096, 32000, 50304, 65536, 128256, 151936, 152064]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.random()
    if kind < 0.75:
        heads, kv_heads, d_qk, d_v, most = rng.choice(_LAYOUTS)
        tokens = _log_uniform(rng, 512, most)
        median = _log_uniform(rng, 100, 1500)
        long_sample = int(tokens * rng.uniform(0.25, 0.75)) if rng.random() < 0.4 else 0
        c = _attn("", tokens, heads, kv_heads, d_qk, d_v, median, round(rng.uniform(0.6, 1.3), 3), 16, 8192,
                  long_sample=long_sample, sigma=rng.choice([0.5, 1.0]), backward=rng.random() < 0.7,
                  row_pad=rng.choice([0, 0, 0, 64]), length_seed=rng.randrange(1 << 30))
    else:
        vocab = rng.choice(_VOCABS) if rng.random() < 0.6 else 8 * _log_uniform(rng, 512, 19000)
        tokens = _log_uniform(rng, 64, 8192)
        c = _ce("", tokens, vocab, rng.randrange(1, max(2, min(64, tokens // 16))),
                rng.choice(["token_mean", "sample_mean", "stable"]), rng.random() < 0.75,
                round(rng.choice([0.0, rng.uniform(0.0, 0.8)]), 3))
    c.pop("name", None)
    return c


# --------------------------------------------------------------------------------------------- inputs

_NORMALIZERS = {"token_mean": hbp.HBP_LOSS_TOKEN_MEAN, "sample_mean": hbp.HBP_LOSS_SAMPLE_MEAN,
                "stable": hbp.HBP_LOSS_STABLE}


def _lengths(case):
    """The pack's sample lengths, the last one cut to fit: a property of the case, not of the inputs' seed."""
    r = np.random.default_rng(case["length_seed"])
    out = [case["long_sample"]] if case["long_sample"] else []
    total = sum(out)
    while total < case["tokens"]:
        n = int(np.clip(np.rint(np.exp(r.normal(math.log(case["median"]), case["spread"]))), case["lo"], case["hi"]))
        n = min(n, case["tokens"] - total)
        out.append(n)
        total += n
    return out


def _prepare_attention(case, seed):
    pa = PackedAttention(_lengths(case), case["tokens"], case["heads"], case["kv_heads"], case["d_qk"], case["d_v"],
                         row_pad=case["row_pad"])
    gen = torch.Generator(device=pa.device).manual_seed(seed)

    def tensor(heads, dim):
        x = pa.buffer(heads, dim)
        x.normal_(0.0, case["sigma"], generator=gen)
        return x

    state = {"kind": "attention", "pa": pa, "q": tensor(pa.Hq, pa.d_qk), "k": tensor(pa.Hkv, pa.d_qk),
             "v": tensor(pa.Hkv, pa.d_v)}
    if case["backward"]:
        state["d_o"] = tensor(pa.Hq, pa.d_v)
        pa.alloc_backward()
    return state


def _prepare_loss(case, seed):
    dev = torch.device("cuda:0")
    T, V, n = case["tokens"], case["vocab"], case["samples"]
    gen = torch.Generator(device=dev).manual_seed(seed)
    logits = torch.empty((T, V), dtype=torch.bfloat16, device=dev).normal_(0.0, 2.0, generator=gen)
    labels = torch.randint(0, V, (T,), dtype=torch.int32, device=dev, generator=gen)
    labels.masked_fill_(torch.rand(T, device=dev, generator=gen) < case["masked"], -100)  # prompt tokens: no loss
    cuts = np.sort(np.random.default_rng(n).choice(np.arange(1, T), n - 1, replace=False)) if n > 1 else []
    cu = torch.from_numpy(np.concatenate([[0], cuts, [T]]).astype(np.int32)).to(dev)
    return {"kind": "loss", "logits": logits, "labels": labels, "cu": cu, "T": T, "V": V, "n": n,
            "normalizer": _NORMALIZERS[case["normalizer"]],
            "t_ave": T * (1.0 - case["masked"]) / n,  # loss tokens per sample, as reduced over all ranks
            "dlogits": torch.empty_like(logits) if case["grad"] else None,
            "loss": torch.empty(1, dtype=torch.float32, device=dev),
            "token_loss": torch.empty(T, dtype=torch.float32, device=dev),
            "workspace": torch.empty(hbp.hbp_packed_ce_workspace_bytes(T, n), dtype=torch.uint8, device=dev)}


def prepare(case, seed):
    return (_prepare_attention if case["kind"] == "attention" else _prepare_loss)(case, seed)


# --------------------------------------------------------------------------------------------- one pass


def run(state):
    if state["kind"] == "attention":
        pa = state["pa"]
        out = pa.forward(state["q"], state["k"], state["v"])
        if "d_o" in state:
            out = out + pa.backward(state["q"], state["k"], state["v"], state["d_o"])
        return out
    s = state
    hbp.hbp_packed_ce(s["logits"], 0, s["T"], s["V"], s["labels"], s["cu"], s["n"], s["normalizer"], s["t_ave"],
                      s["dlogits"], s["loss"], s["token_loss"], s["workspace"],
                      int(torch.cuda.current_stream().cuda_stream))
    return [s["loss"], s["token_loss"]] + ([s["dlogits"]] if s["dlogits"] is not None else [])


# --------------------------------------------------------------------------------- what a pass has to do


def work(case):
    """Bytes: every input read and every output written once.  Flops: causal pairs inside samples only, two
    products forward and five backward (the scores again, dP, dV, dK, dQ)."""
    if case["kind"] == "attention":
        T, h, kv, d, e = case["tokens"], case["heads"], case["kv_heads"], case["d_qk"], case["d_v"]
        pairs = sum(s * (s + 1) // 2 for s in _lengths(case))
        q, k, v, o, rows = 2 * T * h * d, 2 * T * kv * d, 2 * T * kv * e, 2 * T * h * e, 4 * T * h
        nbytes, flops = q + k + v + o + rows, h * pairs * 2 * (d + e)
        if case["backward"]:
            nbytes += q + k + v + 2 * o + rows + q + k + v
            flops += h * pairs * 2 * (3 * d + 2 * e)
        return {"bytes": nbytes, "flops": flops}
    row = 2 * case["vocab"]  # a row without a loss is not read; its gradient row is written as zeros
    nbytes = case["tokens"] * ((1.0 - case["masked"]) * row + (row if case["grad"] else 0) + 8)
    return {"bytes": nbytes, "flops": 6.0 * case["tokens"] * case["vocab"] * (1.0 - case["masked"])}


def tolerance(case):
    if case["kind"] == "attention":
        # bf16 probabilities and outputs: O 2.0e-3, gradients 2.3e-3 to 2.5e-3 off the same path in 64 bits
        return {"rel": 1e-2}
    # gradients stored in bf16 are 9.6e-4 off the same path in 64 bits; losses alone are 32-bit sums (4e-8)
    return {"rel": 4e-3} if case["grad"] else {"rel": 1e-5}


# ------------------------------------------------------------------------------------ the same in 64 bits


def _exact_attention(case, seed):
    if work(case)["flops"] > 2e14:
        return None  # the 131072-token pack: too long in 64 bits
    state = prepare(case, seed)
    pa, h, kv = state["pa"], case["heads"], case["kv_heads"]
    g, d, e, scale = h // kv, case["d_qk"], case["d_v"], 1.0 / math.sqrt(case["d_qk"])
    f64, dev = torch.float64, pa.device

    def out(heads, dim):
        return torch.empty((case["tokens"], heads, dim), dtype=f64, device=dev)

    o, lse = out(h, e), torch.empty((h, case["tokens"]), dtype=f64, device=dev)
    dq, dk, dv = (out(h, d), out(kv, d), out(kv, e)) if case["backward"] else (None, None, None)
    start = 0
    for n in _lengths(case):
        k = state["k"][start:start + n].transpose(0, 1).to(f64).contiguous()  # [kv, n, d]
        v = state["v"][start:start + n].transpose(0, 1).to(f64).contiguous()
        kt, vt = k.transpose(1, 2).contiguous(), v.transpose(1, 2).contiguous()
        gk, gv = torch.zeros_like(k), torch.zeros_like(v)
        step = max(1, min(n, (1 << 27) // (h * n)))  # scores of `step` rows of every head: at most 1 GiB
        for a in range(0, n, step):
            b = min(a + step, n)
            rows = slice(start + a, start + b)

            def by_kv_head(t):  # [rows, h, dim] -> [kv, g * rows, dim]
                return t.transpose(0, 1).reshape(kv, g * (b - a), -1).to(f64)

            def by_row(t):
                return t.reshape(h, b - a, -1).transpose(0, 1)

            q = by_kv_head(state["q"][rows])
            s = torch.matmul(q, kt[:, :, :b].contiguous()).mul_(scale)
            later = torch.arange(b, device=dev)[None, :] > torch.arange(a, b, device=dev)[:, None]
            s.view(h, b - a, b).masked_fill_(later, -math.inf)
            log_sum = torch.logsumexp(s, dim=-1, keepdim=True)
            p = s.sub_(log_sum).exp_()
            po = torch.matmul(p, v[:, :b].contiguous())
            o[rows], lse[:, rows] = by_row(po), log_sum.view(h, b - a)
            if case["backward"]:
                go = by_kv_head(state["d_o"][rows])
                gv[:, :b] += torch.matmul(p.transpose(1, 2).contiguous(), go)
                ds = torch.matmul(go, vt[:, :, :b].contiguous()).sub_((go * po).sum(-1, keepdim=True)).mul_(p)
                dq[rows] = by_row(torch.matmul(ds, k[:, :b].contiguous()).mul_(scale))
                gk[:, :b] += torch.matmul(ds.transpose(1, 2).contiguous(), q).mul_(scale)
        if case["backward"]:
            dk[start:start + n], dv[start:start + n] = gk.transpose(0, 1), gv.transpose(0, 1)
        start += n
    return (o, lse, dq, dk, dv) if case["backward"] else (o, lse)


def _exact_loss(case, seed):
    s = prepare(case, seed)
    labels, T, n = s["labels"].long(), s["T"], s["n"]
    has = (labels >= 0) & (labels < s["V"])
    sample = torch.bucketize(torch.arange(T, device=labels.device), s["cu"][1:].long(), right=True)
    count = torch.zeros(n, dtype=torch.float64, device=labels.device).index_add_(0, sample, has.double())
    if case["normalizer"] == "token_mean":
        w = (1.0 / count.sum().clamp(min=1.0)).expand(T)
    elif case["normalizer"] == "sample_mean":
        w = (1.0 / (count.clamp(min=1.0) * n))[sample]
    else:
        w = torch.full((T,), 1.0 / (n * s["t_ave"]), dtype=torch.float64, device=labels.device)
    w = torch.where(has, w, torch.zeros_like(w))
    token_loss = torch.zeros(T, dtype=torch.float64, device=labels.device)
    grad = torch.empty(s["logits"].shape, dtype=torch.float64, device=labels.device) if case["grad"] else None
    for a in range(0, T, 512):
        rows = slice(a, min(a + 512, T))
        z = s["logits"][rows].double()
        lse, at = torch.logsumexp(z, dim=-1), labels[rows].clamp(0, s["V"] - 1)[:, None]
        token_loss[rows] = torch.where(has[rows], lse - z.gather(1, at)[:, 0], 0.0)
        if grad is not None:
            z.sub_(lse[:, None]).exp_().scatter_add_(1, at, torch.full_like(at, -1, dtype=torch.float64))
            grad[rows] = z.mul_(w[rows, None])
    loss = (w * token_loss).sum().reshape(1)
    return [loss, token_loss] + ([grad] if grad is not None else [])


def exact(case, seed):
    """What `run` gives for these inputs, in 64 bits and plain torch; None where that takes too long."""
    return (_exact_attention if case["kind"] == "attention" else _exact_loss)(case, seed)
