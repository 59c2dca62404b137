"""Work that programs hand to this library, as measurable cases.

A serving or RL-sampling program scores and pools the prompts it prefills: a lone prompt that
arrives online, a chunk of a running prefill, a batch of equal or log-uniform lengths, one very
long context.  It then predicts lengths with the small head, and trains that head on (pooled
vector, length) pairs.  The listed cases are those calls on the model shapes the library is built
for (Llama-3-8B-, Llama-3.2-1B- and Qwen2.5-1.5B-like), each through the public entry point;
``draw`` gives more of the same ranges.

A case is a dict of plain values.  ``kind`` names the call; batches are ``B`` prompts whose lengths
are spread evenly in the logarithm over [lo, hi] (equal lengths when lo == hi).
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2608_15592_amd as estp
from paper_2608_15592_amd.path import alloc_buffers

# hidden size, vocabulary, query heads, KV heads, head size
MODELS = {
    "llama-8b": (4096, 128256, 32, 8, 128),
    "llama-1b": (2048, 128256, 32, 8, 64),
    "qwen-1.5b": (1536, 151936, 12, 2, 128),
    "tiny": (64, 1000, 2, 2, 32),
}


def listed():
    return [
        # one short prompt arrives at an online scheduler: the whole path, latency counts
        {"name": "path_online", "kind": "path", "model": "llama-8b", "dtype": "bf16", "B": 1, "lo": 61, "hi": 61,
         "L": 1, "hidden": 1024, "bins": 16, "norm": "zscore"},
        # the smallest fp32 configuration: launches and host work are all there is
        {"name": "path_tiny_f32", "kind": "path", "model": "tiny", "dtype": "f32", "B": 1, "lo": 128, "hi": 128,
         "L": 1, "hidden": 32, "bins": 1, "norm": "none"},
        # one chunk of a chunked prefill
        {"name": "entropy_chunk", "kind": "entropy", "model": "llama-8b", "dtype": "bf16", "n_tok": 719,
         "mode": False},
        # a batch of 16 x 512 tokens, each token's most probable next token asked for as well
        {"name": "entropy_qwen_mode", "kind": "entropy", "model": "qwen-1.5b", "dtype": "bf16", "n_tok": 8192,
         "mode": True},
        # a full prefill batch of 32 x 2048 tokens: the largest call
        {"name": "entropy_llama", "kind": "entropy", "model": "llama-8b", "dtype": "bf16", "n_tok": 65536,
         "mode": False},
        # a burst of a few prompts of mixed length
        {"name": "importance_burst", "kind": "importance", "model": "qwen-1.5b", "B": 9, "lo": 45, "hi": 1021, "L": 1,
         "lse": False},
        # the full prefill batch, importance summed over the last four layers
        {"name": "importance_llama", "kind": "importance", "model": "llama-8b", "B": 32, "lo": 2048, "hi": 2048,
         "L": 4, "lse": False},
        # a ragged batch whose prefill attention already returned its row log-sum-exps
        {"name": "importance_lse_ragged", "kind": "importance", "model": "llama-1b", "B": 64, "lo": 32, "hi": 4096,
         "L": 2, "lse": True},
        # one long reasoning context
        {"name": "importance_long", "kind": "importance", "model": "llama-8b", "B": 1, "lo": 32768, "hi": 32768,
         "L": 1, "lse": False},
        # pooling of an RL sampling batch
        {"name": "pool_ragged", "kind": "pool", "dtype": "bf16", "d": 4096, "B": 256, "lo": 32, "hi": 4096,
         "norm": "zscore"},
        # lengths and the shortest-job-first order of that batch
        {"name": "predict_batch", "kind": "predict", "d": 4096, "hidden": 1024, "bins": 16, "B": 256},
        # one optimiser step of the head on a batch of pooled vectors
        {"name": "head_train", "kind": "train", "d": 4096, "hidden": 1024, "bins": 16, "B": 64},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _lengths_case(rng, lo, hi, b_hi, tok_hi):
    """Prompts between lo and hi, half the time of equal length, at most tok_hi tokens in all."""
    a, b = sorted((_log_int(rng, lo, hi), _log_int(rng, lo, hi)))
    if rng.random() < 0.5:
        a = b
    B = _log_int(rng, 1, b_hi)
    while B > 1 and int(_lengths(B, a, b).sum()) > tok_hi:
        B = B // 2
    return {"B": B, "lo": a, "hi": b}


def draw(rng):
    kind = rng.choice(["path", "entropy", "entropy", "importance", "importance", "pool", "predict", "train"])
    models = ["llama-8b", "llama-1b", "qwen-1.5b"]
    if kind == "path":
        tiny = rng.random() < 0.25
        case = {"kind": kind, "model": "tiny" if tiny else rng.choice(models), "dtype": "f32" if tiny else "bf16"}
        case.update(_lengths_case(rng, 7, 700, 8, 2048))
        case.update(L=rng.choice([1, 2, 4]), hidden=32 if tiny else rng.choice([256, 1024]),
                    bins=rng.choice([1, 16, 50]), norm=rng.choice(["none", "zscore", "minmax"]))
        return case
    if kind == "entropy":
        return {"kind": kind, "model": rng.choice(models), "dtype": "bf16", "n_tok": _log_int(rng, 5, 60000),
                "mode": rng.random() < 0.4}
    if kind == "importance":
        case = {"kind": kind, "model": rng.choice(models)}
        case.update(_lengths_case(rng, 32, 16384, 128, 65536))
        case.update(L=rng.choice([1, 1, 2, 4]), lse=rng.random() < 0.3)
        # the batch shrinks to the listed calls' work
        while case["B"] > 1 and work(case)["flops"] > 2.2e12:
            case["B"] = case["B"] // 2
        return case
    if kind == "pool":
        case = {"kind": kind, "dtype": rng.choice(["bf16", "bf16", "f32"]), "d": rng.choice([1536, 2048, 4096])}
        case.update(_lengths_case(rng, 32, 32768, 256, 131072))
        case.update(norm=rng.choice(["none", "zscore", "minmax"]))
        return case
    B = _log_int(rng, 1, 600)
    return {"kind": kind, "d": rng.choice([1536, 2048, 4096]), "hidden": rng.choice([256, 512, 1024]),
            "bins": rng.choice([1, 16, 50, 100] if kind == "predict" else [10, 16, 50, 100]), "B": B}


# ----------------------------------------------------------------------------- inputs


def _lengths(B, lo, hi):
    if lo == hi:
        return np.full(B, lo, dtype=np.int64)
    n = [int(round(lo * (hi / lo) ** ((i + 0.5) / B))) for i in range(B)]
    random.Random(B).shuffle(n)
    return np.asarray(n, dtype=np.int64)


def _cu(lengths):
    cu = np.zeros(len(lengths) + 1, dtype=np.int32)
    np.cumsum(lengths, out=cu[1:])
    return torch.from_numpy(cu).cuda()


def _dtype(case):
    return torch.float32 if case.get("dtype", "bf16") == "f32" else torch.bfloat16


def _hidden(g, n, d, dtype):
    """Final-layer hidden states after the norm: rows of RMS 1, 5% of them outliers of 4 times that."""
    out = torch.empty(n, d, dtype=dtype, device="cuda")
    for i in range(0, n, 16384):
        x = torch.randn(min(16384, n - i), d, generator=g, device="cuda")
        x *= torch.rsqrt(x.square().mean(dim=1, keepdim=True))
        x *= 1.0 + 3.0 * (torch.rand(x.shape[0], 1, generator=g, device="cuda") < 0.05)
        out[i:i + x.shape[0]] = x.to(dtype)
    return out


def _lm_head(g, V, d, dtype):
    out = torch.empty(V, d, dtype=dtype, device="cuda")
    for i in range(0, V, 16384):
        out[i:i + 16384] = (0.02 * torch.randn(min(16384, V - i), d, generator=g, device="cuda")).to(dtype)
    return out


def _qk(g, L, n, Hq, Hkv, dh, dtype):
    """Post-RoPE queries and keys; each (layer, query head) has a sharpness of its own in [0.5, 2]."""
    Q = torch.empty(L, n, Hq, dh, dtype=dtype, device="cuda")
    K = torch.empty(L, n, Hkv, dh, dtype=dtype, device="cuda")
    for l in range(L):
        sharp = 0.5 + 1.5 * torch.rand(Hq, 1, generator=g, device="cuda")
        for i in range(0, n, 16384):
            m = min(16384, n - i)
            Q[l, i:i + m] = (sharp * torch.randn(m, Hq, dh, generator=g, device="cuda")).to(dtype)
            K[l, i:i + m] = torch.randn(m, Hkv, dh, generator=g, device="cuda").to(dtype)
    return Q, K


def _head(g, d, hidden, bins):
    W1 = 0.02 * torch.randn(hidden, d, generator=g, device="cuda")
    b1 = 0.02 * torch.randn(hidden, generator=g, device="cuda")
    W2 = 0.02 * torch.randn(bins, hidden, generator=g, device="cuda")
    b2 = 0.02 * torch.randn(bins, generator=g, device="cuda")
    edges = torch.arange(bins + 1, dtype=torch.float32, device="cuda") * (4096.0 / bins)
    return W1, b1, W2, b2, edges, (edges[:-1] + edges[1:]) / 2


def _row_lse(Q, K, lengths):
    """Natural-log row normalisers [L, Hq, n_tok], as a prefill attention returns them."""
    L, n, Hq, dh = Q.shape
    Hkv, G = K.shape[2], Hq // K.shape[2]
    out = torch.empty(L, Hq, n, dtype=torch.float32, device="cuda")
    for l in range(L):
        at = 0
        for N in lengths.tolist():
            for h in range(Hkv):
                k = K[l, at:at + N, h].float().t().contiguous()
                for i in range(0, N, 2048):
                    m = min(2048, N - i)
                    q = Q[l, at + i:at + i + m, h * G:(h + 1) * G].float().reshape(m * G, dh)
                    s = (q @ k[:, :i + m]).view(m, G, i + m) / math.sqrt(dh)
                    later = torch.arange(i + m, device="cuda") > torch.arange(i, i + m, device="cuda")[:, None]
                    s.masked_fill_(later[:, None, :], -math.inf)
                    out[l, h * G:(h + 1) * G, at + i:at + i + m] = torch.logsumexp(s, dim=2).t()
            at += N
    return out


def prepare(case, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    kind = case["kind"]
    st = {"case": case}
    if kind in ("path", "importance", "pool"):
        lengths = _lengths(case["B"], case["lo"], case["hi"])
        n = int(lengths.sum())
        st.update(lengths=lengths, cu=_cu(lengths), max_seqlen=int(lengths.max()))
    if kind == "path":
        d, V, Hq, Hkv, dh = MODELS[case["model"]]
        dt = _dtype(case)
        st["X"] = _hidden(g, n, d, dt)
        st["W"] = _lm_head(g, V, d, dt)
        st["Q"], st["K"] = _qk(g, case["L"], n, Hq, Hkv, dh, dt)
        W1, b1, W2, b2, _, centres = _head(g, d, case["hidden"], case["bins"])
        st["head"] = (W1, b1, W2, b2, centres)
        st["bufs"] = alloc_buffers(n, case["B"], st["max_seqlen"], d, V, case["L"], Hq, Hkv, dh, case["hidden"],
                                   case["bins"], "cuda", dt)
    elif kind == "entropy":
        d, V = MODELS[case["model"]][:2]
        st["X"] = _hidden(g, case["n_tok"], d, _dtype(case))
        st["W"] = _lm_head(g, V, d, _dtype(case))
        st["mode"] = torch.empty(case["n_tok"], dtype=torch.int32, device="cuda") if case["mode"] else None
    elif kind == "importance":
        Hq, Hkv, dh = MODELS[case["model"]][2:]
        st["Q"], st["K"] = _qk(g, case["L"], n, Hq, Hkv, dh, torch.bfloat16)
        st["lse"] = _row_lse(st["Q"], st["K"], lengths) if case["lse"] else None
    elif kind == "pool":
        st["X"] = _hidden(g, n, case["d"], _dtype(case))
        # importance of mean 1/N with a heavy tail, entropy of a few nats
        s = -torch.log(1.0 - torch.rand(n, generator=g, device="cuda"))
        st["S"] = s / torch.repeat_interleave(torch.from_numpy(lengths).cuda(), torch.from_numpy(lengths).cuda())
        st["H"] = 11.0 * torch.rand(n, generator=g, device="cuda").sqrt()
    else:
        st["pooled"] = torch.randn(case["B"], case["d"], generator=g, device="cuda") / 8.0
        W1, b1, W2, b2, edges, centres = _head(g, case["d"], case["hidden"], case["bins"])
        if kind == "predict":
            st["head"] = (W1, b1, W2, b2, centres)
        else:  # in the middle of training: moments of earlier steps' size
            st.update(edges=edges, centres=centres, y=4096.0 * torch.rand(case["B"], generator=g, device="cuda"))
            st["theta"] = torch.cat([W1.flatten(), b1, W2.flatten(), b2])
            st["m"] = 10.0 * torch.randn(st["theta"].numel(), generator=g, device="cuda")
            st["v"] = 100.0 + 900.0 * torch.rand(st["theta"].numel(), generator=g, device="cuda")
    return st


LAMBDA1, LAMBDA2, ALPHA = 0.5, 0.5, 1.0
TRAIN = {"step": 100, "lambda3": 0.5, "lr": 1e-3}


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "path":
        out = estp.run_path(st["X"], st["W"], st["Q"], st["K"], st["cu"], st["max_seqlen"], LAMBDA1, LAMBDA2, ALPHA,
                            case["norm"], head=st["head"], bufs=st["bufs"])
        return {k: v for k, v in out.items() if v is not None}
    if kind == "entropy":
        H = estp.token_entropy(st["X"], st["W"], vocab_argmax=st["mode"])
        return {"H": H} if st["mode"] is None else {"H": H, "vocab_argmax": st["mode"]}
    if kind == "importance":
        if st["lse"] is not None:
            return estp.attn_importance_from_lse(st["Q"], st["K"], st["lse"], st["cu"], st["max_seqlen"])
        return estp.attn_importance(st["Q"], st["K"], st["cu"], st["max_seqlen"])
    if kind == "pool":
        pooled, e, top = estp.combine_pool(st["X"], st["S"], st["H"], st["cu"], st["max_seqlen"], LAMBDA1, LAMBDA2,
                                           ALPHA, case["norm"])
        return {"pooled": pooled, "e": e, "top": top}
    if kind == "predict":
        yhat, bins, order = estp.predict(st["pooled"], *st["head"])
        return {"yhat": yhat, "order": order} if bins is None else {"yhat": yhat, "bin": bins, "order": order}
    loss = estp.head_train_step(st["pooled"], st["y"], st["edges"], st["centres"], st["theta"], st["m"], st["v"],
                                hidden=case["hidden"], **TRAIN)
    return {"loss": loss, "theta": st["theta"], "m": st["m"], "v": st["v"]}


# ----------------------------------------------------------------------------- what a pass cannot do without


def work(case):
    kind = case["kind"]
    if kind in ("path", "importance", "pool"):
        lengths = _lengths(case["B"], case["lo"], case["hi"])
        n, pairs = int(lengths.sum()), int((lengths * (lengths + 1) // 2).sum())
    if kind == "entropy":
        d, V = MODELS[case["model"]][:2]
        n = case["n_tok"]
        return {"bytes": 2 * (n + V) * d + 4 * n * (2 if case["mode"] else 1), "flops": 2 * n * V * d}
    if kind == "importance":
        Hq, Hkv, dh = MODELS[case["model"]][2:]
        return {"bytes": case["L"] * n * (2 * (Hq + Hkv) * dh + (4 * Hq if case["lse"] else 0)) + 4 * n,
                "flops": 2 * dh * Hq * case["L"] * pairs}
    if kind == "pool":
        es = 4 if case["dtype"] == "f32" else 2
        return {"bytes": n * case["d"] * es + 12 * n + 4 * case["B"] * case["d"], "flops": 2 * n * case["d"]}
    B, hidden, K = case["B"], case["hidden"], case["bins"]
    if kind == "path":
        d, V, Hq, Hkv, dh = MODELS[case["model"]]
        es = 4 if case["dtype"] == "f32" else 2
        head = hidden * (d + 1) + K * (hidden + 1)
        return {"bytes": es * ((n + V) * d + case["L"] * n * (Hq + Hkv) * dh) + 12 * n + 4 * (B * d + head),
                "flops": 2 * n * V * d + 2 * dh * Hq * case["L"] * pairs + 2 * n * d + 2 * B * head}
    d = case["d"]
    head = hidden * (d + 1) + K * (hidden + 1)
    if kind == "predict":
        return {"bytes": 4 * (B * d + head + 3 * B), "flops": 2 * B * head}
    return {"bytes": 4 * (B * d + 6 * head + B), "flops": 2 * B * (2 * head + K * hidden) + 10 * head}


def tolerance(case):
    """Inputs may be bf16, but every product and sum is 32-bit: about four times the distance from the
    64-bit values that the library's calls show (another order of those sums shows as much)."""
    kind = case["kind"]
    if kind == "path":  # errors of the scores travel into the weights and the pooled vectors
        return {"rel": 2e-6, "max": 1e-4, "differ": 0.02}
    if kind == "entropy":  # logits that tie within their rounding may change the mode
        return {"rel": 8e-7, "max": 1e-5, "differ": 1e-3}
    if kind == "importance":
        return {"rel": 1.2e-6, "max": 1e-4}
    if kind == "pool":
        return {"rel": 1.5e-6, "max": 1e-4, "differ": 0.02}
    if kind == "predict":  # neighbours in the order whose lengths agree to the last bits may swap
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.02}
    return {"rel": 2e-6, "max": 1e-4}


# ----------------------------------------------------------------------------- 64-bit values


def _entropy64(X, W):
    W = W.double().t().contiguous()
    H = torch.empty(X.shape[0], dtype=torch.float64, device="cuda")
    mode = torch.empty(X.shape[0], dtype=torch.int64, device="cuda")
    for i in range(0, X.shape[0], 2048):
        z = X[i:i + 2048].double() @ W
        mode[i:i + 2048] = z.argmax(dim=1)
        z -= z.logsumexp(dim=1, keepdim=True)
        H[i:i + 2048] = -(z * z.exp()).sum(dim=1)
    return H, mode


def _importance64(Q, K, lengths, lse):
    L, n, Hq, dh = Q.shape
    Hkv, G = K.shape[2], Hq // K.shape[2]
    S = torch.zeros(n, dtype=torch.float64, device="cuda")
    for l in range(L):
        at = 0
        for N in lengths.tolist():
            for h in range(Hkv):
                k = K[l, at:at + N, h].double().t().contiguous()
                for i in range(0, N, 1024):
                    m = min(1024, N - i)
                    q = Q[l, at + i:at + i + m, h * G:(h + 1) * G].double().reshape(m * G, dh)
                    s = (q @ k[:, :i + m]).view(m, G, i + m) / math.sqrt(dh)
                    later = torch.arange(i + m, device="cuda") > torch.arange(i, i + m, device="cuda")[:, None]
                    s.masked_fill_(later[:, None, :], -math.inf)
                    if lse is None:
                        s -= torch.logsumexp(s, dim=2, keepdim=True)
                    else:
                        s -= lse[l, h * G:(h + 1) * G, at + i:at + i + m].t().double()[:, :, None]
                    S[at:at + i + m] += s.exp_().sum(dim=(0, 1)) / (N * Hq)
            at += N
    return S


def _pool64(X, S, H, lengths, norm):
    pooled = torch.empty(len(lengths), X.shape[1], dtype=torch.float64, device="cuda")
    e = torch.empty(X.shape[0], dtype=torch.float64, device="cuda")
    top = torch.empty(len(lengths), dtype=torch.int64, device="cuda")
    at = 0
    for b, N in enumerate(lengths.tolist()):
        s, h = S[at:at + N].double(), H[at:at + N].double()
        if norm == "zscore":
            s, h = ((v - v.mean()) / (v.std(correction=0) + 1e-6) for v in (s, h))
        elif norm == "minmax":
            s, h = ((v - v.min()) / (v.max() - v.min() + 1e-6) for v in (s, h))
        w = torch.softmax((LAMBDA1 * s + LAMBDA2 * h) / ALPHA, dim=0)
        e[at:at + N] = w
        top[b] = at + w.argmax()
        pooled[b] = w @ X[at:at + N].double()
        at += N
    return pooled, e, top


def _predict64(pooled, W1, b1, W2, b2, centres):
    o = torch.relu(pooled.double() @ W1.double().t() + b1.double()) @ W2.double().t() + b2.double()
    if W2.shape[0] == 1:
        y, bins = o[:, 0], None
    else:
        y, bins = torch.softmax(o, dim=1) @ centres.double(), o.argmax(dim=1)
    return y, bins, torch.sort(y, stable=True).indices


def _train64(st, case):
    d, hidden, K, B = case["d"], case["hidden"], case["bins"], case["B"]
    th = st["theta"].double()
    n1 = hidden * d
    W1, b1 = th[:n1].view(hidden, d), th[n1:n1 + hidden]
    W2, b2 = th[n1 + hidden:n1 + hidden + K * hidden].view(K, hidden), th[n1 + hidden + K * hidden:]
    x, y, c = st["pooled"].double(), st["y"].double(), st["centres"].double()
    z = x @ W1.t() + b1
    a = torch.relu(z)
    logp = torch.log_softmax(a @ W2.t() + b2, dim=1)
    p = logp.exp()
    yhat = p @ c
    k = torch.arange(K, device="cuda")
    i = (st["edges"][1:K].double()[None, :] <= y[:, None]).sum(dim=1)
    lab = torch.softmax(-(k[None, :] - i[:, None]).abs().double(), dim=1)
    lam, r = TRAIN["lambda3"], y - yhat
    loss = lam * -(lab * logp).sum(dim=1).mean() + (1.0 - lam) * r.square().mean()
    dO = (lam * (p - lab) - 2.0 * (1.0 - lam) * r[:, None] * p * (c[None, :] - yhat[:, None])) / B
    dZ = (dO @ W2) * (z > 0)
    g = torch.cat([(dZ.t() @ x).flatten(), dZ.sum(dim=0), (dO.t() @ a).flatten(), dO.sum(dim=0)])
    # the library takes its hyperparameters as 32-bit floats
    b1_, b2_, eps, wd, lr = (float(np.float32(h)) for h in (0.9, 0.999, 1e-8, 0.01, TRAIN["lr"]))
    t = TRAIN["step"]
    m = b1_ * st["m"].double() + (1.0 - b1_) * g
    v = b2_ * st["v"].double() + (1.0 - b2_) * g * g
    th = th * (1.0 - lr * wd) - lr * (m / (1.0 - b1_ ** t)) / ((v / (1.0 - b2_ ** t)).sqrt() + eps)
    return {"loss": loss.reshape(1), "theta": th, "m": m, "v": v}


def exact(case, seed):
    st = prepare(case, seed)
    kind = case["kind"]
    if kind == "path":
        H = _entropy64(st["X"], st["W"])[0]
        S = _importance64(st["Q"], st["K"], st["lengths"], None)
        pooled, e, top = _pool64(st["X"], S, H, st["lengths"], case["norm"])
        y, bins, order = _predict64(pooled, *st["head"])
        out = {"H": H, "S": S, "pooled": pooled, "e": e, "top": top, "yhat": y, "bin": bins, "order": order}
        return {k: v for k, v in out.items() if v is not None}
    if kind == "entropy":
        H, mode = _entropy64(st["X"], st["W"])
        return {"H": H, "vocab_argmax": mode} if case["mode"] else {"H": H}
    if kind == "importance":
        return _importance64(st["Q"], st["K"], st["lengths"], st["lse"])
    if kind == "pool":
        pooled, e, top = _pool64(st["X"], st["S"], st["H"], st["lengths"], case["norm"])
        return {"pooled": pooled, "e": e, "top": top}
    if kind == "predict":
        y, bins, order = _predict64(st["pooled"], *st["head"])
        return {"yhat": y, "order": order} if bins is None else {"yhat": y, "bin": bins, "order": order}
    return _train64(st, case)
