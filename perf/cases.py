"""The work that the retrieval index is used for, as cases that can be timed.

Shapes are the ones of ``workloads`` (LLaMA-3.1-8B- and Qwen2.5-7B-shaped
layers, long-context decode) and ragged ones around them.  Inputs follow the
same score model, drawn on the GPU: latent tokens with a power-law spectrum and
a few outlier coordinates, projected to keys, queries and values.  The factors
a program keeps come from float64 linear algebra here, so that a case measures
one call and not the ones before it.

Kinds of case ("do"):
  step       one decode step: append the newest key's codes, score and select
             over the whole cache, attention over each row's list
  score      saki_score_topk: decode (few queries), batched decode, prefill
  attend     saki_attend over lists that are at hand
  build      saki_build_index over the whole cache
  recall     saki_recall of lists that are at hand
  calibrate  moments on the GPU, factors on the host, factors back on the GPU
"""
from __future__ import annotations

import numpy as np
import torch

from paper_2608_03228_amd import saki as S

D_HEAD = 128   # head dimension of every configuration
LATENT = 512
THETA = 500000.0
DEV = "cuda"
_ES = {"f32": 4, "bf16": 2, "fp8": 1}


# ---------------------------------------------------------------- the cases

def _case(do, **kw):
    c = {"do": do, "B": 1, "layers": 1, "H_q": 32, "H_kv": 8, "N": 4096, "cap": 0, "Q": 1,
         "q_start": -1, "r": 32, "sketch": "bf16", "keys": "f32", "shared": False, "k": 64,
         "recon": False, "want_exact": False, "T": 512}
    c.update(kw)
    c["cap"] = max(c["cap"], c["N"])
    return c


def listed():
    return [
        # a decode step early in a conversation: short ragged cache, latency counts
        _case("step", name="decode_step_4k", N=4001, cap=8192),
        # batched decode with the smallest index: one fp8 code set per KV head,
        # bf16 key cache, the selected keys reconstructed from their codes
        _case("step", name="decode_step_shared_fp8", B=4, N=100003, cap=131072, sketch="fp8",
              keys="bf16", shared=True, recon=True),
        # long-context decode: one query per head over 2^20 keys
        _case("score", name="decode_1m", N=1 << 20),
        # Qwen-shaped batched decode: 8 sequences, 16 queries per head
        _case("score", name="decode_batch_131k", B=8, H_q=28, H_kv=4, N=131072, Q=16),
        # prefill of one LLaMA-shaped layer, causal rows 64 .. 4095
        _case("score", name="prefill_layer", Q=4032, q_start=64),
        # the same for all 32 layers in one call
        _case("score", name="prefill_sweep", layers=32, Q=4032, q_start=64),
        # a second part of a ragged prompt, float32 codes at rank 64
        _case("score", name="prefill_ragged_f32", B=2, H_q=8, H_kv=2, N=2777, Q=2477, q_start=300,
              r=64, sketch="f32"),
        # attention of a layer's prefill rows over their selected keys
        _case("attend", name="attend_prefill", Q=4032, q_start=64),
        # index of a batch of long prompts
        _case("build", name="build_batch_131k", B=8, H_q=28, H_kv=4, N=131072),
        # quality of an index over a layer's prefill rows
        _case("recall", name="recall_layer", Q=4032, q_start=64),
        # quality of a long-context decode step
        _case("recall", name="recall_decode_1m", N=1 << 20),
        # calibration of one layer
        _case("calibrate", name="calibrate_layer"),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    H_q, H_kv = rng.choice([(32, 8), (28, 4), (8, 2), (16, 16), (8, 1)])
    do = rng.choice(["step", "step", "score_decode", "score_batch", "score_prefill",
                     "score_prefill", "attend", "build", "recall_prefill", "recall_decode",
                     "calibrate"])
    sketch = rng.choice(["bf16", "bf16", "fp8", "f32"])
    r = rng.choice([16, 32, 32, 64, 128])
    keys = rng.choice(["f32", "bf16"])
    k = rng.choice([64, 64, 64, 32, 10])
    heads = dict(H_q=H_q, H_kv=H_kv)
    if do in ("step", "score_decode"):
        B = rng.choice([1, 1, 2, 4, 8])
        N = _log(rng, 300, (1 << 19) // B)
        return _case(do.split("_")[0], B=B, **heads, N=N, cap=N + rng.choice([0, 1, 500, N // 3]),
                     Q=rng.choice([1, 1, 1, 2, 5]), r=r, sketch=sketch, keys=keys, k=k,
                     shared=rng.random() < 0.4, recon=rng.random() < 0.3)
    if do == "score_batch":
        B = rng.choice([1, 2, 4, 8])
        N = _log(rng, 16384, 131072)
        return _case("score", B=B, **heads, N=N, Q=_log(rng, 16, 64), r=r, sketch=sketch, k=k)
    if do == "score_prefill":
        B = rng.choice([1, 1, 2, 4])
        N = _log(rng, 80, 8192)
        causal = rng.random() < 0.75
        start = rng.randrange(0, N // 2) if causal else -1
        Q = N - start if causal else _log(rng, 16, 2048)
        return _case("score", B=B, **heads, N=N, Q=Q, q_start=start, r=r, sketch=sketch, k=k,
                     shared=rng.random() < 0.25)
    if do == "attend":
        N = _log(rng, 200, 8192)
        start = rng.randrange(0, N // 2)
        return _case("attend", B=rng.choice([1, 1, 2]), **heads, N=N, Q=N - start, q_start=start,
                     r=r, sketch=sketch, keys=keys, k=k, recon=rng.random() < 0.4)
    if do == "build":
        B = rng.choice([1, 2, 4])
        return _case("build", B=B, **heads, N=_log(rng, 300, (1 << 18) // B), r=r, sketch=sketch,
                     keys=keys, shared=rng.random() < 0.3)
    if do == "recall_prefill":
        N = _log(rng, 100, 6000)
        start = rng.randrange(0, N // 2)
        return _case("recall", B=rng.choice([1, 1, 2]), **heads, N=N, Q=N - start, q_start=start,
                     keys=keys, k=k, want_exact=rng.random() < 0.3)
    if do == "recall_decode":
        B = rng.choice([1, 2, 4])
        return _case("recall", B=B, **heads, N=_log(rng, 1000, (1 << 18) // B),
                     Q=rng.choice([1, 2, 16]), keys=keys, k=k, want_exact=rng.random() < 0.5)
    return _case("calibrate", **heads, T=_log(rng, 256, 2048), r=r)


# ---------------------------------------------------------------- inputs

def _weights(g, heads):
    col = torch.arange(1, LATENT + 1, device=DEV, dtype=torch.float32) ** -0.5
    return torch.randn((heads * D_HEAD, LATENT), generator=g, device=DEV) * col


def _project(x, w):  # [n, LATENT] x [heads * d, LATENT] -> [heads, n, d]
    return (x @ w.T).view(x.shape[0], -1, D_HEAD).transpose(0, 1)


def _inputs(c, seed, values=False):
    """Keys [B, layers * H_kv, cap, d], queries [B, layers * H_q, Q, d], q_pos,
    calibration tokens of one layer's heads (the layers of a call share the
    projections and have tokens of their own)."""
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * seed + 17)
    L, H_q, H_kv, N, Q = c["layers"], c["H_q"], c["H_kv"], c["N"], c["Q"]
    std = torch.arange(1, LATENT + 1, device=DEV, dtype=torch.float32) ** -0.5
    out = torch.randperm(LATENT, generator=g, device=DEV)[:4]
    std[out] *= 20.0
    wq, wk, wv = (_weights(g, h) for h in (H_q, H_kv, H_kv))

    def tokens(n):
        return torch.randn((n, LATENT), generator=g, device=DEV) * std

    kt = torch.bfloat16 if c["keys"] == "bf16" else torch.float32
    s = {}
    xc = tokens(c["T"])
    # queries scaled so that the logits spread as attention's do (softmax
    # weights over many of a list's keys); which keys are selected does not change
    wq *= 4.0 * D_HEAD ** 0.5 / (_project(xc, wq)[0] @ _project(xc, wk)[0].T).std()
    s["q_cal"], s["k_cal"] = _project(xc, wq).contiguous(), _project(xc, wk).contiguous()
    if c["do"] == "calibrate":
        return s
    keys = torch.zeros((c["B"], L * H_kv, c["cap"], D_HEAD), dtype=kt, device=DEV)
    q = torch.empty((c["B"], L * H_q, Q, D_HEAD), device=DEV)
    vals = torch.zeros((c["B"], L * H_kv, c["cap"], D_HEAD), device=DEV) if values else None
    for b in range(c["B"]):
        for layer in range(L):
            kv = slice(layer * H_kv, (layer + 1) * H_kv)
            for n0 in range(0, N, 65536):
                n1 = min(N, n0 + 65536)
                x = tokens(n1 - n0)
                keys[b, kv, n0:n1] = _project(x, wk).to(kt)
                if values:
                    vals[b, kv, n0:n1] = _project(x, wv)
                if c["q_start"] >= 0 and n1 > c["q_start"]:  # the sequence's own tokens
                    m = max(n0, c["q_start"])
                    q[b, layer * H_q:(layer + 1) * H_q, m - c["q_start"]:n1 - c["q_start"]] = \
                        _project(x[m - n0:], wq)
            if c["q_start"] < 0:  # fresh tokens that see the whole cache
                q[b, layer * H_q:(layer + 1) * H_q] = _project(tokens(Q), wq)
    s.update(keys=keys, q=q, values=vals)
    s["q_pos"] = (torch.arange(c["q_start"], c["q_start"] + Q, dtype=torch.int32, device=DEV)
                  if c["q_start"] >= 0 else None)
    return s


def _factors64(q_cal, k_cal, r, shared):
    """B_q, B_k [H_q (or H_kv), d, r] and mu [H_kv, d] in float64 (host): with
    Sigma_k = L L^T and the eigenvectors V, values s^2 of L^T Sigma_q L,
    B_q = L V_r s^-1/2 and B_k = L^-T V_r s^1/2, the largest entry of each
    B_k column positive."""
    q, k = q_cal.double().cpu().numpy(), k_cal.double().cpu().numpy()
    H_q, T, _ = q.shape
    H_kv = k.shape[0]
    G = H_q // H_kv
    mu = k.mean(axis=1)
    Bq, Bk = [], []
    for g in range(H_kv):
        kc = k[g] - mu[g]
        Lk = np.linalg.cholesky(kc.T @ kc / T)
        sq = [q[h].T @ q[h] / T for h in range(g * G, (g + 1) * G)]
        for m in [sum(sq) / G] if shared else sq:
            w, V = np.linalg.eigh(Lk.T @ m @ Lk)
            V, s = V[:, ::-1][:, :r], np.sqrt(w[::-1][:r])
            bq, bk = Lk @ V / np.sqrt(s), np.linalg.solve(Lk.T, V) * np.sqrt(s)
            sign = np.sign(bk[np.abs(bk).argmax(axis=0), np.arange(r)])
            Bq.append(bq * sign)
            Bk.append(bk * sign)
    return np.stack(Bq), np.stack(Bk), mu


def _with_factors(c, s):
    Bq, Bk, mu = _factors64(s["q_cal"], s["k_cal"], c["r"], c["shared"])
    G = c["H_q"] // c["H_kv"]
    s["B_k"] = torch.from_numpy(np.tile(Bk.astype(np.float32), (c["layers"], 1, 1))).to(DEV)
    s["B_q"] = torch.from_numpy(np.tile(np.repeat(Bq, G if c["shared"] else 1, axis=0).astype(np.float32),
                                        (c["layers"], 1, 1))).to(DEV)
    s["mu"] = torch.from_numpy(np.tile(mu.astype(np.float32), (c["layers"], 1))).to(DEV)
    return s


def _heads(c):
    H_q, H_kv = c["layers"] * c["H_q"], c["layers"] * c["H_kv"]
    return H_q, H_kv, H_kv if c["shared"] else H_q  # query heads, KV heads, code sets


def _kv(c, h):
    return h // (c["H_q"] // c["H_kv"])


def _visible(c, s):
    """Keys each query row sees, as a limit per row."""
    if s["q_pos"] is None:
        return torch.full((c["Q"],), c["N"], device=DEV)
    return s["q_pos"].long() + 1


def _lists(c, s):
    """Lists [B, H_q, Q, k] as an index finds them (float32 products of the
    factors), the best first, -1 past a row's keys."""
    H_q, _, _ = _heads(c)
    out = torch.full((c["B"], H_q, c["Q"], c["k"]), -1, dtype=torch.int32, device=DEV)
    lim = _visible(c, s)
    j = torch.arange(c["N"], device=DEV)
    m = min(c["k"], c["N"])
    step = max(1, (1 << 28) // c["N"])
    for b in range(c["B"]):
        for h in range(H_q):
            g = _kv(c, h)
            hk = g if c["shared"] else h
            kc = s["keys"][b, g, :c["N"]].float() - s["mu"][g]
            w = s["q"][b, h] @ s["B_q"][h] @ s["B_k"][hk].T
            for i in range(0, c["Q"], step):
                sc = w[i:i + step] @ kc.T
                if s["q_pos"] is not None:
                    sc.masked_fill_(j[None] >= lim[i:i + step, None], -float("inf"))
                v, x = sc.topk(m, dim=1)
                out[b, h, i:i + step, :m] = torch.where(v == -float("inf"), -1, x).int()
    return out


def prepare(c, seed):
    do = c["do"]
    s = _inputs(c, seed, values=do in ("step", "attend"))
    s["case"] = c
    if do == "calibrate":
        H_q, H_kv = c["H_q"], c["H_kv"]
        s["moments"] = [torch.empty(n, dtype=torch.float64, device=DEV) for n in
                        ((H_q, D_HEAD, D_HEAD), (H_kv, D_HEAD, D_HEAD), (H_kv, D_HEAD))]
        s["host"] = [torch.empty(m.shape, dtype=torch.float64).pin_memory() for m in s["moments"]]
        return s
    _with_factors(c, s)
    H_q, H_kv, sets = _heads(c)
    B, N, cap, Q, r, k, sk = (c[x] for x in ("B", "N", "cap", "Q", "r", "k", "sketch"))
    if do in ("step", "score", "build") or c["recon"]:
        s["index"] = torch.zeros(S.saki_index_bytes(B, sets, cap, r, sk), dtype=torch.uint8, device=DEV)
        if do != "build":  # codes of the cached keys; a step appends the last one
            n = N - 1 if do == "step" else N
            S.saki_build_index(s["keys"], s["B_k"], s["mu"], r, sk, sets, index=s["index"],
                               n_begin=0, n_count=n)
    if do in ("step", "score"):
        s["ws"] = torch.empty(S.saki_score_topk_workspace_bytes(B, H_q, Q, N, r, k, sk, sets),
                              dtype=torch.uint8, device=DEV)
        s["top_idx"] = torch.empty((B, H_q, Q, k), dtype=torch.int32, device=DEV)
        s["top_score"] = torch.empty((B, H_q, Q, k), device=DEV)
    if do in ("attend", "recall"):
        s["top_idx"] = _lists(c, s)
    if do in ("step", "attend"):
        s["out"] = torch.empty((B, H_q, Q, D_HEAD), device=DEV)
    if do == "recall":
        s["ws"] = torch.empty(max(1, S.saki_recall_workspace_bytes(B, H_q, H_kv, Q, N, D_HEAD, k)),
                              dtype=torch.uint8, device=DEV)
        s["hits"] = torch.empty((B, H_q, Q), dtype=torch.int32, device=DEV)
        s["exact_idx"] = (torch.empty((B, H_q, Q, k), dtype=torch.int32, device=DEV)
                          if c["want_exact"] else None)
    return s


# ---------------------------------------------------------------- one pass

def _codes(c, index):
    """The index buffer as its values (fp8 codes as bytes)."""
    return index if c["sketch"] == "fp8" else index.view(
        torch.bfloat16 if c["sketch"] == "bf16" else torch.float32)


def _score(c, s):
    _, H_kv, sets = _heads(c)
    return S.saki_score_topk(s["index"], c["sketch"], s["q"], s["B_q"], s["mu"], H_kv, c["cap"],
                             c["N"], c["r"], q_pos=s["q_pos"], k=c["k"], ws=s["ws"],
                             top_idx=s["top_idx"], top_score=s["top_score"], index_heads=sets)


def _attend(c, s):
    H_q, _, _ = _heads(c)
    _, _, sets = _heads(c)
    if c["recon"]:
        return S.saki_attend(s["values"], s["q"], s["top_idx"], c["N"], index=s["index"],
                             sketch=c["sketch"], B_q=s["B_q"], mu=s["mu"], r=c["r"],
                             index_heads=sets, q_pos=s["q_pos"], rope_theta=THETA, out=s["out"])
    return S.saki_attend(s["values"], s["q"], s["top_idx"], c["N"], keys=s["keys"],
                         q_pos=s["q_pos"], rope_theta=THETA, out=s["out"])


def run(s):
    c = s["case"]
    do = c["do"]
    if do == "calibrate":
        S.saki_calibration_moments(s["q_cal"], s["k_cal"], *s["moments"])
        for h, m in zip(s["host"], s["moments"]):
            h.copy_(m, non_blocking=True)
        torch.cuda.current_stream().synchronize()  # the factorisation reads them
        f = S.saki_calibrate_from_moments(*(h.numpy() for h in s["host"]), c["r"], with_sigma=False)
        return [torch.from_numpy(f[x]).to(DEV) for x in ("B_q", "B_k", "mu")]
    _, _, sets = _heads(c)
    if do == "build":
        S.saki_build_index(s["keys"], s["B_k"], s["mu"], c["r"], c["sketch"], sets, index=s["index"],
                           n_begin=0, n_count=c["N"])
        return _codes(c, s["index"])
    if do == "step":
        S.saki_build_index(s["keys"], s["B_k"], s["mu"], c["r"], c["sketch"], sets, index=s["index"],
                           n_begin=c["N"] - 1, n_count=1)
        idx, sc = _score(c, s)
        return {"idx": idx, "score": sc, "out": _attend(c, s), "codes": _codes(c, s["index"])}
    if do == "score":
        idx, sc = _score(c, s)
        return {"idx": idx, "score": sc}
    if do == "attend":
        return _attend(c, s)
    hits, exact_idx = S.saki_recall(s["keys"], s["q"], s["top_idx"], c["N"], q_pos=s["q_pos"],
                                    k=c["k"], ws=s["ws"], hits=s["hits"], exact_idx=s["exact_idx"],
                                    want_exact=c["want_exact"])
    return {"hits": hits, "exact_idx": exact_idx} if c["want_exact"] else hits


# ---------------------------------------------------------------- what a pass cannot do without

def work(c):
    H_q, H_kv, sets = _heads(c)
    B, N, Q, r, k, T = (c[x] for x in ("B", "N", "Q", "r", "k", "T"))
    es, kb, d = _ES[c["sketch"]], 2 if c["keys"] == "bf16" else 4, D_HEAD
    rows = B * H_q * Q
    if c["q_start"] >= 0:
        pairs = B * H_q * sum(min(N, c["q_start"] + i + 1) for i in range(Q))
    else:
        pairs = rows * N
    lists, factors = rows * k * 4, H_q * d * r * 4 + H_kv * d * 4
    code = B * sets * N * r * es
    queries = rows * d * 4
    score = {"bytes": code + queries + factors + 2 * lists, "flops": 2 * r * pairs + 2 * d * r * rows}
    # a selected key and value of every row, each read once however many rows share it
    picked = min(rows * k, B * H_kv * N)
    att_key = picked * (r * es if c["recon"] else d * kb)
    att = {"bytes": att_key + picked * d * 4 + 2 * queries + lists, "flops": 4 * d * rows * k}
    if c["do"] == "score":
        return score
    if c["do"] == "attend":
        return att
    if c["do"] == "step":
        return {"bytes": score["bytes"] + att["bytes"] + B * H_kv * d * kb + B * sets * r * es,
                "flops": score["flops"] + att["flops"] + 2 * d * r * B * sets}
    if c["do"] == "build":
        return {"bytes": B * H_kv * N * d * kb + code + sets * d * r * 4 + H_kv * d * 4,
                "flops": 2 * d * r * B * sets * N}
    if c["do"] == "recall":
        return {"bytes": B * H_kv * N * d * kb + queries + lists * (2 if c["want_exact"] else 1) + rows * 4,
                "flops": 2 * d * pairs}
    return {"bytes": (H_q + H_kv) * T * d * 4 + (H_q + H_kv) * d * d * 8 + factors + H_q * d * r * 4,
            "flops": 2 * d * d * T * (H_q + H_kv) + H_q * 10 * d ** 3}


def tolerance(c):
    """About four times what float32 sums in another order were measured to
    change (64-bit sums over operands rounded as they are stored)."""
    if c["do"] == "build":  # a code near a rounding midpoint may round away: one step of its type
        return {"f32": {"rel": 4e-7, "max": 1.2e-5}, "bf16": {"rel": 6e-5, "max": 3e-2},
                "fp8": {"rel": 0.0, "differ": 5e-5}}[c["sketch"]]
    if c["do"] == "recall":  # decided exactly
        return "exact"
    if c["do"] == "calibrate":  # eigenvectors of close eigenvalues turn with the rounding
        return {"rel": 1e-6, "max": 1e-4}
    if c["do"] == "attend":
        return {"rel": 2e-5, "max": 2e-3}
    if c["do"] == "step":  # a list that ends with another key changes its whole output row
        return {"rel": 1e-2, "max": 0.2, "differ": 5e-3}
    if c["sketch"] == "f32":  # near ties change places
        return {"rel": 1e-6, "max": 6e-6, "differ": 1e-3}
    # an element of the query sketch near a midpoint of bf16 may round away
    return {"rel": 2.4e-4, "max": 2.4e-2, "differ": 3e-3}


# ---------------------------------------------------------------- the same in 64 bits

def _rope64(x, pos):
    half = D_HEAD // 2
    inv = THETA ** (-2.0 * torch.arange(half, dtype=torch.float64, device=DEV) / D_HEAD)
    a = pos.double()[..., None] * inv
    co, si = torch.cos(a), torch.sin(a)
    return torch.cat([x[..., :half] * co - x[..., half:] * si,
                      x[..., half:] * co + x[..., :half] * si], dim=-1)


def _exact_score(c, s):
    H_q, _, _ = _heads(c)
    idx = torch.full((c["B"], H_q, c["Q"], c["k"]), -1, dtype=torch.int32, device=DEV)
    val = torch.full((c["B"], H_q, c["Q"], c["k"]), -float("inf"), dtype=torch.float64, device=DEV)
    lim = _visible(c, s)
    j = torch.arange(c["N"], device=DEV)
    m = min(c["k"], c["N"])
    step = max(1, (1 << 27) // c["N"])
    for b in range(c["B"]):
        for h in range(H_q):
            g = _kv(c, h)
            hk = g if c["shared"] else h
            mu = s["mu"][g].double()
            codes = (s["keys"][b, g, :c["N"]].double() - mu) @ s["B_k"][hk].double()
            q = s["q"][b, h].double()
            z, bb = q @ s["B_q"][h].double(), q @ mu
            for i in range(0, c["Q"], step):
                sc = z[i:i + step] @ codes.T + bb[i:i + step, None]
                if s["q_pos"] is not None:
                    sc.masked_fill_(j[None] >= lim[i:i + step, None], -float("inf"))
                v, x = sc.topk(m, dim=1)
                idx[b, h, i:i + step, :m] = torch.where(v == -float("inf"), -1, x).int()
                val[b, h, i:i + step, :m] = v
    return idx, val


def _exact_codes(c, s, cap):
    """Codes in the index's order: tiles of 64 keys, 16-byte pieces of a key's
    code, a piece of all 64 keys together."""
    _, _, sets = _heads(c)
    r, e = c["r"], 16 // _ES[c["sketch"]]
    tiles = -(-cap // 64)
    out = torch.zeros((c["B"], sets, tiles * 64, r), dtype=torch.float64, device=DEV)
    for b in range(c["B"]):
        for h in range(sets):
            g = h if c["shared"] else _kv(c, h)
            out[b, h, :c["N"]] = (s["keys"][b, g, :c["N"]].double() - s["mu"][g].double()) @ s["B_k"][h].double()
    return out.view(c["B"], sets, tiles, 64, r // e, e).transpose(3, 4).reshape(-1)


def exact(c, seed):
    if c["do"] == "recall":
        return None  # whole numbers
    s = _inputs(c, seed, values=c["do"] == "attend")
    if c["do"] == "calibrate":
        Bq, Bk, mu = _factors64(s["q_cal"], s["k_cal"], c["r"], False)
        return [Bq, Bk, mu]
    if c["layers"] * c["B"] * c["H_q"] > 512:
        return None  # too long
    _with_factors(c, s)
    if c["do"] == "build":
        return None if c["sketch"] == "fp8" else _exact_codes(c, s, c["cap"])
    if c["do"] in ("score", "step"):
        idx, val = _exact_score(c, s)
        if c["do"] == "score":
            return {"idx": idx, "score": val}
        # which keys a list ends with depends on the codes' rounding: no
        # 64-bit value of the attention that follows it
        return {"idx": idx, "score": val, "out": None, "codes": None}
    if c["recon"]:
        return None  # depends on the codes' rounding
    lists = _lists(c, s)
    H_q, _, _ = _heads(c)
    pos = s["q_pos"] if s["q_pos"] is not None else torch.full((c["Q"],), c["N"] - 1, device=DEV)
    out = torch.zeros((c["B"], H_q, c["Q"], D_HEAD), dtype=torch.float64, device=DEV)
    for b in range(c["B"]):
        for h in range(H_q):
            g = _kv(c, h)
            kr = _rope64(s["keys"][b, g].double(), torch.arange(c["cap"], device=DEV))
            v = s["values"][b, g].double()
            qr = _rope64(s["q"][b, h].double(), pos)
            for i in range(0, c["Q"], 512):
                x = lists[b, h, i:i + 512].long()
                ok, x = x >= 0, x.clamp(min=0)
                sc = (kr[x] * qr[i:i + 512, None]).sum(-1) / D_HEAD ** 0.5
                sc.masked_fill_(~ok, -float("inf"))
                out[b, h, i:i + 512] = (torch.softmax(sc, dim=1)[..., None] * v[x]).sum(1)
    return out
