"""Performance cases: the work that a serving program has this package do, layer by layer.

A program holds a ``PrefillEngine`` (paged pools, block cache), plans each batch once and then
runs, for every layer, the Q/K/V producer (or the KV scatter, when its own model makes K and V)
and the prefix-cached attention.  Most cases are one such layer call on a planned batch; one is a
whole decode step with its host planning.  Layer shapes and length laws are those of
``workloads/configs.py`` (plus one multi-head shape of head_dim 64, the other head_dim and group
size that the kernels take).

Kinds: ``attn`` (PrefillEngine.attention), ``qkv`` (PrefillEngine.project / project_to_pool),
``scatter`` (PrefillEngine.scatter), ``step`` (prepare from kept hashes, project_to_pool,
attention, release).
"""

from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2606_21238_amd import hash_blocks_batch
from paper_2606_21238_amd.engine import PrefillEngine

VOCAB = 128256
THETA = 1.0e6
MAX_HISTORY = 32768        # tokens of the longest cached history

# (query heads, KV heads, head_dim) -> hidden size of a layer of that shape
HIDDEN = {(4, 2, 64): 256, (16, 16, 64): 1024, (32, 8, 128): 4096, (40, 8, 128): 5120, (64, 8, 128): 8192}


def _case(kind, shape, n, cached, suffix, ragged=True, miss=0.0, lens=1, rows=False, name=None):
    """n requests: `cached` tokens of history in the cache (median; whole blocks), `suffix` new
    tokens (mean); ragged: lognormal histories and uniform suffixes instead of equal ones; miss:
    share of requests whose history is not cached any more and is computed again; lens: seed of
    the lengths; rows: K and V of a `qkv` case as rows (then scattered) instead of into the pool."""
    c = dict(kind=kind, hq=shape[0], hkv=shape[1], d=shape[2], n=n, cached=cached, suffix=suffix,
             ragged=ragged, miss=miss, lens=lens)
    if kind == "qkv":
        c["rows"] = rows
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one request of a small layer, latency only
        _case("attn", (4, 2, 64), 1, 256, 64, ragged=False, name="attn_tiny"),
        # decode: one new token for each of 64 running sessions with lognormal histories
        _case("attn", (32, 8, 128), 64, 1808, 1, lens=1008, name="attn_decode"),
        # short new turns over cached histories (read-bound)
        _case("attn", (32, 8, 128), 16, 1808, 32, ragged=False, lens=1003, name="attn_short"),
        # questions about cached documents
        _case("attn", (40, 8, 128), 8, 8192, 128, ragged=False, name="attn_question"),
        # conversation batch: turns of mixed length, a quarter of the histories evicted
        _case("attn", (32, 8, 128), 16, 1808, 272, miss=0.25, lens=7, name="attn_turns"),
        # uncached prompts on a multi-head layer of head_dim 64
        _case("attn", (16, 16, 64), 12, 0, 1100, lens=3, name="attn_prefill64"),
        # long documents cached, long new suffix (the headline workload)
        _case("attn", (64, 8, 128), 4, 32768, 2048, ragged=False, name="attn_longctx"),
        # the producer of a decode step: one token per session, weights read once
        _case("qkv", (32, 8, 128), 64, 1808, 1, lens=1008, name="qkv_decode"),
        # the producer for a batch of questions, K and V as rows
        _case("qkv", (40, 8, 128), 8, 8192, 128, lens=5, rows=True, name="qkv_question"),
        # the producer of a prefill batch: some documents missed the cache
        _case("qkv", (40, 8, 128), 8, 8192, 128, ragged=False, miss=0.3, lens=12, name="qkv_prefill"),
        # K/V of a prefill batch from the program's own model into the pool
        _case("scatter", (32, 8, 128), 8, 8192, 128, miss=0.3, lens=9, name="scatter_prefill"),
        # a whole decode step: plan from kept hashes, copy, produce, attend, release
        _case("step", (32, 8, 128), 64, 1808, 1, lens=1008, name="step_decode"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["attn", "attn", "attn", "attn", "qkv", "qkv", "scatter", "step"])
    while True:
        shape = rng.choice(sorted(HIDDEN))
        n = _log_int(rng, 1, 64)
        cached = 0 if rng.random() < 0.15 else _log_int(rng, 64, MAX_HISTORY)
        suffix = 1 if kind == "step" or rng.random() < 0.2 else _log_int(rng, 1, 4096)
        c = _case(kind, shape, n, cached, suffix, ragged=rng.random() < 0.8,
                  miss=rng.choice([0.0, 0.0, 0.25]) if kind != "step" else 0.0,
                  lens=rng.randrange(1 << 30), rows=rng.random() < 0.5)
        P, S = lengths(c)
        w = work(c)
        if sum(P) + sum(S) <= 160_000 and sum(S) <= 40_000 and w["flops"] <= 3e12 and w["bytes"] <= 2e9:
            return c


def lengths(case):
    """(cached tokens, computed tokens) of every request."""
    rng = random.Random(case["lens"])
    P, S = [], []
    for _ in range(case["n"]):
        p, s = case["cached"], case["suffix"]
        if case["ragged"]:
            if p:
                p = max(16, min(int(rng.lognormvariate(math.log(p), 0.8)), 9 * p, MAX_HISTORY))
            if s > 1:
                s = rng.randint(max(1, s // 4), s * 7 // 4)
        p = p // 16 * 16
        if rng.random() < case["miss"]:
            p, s = 0, p + s
        P.append(p)
        S.append(s)
    return P, S


def work(case):
    P, S = lengths(case)
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    t = sum(S)
    attn = {"bytes": sum(4.0 * s * hq * d + 4.0 * (p + s) * hkv * d for p, s in zip(P, S)),
            "flops": sum(4.0 * d * hq * (s * p + s * (s + 1) / 2) for p, s in zip(P, S))}
    if case["kind"] == "attn":
        return attn
    if case["kind"] == "scatter":
        return {"bytes": 8.0 * t * hkv * d + 4.0 * t, "flops": 0}
    h, n_out = HIDDEN[hq, hkv, d], (hq + 2 * hkv) * d
    qkv = {"bytes": 2.0 * (t * h + n_out * h + t * n_out), "flops": 2.0 * t * h * n_out}
    if case["kind"] == "qkv":
        return qkv
    return {k: attn[k] + qkv[k] for k in attn}


def tolerance(case):
    if case["kind"] == "scatter":
        return "exact"
    # bf16 outputs; attention also rounds its probabilities to bf16, a producer rounds the
    # projection before the rotation.  Against 64 bits one layer call reads 1.6e-3 to 2.3e-3, the
    # decode step (rotated queries and keys rounded, then attended) 3.3e-3.
    return {"rel": 1e-2, "max": 0.05}


def _tokens(case, seed):
    rng = np.random.default_rng([seed, 1])
    P, S = lengths(case)
    return [rng.integers(0, VOCAB, p + s, dtype=np.int32) for p, s in zip(P, S)], P, S


def _tensors(case, seed, history):
    """Device tensors, N(0, 1) in bf16 as the configurations say (weights N(0, 1 / hidden)); the
    cached K and V only where `history`."""
    P, S = lengths(case)
    hq, hkv, d, t = case["hq"], case["hkv"], case["d"], sum(S)
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device="cuda", dtype=torch.bfloat16)

    kind, r = case["kind"], {}
    if kind in ("qkv", "step"):
        h = HIDDEN[hq, hkv, d]
        r["x"] = normal(t, h)
        r["w"] = normal((hq + 2 * hkv) * d, h) * h ** -0.5
    else:
        r["k_new"], r["v_new"] = normal(t, hkv, d), normal(t, hkv, d)
        if kind == "attn":
            r["q"] = normal(t, hq, d)
    if history:
        r["k_old"], r["v_old"] = normal(sum(P), hkv, d), normal(sum(P), hkv, d)
    return r


def prepare(case, seed):
    toks, P, S = _tokens(case, seed)
    hq, hkv, d, kind, t = case["hq"], case["hkv"], case["d"], case["kind"], sum(S)
    history = kind in ("attn", "step")
    st = _tensors(case, seed, history)
    blocks = sum(-(-len(x) // 16) for x in toks)
    pool = blocks + 2 * case["n"]
    eng = PrefillEngine(hq, hkv, d, blocks + case["n"], pool, case["n"], policy="arc", pool_fill=0,
                        initial_order=np.random.default_rng([seed, 2]).permutation(pool).astype(np.int32))
    if sum(P):          # the histories were prefilled earlier: blocks in the cache, K/V in the pool
        cached = [x[:p] for x, p in zip(toks, P) if p]
        db = eng.prepare(cached)
        if history:
            eng.scatter(db, st.pop("k_old"), st.pop("v_old"))
        eng.release()
    if kind == "step":
        st["hashes"] = hash_blocks_batch(toks)
        st["n_tokens"] = np.array([len(x) for x in toks], dtype=np.int64)
    else:
        st["db"] = db = eng.prepare(toks)
        eng.release()
        assert db.plan.prefix_lens.tolist() == P
    if kind == "attn":  # the batch's own K and V, as the layer's producer left them in the pool
        eng.scatter(db, st.pop("k_new"), st.pop("v_new"))
    if kind != "scatter":
        st.setdefault("q", torch.empty(t, hq, d, dtype=torch.bfloat16, device="cuda"))
        st["out"] = torch.empty_like(st["q"])
    if case.get("rows"):
        st["k"] = torch.empty(t, hkv, d, dtype=torch.bfloat16, device="cuda")
        st["v"] = torch.empty_like(st["k"])
    st.update(case=dict(case), eng=eng, k_pool=eng.k_pool.view(torch.bfloat16), v_pool=eng.v_pool.view(torch.bfloat16))
    return st


def run(st):
    eng, kind = st["eng"], st["case"]["kind"]
    if kind == "attn":
        eng.attention(st["db"], st["q"], st["out"])
        return st["out"]
    if kind == "scatter":
        eng.scatter(st["db"], st["k_new"], st["v_new"])
        return {"k_pool": st["k_pool"], "v_pool": st["v_pool"]}
    if kind == "qkv":
        if st["case"]["rows"]:
            eng.project(st["db"], st["x"], st["w"], st["q"], st["k"], st["v"], THETA)
            return {"q": st["q"], "k": st["k"], "v": st["v"]}
        eng.project_to_pool(st["db"], st["x"], st["w"], st["q"], THETA)
        return {"q": st["q"], "k_pool": st["k_pool"], "v_pool": st["v_pool"]}
    db = eng.prepare(None, hashes=st["hashes"], n_tokens=st["n_tokens"])
    eng.project_to_pool(db, st["x"], st["w"], st["q"], THETA)
    eng.attention(db, st["q"], st["out"])
    eng.release()
    return {"out": st["out"], "q": st["q"], "k_pool": st["k_pool"], "v_pool": st["v_pool"]}


# ---- the same values in 64 bits, in plain torch ----------------------------------------------

def _project64(case, x, w, P, S):
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    y = (x.double() @ w.double().t()).view(x.shape[0], hq + 2 * hkv, d)
    pos = torch.cat([torch.arange(p, p + s, device="cuda", dtype=torch.float64) for p, s in zip(P, S)])
    freq = THETA ** (-2.0 * torch.arange(d // 2, device="cuda", dtype=torch.float64) / d)
    a = (pos[:, None] * freq)[:, None, :]
    u = y[:, :hq + hkv]
    lo, hi = u[..., :d // 2], u[..., d // 2:]
    rot = torch.cat([lo * a.cos() - hi * a.sin(), hi * a.cos() + lo * a.sin()], dim=2)
    return rot[:, :hq], rot[:, hq:], y[:, hq + hkv:]


def _attend64(case, q, k_old, v_old, k_new, v_new, P, S):
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    out = torch.empty(sum(S), hq, d, dtype=torch.float64, device="cuda")
    po = so = 0
    for p, s in zip(P, S):
        k = torch.cat([k_old[po:po + p].double(), k_new[so:so + s].double()])
        v = torch.cat([v_old[po:po + p].double(), v_new[so:so + s].double()])
        hidden = torch.arange(p + s, device="cuda")[None, :] > torch.arange(p, p + s, device="cuda")[:, None]
        for h in range(hq):
            kh, vh = k[:, h * hkv // hq].contiguous(), v[:, h * hkv // hq].contiguous()
            sc = (q[so:so + s, h].double().contiguous() @ kh.t()) * d ** -0.5
            sc.masked_fill_(hidden, -math.inf)
            out[so:so + s, h] = torch.softmax(sc, dim=1) @ vh
        po, so = po + p, so + s
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind == "scatter":
        return None
    P, S = lengths(case)
    t = _tensors(case, seed, kind != "qkv")
    if kind == "attn":
        return _attend64(case, t["q"], t["k_old"], t["v_old"], t["k_new"], t["v_new"], P, S)
    q, k, v = _project64(case, t["x"], t["w"], P, S)
    if kind == "qkv":
        return {"q": q, "k": k, "v": v} if case["rows"] else {"q": q, "k_pool": None, "v_pool": None}
    return {"out": _attend64(case, q, t["k_old"], t["v_old"], k, v, P, S), "q": q, "k_pool": None, "v_pool": None}
