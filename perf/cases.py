"""The work that is timed when the speed of this library is followed from one version to the next.

Every case is one pass through public entry points of `paper_2603_22910_amd.binding`, with inputs that
were put on the GPU beforehand.  The layers are this repository's own: a 7B-shaped multi-head layer
(H_q = H_kv = 32, d = 128, half or a quarter of the dims retained), an 8B-shaped grouped-query layer
(H_q = 32, H_kv = 8, d = 128, with the paper's retained widths 0, 64, 384 and 512) and the small fp32 layer of
configuration 0.

A case is a dict of plain values:
  kind              "decode", "prefill", "append" or "compress"
  hq, hkv, d, m     layer shape; m = retained flattened dims of the target layer
  dtype             "bf16" or "f32"
  batch, len_lo, len_hi, len_seed
                    sequences and their lengths: len_lo each if len_lo == len_hi, else log-uniform draws
  mode              decode: "fused", "packed" (weights laid out once), "absorbed" or "absorb_v"
  rope, window      the paper's own inference: rotary embedding after the rebuild, first 4 + latest 128
                    tokens uncompressed
  t_q, pos0         prefill: queries of the chunk, cached tokens in front of it
  n_new             append: new tokens of each sequence
"""
from __future__ import annotations

import hashlib
import math
import random

import numpy as np
import torch

from paper_2603_22910_amd import binding as ek

DEV = "cuda:0"
N_SINK, N_RECENT = 4, 128
MHA = dict(hq=32, hkv=32, d=128, dtype="bf16")
GQA = dict(hq=32, hkv=8, d=128, dtype="bf16")
F32 = dict(hq=8, hkv=8, d=64, dtype="f32")
TORCH_DTYPE = {"bf16": torch.bfloat16, "f32": torch.float32}


def _decode(layer, m, mode, batch, lo, hi, len_seed=0, rope=False, window=False):
    return dict(kind="decode", **layer, m=m, mode=mode, batch=batch, len_lo=lo, len_hi=hi, len_seed=len_seed,
                rope=rope, window=window)


def _prefill(layer, m, t_q, pos0, rope=False):
    return dict(kind="prefill", **layer, m=m, t_q=t_q, pos0=pos0, rope=rope)


def _append(layer, m, batch, lo, hi, len_seed, n_new):
    return dict(kind="append", **layer, m=m, batch=batch, len_lo=lo, len_hi=hi, len_seed=len_seed, n_new=n_new)


def _compress(layer, m, batch, lo, hi, len_seed):
    return dict(kind="compress", **layer, m=m, batch=batch, len_lo=lo, len_hi=hi, len_seed=len_seed)


def listed():
    return [
        # the cache writes of one decode step of a serving batch: anchor, target and window rows
        dict(name="append_gqa_b32", **_append(GQA, 512, 32, 200, 900, 1, 1)),
        # the full -> compressed switch of a layer when memory runs short
        dict(name="compress_mha_b8", **_compress(MHA, 2048, 8, 1000, 12000, 2)),
        # configuration 0: the fp32 layer
        dict(name="decode_f32_b1_l512", **_decode(F32, 256, "fused", 1, 512, 512)),
        # one user, short context, the paper's inference set-up: the latency of a single token
        dict(name="decode_gqa_b1_l1000_rope_window", **_decode(GQA, 512, "fused", 1, 1000, 1000, rope=True, window=True)),
        # the paper's throughput set-up: batch 8, contexts up to 36K, rotary embedding and window
        dict(name="decode_gqa_b8_ragged_rope_window", **_decode(GQA, 384, "fused", 8, 2048, 36864, 3, rope=True, window=True)),
        # configuration 1: a batch of equal contexts
        dict(name="decode_mha_b8_l4096", **_decode(MHA, 2048, "fused", 8, 4096, 4096)),
        # configuration 4: a large ragged serving batch, weights laid out once at load time (the largest case)
        dict(name="decode_mha_b32_ragged_packed", **_decode(MHA, 2048, "packed", 32, 1024, 65536, 4)),
        # the other association order on a small batch
        dict(name="decode_gqa_b2_l1500_absorbed", **_decode(GQA, 512, "absorbed", 2, 1500, 1500)),
        # configuration 2: long contexts in the other association order
        dict(name="decode_mha_b4_l32768_absorbed", **_decode(MHA, 1024, "absorbed", 4, 32768, 32768)),
        # configuration 3 with the paper's extras: one very long context, values in the other order
        dict(name="decode_gqa_b1_l131072_absorb_v", **_decode(GQA, 512, "absorb_v", 1, 131072, 131072, rope=True, window=True)),
        # configuration 4's prefill chunk: a whole prompt at once
        dict(name="prefill_mha_8192", **_prefill(MHA, 2048, 8192, 0)),
        # a chunk of a prompt behind what is cached already; retained prefix ends inside a head (m = 64)
        dict(name="prefill_gqa_500_at_7000_rope", **_prefill(GQA, 64, 500, 7000, rope=True)),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    kind = rng.choice(["append", "compress", "f32", "decode", "decode", "paper", "absorbed", "absorb_v", "prefill", "prefill"])
    seed = rng.randrange(1 << 16)
    layer, m = rng.choice([(MHA, 2048), (MHA, 1024), (GQA, 512), (GQA, 384)])
    if kind == "append":
        return _append(layer, m, _log_int(rng, 1, 64), 100, 800, seed, _log_int(rng, 1, 64))
    if kind == "compress":
        return _compress(layer, m, _log_int(rng, 1, 16), 100, _log_int(rng, 500, 16000), seed)
    if kind == "f32":
        return _decode(F32, rng.choice([0, 128, 256]), "fused", _log_int(rng, 1, 4), 64, _log_int(rng, 100, 3000), seed)
    if kind == "prefill":
        if layer is GQA:
            m = rng.choice([0, 64, 384, 512])
        t_q = _log_int(rng, 16, 8192)
        return _prefill(layer, m, t_q, rng.choice([0, _log_int(rng, 100, 24000)]), rope=rng.random() < 0.5)
    # decode: cached tokens of the whole batch, spread over sequences of unequal length
    if kind in ("paper", "absorb_v"):
        layer, m = GQA, rng.choice([0, 64, 384, 512])
    batch = _log_int(rng, 1, 32)
    mean = _log_int(rng, 300, 40000)
    mean = max(200, min(mean, 200000 // batch))
    lo, hi = (mean, mean) if rng.random() < 0.3 else (max(100, mean // 3), mean * 2)
    extras = kind in ("paper", "absorb_v")
    mode = {"decode": rng.choice(["fused", "packed"]), "paper": "fused", "absorbed": "absorbed", "absorb_v": "absorb_v"}[kind]
    return _decode(layer, m, mode, batch, lo, hi, seed, rope=extras, window=extras)


# ---- inputs ------------------------------------------------------------------------------------
def _lengths(case):
    if case["kind"] == "prefill":
        return [case["pos0"] + case["t_q"]]
    lo, hi = case["len_lo"], case["len_hi"]
    if lo == hi:
        return [lo] * case["batch"]
    r = random.Random(case["len_seed"])
    return [min(hi, int(lo * (hi / lo) ** r.random())) for _ in range(case["batch"])]


def _randn(seed, tag, *shape, dtype=torch.float32):
    h = hashlib.sha256(f"{seed}/{tag}".encode()).digest()
    g = torch.Generator(device=DEV)
    g.manual_seed(int.from_bytes(h[:8], "little") >> 1)
    return torch.randn(*shape, generator=g, device=DEV, dtype=dtype)


class _Inputs:
    """Caches, weights and queries of one layer pair, drawn on the GPU from the seed alone: anchor rows
    N(0, 1), retained rows correlated with them, weights N(0, 1/sqrt(d_in)), queries N(0, 1)."""

    def __init__(self, case, seed):
        td = TORCH_DTYPE[case["dtype"]]
        self.D = D = case["hkv"] * case["d"]
        self.m = m = case["m"]
        self.d_in, self.d_out = D + m, D - m
        self.lens = _lengths(case)
        extra = case.get("n_new", 0)
        caps = [(n + extra + 255) // 256 * 256 for n in self.lens]
        self.starts = [sum(caps[:b]) for b in range(len(caps))]
        self.caps = caps
        self.pool = sum(caps)
        cache = {}
        for t in ("k", "v"):
            a = _randn(seed, t + "_a", self.pool, D, dtype=td)
            cache[t] = a
            if case["kind"] == "compress":
                continue
            r = a @ (_randn(seed, t + "_m1", D, m) / math.sqrt(D)).to(td)
            if m:
                r += _randn(seed, t + "_e1", self.pool, m, dtype=td) * 0.1
            cache[t + "_r"] = r
        self.k_a, self.v_a = cache["k"], cache["v"]
        self.k_r, self.v_r = cache.get("k_r"), cache.get("v_r")
        if case["kind"] in ("decode", "prefill"):
            std = 1.0 / math.sqrt(self.d_in)
            self.w_k = (_randn(seed, "w_k", self.d_in, self.d_out) * std).to(td)
            self.w_v = (_randn(seed, "w_v", self.d_in, self.d_out) * std).to(td)
            n_q = case["t_q"] if case["kind"] == "prefill" else case["batch"]
            self.q = _randn(seed, "q", n_q, case["hq"], case["d"]).to(td)
        self.rope = None
        if case.get("rope"):
            i = torch.arange(case["d"] // 2, dtype=torch.float64, device=DEV)
            n = max(self.lens)
            ang = torch.arange(n, dtype=torch.float64, device=DEV)[:, None] * 10000.0 ** (-2.0 * i / case["d"])[None, :]
            self.rope = (torch.cos(ang).float(), torch.sin(ang).float())
        self.win = None
        if case.get("window") or case["kind"] == "append":
            shape = (len(self.lens), N_SINK + N_RECENT, D)
            self.win = (_randn(seed, "win_k", *shape).to(td), _randn(seed, "win_v", *shape).to(td))

    def cache(self, full):
        k, v, width = (self.k_a, self.v_a, self.D) if full else (self.k_r, self.v_r, self.m)
        if width == 0:
            k = v = None
        return ek.LayerCache(k, v, width, self.pool, self.starts, self.lens, self.caps)


MODE_FLAGS = {"fused": 0, "packed": ek.FLAG_W_PACKED, "absorbed": ek.FLAG_ABSORBED, "absorb_v": ek.FLAG_ABSORB_V}


def prepare(case, seed):
    """The caches, the weights in the layout that the mode takes, and a workspace: what a serving
    program holds before the call."""
    x = _Inputs(case, seed)
    kind = case["kind"]
    s = dict(case=case, x=x, kind=kind)
    flags = MODE_FLAGS[case["mode"]] if kind == "decode" else 0
    s["shape"] = shape = ek.make_shape(case["hq"], case["hkv"], case["d"], case["m"], case["dtype"], flags=flags)
    if kind == "compress":
        s["full"] = x.cache(True)
        td = TORCH_DTYPE[case["dtype"]]
        s["out"] = tuple(torch.zeros(x.pool, x.m, dtype=td, device=DEV) for _ in range(2))
        s["dst"] = ek.LayerCache(*s["out"], x.m, x.pool, x.starts, [0] * len(x.lens), x.caps)
        return s
    s["anchor"], s["target"] = x.cache(True), x.cache(False)
    if kind == "append":
        n = case["n_new"] * len(x.lens)
        td = TORCH_DTYPE[case["dtype"]]
        s["new"] = [_randn(seed, "new" + t, n, x.D).to(td) for t in ("k_a", "v_a", "k_t", "v_t")]
        s["n_new"] = np.full(len(x.lens), case["n_new"], dtype=np.int32)
        s["len0"] = np.asarray(x.lens, dtype=np.int32)
        return s
    w_k, w_v = x.w_k, x.w_v
    if kind == "decode" and case["mode"] == "packed":
        w_k, w_v = (torch.empty(x.d_out, x.d_in, dtype=w.dtype, device=DEV) for w in (x.w_k, x.w_v))
        ek.pack_weights(shape, x.w_k, w_k)
        ek.pack_weights(shape, x.w_v, w_v)
    elif case["m"] % case["d"] and not flags:      # a split head: selector columns put in front once
        n = ek.augmented_weight_elems(shape)
        w_k, w_v = (torch.empty(n, dtype=x.w_k.dtype, device=DEV) for _ in range(2))
        ek.augment_weights(shape, x.w_k, x.w_v, w_k, w_v)
        shape.flags |= ek.FLAG_W_AUGMENTED
    s["w"] = (w_k, w_v)
    n_q = case["t_q"] if kind == "prefill" else 0
    need = ek.workspace_bytes(shape, len(x.lens), sum(x.lens), n_q)
    s["workspace"] = torch.empty(need, dtype=torch.uint8, device=DEV)
    s["out"] = torch.empty_like(x.q)
    s["lse"] = torch.empty(x.q.shape[:2], dtype=torch.float32, device=DEV)
    return s


def run(state):
    s, case, x = state, state["case"], state["x"]
    kind = s["kind"]
    if kind == "append":
        # the same step each time: the sequences are as long as they were before it
        s["anchor"].seq_len[:] = s["len0"]
        s["target"].seq_len[:] = s["len0"]
        ka, va, kt, vt = s["new"]
        ek.cache_append(s["shape"], s["anchor"], ka, va, s["n_new"])
        ek.cache_append(s["shape"], s["target"], kt, vt, s["n_new"])
        ek.window_append(s["shape"], x.win[0], x.win[1], N_SINK, N_RECENT, s["len0"], kt, vt, s["n_new"])
        return [x.k_a, x.v_a, x.k_r, x.v_r, *x.win]
    if kind == "compress":
        ek.cache_compress(s["shape"], s["full"], s["dst"])
        return list(s["out"])
    w_k, w_v = s["w"]
    args = (s["shape"], s["anchor"], s["target"], w_k, w_v)
    if kind == "prefill":
        if x.rope is None:
            ek.prefill_attn(*args, 0, x.q, case["t_q"], case["pos0"], s["out"], s["lse"], s["workspace"])
        else:
            ek.prefill_attn_ex(*args, 0, x.q, case["t_q"], case["pos0"], s["out"], s["lse"], s["workspace"], rope=x.rope)
    elif x.rope is None and x.win is None:
        ek.decode_attn(*args, x.q, s["out"], s["lse"], s["workspace"])
    else:
        win = None if x.win is None else (*x.win, N_SINK, N_RECENT)
        ek.decode_attn_ex(*args, x.q, s["out"], s["lse"], s["workspace"], rope=x.rope, window=win)
    return [s["out"], s["lse"]]


# ---- what a pass cannot do without ---------------------------------------------------------------
def work(case):
    es = 2 if case["dtype"] == "bf16" else 4
    D, m = case["hkv"] * case["d"], case["m"]
    d_in, d_out = D + m, D - m
    lens = _lengths(case)
    total = sum(lens)
    if case["kind"] == "append":
        n = case["n_new"] * len(lens)
        # full rows read and written for the anchor; the target's rows read once, its first m dims and
        # the window's copy written
        kept = len(lens) * min(case["n_new"], N_RECENT)
        return {"bytes": 2 * es * (n * (D + D + D + m) + kept * D), "flops": 0}
    if case["kind"] == "compress":
        return {"bytes": 2 * 2 * es * total * m, "flops": 0}
    weights = 2 * d_in * d_out * es
    caches = 2 * total * d_in * es
    G = case["hq"] // case["hkv"]
    if case["kind"] == "prefill":
        t, p = case["t_q"], case["pos0"]
        pairs = t * p + t * (t + 1) // 2
        q = 2 * t * case["hq"] * case["d"] * es
        return {"bytes": weights + caches + q, "flops": 4 * total * d_in * d_out + 4 * pairs * case["hq"] * case["d"]}
    b = len(lens)
    q = 2 * b * case["hq"] * case["d"] * es
    # attention itself, and the product in the association order that the mode stands for
    attn = 4 * total * case["hq"] * case["d"]
    side = 2 * total * d_in * d_out                    # one of keys / values rebuilt
    other = 2 * total * d_in * case["hq"] + 2 * b * d_in * d_out * G
    flops = {"fused": attn + 2 * side, "packed": attn + 2 * side, "absorbed": 2 * other,
             "absorb_v": attn // 2 + side + other}[case["mode"]]
    win = 2 * 2 * b * (N_SINK + N_RECENT) * D if case["window"] else 0
    rope = 2 * max(lens) * (case["d"] // 2) * 4 if case["rope"] else 0
    return {"bytes": weights + caches + q + win + rope, "flops": flops}


def tolerance(case):
    if case["kind"] in ("append", "compress"):
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-4}
    # bf16 outputs of fp32 sums; the absorbed queries and the prefill probabilities are rounded to bf16 inside
    rel = 1e-2 if case["kind"] == "prefill" or case["mode"] == "absorbed" else 6e-3
    return {"rel": rel, "max": 0.1}


# ---- the same in 64 bits, in plain torch ----------------------------------------------------------
def _full_rows(x, t, lo, hi):
    """Rebuilt full-width rows [lo, hi) of the pool in float64."""
    a = (x.k_a if t == "k" else x.v_a)[lo:hi].double()
    r = (x.k_r if t == "k" else x.v_r)[lo:hi].double()
    w = (x.w_k if t == "k" else x.w_v).double()
    return torch.cat([r, torch.cat([a, r], 1) @ w], 1)


def _rotate(x, rows, p0):
    """rows [n, H_kv, d] at positions p0 .. p0 + n - 1."""
    n, h = rows.shape[0], rows.shape[2] // 2
    c, s = (t[p0:p0 + n].double()[:, None, :] for t in x.rope)
    a, b = rows[..., :h], rows[..., h:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def exact(case, seed):
    if case["kind"] not in ("decode", "prefill"):
        return None
    x = _Inputs(case, seed)
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    G, scale = hq // hkv, 1.0 / math.sqrt(d)
    chunk = 8192
    outs, lses = [], []
    for b, L in enumerate(x.lens):
        s0 = x.starts[b]
        ks, vs = [], []
        q = x.q.double() if case["kind"] == "prefill" else x.q[b].double()
        scores = []
        for p in range(0, L, chunk):
            n = min(chunk, L - p)
            k, v = (_full_rows(x, t, s0 + p, s0 + p + n) for t in ("k", "v"))
            if case.get("window"):
                pos = torch.arange(p, p + n, device=DEV)
                inside = (pos < N_SINK) | (pos >= L - N_RECENT)
                pi = pos[inside]
                row = torch.where(pi < N_SINK, pi, N_SINK + (pi - N_SINK) % N_RECENT)
                k[inside], v[inside] = x.win[0][b][row].double(), x.win[1][b][row].double()
            k, v = k.view(n, hkv, d), v.view(n, hkv, d)
            if x.rope is not None:
                k = _rotate(x, k, p)
            if case["kind"] == "prefill":
                ks.append(k)
                vs.append(v)
            else:
                # [hq, n]; running softmax over the chunks
                kq = torch.stack([(k[:, h // G] @ q[h]) for h in range(hq)]) * scale
                mx = kq.amax(1)
                e = torch.exp(kq - mx[:, None])
                o = torch.stack([e[h] @ v[:, h // G] for h in range(hq)])
                scores.append((mx, e.sum(1), o))
        if case["kind"] == "prefill":
            k, v = torch.cat(ks), torch.cat(vs)
            t_q, p0 = case["t_q"], case["pos0"]
            out = torch.empty(t_q, hq, d, dtype=torch.float64, device=DEV)
            lse = torch.empty(t_q, hq, dtype=torch.float64, device=DEV)
            key = torch.arange(L, device=DEV)
            for h in range(hq):
                kh, vh = k[:, h // G].t().contiguous(), v[:, h // G].contiguous()
                for i in range(0, t_q, 2048):
                    j = min(t_q, i + 2048)
                    sc = (q[i:j, h].contiguous() @ kh) * scale
                    sc.masked_fill_(key[None, :] > torch.arange(p0 + i, p0 + j, device=DEV)[:, None], -math.inf)
                    lse[i:j, h] = torch.logsumexp(sc, 1)
                    out[i:j, h] = torch.softmax(sc, 1) @ vh
            return [out, lse]
        M = torch.stack([t[0] for t in scores]).amax(0)
        l = sum(t[1] * torch.exp(t[0] - M) for t in scores)
        o = sum(t[2] * torch.exp(t[0] - M)[:, None] for t in scores)
        outs.append(o / l[:, None])
        lses.append(M + torch.log(l))
    return [torch.stack(outs), torch.stack(lses)]
