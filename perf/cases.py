"""The work that a program has this framework do, as measured cases.

Every case is one pass over one depth window of a cache through the public
``DeviceCache`` methods, the way a serving loop drives them: it holds the
cache, the queries, the outputs and the workspaces, and calls per layer.

* ``decode``    attention of the decode queries over the factorized cache, with
                or without the Eq. 3 probe, fp16 or 8-bit blockwise coefficients
* ``append``    a decode step that routes and appends the new token first
* ``features``  a decode step that also collects the router's attention features
* ``prefill``   routing and compression of a prompt's dense keys and values
* ``sketch``    the bases of a window from its prefill
* ``budget``    re-routing of the whole context under a memory budget
* ``unfused``   the comparison path: rebuild the cache, then dense attention

Inputs follow the synthetic workloads of ``synth/``: orthonormal fp16 bases,
N(0, 1) coefficients, categorical routed ranks, uniform int4 codes and scales.
"""
from __future__ import annotations

import math
import random
from types import SimpleNamespace

import numpy as np
import torch

from paper_2607_06523_amd import DeviceCache, ProbeRef

D = 128
DEV = "cuda"

_BASE = {"kind": "decode", "batch": 1, "tokens": 65536, "ragged": False, "layers": 4, "kv_heads": 8, "group": 4,
         "rank": 48, "levels": "0,4,8,16", "probs": "0.75,0.12,0.08,0.05", "q": "bf16", "coef": "f16",
         "salient": 0.0, "probe_heads": 0, "probe_pos": 1}
_L70B = {"levels": "0,4,8,16,32", "probs": "0.70,0.12,0.10,0.06,0.02"}
_L3 = {"levels": "0,8,16", "probs": "0.80,0.15,0.05"}


def listed():
    def case(name, **kw):
        return {**_BASE, "name": name, **kw}
    return [
        # the smallest call: a short context of a small model, bound by launches and latency
        case("decode-4k", tokens=4096, layers=2, kv_heads=2, rank=32, q="f16", **_L3),
        # the headline: one 64K sequence of an 8B-class decoder, windows of 4 layers
        case("decode-64k"),
        # a serving batch of ragged lengths (8K..16K tokens each), windows of 2 layers
        case("decode-batch16", batch=16, tokens=16384, ragged=True, layers=2, rank=32, **_L3),
        # the largest: a 70B-class decoder at 2 x 128K with a probed KV head
        case("decode-70b-probe", batch=2, tokens=131072, group=8, rank=64, probe_heads=1, **_L70B),
        # the 8-bit blockwise coefficient form of the headline
        case("decode-64k-int8", coef="int8"),
        # wide bases and groups: 16 query heads per KV head, r_b 96, 16K tokens
        case("decode-g16-r96", tokens=16384, layers=2, kv_heads=4, group=16, rank=96, **_L70B),
        # the decode step of a running sequence: route and append the new token, then attend
        case("append-64k", kind="append"),
        # a step that also gathers the attention mass and spike of every token
        case("features-64k", kind="features"),
        # a 32K prompt entering the cache
        case("prefill-32k", kind="prefill", tokens=32768),
        # a window's bases from a 64K prompt
        case("sketch-64k", kind="sketch"),
        # every window of a 32-layer model (8 windows of 4) re-routed to a budget at 64K
        case("budget-64k", kind="budget", layers=32, levels="0,16", probs="0.9,0.1"),
        # the rebuild-then-attend comparison of a 64K layer
        case("unfused-64k", kind="unfused", layers=1),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any kind, sizes over the whole range the listed cases span."""
    kind = rng.choice(["decode"] * 5 + ["append", "features", "prefill", "sketch", "budget", "unfused"])
    c = dict(_BASE, kind=kind)
    c["q"] = rng.choice(["bf16", "f16"])
    c["kv_heads"] = rng.choice([1, 2, 4, 8])
    c["group"] = rng.choice([1, 2, 4, 4, 4, 8])
    c["rank"] = rng.choice([16, 32, 32, 48, 48, 64])
    c["batch"] = rng.choice([1, 1, 1, 2, 3, 16])
    c["layers"] = rng.choice([1, 2, 4])
    if kind in ("decode", "unfused") and rng.random() < 0.25:      # shapes of the general kernel
        c["group"] = rng.choice([8, 16])
        c["rank"] = rng.choice([80, 96, 128])
    if kind == "decode" and c["group"] <= 4 and c["rank"] <= 64 and rng.random() < 0.3:
        c["coef"] = "int8"
    if kind == "prefill" and rng.random() < 0.3:
        c["coef"] = "int8"
    c.update(rng.choice([{}, _L3, _L70B if c["group"] >= 8 else {}]))
    if kind == "budget":
        c.update(levels=rng.choice(["0,8", "0,16", "4,16"]), probs="0.9,0.1", layers=rng.choice([4, 8, 32]))
    if kind == "decode" and rng.random() < 0.3:
        c["probe_heads"] = rng.choice([1, min(2, c["kv_heads"])])
        if c["coef"] == "f16" and rng.random() < 0.3:
            c["probe_pos"] = rng.choice([2, 3])
    if rng.random() < 0.2:
        c["salient"] = 0.02
    cap = 131072 if kind in ("decode", "append", "features") else 65536
    if kind in ("prefill", "sketch"):
        cap = 24576 if kind == "prefill" else 49152
    c["tokens"] = _log(rng, 1000, cap)
    if rng.random() < 0.3:                                          # the round sizes are common too
        c["tokens"] = 1 << int(math.log2(c["tokens"]))
    c["ragged"] = c["batch"] > 1 and rng.random() < 0.7
    total = 262144 if kind == "decode" else cap
    if c["batch"] * c["tokens"] > total:
        c["tokens"] = max(500, total // c["batch"] - rng.randrange(64))
    if kind == "budget":
        c["kv_heads"] = min(c["kv_heads"], 64 * 4 // c["layers"])
    return c


# ---- shapes -----------------------------------------------------------------------------------

def _lens(case):
    if not case["ragged"]:
        return [case["tokens"]] * case["batch"]
    r = random.Random("%d/%d" % (case["batch"], case["tokens"]))
    return [r.randint(max(1, case["tokens"] // 2), case["tokens"]) for _ in range(case["batch"])]


def _levels(case):
    return tuple(int(x) for x in case["levels"].split(","))


def _probs(case):
    return [float(x) for x in case["probs"].split(",")]


def _mean_rank(case):
    s = case["salient"]
    return (1 - s) * sum(p * l for p, l in zip(_probs(case), _levels(case))) + s * _levels(case)[-1]


def _rng(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * (seed + 1) + 17)
    return g


def _bases(seed, n, rank):
    """n orthonormal [rank, D] row bases, fp16."""
    r = np.random.default_rng(seed + 99)
    q = np.linalg.qr(r.standard_normal((n, D, rank)))[0]
    return torch.from_numpy(np.ascontiguousarray(q.transpose(0, 2, 1))).to(DEV).half()


def _rank_codes(case, lens, n, g):
    """Routed levels [n, T] (n = windows x heads); salient spans carry the top level everywhere."""
    T = sum(lens)
    cum = torch.tensor(np.cumsum(_probs(case))[:-1], device=DEV, dtype=torch.float32)
    code = torch.bucketize(torch.rand((n, T), generator=g, device=DEV), cum, right=True).to(torch.uint8)
    if case["salient"] > 0:
        span = torch.rand(T // 64 + 1, generator=g, device=DEV) < case["salient"]
        code[:, span.repeat_interleave(64)[:T]] = len(_levels(case)) - 1
    return code


def _room(case, T):
    """Residual entries a slab has room for: the expected ones and a margin, so that inputs of every
    seed have one shape."""
    top, s = _levels(case)[-1], case["salient"]
    n = T * _mean_rank(case) + 8 * top * math.sqrt(T) + 512 * top * math.sqrt(s * T / 64 + (s > 0))
    return -(-(min(int(n), T * top) + 512) // 256) * 256


def _entries(code, levels, layers, room, g):
    """Offsets [H, T+1], and per (layer, Z, head) channels, packed codes; distinct channels per
    token, largest |code| first, then by channel."""
    H, T = code.shape
    rho = torch.tensor(levels, device=DEV, dtype=torch.int64)[code.long()]
    off = torch.zeros((H, T + 1), dtype=torch.int64, device=DEV)
    off[:, 1:] = rho.cumsum(1)
    stride = max(room, -(-(int(off[:, -1].max()) + 512) // 256) * 256)
    idx = torch.zeros((layers, 2, H, stride), dtype=torch.uint8, device=DEV)
    nib = torch.zeros((layers, 2, H, stride), dtype=torch.uint8, device=DEV)
    for h in range(H):
        for k, r in enumerate(levels):
            tok = torch.nonzero(code[h] == k).flatten() if r else code.new_zeros(0)
            if tok.numel() == 0:
                continue
            shape = (layers, 2, tok.numel(), 1)
            ri = lambda lo, hi, s: torch.randint(lo, hi, s, generator=g, device=DEV, dtype=torch.int32)
            j = torch.arange(r, device=DEV, dtype=torch.int32)
            ch = (ri(0, D, shape) + j * (2 * ri(0, D // 2, shape) + 1)) % D
            q = ri(-7, 8, (layers, 2, tok.numel(), r))
            key = torch.sort(((7 - q.abs()) * 256 + ch) * 2 + (q < 0), dim=-1).values
            mag, ch, neg = 7 - key // 512, (key // 2) % 256, key % 2
            q = torch.where(neg == 1, -mag, mag)
            pos = (off[h][tok][:, None] + j).flatten()
            idx[:, :, h, pos] = ch.flatten(2).to(torch.uint8)
            nib[:, :, h, pos] = (q & 15).flatten(2).to(torch.uint8)
    return off, stride, idx, nib[..., 0::2] | (nib[..., 1::2] << 4)


def _cache(case, seed, g, filled=True, entries=True):
    """A DeviceCache of the case's shape; ``filled``: with coefficients and residuals."""
    lens, levels, L, H, rb = _lens(case), _levels(case), case["layers"], case["kv_heads"], case["rank"]
    T, B = sum(lens), len(lens)
    window = 4 if case["kind"] == "budget" else L
    M, T16 = L // window, -(-sum(lens) // 16) * 16
    i8 = case["coef"] == "int8"
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    filled = filled and entries
    stride = 512
    idx = val = np.zeros((0,), np.uint8)
    if entries:
        code = _rank_codes(case, lens, M * H, g)
        if filled:
            off, stride, idx, val = _entries(code, levels, L, _room(case, T), g)
        else:                                     # room for whatever the router assigns
            stride = -(-(T * levels[-1] + 512) // 256) * 256
            off = torch.zeros((H, T + 1), dtype=torch.int64, device=DEV)
            idx = torch.zeros((L, 2, H, stride), dtype=torch.uint8, device=DEV)
            val = torch.zeros((L, 2, H, stride // 2), dtype=torch.uint8, device=DEV)
    e16, e8 = np.zeros((L, H, 0, rb), np.uint16), np.zeros((L, H, 0, rb), np.int8)
    host = SimpleNamespace(
        basis=np.zeros((0,), np.uint16), coef_format=case["coef"], coef_k=e8 if i8 else e16,
        coef_v=np.zeros((L, H, 0, rb, 16), np.int8 if i8 else np.uint16), coef_scale_k=np.zeros((0,), np.uint16),
        coef_scale_v=np.zeros((0,), np.uint16), rank_code=np.zeros((0,), np.uint8), res_off=np.zeros((0,), np.uint32),
        res_idx=np.zeros((0,), np.uint8), res_val=np.zeros((0,), np.uint8), res_scale=np.zeros((0,), np.uint16),
        q_dtype=case["q"], q_bits=np.zeros((0,), np.uint16), cu_seqlens=cu, n_layers=L, window=window,
        n_kv_heads=H, n_q_heads=H * case["group"], head_dim=D, basis_rank=rb, levels=levels, res_stride=stride)
    dc = DeviceCache(host)
    dc.basis = _bases(seed, B * M * H * 2, rb).view(B, M, H, 2, rb, D)
    if entries:
        dc.rank_code = code.view(M, H, T)
        dc.res_off = off.to(torch.int32).view(M, H, T + 1)
        dc.res_idx, dc.res_val = idx, val
        if i8:
            dc.coef_k = torch.zeros((L, H, T16 // 16, rb // 16, 16, 16), dtype=torch.int8, device=DEV)
            dc.coef_v = torch.zeros((L, H, T16 // 16, rb, 16), dtype=torch.int8, device=DEV)
            dc.coef_scale_k = torch.zeros((L, H, rb // 16, T), dtype=torch.float16, device=DEV)
            dc.coef_scale_v = torch.zeros((L, H, rb // 16, T), dtype=torch.float16, device=DEV)
        else:
            dc.coef_k = torch.zeros((L, H, T16 // 16, rb // 8, 16, 8), dtype=torch.float16, device=DEV)
            dc.coef_v = torch.zeros((L, H, T16 // 8, rb, 8), dtype=torch.float16, device=DEV)
        dc.res_scale = torch.zeros((L, 2, H, T), dtype=torch.float16, device=DEV)
    if filled:
        if i8:
            for t in (dc.coef_k, dc.coef_v):
                t.copy_((torch.randn(t.shape, generator=g, device=DEV) * 8).round_().clamp_(-127, 127))
            for t in (dc.coef_scale_k, dc.coef_scale_v):
                t.copy_(0.11 + 0.03 * torch.rand(t.shape, generator=g, device=DEV))
        else:
            dc.coef_k.normal_(generator=g)
            dc.coef_v.normal_(generator=g)
        if T16 > T:                               # padding tokens are zero
            pad = T16 - T
            dc.coef_k[:, :, -1, :, 16 - pad:] = 0
            if i8:
                dc.coef_v[:, :, -1, :, 16 - pad:] = 0
            else:
                v = dc.coef_v.view(L, H, T16 // 8, rb, 8)
                v[:, :, -1, :, 8 - min(pad, 8):] = 0
                if pad > 8:
                    v[:, :, -2, :, 16 - pad:] = 0
        dc.res_scale.copy_(0.01 + 0.09 * torch.rand(dc.res_scale.shape, generator=g, device=DEV))
    dc.set_split(0)
    return dc


def _queries(case, n, g):
    dt = torch.bfloat16 if case["q"] == "bf16" else torch.float16
    shape = (n, case["batch"], case["kv_heads"] * case["group"], D)
    return (torch.randn(shape, generator=g, device=DEV) / math.sqrt(D)).to(dt)


def _dense(case, dc, g, layers):
    """Dense keys and values near the bases' span (with a full-rank remainder), per layer [T, H, D]."""
    lens = _lens(case)
    out = []
    for _ in range(layers):
        kv = []
        for z in range(2):
            rows = []
            for b, n in enumerate(lens):
                a = torch.randn((case["kv_heads"], n, case["rank"]), generator=g, device=DEV)
                x = torch.bmm(a, dc.basis[b, 0, :, z].float())
                rows.append(x.add_(torch.randn(x.shape, generator=g, device=DEV), alpha=0.25).half())
            kv.append(torch.cat(rows, 1).transpose(0, 1).contiguous())
        out.append(kv)
    return out


def _router(case, g, M, H, T):
    """Router features, weights and thresholds."""
    phi = torch.empty((M, H, T, 4), device=DEV)
    phi[..., 0].exponential_(1.0, generator=g)
    phi[..., 1].exponential_(2.0, generator=g)
    phi[..., 2] = (torch.rand((M, H, T), generator=g, device=DEV) < 0.05).float()
    phi[..., 3].uniform_(0.0, 0.2, generator=g)
    u = 0.25 + 1.25 * torch.rand((M, 4), generator=g, device=DEV)
    th = (2.0 + 4.0 * torch.rand((M, len(_levels(case)) - 1), generator=g, device=DEV)).sort(1).values.contiguous()
    return phi, u, th


def prepare(case, seed):
    g = _rng(case, seed)
    kind, L, H, G = case["kind"], case["layers"], case["kv_heads"], case["group"]
    lens = _lens(case)
    B, T = len(lens), sum(lens)
    s = {"case": case}
    outs = lambda: [torch.empty((B, H * G, D), dtype=torch.float32, device=DEV) for _ in range(L)]
    if kind == "decode":
        s["dc"] = dc = _cache(case, seed, g)
        s["q"], s["outs"] = _queries(case, L, g), outs()
        n = case["probe_heads"]
        if n:
            heads = [(1 + 3 * i) % H for i in range(n)]
            heads = heads if len(set(heads)) == n else list(range(n))
            T16 = -(-T // 16) * 16
            refs, errs = [], []
            for _ in range(L):
                k = torch.randn((n, T, D), generator=g, device=DEV, dtype=torch.float16)
                v = torch.randn((n, T16 // 16, D, 16), generator=g, device=DEV, dtype=torch.float16)
                if T16 > T:
                    v[:, -1, :, 16 - (T16 - T):] = 0
                qp = _queries(case, case["probe_pos"] - 1, g) if case["probe_pos"] > 1 else None
                refs.append(ProbeRef(heads, k, v, q_prev=qp))
                errs.append(torch.empty((B, n * G), dtype=torch.float32, device=DEV))
            s["probes"], s["errs"] = refs, errs
        s["ws"] = dc.workspace(s["probes"][0] if n else None)
    elif kind == "append":
        s["dc"] = dc = _cache(case, seed, g)
        s["q"], s["outs"] = _queries(case, L, g), outs()
        s["phi"], s["u"], s["th"] = _router(case, g, 1, H, T)
        s["x"] = [[torch.randn((B, H, D), generator=g, device=DEV, dtype=torch.float16) for _ in range(2)]
                  for _ in range(L)]
    elif kind == "features":
        s["dc"] = dc = _cache(case, seed, g)
        s["q"], s["outs"] = _queries(case, L, g), outs()
        s["phi"] = torch.zeros((1, H, T, 4), dtype=torch.float32, device=DEV)
    elif kind == "prefill":
        s["dc"] = dc = _cache(case, seed, g, filled=False)
        s["phi"], s["u"], s["th"] = _router(case, g, 1, H, T)
        s["x"] = _dense(case, dc, g, L)
    elif kind == "sketch":
        s["dc"] = dc = _cache(case, seed, g, entries=False)
        x = torch.empty((B, L, 2, max(lens), H, D), dtype=torch.float16, device=DEV)
        for l, kv in enumerate(_dense(dict(case, ragged=False), dc, g, L)):
            for z in range(2):
                x[:, l, z] = kv[z].view(B, case["tokens"], H, D)[:, :max(lens)]
        s["x"] = [x[b, :, :, :n].contiguous() for b, n in enumerate(lens)]
        s["om"] = [torch.randn((L * n, case["rank"]), generator=g, device=DEV, dtype=torch.float16) for n in lens]
    elif kind == "budget":
        s["dc"] = dc = _cache(case, seed, g, entries=False)
        M = L // 4
        s["phi"], s["u"], _ = _router(case, g, M, H, T)
        lo, hi = _levels(case)
        s["entries"] = torch.full((M, H), T * lo + T * (hi - lo) // 10, dtype=torch.int64, device=DEV)
        s["codes"] = torch.empty((M, H, T), dtype=torch.uint8, device=DEV)
        s["offs"] = torch.empty((M, H, T + 1), dtype=torch.int32, device=DEV)
    elif kind == "unfused":
        s["dc"] = dc = _cache(case, seed, g)
        s["q"], s["outs"] = _queries(case, L, g), outs()
        T16 = -(-T // 16) * 16
        s["k"] = torch.empty((H, T, D), dtype=torch.float16, device=DEV)
        s["v"] = torch.empty((H, T16 // 16, D, 16), dtype=torch.float16, device=DEV)
    return s


def run(s):
    case, dc = s["case"], s["dc"]
    kind, L = case["kind"], case["layers"]
    if kind == "decode":
        if not case["probe_heads"]:
            return [dc.decode(l, q=s["q"][l], out=s["outs"][l], workspace=s["ws"]) for l in range(L)]
        return [dc.decode(l, q=s["q"][l], out=s["outs"][l], workspace=s["ws"], probe=s["probes"][l],
                          err=s["errs"][l], with_ref=False)[:2] for l in range(L)]
    if kind == "append":
        # the newest sequence's token is routed here; earlier sequences' slots hold their routed rank
        dc.route_range(s["phi"], s["u"], s["th"], dc.total_tokens - 1, dc.total_tokens)
        outs = [dc.decode_append(l, s["x"][l][0], s["x"][l][1], q=s["q"][l], out=s["outs"][l]) for l in range(L)]
        return {"out": outs, "codes": dc.rank_code, "off": dc.res_off, "k": dc.coef_k, "v": dc.coef_v,
                "idx": dc.res_idx, "val": dc.res_val, "scale": dc.res_scale}
    if kind == "features":
        s["phi"].zero_()                                            # a new feature interval
        outs = [dc.decode_features(l, s["phi"], q=s["q"][l], out=s["outs"][l]) for l in range(L)]
        return {"out": outs, "phi": s["phi"]}
    if kind == "prefill":
        T = dc.total_tokens
        dc.route_range(s["phi"], s["u"], s["th"], 0, T)
        for l in range(L):
            dc.compress(l, s["x"][l][0], s["x"][l][1], 0, T)
        r = {"codes": dc.rank_code, "off": dc.res_off, "k": dc.coef_k, "v": dc.coef_v, "idx": dc.res_idx,
             "val": dc.res_val, "scale": dc.res_scale}
        if case["coef"] == "int8":
            r.update(ks=dc.coef_scale_k, vs=dc.coef_scale_v)
        return r
    if kind == "sketch":
        for b in range(dc.batch):
            dc.sketch_basis(0, b, s["x"][b], s["om"][b])
        return dc.basis
    if kind == "budget":
        return dc.route_budget(s["phi"], s["u"], s["entries"], 0, dc.total_tokens, s["codes"], s["offs"])
    outs = []
    for l in range(L):
        dc.materialize(l, s["k"], s["v"])
        outs.append(dc.dense_decode(s["k"], s["v"], s["q"][l], out=s["outs"][l]))
    return {"out": outs, "k": s["k"], "v": s["v"]}


def work(case):
    lens, L, H, G, rb = _lens(case), case["layers"], case["kv_heads"], case["group"], case["rank"]
    T, B, kind = sum(lens), len(lens), case["kind"]
    rho = _mean_rank(case)
    coef = 2 * rb if case["coef"] == "f16" else rb + rb // 8
    basis = B * H * 2 * rb * D * 2
    # a layer's compressed factors: both coefficient rows, scales and entries, the offsets, the bases
    factors = H * T * (2 * coef + 2 * 2 + 2 * 1.5 * rho + 4) + basis
    qo = B * H * G * D * 6
    attend = 4.0 * T * H * G * (rb + rho)
    if kind in ("decode", "append", "features"):
        w = {"bytes": L * (factors + qo), "flops": L * attend}
        if kind == "append":
            w["bytes"] += L * 2 * B * H * D * 2
        if kind == "features":
            w["bytes"] += H * T * 16                 # the two feature columns, read and written once
        n = case["probe_heads"]
        w["bytes"] += L * n * T * D * 4
        w["flops"] += L * n * case["probe_pos"] * T * G * 4.0 * D
        return w
    if kind == "prefill":
        return {"bytes": H * T * (16 + 1 + 4) + L * (factors + 2 * T * H * D * 2), "flops": L * 2.0 * T * H * 4 * D * rb}
    if kind == "sketch":
        return {"bytes": L * T * (2 * H * D + rb) * 2 + basis, "flops": 2.0 * L * T * 2 * H * D * rb}
    if kind == "budget":
        return {"bytes": (L // 4) * H * T * (16 + 1 + 4), "flops": (L // 4) * H * T * 7.0}
    dense = 2 * H * T * D * 2
    return {"bytes": L * (factors + 2 * dense + qo), "flops": L * (2.0 * 2 * T * H * D * rb + 4.0 * T * H * G * D)}


def tolerance(case):
    kind = case["kind"]
    if kind in ("prefill", "budget"):
        return "exact"                       # defined bit for bit by their order of operations
    if kind == "sketch":
        return {"rel": 1e-5}                 # fp16 bases of float64 sums: an entry may round the other way
    if kind == "unfused":
        return {"rel": 5e-5}                 # fp16 rebuilt rows: some entries round the other way
    return {"rel": 2e-6}                     # float32 sums: 2e-7 to 5e-7 from 64 bits


# ---- the same values in 64 bits ------------------------------------------------------------------

def _key_rows(t, T):        # [H, NB, R/e, 16, e] -> [H, T, R]
    H, NB, ng, b, e = t.shape
    return t.transpose(2, 3).reshape(H, NB * b, ng * e)[:, :T]


def _val_rows(t, T):        # [H, NB, R, e] -> [H, T, R]
    H, NB, R, e = t.shape
    return t.transpose(2, 3).reshape(H, NB * e, R)[:, :T]


def _rows64(dc, l, z, h):
    """Coefficients [T, r_b] and dense residuals [T, D] of one (layer, Z, head), float64."""
    T, rb = dc.total_tokens, dc.basis_rank
    c = (_key_rows if z == 0 else _val_rows)((dc.coef_k if z == 0 else dc.coef_v)[l, h:h + 1], T)[0].double()
    if dc.coef_format == "int8":
        sc = (dc.coef_scale_k if z == 0 else dc.coef_scale_v)[l, h].double()
        c = c * sc.t().repeat_interleave(16, 1)
    off = dc.res_off.view(-1, T + 1)[h].long()
    n = int(off[-1])
    tok = torch.repeat_interleave(torch.arange(T, device=DEV), off[1:] - off[:-1])
    b = dc.res_val[l, z, h].long()
    q = torch.stack([b & 15, b >> 4], 1).flatten()[:n]
    q = torch.where(q > 7, q - 16, q)
    r = torch.zeros((T, D), dtype=torch.float64, device=DEV)
    r[tok, dc.res_idx[l, z, h, :n].long()] = q.double() * dc.res_scale[l, z, h].double()[tok]
    return c, r


def _rebuilt64(dc, l, z, h):
    c, r = _rows64(dc, l, z, h)
    cu = [int(x) for x in dc.cu_host]
    for b in range(dc.batch):
        r[cu[b]:cu[b + 1]] += c[cu[b]:cu[b + 1]] @ dc.basis[b, 0, h, z].double()
    return r


def _attend64(q, k, v, cu, G, trim=0):
    """q [B, G, D] over one head's [T, D] rows: (out [B, G, D], probabilities [T, G])."""
    out = torch.zeros((len(cu) - 1, G, D), dtype=torch.float64, device=DEV)
    prob = torch.zeros((k.shape[0], G), dtype=torch.float64, device=DEV)
    for b in range(len(cu) - 1):
        lo, hi = cu[b], max(cu[b], cu[b + 1] - trim)
        if hi > lo:
            p = torch.softmax(k[lo:hi] @ q[b].double().t() / math.sqrt(D), 0)
            prob[lo:hi] = p
            out[b] = p.t() @ v[lo:hi]
    return out, prob


def exact(case, seed):
    kind, L, H, G, rb = case["kind"], case["layers"], case["kv_heads"], case["group"], case["rank"]
    if kind in ("prefill", "budget", "append"):
        return None                          # whole values, or a state that the pass itself rewrites
    s = prepare(case, seed)
    dc = s["dc"]
    cu, B, T = [int(x) for x in dc.cu_host], dc.batch, dc.total_tokens
    if kind == "sketch":
        got = torch.empty(dc.basis.shape, dtype=torch.float64, device=DEV)
        for b in range(B):
            om = s["om"][b].double()
            n = s["x"][b].shape[2]
            for h in range(H):
                for z in range(2):
                    y = om.t() @ s["x"][b][:, z, :, h].reshape(L * n, D).double()
                    top = y.norm(dim=1).max()
                    rows = []
                    for i in range(rb):
                        v = y[i].clone()
                        for w in rows:
                            v -= (v @ w) * w
                        nv = v.norm()
                        rows.append(v / nv if float(nv) > 1e-9 * float(top) else v * 0)
                    got[b, 0, h, z] = torch.stack(rows)
        return got
    outs = [torch.zeros((B, H * G, D), dtype=torch.float64, device=DEV) for _ in range(L)]
    mass = torch.zeros((H, T), dtype=torch.float64, device=DEV)
    spike = torch.zeros((H, T), dtype=torch.float64, device=DEV)
    errs, dense = [], []
    for l in range(L):
        q = s["q"][l]
        probe = s["probes"][l] if case["probe_heads"] else None
        cols = []
        dense = []
        for h in range(H):
            k, v = _rebuilt64(dc, l, 0, h), _rebuilt64(dc, l, 1, h)
            if kind == "unfused":
                dense.append((k, v))
                k, v = k.half().double(), v.half().double()
            outs[l][:, h * G:(h + 1) * G], p = _attend64(q[:, h * G:(h + 1) * G], k, v, cu, G)
            if kind == "features":
                mass[h] += p.sum(1)
                spike[h] = torch.maximum(spike[h], p.max(1).values)
            if probe is not None and h in probe.kv_heads:
                i = probe.kv_heads.index(h)
                kr, vr = probe.k_ref[i].double(), _val_rows(probe.v_ref[i:i + 1], T)[0].double()
                num = torch.zeros((B, G), dtype=torch.float64, device=DEV)
                den = num.clone()
                for j in range(case["probe_pos"]):
                    qj = (q if j == 0 else probe.q_prev[j - 1])[:, h * G:(h + 1) * G]
                    o, r = _attend64(qj, k, v, cu, G, j)[0], _attend64(qj, kr, vr, cu, G, j)[0]
                    num += (r - o).square().sum(2)
                    den += r.square().sum(2)
                cols.append((i, num.sqrt() / (den.sqrt() + probe.eps)))
        errs.append(torch.cat([c for _, c in sorted(cols, key=lambda x: x[0])], 1) if cols else None)
    if kind == "features":
        phi = torch.zeros((1, H, T, 4), dtype=torch.float64, device=DEV)
        phi[0, :, :, 0], phi[0, :, :, 1] = mass, spike
        return {"out": outs, "phi": phi}
    if kind == "unfused":
        T16 = -(-T // 16) * 16
        k = torch.stack([a for a, _ in dense])
        v = torch.zeros((H, T16, D), dtype=torch.float64, device=DEV)
        v[:, :T] = torch.stack([b for _, b in dense])
        return {"out": outs, "k": k, "v": v.view(H, T16 // 16, 16, D).transpose(2, 3).contiguous()}
    return [(o, e) for o, e in zip(outs, errs)] if case["probe_heads"] else outs
