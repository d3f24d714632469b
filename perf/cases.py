"""The calls whose speed matters to a user of this package, as timed cases.

A serving program holds a paged KV cache per layer and, for every token it
decodes, appends the new token's K and V and runs decode attention over the
batch; now and then it moves blocks between the GPU cache and a host cache, and
part of the batch may be decoded by the host CPU. The cases cover those calls
through the package's public entry points, from one short request to the
largest layer, with the head counts, length mixes, cache layouts and launch
forms that such programs use.

A case is a dict of plain values:

* ``op``: ``decode`` (one ``decode_attention``), ``append`` (one ``kv_append``),
  ``copy`` (one ``copy_blocks``), ``layers`` (append and decode of several layers
  replayed from one HIP graph) or ``cpu`` (one ``cpu_decode_attention``);
* ``hq``, ``hkv``: query and kv heads; head_dim is 128 and a block 16 tokens;
* ``batch``, ``mix``, ``lo``, ``hi``: requests and their cached lengths (``uniform``
  in [lo, hi], ``lognormal`` with median lo and sigma 0.6 clipped to [128, hi],
  ``skew``: 8 requests of hi tokens among requests uniform in [16, lo]), drawn
  from ``lens_seed``;
* ``layout``: ``interleaved`` (``new_kv_cache``) or ``dense`` (two allocations).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2411_01142_amd as neo

D = 128   # head dim
BS = 16   # tokens per block


def _decode(name, hq, hkv, batch, mix, lo, hi, layout="interleaved"):
    return {"name": name, "op": "decode", "hq": hq, "hkv": hkv, "batch": batch, "mix": mix,
            "lo": lo, "hi": hi, "layout": layout, "lens_seed": 11}


def listed():
    return [
        # One interactive user of an 8B-shaped model, a chat of under a thousand
        # tokens: the smallest call, where launch and latency are everything.
        _decode("one_short", 32, 8, 1, "uniform", 877, 877),
        # One user with a long document in context: a single sequence has to fill
        # the whole chip.
        _decode("one_long", 32, 8, 1, "uniform", 50021, 50021),
        # A small batch of a 7B-shaped layer without grouped heads (config 1).
        _decode("mha_small", 32, 32, 4, "uniform", 64, 512),
        # Ordinary serving batches of an 8B-shaped layer (config 2), and
        # summarisation-like lengths over two separate dense caches (config 3).
        _decode("serve_64", 32, 8, 64, "uniform", 512, 2048),
        _decode("summarise_256", 32, 8, 256, "lognormal", 1500, 8192, "dense"),
        # The largest: a 70B-shaped layer with code-generation-like lengths
        # (config 4), and one GPU's share of it at 8-way tensor parallelism
        # (config 6).
        _decode("layer70b_512", 64, 8, 512, "uniform", 256, 4096),
        _decode("layer70b_tp8", 8, 1, 512, "uniform", 256, 4096),
        # Many short requests next to a few very long ones (config 5).
        _decode("skewed_1024", 32, 8, 1024, "skew", 256, 32768),
        # The token loop of a small-batch server: append and decode of eight
        # layers captured once in a HIP graph and replayed per token.
        {"name": "token_graph", "op": "layers", "layers": 8, "hq": 32, "hkv": 8, "batch": 13,
         "mix": "uniform", "lo": 100, "hi": 1500, "layout": "interleaved", "lens_seed": 12},
        # The cache write of a large batch, one layer, by itself.
        {"name": "append_256", "op": "append", "hq": 32, "hkv": 8, "batch": 256,
         "mix": "uniform", "lo": 64, "hi": 1024, "layout": "interleaved", "lens_seed": 13},
        # One request of about 4 000 tokens swapped out to a pinned host cache.
        {"name": "swap_out", "op": "copy", "way": "out", "hkv": 8, "blocks": 253,
         "layout": "interleaved"},
        # The requests whose KV lives in host memory, decoded by the host CPU.
        {"name": "host_16", "op": "cpu", "hq": 32, "hkv": 8, "batch": 16, "mix": "uniform",
         "lo": 256, "hi": 2048, "layout": "dense", "lens_seed": 14},
    ]


def draw(rng):
    """One more case of the ranges above."""
    def logu(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choices(["decode", "layers", "append", "copy", "cpu"], [14, 2, 2, 2, 1])[0]
    layout = rng.choice(["interleaved", "interleaved", "dense"])
    if op == "copy":
        way = rng.choice(["out", "in", "device"])
        return {"op": op, "way": way, "hkv": rng.choice([1, 2, 8, 8, 16, 32]),
                "blocks": logu(4, 1000 if way != "device" else 8000), "layout": layout}
    hkv = rng.choice([1, 2, 4, 8, 8, 8, 16, 32])
    group = rng.choice([g for g in (1, 2, 4, 4, 8, 8, 16) if hkv * g <= 128])
    most = {"decode": 3e9, "layers": 5e8, "append": 1e9, "cpu": 2e8}[op]  # bytes of K and V
    batch = logu(1, {"decode": 1000, "layers": 64, "append": 600, "cpu": 32}[op])
    mean = min(logu(40, 60000), most / (batch * hkv * 512))
    mean = max(mean, 17)
    mix = rng.choice(["uniform", "uniform", "lognormal"]) if mean >= 256 else "uniform"
    if batch >= 64 and mean >= 600 and rng.random() < 0.4:
        # the same tokens, half of them in eight long requests
        mix, lo, hi = "skew", int(mean), int(batch * mean / 16)
    elif mix == "lognormal":
        lo, hi = int(mean / 1.3), int(mean * 5)
    else:
        spread = rng.choice([0.0, 0.5, 0.8])
        lo, hi = max(1, int(mean * (1 - spread))), int(mean * (1 + spread))
    case = {"op": op, "hq": hkv * group, "hkv": hkv, "batch": batch, "mix": mix, "lo": lo,
            "hi": hi, "layout": "dense" if op == "cpu" else layout,
            "lens_seed": rng.randrange(1 << 20)}
    if op == "layers":
        case["layers"] = rng.randint(2, 8)
    return case


# ------------------------------------------------------------------ inputs

def _lens(case):
    """Cached length of each request, the token being decoded included."""
    r = np.random.default_rng(case["lens_seed"])
    B, lo, hi = case["batch"], case["lo"], case["hi"]
    if case["mix"] == "lognormal":
        x = r.lognormal(mean=math.log(lo), sigma=0.6, size=B)
        return np.clip(np.rint(x), min(128, hi), hi).astype(np.int32)
    if case["mix"] == "skew":
        x = r.integers(16, max(16, lo), size=B, endpoint=True)
        x[r.choice(B, size=8, replace=False)] = hi
        return x.astype(np.int32)
    return r.integers(lo, hi, size=B, endpoint=True).astype(np.int32)


def _table(lens, seed):
    """(block table, blocks in the pool): every request's blocks scattered over a
    pool with 5 % spare blocks, as after some time of serving; -1 where unused."""
    nblk = (lens.astype(np.int64) + BS - 1) // BS
    pool = int(nblk.sum()) + math.ceil(0.05 * int(nblk.sum()))
    perm = np.random.default_rng(seed).permutation(pool).astype(np.int32)
    table = np.full((len(lens), int(nblk.max())), -1, np.int32)
    used = np.arange(table.shape[1])[None, :] < nblk[:, None]
    table[used] = perm[:int(nblk.sum())]
    return table, pool


def _normal(shape, gen, device="cuda"):
    return torch.randn(shape, generator=gen, device=device, dtype=torch.bfloat16)


def _caches(blocks, hkv, layout, gen, pinned=False):
    """K and V caches filled with N(0, 1) values."""
    if layout == "interleaved":
        k, v = neo.new_kv_cache(blocks, hkv, device="cuda")
    else:
        k = torch.empty((blocks, hkv, D // 8, BS, 8), dtype=torch.bfloat16, device="cuda")
        v = torch.empty((blocks, hkv, D, BS), dtype=torch.bfloat16, device="cuda")
    for c in (k, v):
        for i in range(0, blocks, 8192):
            part = c[i:i + 8192]
            part.copy_(_normal(part.shape, gen))
    if pinned:
        hk = torch.empty(k.shape, dtype=k.dtype, pin_memory=True)
        hv = torch.empty(v.shape, dtype=v.dtype, pin_memory=True)
        k, v = hk.copy_(k), hv.copy_(v)
    return k, v


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _batch(case, seed, layers=1):
    gen = _gen(seed)
    lens = _lens(case)
    table, pool = _table(lens, seed)
    B, hq, hkv = case["batch"], case["hq"], case["hkv"]
    kv = [_caches(pool, hkv, case["layout"], gen) for _ in range(layers)]
    return {"q": [_normal((B, hq, D), gen) for _ in range(layers)],
            "k_new": [_normal((B, hkv, D), gen) for _ in range(layers)],
            "v_new": [_normal((B, hkv, D), gen) for _ in range(layers)],
            "k": [k for k, _ in kv], "v": [v for _, v in kv],
            "table": torch.from_numpy(table).cuda(), "lens": torch.from_numpy(lens).cuda()}


def _copy_setup(case, seed):
    gen = _gen(seed)
    n, hkv, way = case["blocks"], case["hkv"], case["way"]
    r = np.random.default_rng(seed)
    src_blocks, dst_blocks = n + n // 4 + 1, n + n // 8 + 3
    src = _caches(src_blocks, hkv, "dense" if way == "in" else case["layout"], gen, way == "in")
    dst = _caches(dst_blocks, hkv, "dense" if way == "out" else case["layout"], gen, way == "out")
    return {"src": src, "dst": dst,
            "src_ids": torch.from_numpy(r.permutation(src_blocks)[:n].astype(np.int32)).cuda(),
            "dst_ids": torch.from_numpy(r.permutation(dst_blocks)[:n].astype(np.int32)).cuda()}


def _token(s, workspace):
    """One token through the layers: each layer's append, then its attention."""
    outs = []
    for q, k, v, kn, vn in zip(s["q"], s["k"], s["v"], s["k_new"], s["v_new"]):
        neo.kv_append(k, v, kn, vn, s["table"], s["lens"])
        outs.append(neo.decode_attention(q, k, v, s["table"], s["lens"], workspace=workspace))
    return outs


def prepare(case, seed):
    op = case["op"]
    if op == "copy":
        return {"op": op, **_copy_setup(case, seed)}
    s = {"op": op, **_batch(case, seed, case.get("layers", 1))}
    if op == "layers":
        ws = neo.new_workspace(case["batch"], case["hq"], case["hkv"])
        _token(s, ws)  # warm-up before the capture
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            outs = _token(s, ws)
        s.update(graph=graph, outs=outs, workspace=ws)
    elif op == "cpu":
        for name in ("q", "k", "v"):
            s[name] = [t.cpu() for t in s[name]]
        s["table"], s["lens"] = s["table"].cpu(), s["lens"].cpu()
    return s


def run(s):
    op = s["op"]
    if op == "decode":
        return neo.decode_attention(s["q"][0], s["k"][0], s["v"][0], s["table"], s["lens"])
    if op == "layers":
        s["graph"].replay()
        return s["outs"]
    if op == "append":
        neo.kv_append(s["k"][0], s["v"][0], s["k_new"][0], s["v_new"][0], s["table"], s["lens"])
        return [s["k"][0], s["v"][0]]
    if op == "copy":
        neo.copy_blocks(*s["src"], *s["dst"], s["src_ids"], s["dst_ids"])
        return list(s["dst"])
    return neo.cpu_decode_attention(s["q"][0], s["k"][0], s["v"][0], s["table"], s["lens"])


# -------------------------------------------------------------- accounting

def work(case):
    if case["op"] == "copy":
        one = case["blocks"] * case["hkv"] * 2 * D * BS * 2  # K and V, bf16
        return {"bytes": 2 * one + 8 * case["blocks"], "flops": 0}
    lens = _lens(case).astype(np.int64)
    B, hq, hkv = case["batch"], case["hq"], case["hkv"]
    append = B * hkv * D * 2 * 2 * 2 + 8 * B  # rows read and written, table entry, length
    if case["op"] == "append":
        return {"bytes": append, "flops": 0}
    tokens = int(lens.sum())
    decode = (tokens * hkv * D * 2 * 2 + B * hq * D * (2 + 4)
              + 4 * int(((lens + BS - 1) // BS).sum()) + 4 * B)
    flops = tokens * hq * D * 4
    if case["op"] == "layers":
        return {"bytes": case["layers"] * (decode + append), "flops": case["layers"] * flops}
    return {"bytes": decode, "flops": flops}


def tolerance(case):
    # Data movement keeps every bit. Attention reads bf16 and sums in fp32, the
    # softmax weights carried with about 16 mantissa bits or more: 1.5e-6 to 3e-6
    # from the 64-bit result in the 2-norm.
    if case["op"] in ("append", "copy"):
        return "exact"
    return {"rel": 1e-5, "max": 2e-4}


def exact(case, seed):
    """What ``run`` returns for these inputs, in 64 bits and without the package's
    kernels: the softmax attention of every request over its gathered rows."""
    if case["op"] in ("append", "copy"):
        return None
    s = _batch(case, seed, case.get("layers", 1))
    lens, table = _lens(case), s["table"].to(torch.int64)
    B, hq, hkv = case["batch"], case["hq"], case["hkv"]
    outs = []
    for q, k, v, kn, vn in zip(s["q"], s["k"], s["v"], s["k_new"], s["v_new"]):
        out = torch.zeros((B, hq, D), dtype=torch.float64, device="cuda")
        for b in range(B):
            L = int(lens[b])
            ids = table[b, :(L + BS - 1) // BS]
            # [blocks, hkv, piece, slot, 8] and [blocks, hkv, dim, slot] to [hkv, token, dim]
            K = k[ids].permute(1, 0, 3, 2, 4).reshape(hkv, -1, D)[:, :L].double()
            V = v[ids].permute(1, 0, 3, 2).reshape(hkv, -1, D)[:, :L].double()
            if case["op"] == "layers":
                K[:, L - 1], V[:, L - 1] = kn[b].double(), vn[b].double()
            Q = q[b].double().reshape(hkv, hq // hkv, D)
            scores = torch.matmul(Q, K.transpose(1, 2).contiguous()) / math.sqrt(D)
            out[b] = torch.matmul(torch.softmax(scores, dim=2), V.contiguous()).reshape(hq, D)
        outs.append(out)
    if case["op"] == "layers":
        return outs
    return outs[0].cpu().numpy() if case["op"] == "cpu" else outs[0]
