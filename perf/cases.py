"""Performance cases of the hybrid-batch decoder layer.

What a scheduler has this library do, iteration after iteration: decode-only
batches while no prompt waits, prefill chunks with and without decodes beside
them, several chunks at once, the per-GPU shares of tensor-parallel layers, the
import of one request's keys and values, and whole-model iterations. Shapes
and length distributions are those of hb_workloads; every call goes through
the Python binding of the C ABI.

A case holds plain values only:
  kind      "layer" (hb_run_iteration), "noalloc" (hb_run_iteration_noalloc),
            "append" (hb_append_kv) or "model" (hb_run_model)
  shape     a layer shape of hb_workloads
  chunks, chunk_lo, chunk_hi, off_lo, off_hi   number of prefill chunks, the
            range of their lengths and of the contexts before them
  decodes, ctx_lo, ctx_hi   number of decodes, the range of their contexts
            (spread over the logarithm)
  mix       seed of the lengths, which thus belong to the case
  out       "f32" or "bf16" layer output
  tokens, context           append: tokens written, position of the first
  layers, vocab             model: decoder layers, LM head rows
"""
import math
import random

import numpy as np
import torch

from hb_workloads import SHAPES
from paper_2503_22562_amd import hb

BLOCK = 16


def _layer(name, shape, chunks, decodes, out, mix, kind="layer"):
    n, clo, chi, olo, ohi = chunks
    d, lo, hi = decodes
    return {"name": name, "kind": kind, "shape": shape, "chunks": n, "chunk_lo": clo, "chunk_hi": chi,
            "off_lo": olo, "off_hi": ohi, "decodes": d, "ctx_lo": lo, "ctx_hi": hi, "mix": mix, "out": out}


def listed():
    return [
        # one user decoding alone: the smallest iteration, weights streamed for one row
        _layer("8b-dec1", "llama3-8b", (0, 0, 0, 0, 0), (1, 1501, 1501), "f32", 1),
        # a lightly loaded tensor-parallel replica, called from a loop that may not allocate
        _layer("70b-tp8-dec8", "llama3-70b-tp8-shard", (0, 0, 0, 0, 0), (8, 512, 8192), "bf16", 2, "noalloc"),
        # an ordinary decode queue with no prompt waiting
        _layer("8b-dec32", "llama3-8b", (0, 0, 0, 0, 0), (32, 256, 8192), "bf16", 3),
        # a long decode queue
        _layer("8b-dec256", "llama3-8b", (0, 0, 0, 0, 0), (256, 256, 8192), "f32", 4),
        # the strictest latency tier: a small chunk beside a decode queue
        _layer("8b-chunk128-dec32", "llama3-8b", (1, 128, 128, 0, 0), (32, 256, 8192), "f32", 5),
        # the usual hybrid batch (the benchmark's workload: chunk 512 behind 3431 tokens, 64 decodes)
        _layer("8b-chunk512-dec64", "llama3-8b", (1, 512, 512, 3431, 3431), (64, 512, 4096), "f32", 6),
        # the share of one of two GPUs, odd lengths throughout
        _layer("8b-tp2-chunk777-dec45", "llama3-8b-tp2-shard", (1, 777, 777, 1234, 1234), (45, 300, 6000), "bf16", 7),
        # the relaxed tier: a whole large chunk of a fresh prompt, no decodes
        _layer("8b-chunk2048", "llama3-8b", (1, 2048, 2048, 0, 0), (0, 0, 0), "f32", 8),
        # a busy replica: four chunks of different prompts and a long decode queue
        _layer("8b-4chunks-dec256", "llama3-8b", (4, 256, 1024, 0, 4096), (256, 300, 8192), "f32", 9),
        # import of one request's cached prefix, unaligned at both ends
        {"name": "8b-append3001", "kind": "append", "shape": "llama3-8b", "tokens": 3001, "context": 517},
        # the largest: long-context prefill of the 70B layer beside long decodes
        _layer("70b-chunk2048-dec32", "llama3-70b", (1, 2048, 2048, 30720, 30720), (32, 32768, 32768), "f32", 10),
        # a whole-model call: embedding, four layers, final norm and a 128K-row head
        dict(_layer("8b-model4-chunk256-dec48", "llama3-8b", (1, 256, 256, 1000, 1000), (48, 256, 4096), "bf16", 11,
                    "model"), layers=4, vocab=128256),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    kind = rng.choice(["layer"] * 7 + ["noalloc", "append", "model"])
    mix = rng.randrange(1 << 30)
    if kind == "append":
        shape = rng.choice(["llama3-8b", "llama3-70b", "llama3-8b-tp2-shard", "llama3-70b-tp8-shard"])
        return {"kind": kind, "shape": shape, "tokens": _log_int(rng, 64, 16384), "context": rng.randrange(0, 4096)}
    if kind == "model":
        c = _layer("", "llama3-8b", (rng.randrange(0, 2), 32, 512, 0, 2048), (_log_int(rng, 1, 64), 64, 4096), "bf16", mix,
                   kind)
        del c["name"]
        return dict(c, layers=rng.randrange(1, 5), vocab=128256)
    shapes = ["llama3-8b"] * 5 + ["llama3-8b-tp2-shard"] * 2 + ["llama3-70b-tp8-shard"] * 2
    shape = rng.choice(shapes + ([] if kind == "noalloc" else ["llama3-70b"]))
    big = shape == "llama3-70b"
    chunks = rng.choice([0, 1, 1, 1, 1] if big else [0, 0, 1, 1, 1, 2, 4])
    top = 2048 // max(1, chunks)
    hi = _log_int(rng, 64, top)
    decodes = _log_int(rng, 1, 32 if big else 256)
    if chunks and rng.random() < 0.2:
        decodes = 0
    if kind == "noalloc":  # within its fixed scratch
        chunks, hi, decodes = min(chunks, 1), min(hi, 128), min(decodes, 64)
    c = _layer("", shape, (chunks, max(1, hi // 3 if chunks > 1 else hi), hi, 0, rng.choice([0, 1024, 8192])),
               (decodes, 100, 8192 if not big else 16384), rng.choice(["f32", "bf16"]), mix, kind)
    del c["name"]
    return c


def _lens(case):
    """(chunk_len, context_len) of each request, chunks first: a function of the case alone."""
    rng = random.Random(case["mix"])
    lens = [(rng.randint(case["chunk_lo"], case["chunk_hi"]), rng.randint(case["off_lo"], case["off_hi"]))
            for _ in range(case["chunks"])]
    return lens + [(1, _log_int(rng, case["ctx_lo"], case["ctx_hi"])) for _ in range(case["decodes"])]


def _normal(gen, shape, std=1.0):
    return torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(0.0, std, generator=gen)


def _weights(gen, s):
    qd, f = s.n_q_heads * s.head_dim, s.ffn_dim
    w = {"w_qkv": _normal(gen, (s.qkv_dim, s.hidden), s.hidden ** -0.5),
         "w_o": _normal(gen, (s.hidden, qd), qd ** -0.5),
         "w_gate_up": _normal(gen, (2 * f, s.hidden), s.hidden ** -0.5),
         "w_down": _normal(gen, (s.hidden, f), f ** -0.5)}
    for name in ("g_attn", "g_ffn"):
        w[name] = 1 + _normal(gen, (s.hidden,), 0.1)
    return w


def _pool(gen, s, blocks):
    """A pool whose every slot holds a cached key / value ~ N(0, 1)."""
    return _normal(gen, (blocks, s.n_kv_heads, 16, s.head_dim)), _normal(gen, (blocks, s.n_kv_heads, 16, s.head_dim))


def _inputs(case, seed):
    """Everything on the device that a case's call reads, from the seed alone."""
    s = SHAPES[case["shape"]]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    perm = np.random.default_rng(seed)
    i = {"shape": s}
    if case["kind"] == "append":
        n = -(-(case["context"] + case["tokens"]) // BLOCK)
        i["blocks"] = n + 16
        i["table"] = perm.permutation(i["blocks"])[:n].astype(np.int32)
        i["pools"] = [_pool(gen, s, i["blocks"])]
        i["k"] = _normal(gen, (case["tokens"], s.n_kv_heads, s.head_dim))
        i["v"] = _normal(gen, (case["tokens"], s.n_kv_heads, s.head_dim))
        i["weights"] = [_weights(gen, s)]
        return i
    lens = _lens(case)
    need = [-(-(c + x) // BLOCK) for c, x in lens]
    i["blocks"] = sum(need) + 16
    ids = perm.permutation(i["blocks"]).astype(np.int32)
    ends = np.cumsum(need)
    i["requests"] = [(c, x, ids[e - n:e].copy()) for (c, x), n, e in zip(lens, need, ends)]
    i["tokens"] = sum(c for c, _ in lens)
    layers = case.get("layers", 1)
    i["weights"] = [_weights(gen, s) for _ in range(layers)]
    i["pools"] = [_pool(gen, s, i["blocks"]) for _ in range(layers)]
    if case["kind"] == "model":
        i["embed"] = _normal(gen, (case["vocab"], s.hidden))
        i["lm_head"] = _normal(gen, (case["vocab"], s.hidden), s.hidden ** -0.5)
        i["g_final"] = 1 + _normal(gen, (s.hidden,), 0.1)
        i["ids"] = torch.randint(0, case["vocab"], (i["tokens"],), dtype=torch.int32, device="cuda", generator=gen)
    else:
        i["x"] = _normal(gen, (i["tokens"], s.hidden))
    return i


def prepare(case, seed):
    st = _inputs(case, seed)
    s, kind = st["shape"], case["kind"]
    st["kind"], st["context"] = kind, case.get("context", 0)
    if kind == "append":
        cfg = hb.make_config(s, 64, 8)
    else:
        cfg = hb.make_config(s, max(64, st["tokens"]), max(8, len(st["requests"])))
    if kind == "model":
        st["model"] = hb.hb_create_model(cfg, st["weights"], st["pools"], st["blocks"], st["embed"], st["g_final"],
                                         st["lm_head"])
        n = len(st["requests"])
        st["logits"] = torch.empty((n, case["vocab"]), dtype=torch.float32, device="cuda")
        st["next"] = torch.empty(n, dtype=torch.int32, device="cuda")
        return st
    (k, v), = st["pools"]
    st["layer"] = hb.hb_create_layer(cfg, st["weights"][0], k, v, st["blocks"])
    if kind != "append":
        out = torch.float32 if case["out"] == "f32" else torch.bfloat16
        st["y"] = torch.empty((st["tokens"], s.hidden), dtype=out, device="cuda")
    return st


def run(state):
    kind = state["kind"]
    if kind == "append":
        hb.hb_append_kv(state["layer"], state["table"], state["context"], state["k"], state["v"])
        return {"pools": state["pools"]}
    if kind == "model":
        hb.hb_run_model(state["model"], state["requests"], state["ids"], state["next"], state["logits"])
        return {"logits": state["logits"], "pools": state["pools"]}
    call = hb.hb_run_iteration_noalloc if kind == "noalloc" else hb.hb_run_iteration
    call(state["layer"], state["requests"], state["x"], state["y"])
    return {"y": state["y"], "pools": state["pools"]}


def work(case):
    s = SHAPES[case["shape"]]
    tok = 2 * s.n_kv_heads * s.head_dim * 2  # bytes of one token's K and V
    if case["kind"] == "append":
        return {"bytes": 2 * case["tokens"] * tok, "flops": 0}
    lens = _lens(case)
    t = sum(c for c, _ in lens)
    pairs = sum(c * x + c * (c + 1) / 2 for c, x in lens)
    layers = case.get("layers", 1)
    flops = layers * (2.0 * t * s.linear_params + 4.0 * s.n_q_heads * s.head_dim * pairs)
    nbytes = layers * (2.0 * s.linear_params + 4.0 * s.hidden  # weights and gains
                       + sum(x for _, x in lens) * tok         # cached K and V read
                       + t * tok)                              # new K and V written
    if case["kind"] == "model":
        nbytes += t * (4 + 2 * s.hidden) + 2.0 * case["vocab"] * s.hidden + 2.0 * s.hidden
        nbytes += len(lens) * (4.0 * case["vocab"] + 4)
        flops += 2.0 * len(lens) * case["vocab"] * s.hidden
    else:
        nbytes += t * s.hidden * (2 + (4 if case["out"] == "f32" else 2))
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["kind"] == "append":
        return "exact"  # a copy
    if case["kind"] == "model":
        # four times what other tiles and K splits change (rel 0.0047, max 0.031):
        # bf16 hidden states between the layers carry every rounding on
        return {"rel": 0.019, "max": 0.13}
    # four times what other tiles, K splits and key splits change (rel up to
    # 0.0013, max 0.0078: one rounding of a bf16 intermediate or output)
    return {"rel": 0.005, "max": 0.032}


# --- the same results in fp64 ---------------------------------------------------
def _k_index(hd):
    """Flat positions of K[slot][dim] inside a stored block of one kv head."""
    s, d = np.meshgrid(np.arange(16), np.arange(hd), indexing="ij")
    i = (((s // 4) % 2) * (hd // 8) + d // 8) * 64 + (4 * (s // 8) + s % 4) * 8 + d % 8
    return torch.from_numpy(i.reshape(-1)).cuda()


def _v_index(hd):
    s, d = np.meshgrid(np.arange(16), np.arange(hd), indexing="ij")
    i = ((s // 8) * hd + d) * 8 + s % 8
    return torch.from_numpy(i.reshape(-1)).cuda()


def _read(pool, index, table, n):
    """[n][n_kv][hd] of the first n positions behind a block table."""
    nb, nkv, _, hd = pool.shape
    rows = pool.view(nb, nkv, 16 * hd)[torch.from_numpy(table).long().cuda()][:, :, index]
    return rows.view(len(table), nkv, 16, hd).transpose(1, 2).reshape(-1, nkv, hd)[:n]


def _write(pool, index, table, start, x):
    nb, nkv, _, hd = pool.shape
    pos = torch.arange(start, start + x.shape[0], device="cuda")
    blk = torch.from_numpy(table).long().cuda()[pos // BLOCK]
    at = index.view(16, hd)[pos % BLOCK]                                          # [n][hd]
    head = torch.arange(nkv, device="cuda")
    flat = (blk[:, None, None] * nkv + head[None, :, None]) * (16 * hd) + at[:, None, :]
    pool.view(-1)[flat.reshape(-1)] = x.reshape(-1)


def _rms(x, g, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * g


def _rope(z, pos, theta):
    hd = z.shape[-1]
    j = torch.arange(hd // 2, dtype=torch.float64, device="cuda")
    phi = (pos.double()[:, None] * theta ** (-2.0 * j / hd)[None, :])[:, None, :]
    c, s = torch.cos(phi), torch.sin(phi)
    u, w = z[..., :hd // 2], z[..., hd // 2:]
    return torch.cat([u * c - w * s, w * c + u * s], -1)


def _layer64(s, w, kp, vp, requests, x):
    """The decoder layer over the batch; kp, vp: fp64 pools, updated."""
    nq, nkv, hd, group = s.n_q_heads, s.n_kv_heads, s.head_dim, s.n_q_heads // s.n_kv_heads
    ki, vi = _k_index(hd), _v_index(hd)
    t = x.shape[0]
    pos = torch.cat([torch.arange(c0, c0 + c, device="cuda") for c, c0, _ in requests])
    qkv = _rms(x, w["g_attn"].double(), s.rms_eps) @ w["w_qkv"].double().T
    q = _rope(qkv[:, :nq * hd].view(t, nq, hd), pos, s.rope_theta)
    k = _rope(qkv[:, nq * hd:(nq + nkv) * hd].view(t, nkv, hd), pos, s.rope_theta)
    v = qkv[:, (nq + nkv) * hd:].view(t, nkv, hd)
    o = torch.empty_like(q)
    at = 0
    for c, ctx, table in requests:
        _write(kp, ki, table, ctx, k[at:at + c])
        _write(vp, vi, table, ctx, v[at:at + c])
        at += c
    at = 0
    for c, ctx, table in requests:
        kc, vc = _read(kp, ki, table, ctx + c), _read(vp, vi, table, ctx + c)
        late = torch.arange(ctx + c, device="cuda")[None, :] > torch.arange(ctx, ctx + c, device="cuda")[:, None]
        for h in range(nkv):
            kh, vh = kc[:, h].contiguous(), vc[:, h].contiguous()
            for g in range(h * group, (h + 1) * group):
                sc = (q[at:at + c, g].contiguous() @ kh.T).mul_(hd ** -0.5)
                sc.masked_fill_(late, -math.inf)
                o[at:at + c, g] = torch.softmax(sc, -1) @ vh
        at += c
    h2 = x + o.view(t, nq * hd) @ w["w_o"].double().T
    f = _rms(h2, w["g_ffn"].double(), s.rms_eps)
    gate = f @ w["w_gate_up"][:s.ffn_dim].double().T
    up = f @ w["w_gate_up"][s.ffn_dim:].double().T
    return h2 + (gate * torch.sigmoid(gate) * up) @ w["w_down"].double().T


def exact(case, seed):
    i = _inputs(case, seed)
    s = i["shape"]
    pools = [(k.double(), v.double()) for k, v in i["pools"]]
    if case["kind"] == "append":
        (kp, vp), = pools
        _write(kp, _k_index(s.head_dim), i["table"], case["context"], i["k"].double())
        _write(vp, _v_index(s.head_dim), i["table"], case["context"], i["v"].double())
        return {"pools": pools}
    model = case["kind"] == "model"
    x = (i["embed"][i["ids"].long()] if model else i["x"]).double()
    for w, (kp, vp) in zip(i["weights"], pools):
        x = _layer64(s, w, kp, vp, i["requests"], x)
    if not model:
        return {"y": x, "pools": pools}
    last = torch.from_numpy(np.cumsum([c for c, _, _ in i["requests"]]) - 1).cuda()
    logits = _rms(x[last], i["g_final"].double(), s.rms_eps) @ i["lm_head"].double().T
    return {"logits": logits, "pools": pools}
