"""Timed cases of the pipeline stage: what a serving program asks of it.

A case is one call of the stage through ``harness.DeviceStage``: a prefill, a
decode or a mixed step over a few consecutive layers, and on a model's last
stage the logits after it. Model shapes, batch sizes, chunk budgets and
context ranges are those of the repository's workloads (``synth.WORKLOADS``,
``bench.py``) and tests. Layers and requests are synthetic: projections
N(0, 0.02^2), gains 1 + N(0, 0.02^2), hidden rows and cached keys and values
N(0, 1), block tables scattered over the pool.

Fields of a case (plain values):
  shape, tp    model shape and the tensor-parallel degree whose one rank's
               share of a layer is held (heads and FFN divided by it)
  dtype        "bf16" or "f32"
  layers       consecutive layers of the stage
  prompts      prefill chunks as "rows@context rows@context ..." ("" for none)
  decodes      sequences that decode one token, with contexts uniform on
               [ctx_lo, ctx_hi]
  logits       the final norm and the vocabulary projection of every decode row
"""

from __future__ import annotations

import math

import numpy as np
import torch

# hidden, query heads, kv heads, head_dim, ffn, layer eps, rotary base, q/k norm
SHAPES = {
    "tiny": (256, 4, 2, 64, 704, 1e-5, 5e5, False),
    "small-qk": (512, 8, 1, 128, 768, 1e-6, 1e6, True),
    "l70": (8192, 64, 8, 128, 28672, 1e-5, 5e5, False),
    "q32": (5120, 64, 8, 128, 25600, 1e-6, 1e6, True),
}
BLOCK = 16
VOCAB = 128256
MAX_TOKENS, MAX_SEQS = 2176, 132  # a serving stage: 2048 prefill + 128 decode rows per step


def _case(name, shape, layers, prompts="", decodes=0, ctx=(0, 0), tp=1, dtype="bf16",
          logits=False):
    c = {"shape": shape, "tp": tp, "dtype": dtype, "layers": layers, "prompts": prompts,
         "decodes": decodes, "ctx_lo": ctx[0], "ctx_hi": ctx[1], "logits": logits}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the two-layer test stage: a decode step of its 4 requests, the
        # smallest call there is (latency and launches)
        _case("tiny decode 4", "tiny", 2, decodes=4, ctx=(16, 80)),
        # ... and the prefill of its 4 prompts of 16-64 tokens in the fp32 mode
        _case("tiny f32 prefill", "tiny", 2, "41@0 17@0 64@0 29@0", dtype="f32"),
        # the fp32 mode as it is used to check a model: prompts, a
        # continuation chunk and decodes in one step (head_dim 128, q/k norm)
        _case("small f32 mixed", "small-qk", 2, "211@0 150@97 61@640", 16, (30, 900),
              dtype="f32"),
        # one interactive request on the 70B-shaped stage
        _case("l70 decode 1", "l70", 4, decodes=1, ctx=(3500, 3500)),
        # the decode workload: 64 requests, contexts 512-2048
        _case("l70 decode 64", "l70", 4, decodes=64, ctx=(512, 2048)),
        # a few requests that migrated or grew to long contexts
        _case("l70 decode long", "l70", 2, decodes=3, ctx=(20000, 65000)),
        # a full serving batch on the last stage: 128 decodes and their logits
        _case("l70 decode 128 logits", "l70", 2, decodes=128, ctx=(1024, 4096), logits=True),
        # one of 8 tensor-parallel ranks, static batch 32 (763-994 tokens)
        _case("l70 tp8 decode 32", "l70", 8, decodes=32, ctx=(763, 994), tp=8),
        # continuous batching: 4 chunks of 512 behind prefixes, 128 decodes
        _case("q32 mixed", "q32", 2, "512@0 512@512 512@1024 512@1536", 128, (256, 4096)),
        # a whole prefill budget: the end of one prompt and the start of another
        _case("l70 prefill 2048", "l70", 2, "1193@2048 855@0"),
        # what is left of a prompt after whole chunks, with a new short one
        _case("l70 prefill tail", "l70", 2, "154@3535 37@0"),
        # KV recomputation of a migrated request: its last whole chunk
        _case("l70 recompute", "l70", 1, "2048@61440"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges: a decode, prefill or mixed step of a
    serving shape (or a rank's share of it), or a step of the small shapes."""
    most = {k: max(work(c)[k] for c in listed()) for k in ("bytes", "flops")}
    while True:
        kind = rng.choice(["decode", "decode", "prefill", "prefill", "mixed", "small", "small"])
        if kind == "small":
            shape = rng.choice(["tiny", "small-qk"])
            dtype = rng.choice(["bf16", "f32"])
            rows, n = _log_int(rng, 1, 420), rng.randint(1, 3)
            chunks = ["%d@%d" % (max(1, rows // n), _log_int(rng, 1, 600) - 1) for _ in range(n)]
            d = rng.choice([0, rng.randint(1, 16)])
            c = _case(None, shape, 2, " ".join(chunks) if d == 0 or rng.random() < 0.5 else "",
                      d, (1, rng.randint(2, 900)), dtype=dtype)
        else:
            shape, tp, layers = rng.choice([("l70", 1, 2), ("q32", 1, 2), ("l70", 2, 3),
                                            ("l70", 4, 4), ("l70", 8, 8)])
            prompts, d, lo, hi = "", 0, 0, 0
            if kind != "decode":
                rows, n = _log_int(rng, 17, 2048), rng.randint(1, 4)
                long = rng.random() < 0.3
                prompts = " ".join("%d@%d" % (max(1, rows // n - rng.randint(0, 7)),
                                              _log_int(rng, 1, 30000 if long else 4096) - 1)
                                   for _ in range(n))
            if kind != "prefill":
                d = _log_int(rng, 1, 128)
                hi = _log_int(rng, 64, min(65000, 600000 // d))
                lo = rng.randint(hi // 4, hi)
            c = _case(None, shape, layers, prompts, d, (lo, hi), tp,
                      logits=kind == "decode" and tp == 1 and rng.random() < 0.3)
        w = work(c)
        if all(w[k] <= most[k] for k in most):
            return c


def _dims(case):
    H, nq, nkv, d, F, eps, theta, qk = SHAPES[case["shape"]]
    tp = case["tp"]
    return H, nq // tp, nkv // tp, d, F // tp, eps, theta, qk


def _lengths(case):
    """(prefill rows, prefill contexts, decode contexts), of the case alone."""
    pairs = [p.split("@") for p in case["prompts"].split()]
    q = np.array([int(a) for a, _ in pairs], np.int32)
    c = np.array([int(b) for _, b in pairs], np.int32)
    r = np.random.default_rng([case["decodes"], case["ctx_lo"], case["ctx_hi"]])
    d = r.integers(case["ctx_lo"], case["ctx_hi"] + 1, size=case["decodes"]).astype(np.int32)
    return q, c, d


def _weight_shapes(case):
    H, nq, nkv, d, F, _, _, qk = _dims(case)
    s = {"attn_norm": (H,), "w_qkv": ((nq + 2 * nkv) * d, H), "w_o": (H, nq * d),
         "ffn_norm": (H,), "w_gate_up": (2 * F, H), "w_down": (H, F)}
    if qk:
        s.update(q_norm=(d,), k_norm=(d,))
    return s


def _normal(seed, key, shape, dtype, mean=0.0, std=1.0):
    g = torch.Generator(device="cuda")
    g.manual_seed((seed * 1_000_003 + key * 7919 + 17) & 0x7FFFFFFFFFFF)
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(mean, std, generator=g)


def _inputs(case, seed):
    """Row-major weights, KV pool, block tables and hidden rows, from the seed."""
    H, nq, nkv, d, F, _, _, _ = _dims(case)
    td = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    layers = []
    for l in range(case["layers"]):
        w = {}
        for i, (name, shp) in enumerate(sorted(_weight_shapes(case).items())):
            gain = len(shp) == 1
            w[name] = _normal(seed, 100 + 16 * l + i, shp, td, 1.0 if gain else 0.0, 0.02)
        layers.append(w)
    q, c, dc = _lengths(case)
    ends = np.concatenate([c + q, dc + 1])
    nblk = (ends + BLOCK - 1) // BLOCK
    num_blocks = int(nblk.sum()) + 3
    ids = np.random.default_rng([seed, 5]).permutation(num_blocks).astype(np.int32)
    tables = np.zeros((len(ends), int(nblk.max())), np.int32)
    at = 0
    for i, n in enumerate(nblk):
        tables[i, :n] = ids[at:at + n]
        at += n
    pool = _normal(seed, 1, (case["layers"], num_blocks, nkv, 2, BLOCK * d), td)
    T = int(q.sum()) + len(dc)
    x = _normal(seed, 2, (T, H), td)
    head = None
    if case["logits"]:
        head = (_normal(seed, 3, (H,), td, 1.0, 0.02), _normal(seed, 4, (VOCAB, H), td, 0.0, 0.02))
    return layers, pool, tables, x, head


def prepare(case, seed):
    from paper_2606_18600_amd import synth
    from paper_2606_18600_amd.harness import DeviceStage, pack_layer, pack_lm_head, model_config

    H, nq, nkv, d, F, eps, theta, qk = _dims(case)
    layers, pool, tables, x, head = _inputs(case, seed)
    q, c, dc = _lengths(case)
    shape = synth.ModelShape(case["shape"], H, nq, nkv, d, F, eps, theta, qk, qk_rms_eps=1e-6)
    longest = int(max(np.concatenate([c + q, dc + 1])))
    max_position = 8192 if longest <= 8192 else 65536
    cfg = model_config(shape, case["dtype"], max_position)
    layers = [pack_layer(cfg, w, free_source=True) for w in layers]
    big = H >= 4096
    st = DeviceStage(shape, case["dtype"], 0, layers, pool.shape[1],
                     MAX_TOKENS if big else max(512, len(x)), MAX_SEQS if big else 32,
                     max_position, kv_pool=pool.reshape(-1), packed=True)
    bt = torch.from_numpy(tables).cuda()
    state = {"stage": st, "q": q, "c": c, "d": dc, "x": x, "out": torch.empty_like(x),
             "pbt": bt[:len(q)].contiguous(), "dbt": bt[len(q):].contiguous(), "pool": pool}
    if head is not None:
        state["norm"], state["head"] = head[0], pack_lm_head(cfg, head[1])
        state["logits"] = torch.empty((len(x), VOCAB), dtype=torch.float32, device="cuda")
        torch.cuda.synchronize()
    return state


def run(s):
    st, x, out = s["stage"], s["x"], s["out"]
    if len(s["q"]) and len(s["d"]):
        st.mixed(s["q"], s["c"], s["pbt"], s["d"], s["dbt"], x, out)
    elif len(s["q"]):
        st.prefill(s["q"], s["c"], s["pbt"], x, out)
    else:
        st.decode(s["d"], s["dbt"], x, out)
    r = {"hidden": out, "kv": s["pool"]}
    if "head" in s:
        r["logits"] = st.lm_head(s["norm"], s["head"], out, logits=s["logits"])
    return r


def work(case):
    H, nq, nkv, d, F, _, _, _ = _dims(case)
    q, c, dc = (a.astype(np.int64) for a in _lengths(case))
    L, es = case["layers"], 2 if case["dtype"] == "bf16" else 4
    T = int(q.sum()) + len(dc)
    params = sum(int(np.prod(s)) for s in _weight_shapes(case).values())
    mats = params - 2 * H
    pairs = int((q * c + q * (q + 1) // 2).sum() + (dc + 1).sum())
    kv_row = 2 * nkv * d * es
    nbytes = L * (params * es + int(c.sum() + dc.sum() + T) * kv_row) + 2 * T * H * es
    flops = L * (2 * T * mats + 4 * d * nq * pairs)
    if case["logits"]:
        nbytes += VOCAB * H * es + T * VOCAB * 4
        flops += 2 * T * VOCAB * H
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # bf16 activations, keys, values and probabilities are rounded several
    # times in each layer (2^-9 each); against 64 bits the step measured
    # 0.002-0.008 where the contexts are given and 0.010-0.013 where a whole
    # prompt passes through two layers, and two implementations that round
    # apart differ by about as much again. The fp32 mode rounds nothing
    # (measured 6e-8 to 1.2e-7); its sums may run in another order.
    if case["dtype"] == "f32":
        return {"rel": 1e-6, "max": 4e-5}
    return {"rel": 2e-2, "max": 0.3}


def _koff(d):
    o, e = np.meshgrid(np.arange(BLOCK), np.arange(d), indexing="ij")
    return torch.from_numpy((e // 32) * 512 + (o + 16 * ((e % 32) // 8)) * 8 + e % 8).cuda()


def _voff(d):
    o, e = np.meshgrid(np.arange(BLOCK), np.arange(d), indexing="ij")
    return torch.from_numpy((e // 32) * 512 + (e % 16 + 16 * (o // 4)) * 8
                            + ((e // 16) % 2) * 4 + o % 4).cuda()


def exact(case, seed):
    """The step in 64 bits: textbook RMSNorm, rotate-half rotary embedding,
    causal grouped-query attention over the gathered cache, SwiGLU."""
    H, nq, nkv, d, F, eps, theta, qk = _dims(case)
    layers, pool, tables, x, head = _inputs(case, seed)
    q, c, dc = _lengths(case)
    pool = pool.double()
    x = x.double()
    koff, voff = _koff(d), _voff(d)
    seqs = [(int(a), int(b)) for a, b in zip(q, c)] + [(1, int(b)) for b in dc]
    pos = torch.cat([torch.arange(b, b + a) for a, b in seqs]).double().cuda()
    inv = theta ** (-2.0 * torch.arange(d // 2, dtype=torch.float64, device="cuda") / d)
    ang = pos[:, None] * inv[None, :]
    cos, sin = ang.cos()[:, None, :], ang.sin()[:, None, :]

    def norm(v, g, e):
        return v / torch.sqrt((v * v).mean(-1, keepdim=True) + e) * g.double()

    def rotate(v):
        a, b = v[..., :d // 2], v[..., d // 2:]
        return torch.cat([a * cos - b * sin, a * sin + b * cos], -1)

    for l, w in enumerate(layers):
        h = norm(x, w["attn_norm"], eps)
        p = (h @ w["w_qkv"].double().T).view(len(x), nq + 2 * nkv, d)
        Q, K, V = p[:, :nq], p[:, nq:nq + nkv], p[:, nq + nkv:]
        if qk:
            Q, K = norm(Q, w["q_norm"], 1e-6), norm(K, w["k_norm"], 1e-6)
        Q, K = rotate(Q), rotate(K)
        att = torch.empty((len(x), nq, d), dtype=torch.float64, device="cuda")
        row = 0
        for i, (n, ctx) in enumerate(seqs):
            at = torch.arange(ctx, ctx + n, device="cuda")
            bt = torch.from_numpy(tables[i].astype(np.int64)).cuda()
            blk, o = bt[at // BLOCK], at % BLOCK
            for k in range(nkv):
                pool[l][blk[:, None], k, 0, koff[o]] = K[row:row + n, k]
                pool[l][blk[:, None], k, 1, voff[o]] = V[row:row + n, k]
            nb = (ctx + n + BLOCK - 1) // BLOCK
            kv = pool[l][bt[:nb]]
            future = torch.arange(nb * BLOCK, device="cuda")[None, :] > at[:, None]
            for k in range(nkv):
                kk = kv[:, k, 0][:, koff].reshape(nb * BLOCK, d)
                vv = kv[:, k, 1][:, voff].reshape(nb * BLOCK, d)
                for g in range(k * (nq // nkv), (k + 1) * (nq // nkv)):
                    s = Q[row:row + n, g] @ kk.T / math.sqrt(d)
                    s.masked_fill_(future, -math.inf)
                    att[row:row + n, g] = torch.softmax(s, -1) @ vv
            row += n
        x = x + att.reshape(len(x), nq * d) @ w["w_o"].double().T
        h = norm(x, w["ffn_norm"], eps)
        gu = h @ w["w_gate_up"].double().T
        gate, up = gu[:, :F], gu[:, F:]
        x = x + (gate * torch.sigmoid(gate) * up) @ w["w_down"].double().T
    r = {"hidden": x, "kv": pool}
    if head is not None:
        r["logits"] = norm(x, head[0], eps) @ head[1].double().T
    return r
