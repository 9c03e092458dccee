"""Work that a user of the library has it do, for timing and for comparing outputs.

Each case is one pass through the public entry points of the binding over a
model shape of ``workloads/configs.py``: prefix prefill (one request or a
varlen batch), chunked prefill over an earlier prefix, a decode step (one to
64 sequences, with a workspace or with the library's static scratch), pack,
assemble, and the whole reconstruction of a small request.  Weights, token
ids, block tables and caches follow ``workloads/gen.py``.

The models keep their real layer shapes and vocabulary; their depth is cut to
a few layers, still many times what the last-level cache holds, so that a
state is quick to make and rounding does not travel through 64 layers.

A case is a dict of plain values:
  kind    prefill | chunk | decode | pack | assemble | reconstruct
  model   tiny | mid | large (``configs.preset``)
  layers  depth
  ctx     tokens per sequence, comma-separated; prefill: the prefix lengths;
          chunk: the end of the chunk; decode: the position decoded at;
          pack, assemble, reconstruct: the tokens the source holds
  start   chunk: where each chunk starts; pack, assemble, reconstruct: the
          split between prefix and suffix
  chunk   pack, assemble, reconstruct: suffix chunk tokens (0: one chunk)
  static  decode: the entry point without a workspace
"""
from __future__ import annotations

import math

import torch

import paper_2608_16477_amd as P
from workloads import configs, gen

DEV = "cuda"
SPARE_PAGES = 32   # pool pages that belong to nobody
GAIN_SIGMA = 0.1   # RMSNorm gains are 1 + N(0, 0.1)


def _text(values):
    return ",".join(str(int(v)) for v in values)


def _ints(text):
    return [int(v) for v in str(text).split(",")]


def listed():
    mid_ctx, mid_prefix = configs.concurrent_lengths(seed=0, n=8)
    many_ctx, _ = configs.concurrent_lengths(seed=1, n=32)
    return [
        # The smallest whole migration: prefill, pack, assembly and one decode
        # step of a 128-token request split at 96; launches and host work.
        dict(name="reconstruct_tiny", kind="reconstruct", model="tiny", layers=2, ctx="128", start="96", chunk=0),
        # The prefix of the large workload: 3000 tokens, not a multiple of 16.
        dict(name="prefill_large_3000", kind="prefill", model="large", layers=3, ctx="3000"),
        # The prefix of the mid workload.
        dict(name="prefill_mid_1536", kind="prefill", model="mid", layers=3, ctx="1536"),
        # Eight requests migrated at once, prefixes of 500 to 7000 tokens.
        dict(name="prefill_mid_varlen8", kind="prefill", model="mid", layers=3, ctx=_text(mid_prefix)),
        # A short prefix, the low end of the evaluated contexts (500 tokens).
        dict(name="prefill_large_500", kind="prefill", model="large", layers=3, ctx="500"),
        # A 256-token chunk of a prefill that is interleaved with decoding.
        dict(name="chunk_large_256", kind="chunk", model="large", layers=3, ctx="3000", start="2744"),
        # The first token after the handover of the large workload.
        dict(name="decode_large_1", kind="decode", model="large", layers=8, ctx="4000", static=False),
        # Eight migrated requests resumed in one batch.
        dict(name="decode_mid_8", kind="decode", model="mid", layers=12, ctx=_text(mid_ctx), static=False),
        # A batch of resident sessions at the target, half the sequence limit.
        dict(name="decode_mid_32", kind="decode", model="mid", layers=12, ctx=_text(many_ctx), static=False),
        # One session through the allocation-free entry point.
        dict(name="decode_mid_1_static", kind="decode", model="mid", layers=12, ctx="2048", static=True),
        # Two completed 32-token chunks leave the source: 16 MiB.
        dict(name="pack_large_64", kind="pack", model="large", layers=64, ctx="8192", start="8128", chunk=32),
        # The large workload's 1000-token suffix, split inside a page.
        dict(name="assemble_large_1000", kind="assemble", model="large", layers=64, ctx="4000", start="3000", chunk=0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    kind = rng.choices(("prefill", "chunk", "decode", "pack", "assemble", "reconstruct"), (6, 4, 6, 2, 2, 1))[0]
    if kind == "prefill":
        model = rng.choice(("mid", "large"))
        n = rng.choice((1, 1, 1, 2, 3, 8))
        return dict(kind=kind, model=model, layers=3, ctx=_text(_log(rng, 16, 8000) for _ in range(n)))
    if kind == "chunk":
        model = rng.choice(("mid", "large"))
        n = rng.choice((1, 1, 1, 2))
        sizes = [rng.choice((64, 128, 256, 256, 512, _log(rng, 1, 1024))) for _ in range(n)]
        start = [_log(rng, 16, 6000) for _ in range(n)]
        return dict(kind=kind, model=model, layers=3, ctx=_text(a + b for a, b in zip(start, sizes)),
                    start=_text(start))
    if kind == "decode":
        model = rng.choice(("mid", "large"))
        n = _log(rng, 1, 64)
        return dict(kind=kind, model=model, layers=12 if model == "mid" else 8,
                    ctx=_text(_log(rng, 500, 8000) for _ in range(n)), static=n <= 8 and rng.random() < 0.3)
    if kind in ("pack", "assemble"):
        model, layers = rng.choice((("mid", 36), ("large", 64)))
        start = _log(rng, 250, 4000)
        return dict(kind=kind, model=model, layers=layers, ctx=str(start + _log(rng, 32, 4096)), start=str(start),
                    chunk=rng.choice((0, 32, 32, 64, 256)))
    start = _log(rng, 16, 500)
    return dict(kind=kind, model=rng.choice(("tiny", "mid")), layers=2, ctx=str(start + _log(rng, 1, 250)),
                start=str(start), chunk=rng.choice((0, 32)))


def draw(rng):
    most = [work(c) for c in listed()]
    top = {k: max(w[k] for w in most) for k in ("bytes", "flops")}
    while True:
        c = _draw_once(rng)
        w = work(c)
        if all(w[k] <= top[k] for k in top):
            return c


# ------------------------------------------------------------------ inputs
def _config(case):
    return configs.preset(case["model"]).with_layers(int(case["layers"]))


def _pages(tokens):
    return (tokens + configs.PAGE - 1) // configs.PAGE


def _pool(cfg, pages, seed, tag, filled):
    if filled:
        return gen.kv_pool_normal(cfg.n_layers, pages, cfg.page_size, cfg.n_kv_heads, cfg.head_dim, seed, DEV, tag)
    return torch.zeros((cfg.n_layers, 2, pages, cfg.page_size, cfg.n_kv_heads, cfg.head_dim),
                       dtype=torch.bfloat16, device=DEV)


def _tables(lens, seed, tag):
    """Block tables of sequences that hold `lens` tokens, and the pool's pages."""
    pages = [_pages(n) for n in lens]
    total = sum(pages) + SPARE_PAGES
    return torch.tensor(gen.disjoint_block_tables(pages, total, max(pages), seed, tag), device=DEV), total


def _weights(cfg, seed, head):
    layers = [gen.layer_weights(cfg, l, seed, 1, DEV, GAIN_SIGMA) for l in range(cfg.n_layers)]
    shapes = gen.global_shapes(cfg)
    embed = gen.normal_bf16(shapes["embed"], gen.SIGMA, DEV, seed, 1, 0xFFFF, 0)
    glob = {"embed": embed,
            "final_norm": gen.normal_bf16(shapes["final_norm"], GAIN_SIGMA, DEV, seed, 1, 0xFFFF, 1, mean=1.0),
            # a prefill computes no logits: it never reads this one
            "lm_head": gen.normal_bf16(shapes["lm_head"], gen.SIGMA, DEV, seed, 1, 0xFFFF, 2) if head else embed}
    return glob, layers


def _suffix_chunks(case):
    a, b = _ints(case["start"])[0], _ints(case["ctx"])[0]
    size = int(case["chunk"]) or b - a
    return [(t, min(size, b - t)) for t in range(a, b, size)]


def _inputs(case, seed):
    """The inputs of a case, without the library's handle and workspace."""
    cfg, kind, ctx = _config(case), case["kind"], _ints(case["ctx"])
    s = {"kind": kind, "cfg": cfg, "ctx": ctx}
    if kind in ("prefill", "chunk", "decode", "reconstruct"):
        s["glob"], s["layers"] = _weights(cfg, seed, kind in ("decode", "reconstruct"))
    if kind == "prefill":
        s["start"] = [0] * len(ctx)
        s["bt"], pages = _tables(ctx, seed, 1)
        s["pool"] = _pool(cfg, pages, seed, 4, False)
    elif kind == "chunk":
        s["start"] = _ints(case["start"])
        s["bt"], pages = _tables(ctx, seed, 1)
        s["pool"] = _pool(cfg, pages, seed, 4, True)      # earlier chunks' K/V
    elif kind == "decode":
        s["bt"], pages = _tables([n + 1 for n in ctx], seed, 1)
        s["pool"] = _pool(cfg, pages, seed, 4, True)      # the resident caches
        s["tokens"] = gen.token_ids(len(ctx), cfg.vocab, seed).to(DEV)
    elif kind == "reconstruct":
        s["start"] = _ints(case["start"])
        s["src_bt"], pages = _tables(ctx, seed, 1)
        s["src"] = _pool(cfg, pages, seed, 4, True)
        s["bt"], pages = _tables([ctx[0] + 1], seed, 2)
        s["pool"] = _pool(cfg, pages, seed, 5, False)
        s["tokens"] = gen.token_ids(1, cfg.vocab, seed, 1).to(DEV)
    else:
        s["bt"], pages = _tables(ctx, seed, 1)
        s["pool"] = _pool(cfg, pages, seed, 4, True)
    if kind in ("pack", "assemble", "reconstruct"):
        s["chunks"] = _suffix_chunks(case)
        n = sum(c for _, c in s["chunks"]) * cfg.s_kv
        if kind == "assemble":
            s["arena"] = gen.normal_bf16((n // 2,), 1.0, DEV, seed, 6)
        else:
            s["arena"] = torch.zeros(n // 2, dtype=torch.bfloat16, device=DEV)
    if kind in ("prefill", "chunk"):
        lens = [b - a for a, b in zip(s["start"], ctx)]
    else:
        lens = s.get("start", [])
    s["cu"] = [0]
    for n in lens:
        s["cu"].append(s["cu"][-1] + n)
    if "glob" in s and kind != "decode":
        s["ids"] = gen.token_ids(s["cu"][-1], cfg.vocab, seed).to(DEV)
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    cfg, kind, n = s["cfg"], s["kind"], len(s["ctx"])
    s["err"] = torch.zeros(1, dtype=torch.int32, device=DEV)
    if "glob" in s:
        s["model"] = P.Model(cfg, s["glob"], s["layers"])
        rows = n if kind == "decode" else s["cu"][-1]
        s["static"] = bool(case.get("static"))
        if not s["static"]:
            s["ws"] = s["model"].workspace(rows, n)
            # the residual stream, the workspace's defined part
            s["resid"] = s["ws"][:rows * cfg.hidden * 4].view(torch.float32).view(rows, cfg.hidden)
    if kind in ("decode", "reconstruct"):
        s["logits"] = torch.empty((n, cfg.vocab), dtype=torch.float32, device=DEV)
    if "chunks" in s:
        at = 0
        s["descs"], s["hdrs"] = [], []
        for t, c in s["chunks"]:
            s["descs"].append(P.ChunkDesc(t, c, at))
            s["hdrs"].append(P.ChunkHeader(7, 3, t, c, at, cfg.n_layers, cfg.n_kv_heads, cfg.head_dim, 2))
            at += c * cfg.s_kv
    return s


def run(s):
    kind = s["kind"]
    if kind == "prefill":
        s["model"].prefill_prefix(s["ids"], s["cu"], s["bt"], s["pool"], s["ws"], s["err"])
        return {"pool": s["pool"], "resid": s["resid"]}
    if kind == "chunk":
        s["model"].prefill_chunk(s["ids"], s["cu"], s["start"], s["bt"], s["pool"], s["ws"], s["err"])
        return {"pool": s["pool"], "resid": s["resid"]}
    if kind == "decode":
        if s["static"]:
            s["model"].decode_step_static(s["tokens"], s["ctx"], s["bt"], s["pool"], s["logits"], s["err"])
            return {"pool": s["pool"], "logits": s["logits"]}
        s["model"].decode_step(s["tokens"], s["ctx"], s["bt"], s["pool"], s["logits"], s["ws"], s["err"])
        return {"pool": s["pool"], "logits": s["logits"], "resid": s["resid"]}
    if kind == "pack":
        P.pallas_pack_suffix_blocks(s["pool"], s["bt"][0], s["descs"], s["arena"], s["err"])
        return s["arena"].view(torch.int32)
    if kind == "assemble":
        P.pallas_assemble_kv(s["pool"], s["bt"][0], s["hdrs"], s["arena"], 7, 3, s["err"])
        return s["pool"].view(torch.int32)
    m = s["model"]
    m.prefill_prefix(s["ids"], s["cu"], s["bt"], s["pool"], s["ws"], s["err"])
    P.pallas_pack_suffix_blocks(s["src"], s["src_bt"][0], s["descs"], s["arena"], s["err"])
    P.pallas_assemble_kv(s["pool"], s["bt"][0], s["hdrs"], s["arena"], 7, 3, s["err"])
    m.decode_step(s["tokens"], s["ctx"], s["bt"], s["pool"], s["logits"], s["ws"], s["err"])
    return {"pool": s["pool"], "logits": s["logits"]}


# ------------------------------------------------------------------ work
def work(case):
    cfg, kind, ctx = _config(case), case["kind"], _ints(case["ctx"])
    H, F, d, L = cfg.hidden, cfg.ffn, cfg.head_dim, cfg.n_layers
    layer = cfg.qkv_out * H + H * cfg.q_dim + 3 * H * F      # weights of a layer
    kv_row = 2 * cfg.kv_dim                                   # K and V values of a token and layer
    total = {"bytes": 0.0, "flops": 0.0}

    def prefill(starts, ends):
        rows = sum(e - s for s, e in zip(starts, ends))
        pairs = sum((e * (e + 1) - s * (s + 1)) // 2 for s, e in zip(starts, ends))   # visible (query, key) pairs
        total["flops"] += (L - 1) * (2.0 * rows * layer + 4.0 * cfg.q_dim * pairs) + 2.0 * rows * H * kv_row
        total["bytes"] += 2.0 * ((L - 1) * layer + H * kv_row)                        # weights
        total["bytes"] += rows * (2.0 * H + 4.0 * H + 2.0 * L * kv_row)               # embedding, residual, K/V
        total["bytes"] += 2.0 * (L - 1) * kv_row * sum(starts)                        # earlier K/V

    def decode(pos):
        n, keys = len(pos), sum(pos)
        total["flops"] += 2.0 * n * (L * layer + cfg.vocab * H) + 4.0 * L * cfg.q_dim * (keys + n)
        total["bytes"] += 2.0 * (L * layer + cfg.vocab * H) + 2.0 * L * kv_row * (keys + n)
        total["bytes"] += n * (2.0 * H + 4.0 * H + 4.0 * cfg.vocab)

    if kind == "prefill":
        prefill([0] * len(ctx), ctx)
    elif kind == "chunk":
        prefill(_ints(case["start"]), ctx)
    elif kind == "decode":
        decode(ctx)
    else:
        start = _ints(case["start"])
        moved = 2.0 * cfg.s_kv * (ctx[0] - start[0])          # read once, written once
        if kind == "reconstruct":
            prefill([0], start)
            decode(ctx)
            moved *= 2
        total["bytes"] += moved
    return total


def tolerance(case):
    if case["kind"] in ("pack", "assemble"):
        return "exact"   # a bit copy
    # bf16 weights, activations and caches with float32 sums.  Against 64 bits
    # the residual and the logits are 1.0e-2 off after two layers and 1.3e-2
    # to 1.6e-2 after 8 and 12; two correct runs differ by up to the sum of
    # their errors.
    if case["kind"] == "decode":
        return {"rel": 3e-2, "max": 0.2}
    return {"rel": 2e-2, "max": 0.15}


# ------------------------------------------------------------------ exact
def _norm(x, gain, eps):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps) * gain.double()


def _project(x, w):
    """x W^T in 64 bits, over a few thousand weight rows at a time."""
    return torch.cat([x @ part.double().T for part in w.split(32768)], -1)


def _rope(x, pos, theta):
    half = x.shape[-1] // 2
    freq = theta ** (-torch.arange(half, device=x.device, dtype=torch.float64) / half)
    a = pos.double()[:, None, None] * freq
    lo, hi = x[..., :half], x[..., half:]
    return torch.cat([lo * a.cos() - hi * a.sin(), hi * a.cos() + lo * a.sin()], -1)


def _attend(q, k, v, pos):
    """q [n][Hq][d] at positions pos, k and v [keys][Hkv][d]: causal."""
    out = torch.empty_like(q)
    grp = q.shape[1] // k.shape[1]
    step = max(1, (1 << 27) // (grp * k.shape[0]))
    keys = torch.arange(k.shape[0], device=q.device)
    for kh in range(k.shape[1]):
        hs = slice(kh * grp, kh * grp + grp)
        for a in range(0, q.shape[0], step):
            qa = q[a:a + step, hs]
            sc = (qa.reshape(-1, q.shape[-1]) @ k[:, kh].T.contiguous()).view(qa.shape[0], grp, -1)
            sc = sc / math.sqrt(q.shape[-1])
            sc.masked_fill_(keys[None, None, :] > pos[a:a + step, None, None], -math.inf)
            w = torch.softmax(sc, -1).view(-1, k.shape[0])
            out[a:a + step, hs] = (w @ v[:, kh].contiguous()).view(qa.shape[0], grp, -1)
    return out


def _slots(table, pos):
    return table[pos // configs.PAGE].long(), pos % configs.PAGE


def _forward(s, ids, cu, start, ctx, pool, whole):
    """The decoder over rows [cu[i], cu[i + 1]) of sequence i at positions
    start[i] .. ctx[i] - 1; K and V go into `pool` (64 bits).  Returns the
    residual entering the last layer, or leaving it when `whole`."""
    cfg = s["cfg"]
    pos = torch.cat([torch.arange(a, b, device=DEV) for a, b in zip(start, ctx)])
    r = s["glob"]["embed"][ids.long()].double()
    for l, w in enumerate(s["layers"]):
        qkv = _project(_norm(r, w["attn_norm"], cfg.rms_eps), w["w_qkv"]).view(r.shape[0], -1, cfg.head_dim)
        q, k, v = qkv.split([cfg.n_q_heads, cfg.n_kv_heads, cfg.n_kv_heads], 1)
        if cfg.qk_norm:
            q, k = _norm(q, w["q_norm"], cfg.rms_eps), _norm(k, w["k_norm"], cfg.rms_eps)
        q, k = _rope(q, pos, cfg.rope_theta), _rope(k, pos, cfg.rope_theta)
        last = l == cfg.n_layers - 1 and not whole
        o = []
        for i in range(len(ctx)):
            rows = slice(cu[i], cu[i + 1])
            page, slot = _slots(s["bt"][i], pos[rows])
            pool[l, 0, page, slot], pool[l, 1, page, slot] = k[rows], v[rows]
            if not last:
                page, slot = _slots(s["bt"][i], torch.arange(ctx[i], device=DEV))
                o.append(_attend(q[rows], pool[l, 0, page, slot], pool[l, 1, page, slot], pos[rows]))
        if last:
            break
        r = r + _project(torch.cat(o).view(r.shape[0], -1), w["w_o"])
        gate, up = _project(_norm(r, w["mlp_norm"], cfg.rms_eps), w["w_gate_up"]).chunk(2, -1)
        r = r + _project(gate * torch.sigmoid(gate) * up, w["w_down"])
    return r


def exact(case, seed):
    s = _inputs(case, seed)
    kind, cfg, ctx = s["kind"], s["cfg"], s["ctx"]
    if kind in ("pack", "assemble"):
        return None   # a bit copy: nothing to round
    pool = s["pool"].double()
    if kind in ("prefill", "chunk"):
        r = _forward(s, s["ids"], s["cu"], s["start"], ctx, pool, False)
        return {"pool": pool, "resid": r}
    if kind == "reconstruct":
        _forward(s, s["ids"], s["cu"], [0], s["start"], pool, False)
        t = torch.arange(s["start"][0], ctx[0], device=DEV)
        page, slot = _slots(s["bt"][0], t)
        spage, sslot = _slots(s["src_bt"][0], t)
        pool[:, :, page, slot] = s["src"][:, :, spage, sslot].double()
    r = _forward(s, s["tokens"], list(range(len(ctx) + 1)), ctx, [n + 1 for n in ctx], pool, True)
    logits = _project(_norm(r, s["glob"]["final_norm"], cfg.rms_eps), s["glob"]["lm_head"])
    if kind == "reconstruct" or case.get("static"):
        return {"pool": pool, "logits": logits}
    return {"pool": pool, "logits": logits, "resid": r}
