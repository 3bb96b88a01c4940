"""What a user of this package has it do, as cases that can be timed and checked.

Two entry points carry a program that drafts blocks with the refiner:

* ``refine``: ``Refiner.refine_block`` (base readout, seed, K Jacobi passes,
  with the refined logits) and ``Refiner.verify_block`` on its block, for a
  batch of blocks;
* ``layer``: one forward of the context layer that produces the hidden states
  (``Layer.forward``, or ``layer_forward_noalloc`` for programs that may not
  allocate).

The sizes are the package's own workloads (``synth/configs.py``: the tiny fp32
refiner and the Qwen3-8B shape at batch 1, 8, 32 and 64), and odd and ragged
ones in the ranges its tests cover.  All values are synthetic with the
distributions of ``synth/``; everything is made on the device from the seed.
"""
from __future__ import annotations

import math

import torch

from paper_2608_02438_amd.xpress import (LAYER_WEIGHT_NAMES, Layer, RefineOut, Refiner,
                                         layer_forward_noalloc, layer_weights_struct)

R = 256                       # the refiner's rank
HD = 128                      # head_dim of the context layer
EPS, THETA = 1e-6, 1e6
QWEN = dict(H=4096, V=151936)
QWEN_LAYER = dict(H=4096, n_heads=32, n_kv=8, ffn=12288)


def _refine(name=None, dtype="bf16", H=4096, V=151936, B=16, batch=1, K=6, mode="greedy",
            seeded=False, h_sigma=1.0, temperature=False, top_k=0, top_p=1.0, early_exit=False,
            p_match=0.8):
    c = dict(kind="refine", dtype=dtype, H=H, V=V, B=B, batch=batch, K=K, mode=mode,
             seeded=seeded, h_sigma=h_sigma, temperature=temperature, top_k=top_k, top_p=top_p,
             early_exit=early_exit, p_match=p_match)
    return dict(c, name=name) if name else c


def _layer(name=None, H=4096, n_heads=32, n_kv=8, ffn=12288, B=16, batch=1, ctx_lo=2048,
           ctx_hi=2048, causal=True, noalloc=False):
    c = dict(kind="layer", H=H, n_heads=n_heads, n_kv=n_kv, ffn=ffn, B=B, batch=batch,
             ctx_lo=ctx_lo, ctx_hi=ctx_hi, causal=causal, noalloc=noalloc)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: the tiny fp32 refiner with the caller's seed ids,
        # where the launches and the chain between them are all there is
        _refine("refine-tiny-f32", dtype="f32", H=256, V=1024, B=8, K=8, seeded=True, p_match=0.7),
        # one user decoding greedily: the latency of a single draft block
        _refine("refine-b1-greedy", **QWEN),
        # a small sampling batch at temperature 1
        _refine("refine-b8-sample", **QWEN, batch=8, mode="sample", h_sigma=1.5625),
        # an odd batch of short blocks, truncated sampling with a temperature
        # of its own per sequence, stopping at each sequence's fixed point
        _refine("refine-b5-topk-topp", **QWEN, B=13, batch=5, mode="sample", h_sigma=1.5625,
                temperature=True, top_k=50, top_p=0.9, early_exit=True),
        # a serving batch, greedy
        _refine("refine-b32-greedy", **QWEN, batch=32),
        # the largest configured batch, greedy and sampled sequences mixed
        _refine("refine-b64x32-mixed", **QWEN, B=32, batch=64, mode="mixed"),
        # full-precision refiner over a ragged vocabulary, mixed sequences
        _refine("refine-f32-ragged", dtype="f32", H=2048, V=33001, B=11, batch=3, mode="mixed",
                temperature=True),
        # a small model's layer under a no-allocation rule, ragged contexts
        _layer("layer-small-noalloc", H=1024, n_heads=16, n_kv=8, ffn=3072, B=7, batch=3,
               ctx_lo=1, ctx_hi=701, noalloc=True),
        # the context layer at the four configured batches: the target's causal
        # forward, and once the drafter's bidirectional block
        _layer("layer-b1-ctx2048", **QWEN_LAYER),
        _layer("layer-b8-ctx4096-bidir", **QWEN_LAYER, batch=8, ctx_lo=4096, ctx_hi=4096,
               causal=False),
        _layer("layer-b32-ctx8192", **QWEN_LAYER, batch=32, ctx_lo=8192, ctx_hi=8192),
        _layer("layer-b64x32-ragged", **QWEN_LAYER, B=32, batch=64, ctx_lo=512, ctx_hi=16384),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the ranges above; never dearer than the largest listed one."""
    top = max(_cost(c) for c in listed())
    while True:
        c = _draw_refine(rng) if rng.random() < 0.5 else _draw_layer(rng)
        if _cost(c) <= top:
            return c


def _draw_refine(rng):
    f32 = rng.random() < 0.2
    mode = rng.choice(["greedy", "sample", "mixed"])
    sampled = mode != "greedy"
    trunc = sampled and rng.random() < 0.3
    return _refine(
        dtype="f32" if f32 else "bf16",
        H=256 * (_log_int(rng, 1, 8) if f32 else _log_int(rng, 4, 16)),
        V=_log_int(rng, 1000, 40000) if f32 else rng.choice([151936, _log_int(rng, 8000, 152064)]),
        B=rng.choice([8, 16, 32, rng.randint(1, 32)]),
        batch=_log_int(rng, 1, 4 if f32 else 64), K=rng.choice([0, 1, 4, 6, 6, 8]), mode=mode,
        seeded=rng.random() < 0.2, h_sigma=1.5625 if sampled else 1.0,
        temperature=sampled and rng.random() < 0.5,
        top_k=rng.randint(1, 200) if trunc and rng.random() < 0.7 else 0,
        top_p=round(rng.uniform(0.5, 0.99), 3) if trunc else 1.0, early_exit=rng.random() < 0.3)


def _draw_layer(rng):
    n_kv = rng.choice([2, 4, 8])
    batch, B = _log_int(rng, 1, 64), rng.choice([8, 16, 32, rng.randint(1, 32)])
    lo = _log_int(rng, 1, 8192)
    return _layer(H=256 * _log_int(rng, 2, 16), n_heads=n_kv * rng.choice([1, 2, 4, 8]), n_kv=n_kv,
                  ffn=256 * _log_int(rng, 4, 48), B=B, batch=batch, ctx_lo=lo,
                  ctx_hi=_log_int(rng, lo, 16384), causal=rng.random() < 0.6,
                  noalloc=batch * B <= 64 and rng.random() < 0.5)


def _cost(c):
    """Seconds of a pass at 4 TB/s and 0.8 PFLOP/s (fp32: 50 TFLOP/s), for bounding draws only."""
    w = work(c)
    return w["bytes"] / 4e12 + w["flops"] / (5e13 if c.get("dtype") == "f32" else 8e14)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _normal(g, shape, sigma, dtype, mean=0.0):
    n = math.prod(shape)
    out = torch.empty(n, dtype=dtype, device="cuda")
    step = 1 << 27
    for i in range(0, n, step):
        x = torch.randn(min(step, n - i), generator=g, device="cuda", dtype=torch.float32)
        out[i:i + step] = x.mul_(sigma).add_(mean)
    return out.view(shape)


def _refine_inputs(c, seed):
    g = _gen(seed)
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    H, V, B, n = c["H"], c["V"], c["B"], c["batch"]
    shapes = dict(W_lm=(V, H), W_h=(R, H), W_g=(R, H), W_e=(V, R), W_in=(R, 3 * R), L=(R, B, B),
                  W_1=(2 * R, R), W_2=(R, 2 * R), W_r=(V, R))
    w = {k: _normal(g, s, 0.02, dt) for k, s in shapes.items()}
    rand = lambda *s: torch.rand(s, generator=g, device="cuda", dtype=torch.float32)  # noqa: E731
    ids = lambda *s: torch.randint(0, V, s, generator=g, device="cuda",  # noqa: E731
                                   dtype=torch.int32)
    i = dict(hidden=_normal(g, (n, B, H), c["h_sigma"], dt), anchor=ids(n), seed_ids=None,
             temp=None, u_draft=None, temperature=None, top_k=None, top_p=None,
             target_logits=None, r_accept=None, u_resample=None)
    if c["seeded"]:
        i["seed_ids"] = ids(n, B)
    if c["mode"] != "greedy":
        i["temp"] = torch.ones(n, dtype=torch.uint8, device="cuda")
        if c["mode"] == "mixed":
            i["temp"][0::2] = 0
        i.update(u_draft=rand(n, B), r_accept=rand(n, B), u_resample=rand(n),
                 target_logits=_normal(g, (n, B + 1, V), 2.0, torch.float32))
        if c["temperature"]:
            i["temperature"] = rand(n) * 0.9 + 0.6
        if c["top_k"]:
            i["top_k"] = torch.full((n,), c["top_k"], dtype=torch.int32, device="cuda")
        if c["top_p"] < 1:
            i["top_p"] = torch.full((n,), c["top_p"], dtype=torch.float32, device="cuda")
    # the target agrees with the drafter's own choice with probability p_match
    own = torch.cat([(x.float() @ w["W_lm"].float().T if dt is torch.float32 else x @ w["W_lm"].T)
                     .argmax(-1) for x in i["hidden"].view(n * B, H).split(256)])
    t = ids(n, B + 1)
    t[:, :B] = torch.where(rand(n, B) < c["p_match"], own.view(n, B).to(torch.int32), t[:, :B])
    i["target_ids"] = t
    return w, i


def _layer_inputs(c, seed):
    g = _gen(seed)
    H, q, kv, f, n = c["H"], c["n_heads"] * HD, c["n_kv"] * HD, c["ffn"], c["batch"]
    bf = torch.bfloat16
    shapes = dict(g_attn=(H,), Wq=(q, H), Wk=(kv, H), Wv=(kv, H), g_q=(HD,), g_k=(HD,), Wo=(H, q),
                  g_mlp=(H,), Wg=(f, H), Wu=(f, H), Wd=(H, f))
    w = {k: _normal(g, s, 0.1, bf, 1.0) if k[0] == "g" else _normal(g, s, 0.02, bf)
         for k, s in shapes.items()}
    ctx = torch.randint(c["ctx_lo"], c["ctx_hi"] + 1, (n,), generator=g, device="cuda",
                        dtype=torch.int32)
    cache = (n, c["ctx_hi"], c["n_kv"], HD)
    return w, dict(x=_normal(g, (n, c["B"], H), 1.0, bf), k_cache=_normal(g, cache, 1.0, bf),
                   v_cache=_normal(g, cache, 1.0, bf), ctx_len=ctx)


class _State:
    pass


def prepare(case, seed):
    c, s = case, _State()
    s.case = c
    n, B = c["batch"], c["B"]
    if c["kind"] == "layer":
        s.w, s.inp = _layer_inputs(c, seed)
        s.h32 = torch.empty((n, B, c["H"]), dtype=torch.float32, device="cuda")
        s.h16 = torch.empty((n, B, c["H"]), dtype=torch.bfloat16, device="cuda")
        size = (c["H"], c["n_heads"], c["n_kv"], c["ffn"])
        if c["noalloc"]:
            s.struct = layer_weights_struct(s.w, *size)
        else:
            s.layer = Layer(s.w, *size, max_batch=n, max_B=B, max_ctx=c["ctx_hi"])
        return s
    w, s.inp = _refine_inputs(c, seed)
    s.ref = Refiner(w, c["H"], R, c["V"], B, n)
    # the token results of a step in one buffer, as a program that copies them
    # to the host in one go keeps them: ids, passes, accepted lengths, next tokens
    s.tokens = torch.zeros(n * (B + 3), dtype=torch.int32, device="cuda")
    s.out = RefineOut(ids=s.tokens[:n * B].view(n, B), iters=s.tokens[n * B:n * (B + 1)],
                      logits=torch.empty((n, B, c["V"]), dtype=torch.float32, device="cuda"),
                      traj=None)
    s.verdict = (s.tokens[n * (B + 1):n * (B + 2)], s.tokens[n * (B + 2):])
    greedy, sampled = _rows(c)
    s.results = {"tokens": s.tokens, "greedy_logits": s.out.logits[greedy],
                 "sampled_logits": s.out.logits[sampled]}
    return s


def run(state):
    s, c, i = state, state.case, state.inp
    if c["kind"] == "layer":
        args = (i["x"], i["k_cache"], i["v_cache"], i["ctx_len"])
        if c["noalloc"]:
            layer_forward_noalloc(s.struct, *args, s.h32, s.h16, causal=c["causal"])
        else:
            s.layer.forward(*args, causal=c["causal"], h_f32=s.h32, h_bf16=s.h16)
        return {"h_f32": s.h32, "h_bf16": s.h16}
    s.ref.refine_block(i["hidden"], i["anchor"], seed_ids=i["seed_ids"], temp=i["temp"],
                       u_draft=i["u_draft"], K=c["K"], early_exit=c["early_exit"],
                       write_logits=True, out=s.out, temperature=i["temperature"],
                       top_k=i["top_k"], top_p=i["top_p"])
    s.ref.verify_block(s.out.ids, i["target_ids"], temp=i["temp"],
                       target_logits=i["target_logits"], r_accept=i["r_accept"],
                       u_resample=i["u_resample"], out=s.verdict)
    return s.results


def _rows(c):
    """The greedy sequences and the sampled ones, as slices of the batch."""
    none, every = slice(0, 0), slice(0, c["batch"])
    return {"greedy": (every, none), "sample": (none, every),
            "mixed": (slice(0, None, 2), slice(1, None, 2))}[c["mode"]]


# ---------------------------------------------------------------------------
# the work of a pass: every input read once, every output written once
# ---------------------------------------------------------------------------
def work(case):
    c = case
    n, B, H = c["batch"], c["B"], c["H"]
    M = n * B
    if c["kind"] == "layer":
        q, kv, f = c["n_heads"] * HD, c["n_kv"] * HD, c["ffn"]
        weights = H * (q + 2 * kv) + q * H + 3 * H * f
        keys = n * (c["ctx_lo"] + c["ctx_hi"]) // 2
        return {"bytes": 2 * weights + 4 * keys * kv + M * H * (2 + 4 + 2),
                "flops": 2 * M * weights + 4 * B * (keys + n * B) * q}
    es, V, K = (2 if c["dtype"] == "bf16" else 4), c["V"], c["K"]
    sampled = {"greedy": 0, "sample": n, "mixed": n // 2}[c["mode"]]
    weights = V * H + (V * R if K else 0) + 2 * R * H + 7 * R * R + R * B * B // 2
    # every weight, hidden state and (for a sampled sequence) one row of target
    # logits at least once, the logits out once; the passes (stopping early, two
    # at least) count by their arithmetic alone, though each one also reads the
    # readout head and the base logits anew: it depends on all of the one before
    passes = min(K, 2) if c["early_exit"] else K
    return {"bytes": weights * es + M * H * es + M * V * 4 + sampled * V * 4,
            "flops": 2 * M * V * H + passes * (2 * M * V * R + 14 * M * R * R)}


def tolerance(case):
    """Relative errors between correct implementations that sum in another
    order, four times what was measured.  The layer with and without its k
    splits: 5.9e-4 of the fp32 output, 1.3e-3 of the bf16 one (roundings of the
    bf16 activations inside).  The refined logits against 64 bits: 4e-7 in
    fp32, up to 4e-6 in bf16 (z on the other side of a rounding); where a
    sampled token falls on the other side of its uniform, that position's
    token part of the readout changes (1.4e-4 for one of 128 positions)."""
    if case["kind"] == "layer":
        return {"rel": 5e-3, "max": 0.04}
    if case["mode"] == "greedy":
        return {"rel": 2e-5, "max": 0.01, "differ": 0.01}
    return {"rel": 5e-4, "max": 0.05, "differ": 0.01}


# ---------------------------------------------------------------------------
# the same values in 64 bits
# ---------------------------------------------------------------------------
def exact(case, seed):
    return _exact_layer(case, seed) if case["kind"] == "layer" else _exact_refine(case, seed)


def _exact_refine(c, seed):
    """Logits of the sequences whose tokens do not hang on a rounding: a
    sampled token is decided by a uniform against sums over the vocabulary, so
    sampled sequences have them only where no sampled token enters."""
    w, i = _refine_inputs(c, seed)
    fixed = c["K"] == 0 or (c["K"] == 1 and c["seeded"])
    greedy, sampled = _rows(c)
    return {"tokens": None, "greedy_logits": _jacobi(c, w, i, greedy),
            "sampled_logits": _jacobi(c, w, i, sampled) if fixed else None}


def _jacobi(c, w, i, rows):
    f64 = torch.float64
    h = i["hidden"][rows].to(f64)
    n, B, V = h.shape[0], c["B"], c["V"]
    if n == 0:
        return torch.empty((0, B, V), dtype=f64, device="cuda")
    d = {k: v.to(f64) for k, v in w.items() if k != "W_lm"}
    s = torch.empty((n, B, V), dtype=f64, device="cuda")
    for v in range(0, V, 16384):
        s[:, :, v:v + 16384] = h @ w["W_lm"][v:v + 16384].to(f64).T.contiguous()
    mean = h.mean(1, keepdim=True).expand_as(h)
    fixed = torch.cat([h @ d["W_h"].T, mean @ d["W_g"].T], -1) @ d["W_in"][:, :2 * R].T
    low = d["L"].tril(-1).permute(1, 2, 0)                       # [k][i][channel]
    y = i["seed_ids"][rows].long() if i["seed_ids"] is not None else s.argmax(-1)
    logits = s
    for _ in range(c["K"]):
        prev = torch.cat([i["anchor"][rows].long()[:, None], y[:, :-1]], 1)
        a = fixed + d["W_e"][prev] @ d["W_in"][:, 2 * R:].T
        mixed = a + (low[None] * a[:, None]).sum(2)
        z = mixed + torch.nn.functional.silu(mixed @ d["W_1"].T) @ d["W_2"].T
        if c["dtype"] == "bf16":
            z = z.to(torch.bfloat16).to(f64)                     # z is stored as the weights are
        logits = s + z @ d["W_r"].T
        y = logits.argmax(-1)
    return logits


def _exact_layer(c, seed):
    w, i = _layer_inputs(c, seed)
    f64 = torch.float64
    d = {k: v.to(f64) for k, v in w.items()}
    n, B, H, nh, nkv = c["batch"], c["B"], c["H"], c["n_heads"], c["n_kv"]
    norm = lambda t, g: t * torch.rsqrt((t * t).mean(-1, keepdim=True) + EPS) * g  # noqa: E731
    inv = THETA ** (-2.0 * torch.arange(HD // 2, dtype=f64, device="cuda") / HD)
    h = torch.empty((n, B, H), dtype=f64, device="cuda")
    hidden = torch.ones((B, B), dtype=torch.bool, device="cuda").triu(1) if c["causal"] else None
    for b, C in enumerate(i["ctx_len"].tolist()):
        x = i["x"][b].to(f64)
        u = norm(x, d["g_attn"])
        ang = (C + torch.arange(B, dtype=f64, device="cuda"))[:, None, None] * inv
        def rope(t):
            p, r = t[..., :HD // 2], t[..., HD // 2:]
            return torch.cat([p * ang.cos() - r * ang.sin(), r * ang.cos() + p * ang.sin()], -1)
        q = rope(norm((u @ d["Wq"].T).view(B, nh, HD), d["g_q"]))
        k = rope(norm((u @ d["Wk"].T).view(B, nkv, HD), d["g_k"]))
        keys = torch.cat([i["k_cache"][b, :C].to(f64), k]).permute(1, 2, 0).contiguous()
        vals = torch.cat([i["v_cache"][b, :C].to(f64), (u @ d["Wv"].T).view(B, nkv, HD)])
        qg = q.view(B, nkv, nh // nkv, HD).permute(1, 2, 0, 3).reshape(nkv, -1, HD)
        sc = (qg @ keys / math.sqrt(HD)).view(nkv, nh // nkv, B, C + B)
        if hidden is not None:
            sc[..., C:].masked_fill_(hidden, -math.inf)
        o = sc.softmax(-1).view(nkv, -1, C + B) @ vals.permute(1, 0, 2).contiguous()
        o = o.view(nkv, nh // nkv, B, HD).permute(2, 0, 1, 3).reshape(B, nh * HD)
        x1 = x + o @ d["Wo"].T
        u2 = norm(x1, d["g_mlp"])
        h[b] = x1 + (torch.nn.functional.silu(u2 @ d["Wg"].T) * (u2 @ d["Wu"].T)) @ d["Wd"].T
    return {"h_f32": h, "h_bf16": h}
