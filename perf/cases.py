"""The work a serving program has this library do, as cases that can be timed.

A cycle of speculative decoding calls the library three times: it drafts
(`Drafter.forward`: the pass and its tree), it accepts after the target has
verified the tree (`Drafter.accept_sample`), and it writes the drafter's cache
rows of the verified positions (`Drafter.kv_update`).  A new prompt is one
larger `kv_update`.  The cases are these calls, each through the entry point
that such a program uses, at the drafter shapes of `fe_synth.configs`, from
the smallest (the tiny fp32 drafter, a pass of a few launches) to the largest
(the 70B-shaped pass and the self-context prefill).

What the outputs are: the pass returns its logits, the probabilities of its
candidates and the tree's structure.  In bf16 it does not return the
candidates' ids: the logits of random weights lie so close that the rounding
of one layer decides which of two ids comes first, so ids say nothing about
correctness that the logits and the candidates' probabilities do not say; in
fp32, for one sequence, the ids and the tree's tokens are returned too.  For drawn
candidates (`draw` in the case) the probabilities are left out as well: which
candidate is drawn turns on the same near-ties.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2509_20416_amd.drafter import DeviceInputs, Drafter

DEV = "cuda:0"
TORCH_TYPE = {"bf16": torch.bfloat16, "f32": torch.float32}
FIELDS = ("attn_norm", "wq", "wk", "wv", "wo", "mlp_norm", "w_gate", "w_up", "w_down")
N_FEAT = 3      # target features per position (low, middle, high)
RMS_EPS = 1e-5

# Drafter widths of the target families the library is used with.
SHAPES = {
    "tiny": dict(hidden=256, hq=4, hkv=4, dim=64, inter=704, vocab=1024, tvocab=1024, theta=10000.0),
    "8b": dict(hidden=4096, hq=32, hkv=8, dim=128, inter=14336, vocab=32000, tvocab=128256,
               theta=500000.0),
    "13b": dict(hidden=5120, hq=40, hkv=40, dim=128, inter=13824, vocab=32000, tvocab=32000,
                theta=10000.0),
    "70b": dict(hidden=8192, hq=64, hkv=8, dim=128, inter=28672, vocab=32000, tvocab=128256,
                theta=500000.0),
}


def _pass(name, shape, **kw):
    c = dict(name=name, kind="pass", dtype="bf16", ctx="cascade", batch=1, plo=1024, phi=1024,
             layers=5, topk=8, graph=True, draw=False, temp=1.0)
    return {**c, **SHAPES[shape], **kw}


def _update(name, shape, **kw):
    c = dict(name=name, kind="update", dtype="bf16", ctx="cascade", batch=1, rows=1024, plo=0, phi=0,
             layers=5)
    return {**c, **SHAPES[shape], **kw}


def listed():
    return [
        # The smallest call: an fp32 drafter of 2 layers, all latency and launches.
        _pass("tiny_f32_b1", "tiny", dtype="f32", layers=2, topk=4, plo=64, phi=64),
        # One user decoding with an 8B-class target: the library's headline call.
        _pass("8b_b1", "8b"),
        # One user of a 13B-class multi-head target with a longer history.
        _pass("13b_b1", "13b", layers=6, plo=2048, phi=2048),
        # One user of a 70B-class target with a long history: the heaviest weights.
        _pass("70b_b1", "70b", plo=4096, phi=4096, topk=10),
        # A small serving batch at temperature 1 with drawn candidates, ragged
        # histories, launched without a graph (the batch changes as requests come and go).
        _pass("8b_b6_sampled", "8b", batch=6, plo=150, phi=3000, graph=False, draw=True),
        # A middling batch of a multi-head drafter.
        _pass("13b_b12", "13b", batch=12, layers=4, plo=100, phi=2000, topk=6),
        # The large serving batch: 32 ragged histories, 7 layers.
        _pass("8b_b32", "8b", batch=32, layers=7, plo=256, phi=8192),
        # After one cycle of one user: the cache rows of its accepted tokens.
        _update("8b_update_cycle", "8b", rows=6, plo=1024, phi=1024),
        # After one cycle of the batch of 32: 1 to 8 rows of each sequence.
        _update("8b_update_b32", "8b", batch=32, rows=147, layers=7, plo=256, phi=2048),
        # A new prompt of 1024 tokens.
        _update("8b_update_prompt", "8b", rows=1024),
        # The same prompt where every layer keys its own input: a prefill of the N layers.
        _update("8b_self_prompt", "8b", rows=1024, ctx="self"),
        # Acceptance of a batch's sampled trees after verification.
        dict(name="accept_b8", kind="accept", batch=8, layers=5, topk=8, vocab=32000, tvocab=128256,
             temp=1.0, drawn=True),
    ]


def _ids_fixed(c):
    """Whether rounding leaves the candidates' order alone: fp32 and a single sequence."""
    return c["dtype"] == "f32" and c["batch"] == 1


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_shape(rng, hmax):
    """Widths of some drafter: head dim 64 or 128, grouped or multi-head, MLP
    and vocabulary of any legal size."""
    dim = rng.choice((64, 128, 128))
    hq = max(2, _log_int(rng, 512, hmax) // dim)
    group = rng.choice([g for g in (1, 2, 4, 8) if hq % g == 0])
    hidden = hq * dim
    inter = 32 * max(8, int(hidden * rng.uniform(2.2, 3.6)) // 32)
    vocab = 16 * _log_int(rng, 64, 2000)
    tvocab = min(131072, int(vocab * rng.uniform(1.0, 4.0)))
    return dict(hidden=hidden, hq=hq, hkv=hq // group, dim=dim, inter=inter, vocab=vocab,
                tvocab=tvocab, theta=rng.choice((10000.0, 500000.0)))


def draw(rng):
    while True:
        kind = rng.choice(("pass", "pass", "pass", "update", "update", "self", "accept"))
        if kind == "pass":
            f32 = rng.random() < 0.2
            s = _draw_shape(rng, 1024 if f32 else 8192)
            phi = _log_int(rng, 16, 8192)
            c = dict(kind="pass", dtype="f32" if f32 else "bf16",
                     ctx=rng.choice(("cascade", "cascade", "cascade", "self")),
                     batch=_log_int(rng, 1, 32), plo=max(1, int(phi * rng.uniform(0.1, 1.0))), phi=phi,
                     layers=rng.randint(2, 8), topk=rng.randint(2, 10), graph=rng.random() < 0.6,
                     draw=rng.random() < 0.25, temp=round(rng.uniform(0.6, 1.0), 2), **s)
        elif kind == "accept":
            c = dict(kind="accept", batch=_log_int(rng, 1, 32), layers=rng.randint(2, 8),
                     topk=rng.randint(2, 10), vocab=16 * _log_int(rng, 64, 2000), tvocab=0, temp=1.0,
                     drawn=rng.random() < 0.7)
            c["tvocab"] = min(131072, int(c["vocab"] * rng.uniform(1.0, 4.0)))
        else:
            s = _draw_shape(rng, 6144)
            rows = _log_int(rng, 1, 2500)
            batch = min(rows, rng.choice((1, 1, 2, 5, 16)))
            c = dict(kind="update", dtype="bf16", ctx="self" if kind == "self" else "cascade",
                     batch=batch, rows=rows, plo=0, phi=0, layers=rng.randint(2, 8), **s)
        if c["kind"] == "accept":
            if c["tvocab"] >= c["vocab"]:
                return c
            continue
        w = work(c)
        if w["bytes"] < 6e9 and w["flops"] < 2.2e12 and c["tvocab"] >= c["vocab"]:
            return c


# ---------------------------------------------------------------------------
# What a program holds before the call.
# ---------------------------------------------------------------------------
def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + salt) & 0x7fffffffffff)
    return g


def _weights(c, seed):
    """Weights of the widths in `c`: N(0, 0.02) matrices, gains about 1, a
    random one-to-one map from draft to target ids."""
    g, dt = _gen(seed, 1), TORCH_TYPE[c["dtype"]]
    d, inter, qd, kvd = c["hidden"], c["inter"], c["hq"] * c["dim"], c["hkv"] * c["dim"]

    def lin(*shape):
        return torch.empty(shape, dtype=dt, device=DEV).normal_(0.0, 0.02, generator=g)

    def gain():
        return torch.empty(d, dtype=torch.float32, device=DEV).normal_(1.0, 0.02, generator=g).to(dt)

    layers = []
    for _ in range(c["layers"]):
        lw = SimpleNamespace(FIELDS=FIELDS, attn_norm=gain(), wq=lin(qd, d), wk=lin(kvd, d),
                             wv=lin(kvd, d), wo=lin(d, qd), mlp_norm=gain(), w_gate=lin(inter, d),
                             w_up=lin(inter, d), w_down=lin(d, inter))
        layers.append(lw)
    if c["vocab"] == c["tvocab"]:
        d2t = np.arange(c["vocab"], dtype=np.int32)
    else:
        d2t = np.sort(np.random.default_rng(int(seed)).choice(c["tvocab"], c["vocab"], replace=False))
    return SimpleNamespace(w_fuse=lin(d, N_FEAT * d), w_in=lin(d, 2 * d), embed=lin(c["tvocab"], d),
                           final_norm=gain(), lm_head=lin(c["vocab"], d), d2t=d2t.astype(np.int32),
                           layers=layers)


def _config(c, **kw):
    g = dict(hidden=512, hq=4, hkv=4, dim=128, inter=1024, theta=10000.0, dtype="bf16", ctx="cascade",
             topk=1)
    g.update(c)
    return SimpleNamespace(hidden=g["hidden"], n_q_heads=g["hq"], n_kv_heads=g["hkv"],
                           head_dim=g["dim"], intermediate=g["inter"], n_layers=g["layers"],
                           draft_vocab=g["vocab"], target_vocab=g["tvocab"], n_feat_levels=N_FEAT,
                           rope_theta=g["theta"], rms_eps=RMS_EPS, dtype=g["dtype"],
                           cascade_ctx=g["ctx"], topk=g["topk"], batch=g["batch"], **kw)


def _lens(c):
    """Prefix length of each sequence, part of the case (so that its work is known)."""
    r = np.random.default_rng(12345 + 7 * c["batch"] + c["phi"])
    return r.integers(c["plo"], c["phi"] + 1, c["batch"]).astype(np.int32)


def _pass_inputs(c, seed):
    g, dt = _gen(seed, 2), TORCH_TYPE[c["dtype"]]
    lens = _lens(c)
    kv = (int(lens.sum()), c["hkv"], c["dim"])
    new = lambda shape: torch.empty(shape, dtype=dt, device=DEV).normal_(generator=g)  # noqa: E731
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    return SimpleNamespace(
        lens=lens, features=new((c["batch"], N_FEAT * c["hidden"])),
        tokens=torch.randint(0, c["tvocab"], (c["batch"],), generator=g, device=DEV, dtype=torch.int32),
        cu=torch.from_numpy(cu).to(DEV), k=[new(kv) for _ in range(c["layers"])],
        v=[new(kv) for _ in range(c["layers"])])


def _update_inputs(c, seed):
    """The verified rows: each sequence appends its share of `rows` to a cache
    of its own that already holds its prefix.  The caches hold zeros where
    nothing has been written (the cascade's rows do not depend on them)."""
    g, dt = _gen(seed, 3), TORCH_TYPE[c["dtype"]]
    share = np.full(c["batch"], c["rows"] // c["batch"], dtype=np.int64)
    share[: c["rows"] % c["batch"]] += 1
    if c["batch"] > 2:  # uneven, as acceptance leaves them
        moved = share[::3] // 2
        share[::3] -= moved
        share[1] += moved.sum()
        over = max(0, int(share[1]) - 8) if c["rows"] <= 8 * c["batch"] else 0
        i = c["batch"] - 1
        share[1] -= over
        while over > 0:
            add = int(min(over, max(0, 8 - share[i])))
            share[i] += add
            over -= add
            i -= 1
    first = _lens(c).astype(np.int64)  # position of the first new row
    pos, dst, row = [], [], 0
    for b in range(c["batch"]):
        pos.append(first[b] + np.arange(share[b]))
        dst.append(row + np.arange(share[b]))  # the rows of this call, one sequence after the other
        row += int(share[b])
    up = lambda a: torch.from_numpy(np.concatenate(a).astype(np.int32)).to(DEV)  # noqa: E731
    return SimpleNamespace(
        features=torch.empty((c["rows"], N_FEAT * c["hidden"]), dtype=dt, device=DEV).normal_(generator=g),
        tokens=torch.randint(0, c["tvocab"], (c["rows"],), generator=g, device=DEV, dtype=torch.int32),
        pos=up(pos), dst=up(dst), share=share,
        max_pos=int(max(p.max() if len(p) else 0 for p in pos)) + 1)


def _accept_inputs(c, seed):
    """A batch's sampled candidates and the target's distributions after every
    node: the target agrees with the draft up to noise, as a trained drafter's does."""
    g = _gen(seed, 4)
    B, N, k, V, Vt = c["batch"], c["layers"], c["topk"], c["vocab"], c["tvocab"]
    rnd = lambda *s: torch.randn(s, generator=g, device=DEV)  # noqa: E731
    d2t = np.sort(np.random.default_rng(int(seed)).choice(Vt, V, replace=False)).astype(np.int32)
    logits = 2.5 * rnd(B, N, V)
    # 23-bit uniforms inside (0, 1), as the library's own generator gives them
    unit = lambda *s: (torch.randint(0, 1 << 23, s, generator=g, device=DEV).double() + 0.5) / (1 << 23)  # noqa: E731
    uni = unit(B, N, V).float()
    z = logits.double() / c["temp"]
    key = z - torch.log(-torch.log(uni.double())) if c["drawn"] else z
    cand = key.topk(k, dim=-1).indices
    order = z.gather(-1, cand).argsort(dim=-1, descending=True, stable=True)
    cand = cand.gather(-1, order)
    t = torch.from_numpy(d2t).to(DEV)
    ids = t[cand].to(torch.int32)
    T = 1 + N * k
    level = torch.cat([torch.zeros(1), torch.arange(N * k) // k + 1]).long().clamp(max=N - 1).to(DEV)
    probs = torch.empty((B, T, Vt), device=DEV)
    for b in range(B):
        zt = torch.full((T, Vt), -4.0, device=DEV) + rnd(T, Vt)
        zt[:, t.long()] = logits[b, level] + 0.7 * rnd(T, V)
        probs[b] = torch.softmax(zt / c["temp"], -1)
    return SimpleNamespace(
        d2t=d2t, logits=logits, uniforms=uni if c["drawn"] else None, topk_draft=cand.to(torch.int32),
        ids=ids, probs=probs, roots=torch.zeros(B, dtype=torch.int32, device=DEV),
        u=unit(B, N * k + 1).float())


def prepare(c, seed):
    if c["kind"] == "pass":
        i = _pass_inputs(c, seed)
        pmax = int(i.lens.max())
        dr = Drafter(_config(c, prefix=pmax), _weights(c, seed), device=DEV, max_batch=c["batch"],
                     max_prefix=pmax, max_topk=c["topk"], graph=c["graph"])
        di = DeviceInputs(batch=c["batch"], features=i.features, next_tokens=i.tokens,
                          prefix_lens=torch.from_numpy(i.lens).to(DEV), cu_prefix=i.cu, kcache=i.k,
                          vcache=i.v, max_prefix=pmax)
        return SimpleNamespace(
            case=c, dr=dr, di=di, out=dr.alloc_outputs(c["batch"], c["topk"], logits=True),
            tree=dr.alloc_tree(c["batch"], c["topk"]),
            so=torch.tensor([seed, 3], dtype=torch.int64, device=DEV) if c["draw"] else None)
    if c["kind"] == "update":
        i = _update_inputs(c, seed)
        dr = Drafter(_config(c, prefix=i.max_pos), _weights(c, seed), device=DEV, max_batch=1,
                     max_prefix=i.max_pos)
        shape = (c["rows"], c["hkv"], c["dim"])
        cache = lambda: [torch.zeros(shape, dtype=TORCH_TYPE[c["dtype"]], device=DEV)  # noqa: E731
                         for _ in range(c["layers"])]
        return SimpleNamespace(case=c, dr=dr, i=i, k=cache(), v=cache())
    i = _accept_inputs(c, seed)
    w = _weights({**c, "hidden": 512, "hq": 4, "hkv": 4, "dim": 128, "inter": 1024, "dtype": "bf16"}, seed)
    w.d2t = i.d2t
    dr = Drafter(_config(c, prefix=16), w, device=DEV, max_batch=c["batch"], max_prefix=16,
                 max_topk=c["topk"])
    tree = dr.alloc_tree(c["batch"], c["topk"])
    lens = torch.ones(c["batch"], dtype=torch.int32, device=DEV)
    di = DeviceInputs(batch=c["batch"], features=None, next_tokens=i.roots, prefix_lens=lens,
                      cu_prefix=None, kcache=[], vcache=[], max_prefix=16)
    dr.build_tree(di, i.ids, c["topk"], out=tree)
    return SimpleNamespace(case=c, dr=dr, i=i, tree=tree)


# ---------------------------------------------------------------------------
# One pass through the entry point.
# ---------------------------------------------------------------------------
def run(s):
    c = s.case
    if c["kind"] == "pass":
        if c["draw"]:
            s.dr.forward(s.di, c["topk"], out=s.out, tree=s.tree, temperature=c["temp"],
                         seed_offset=s.so)
        elif c["temp"] != 1.0:
            s.dr.forward(s.di, c["topk"], out=s.out, tree=s.tree, temperature=c["temp"])
        else:
            s.dr.forward(s.di, c["topk"], out=s.out, tree=s.tree)
        t = s.tree
        got = {"logits": s.out["logits"], "depth": t["depth"], "mask": t["mask"],
               "parents": t["parents"], "positions": t["positions"], "retrieve": t["retrieve"]}
        if not c["draw"]:
            got["topk_probs"] = s.out["topk_probs"]
            if _ids_fixed(c):
                got["topk_ids"] = s.out["topk_ids"]
                got["tokens"] = t["tokens"]
        return got
    if c["kind"] == "update":
        i = s.i
        s.dr.kv_update(i.features, i.tokens, i.pos, i.dst, s.k, s.v)
        return {"k": s.k, "v": s.v}
    i = s.i
    return s.dr.accept_sample(s.tree, i.topk_draft, i.logits, i.probs, i.u, temperature=c["temp"],
                              draft_uniforms=i.uniforms, topk=c["topk"])


# ---------------------------------------------------------------------------
# The same in 64 bits, in plain torch.
# ---------------------------------------------------------------------------
def _norm(x, gamma):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + RMS_EPS) * gamma.double()


def _lin(x, w):
    return x @ w.double().t()


def _rope(x, pos, theta):
    """Rotary embedding of x [rows, heads, D] at positions pos [rows]."""
    D = x.shape[-1]
    m = torch.arange(D // 2, dtype=torch.float64, device=DEV)
    ang = pos.double()[:, None] * torch.pow(torch.tensor(float(theta), dtype=torch.float64, device=DEV), -2.0 * m / D)
    cos, sin = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    a, b = x[..., : D // 2], x[..., D // 2:]
    return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)


def _attend(q, k, v, mask=None):
    """q [m, Hq, D] over k, v [n, Hkv, D] -> [m, Hq * D]; mask [m, n] of the keys seen."""
    g = q.shape[1] // k.shape[1]
    k, v = (t.repeat_interleave(g, 1).transpose(0, 1).contiguous() for t in (k, v))  # [Hq, n, D]
    out = []
    for h in range(q.shape[1]):
        s = (q[:, h].contiguous() @ k[h].t()) / math.sqrt(q.shape[-1])
        if mask is not None:
            s = s.masked_fill(~mask, -math.inf)
        out.append(torch.softmax(s, -1) @ v[h])
    return torch.stack(out, 1).reshape(q.shape[0], -1)


def _mlp(x, lw):
    n = _norm(x, lw.mlp_norm)
    return x + _lin(torch.nn.functional.silu(_lin(n, lw.w_gate)) * _lin(n, lw.w_up), lw.w_down)


def _x0(w, features, tokens):
    g = _lin(features.double(), w.w_fuse)
    return _lin(torch.cat([g, w.embed[tokens.long()].double()], -1), w.w_in)


def _exact_pass(c, seed):
    i, w = _pass_inputs(c, seed), _weights(c, seed)
    B, hq, hkv, D = c["batch"], c["hq"], c["hkv"], c["dim"]
    lens = torch.from_numpy(i.lens).to(DEV)
    xs = [_x0(w, i.features, i.tokens)]
    for l, lw in enumerate(w.layers):
        ctx = xs if c["ctx"] == "cascade" else xs[-1:]
        q = _rope(_lin(_norm(xs[-1], lw.attn_norm), lw.wq).view(B, hq, D), lens + len(ctx) - 1, c["theta"])
        ks, vs = [], []
        for j, x in enumerate(ctx):
            n = _norm(x, lw.attn_norm)
            ks.append(_rope(_lin(n, lw.wk).view(B, hkv, D), lens + j, c["theta"]))
            vs.append(_lin(n, lw.wv).view(B, hkv, D))
        ao, row = [], 0
        for b in range(B):
            P = int(i.lens[b])
            k = torch.cat([i.k[l][row:row + P].double()] + [t[b:b + 1] for t in ks])
            v = torch.cat([i.v[l][row:row + P].double()] + [t[b:b + 1] for t in vs])
            ao.append(_attend(q[b:b + 1], k, v))
            row += P
        xs.append(_mlp(xs[-1] + _lin(torch.cat(ao), lw.wo), lw))
    logits = torch.stack([_lin(_norm(x, w.final_norm), w.lm_head) for x in xs[1:]], 1)
    got = {"logits": logits, "depth": None, "mask": None, "parents": None, "positions": None,
           "retrieve": None}
    if not c["draw"]:
        got["topk_probs"] = torch.softmax(logits / c["temp"], -1).topk(c["topk"], dim=-1).values
        if _ids_fixed(c):
            got["topk_ids"] = got["tokens"] = None
    return got


def _exact_update(c, seed):
    i, w = _update_inputs(c, seed), _weights(c, seed)
    hq, hkv, D, M = c["hq"], c["hkv"], c["dim"], c["rows"]
    x = _x0(w, i.features, i.tokens)
    got = {"k": [], "v": []}
    if c["ctx"] == "self":  # row m sees the rows of its sequence up to itself
        b = torch.from_numpy(np.repeat(np.arange(len(i.share)), i.share)).to(DEV)
        r = torch.arange(M, device=DEV)
        mask = (b[:, None] == b[None]) & (r[None] <= r[:, None])
    for lw in w.layers:
        n = _norm(x, lw.attn_norm)
        k = _rope(_lin(n, lw.wk).view(M, hkv, D), i.pos, c["theta"])
        v = _lin(n, lw.wv).view(M, hkv, D)
        got["k"].append(k)
        got["v"].append(v)
        if c["ctx"] == "self":
            q = _rope(_lin(n, lw.wq).view(M, hq, D), i.pos, c["theta"])
            x = _mlp(x + _lin(_attend(q, k, v, mask), lw.wo), lw)
    return got


def exact(c, seed):
    if c["kind"] == "pass":
        return _exact_pass(c, seed)
    if c["kind"] == "update":
        return _exact_update(c, seed)
    return None  # acceptance gives whole numbers


# ---------------------------------------------------------------------------
# What a pass cannot do without, and how far apart two correct ones are.
# ---------------------------------------------------------------------------
def work(c):
    if c["kind"] == "accept":
        # the draft's and the target's row of every level that the walk can
        # visit, the uniforms of the candidates, the tree
        B, N, k, T = c["batch"], c["layers"], c["topk"], 1 + c["layers"] * c["topk"]
        rows = B * (N * c["vocab"] + (N + 1) * c["tvocab"])
        return {"bytes": 4 * (rows + B * (4 * T + N * (k + 2))), "flops": 4 * rows}
    es = 2 if c["dtype"] == "bf16" else 4
    d, inter, N, V = c["hidden"], c["inter"], c["layers"], c["vocab"]
    qd, kvd = c["hq"] * c["dim"], c["hkv"] * c["dim"]
    fc = N_FEAT * d * d + 2 * d * d
    layer = d * (2 * qd + 2 * kvd) + 3 * d * inter
    if c["kind"] == "update":
        M = c["rows"]
        mats = fc + N * (layer if c["ctx"] == "self" else 2 * d * kvd)
        if c["ctx"] == "self":  # the last layer only writes its keys and values
            mats -= layer - 2 * d * kvd
        flops = 2 * M * mats
        if c["ctx"] == "self":
            share = M / c["batch"]
            flops += (N - 1) * 4 * qd * M * share / 2
        return {"bytes": es * (mats + M * (N_FEAT * d + d + 2 * N * kvd)), "flops": flops}
    B, lens = c["batch"], _lens(c)
    flops = 2 * B * fc + 2 * B * N * V * d
    for i in range(1, N + 1):
        nctx = i if c["ctx"] == "cascade" else 1
        flops += 2 * B * (layer + (nctx - 1) * 2 * d * kvd)
        flops += 4 * qd * (int(lens.sum()) + nctx * B)
    nbytes = es * (fc + N * layer + V * d + 2 * N * kvd * int(lens.sum()) + B * (N_FEAT + 1) * d)
    T = 1 + N * c["topk"]
    nbytes += 4 * B * N * V + B * (T * (16 + T) + 4 * (N * (c["topk"] - 1) + 1) * (N + 1))
    return {"bytes": nbytes, "flops": flops}


def tolerance(c):
    """About four times the distance to exact() that the path shows: logits
    0.0045 to 0.0053 and probabilities up to 0.009 (bf16 activations through 2 to 8 layers), cache
    rows 0.0029 after one norm and 0.0056 after four layers, fp32 sums 4e-7
    (more over the wider sums that `draw` reaches)."""
    if c["kind"] == "accept":
        return "exact"
    if c["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3, "differ": 0.0}
    if c["kind"] == "update" and c["ctx"] != "self":
        return {"rel": 0.012, "max": 0.1, "differ": 0.0}
    return {"rel": 0.02, "max": 0.2, "differ": 0.0}
