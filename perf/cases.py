"""The work that a user of this library has it do, as cases that can be timed and compared.

A case is a dict of plain sizes; `listed()` names the ones that stand for the real uses, `draw()` gives further ones of
the same ranges, `prepare()` builds what a decoding program holds before the call (weights, paged cache, candidate
tokens), `run()` is one pass through the public entry points of `Session`, `exact()` the same values in 64 bits from
plain torch.  Sizes come from the workload configurations of `synth/configs.py` (7B, 13B and 33B LLaMA shapes, the tiny
fp32 shape); single uses run a few decoder layers of those shapes, since every layer of a model does the same work.

Weights are random of the width that initialisation gives.  The rows of the LM head and of the draft heads' vocabulary
projections are scaled by u^(-1/2), u uniform: logits of trained models are peaked, and the greedy token or the order of
the candidates then does not hang on the last bits of near-equal logits, as it would with identically spread rows.
"""
from __future__ import annotations

import heapq
import math
import zlib
from types import SimpleNamespace

import torch

from paper_2402_05109_amd.session import Session

DEV = "cuda:0"
STD = 0.02
EPS, THETA = 1e-6, 10000.0


# ---- cases -------------------------------------------------------------------------------------------------------
# kind      what one pass is
# verify    tree_verify_forward over B rows x T tree nodes behind `ctx` cached tokens (T = 1: plain decoding)
# prefill   Session.reset + Session.prefill of a prompt of `ctx` tokens in chunks of `chunk`
# draft     hydra_draft_tree: `K` heads of `mlp` layers expand the tree of T nodes for B rows
# prefix    hydra_prefix_attention: the Hydra++ layer over the tokens a step accepted
# tail      accept_typical (seeded uniform numbers) + kv_compact over all layers of the cache
# generate  Session.generate: the decoding loop itself, fp32, draft / verify / accept / compact and the read-back
_7B = dict(H=32, Dh=128, F=11008, V=32000)
_13B = dict(H=40, Dh=128, F=13824, V=32000)
_33B = dict(H=52, Dh=128, F=17920, V=32000)


def listed():
    return [
        # the headline: one request of the 7B shape, the whole verification call of a decoding step, 64-node tree
        dict(name="verify_7b_full", kind="verify", NL=32, **_7B, B=1, T=64, ctx=776, logits=1),
        # a full serving batch: 16 requests x 64 nodes, 1024-token contexts
        dict(name="verify_7b_batch16", kind="verify", NL=8, **_7B, B=16, T=64, ctx=1024, logits=1),
        # a small batch of the largest shape at a long context
        dict(name="verify_33b_batch4", kind="verify", NL=3, **_33B, B=4, T=64, ctx=2048, logits=1),
        # one request of the middle shape near the longest context, the smaller tree, odd length
        dict(name="verify_13b_long", kind="verify", NL=4, **_13B, B=1, T=32, ctx=3891, logits=1),
        # plain autoregressive decoding, the baseline that every user also runs: one node, greedy token only
        dict(name="decode_7b", kind="verify", NL=8, **_7B, B=1, T=1, ctx=701, logits=0),
        # the small trees that pay at larger batches; 96 rows, odd context
        dict(name="verify_7b_batch8_t12", kind="verify", NL=4, **_7B, B=8, T=12, ctx=517, logits=1),
        # reading a prompt: 1000 tokens in chunks of 128, the last one ragged
        dict(name="prefill_7b", kind="prefill", NL=2, **_7B, B=1, ctx=1000, chunk=128),
        # drafting for one request: Hydra heads
        dict(name="draft_7b", kind="draft", **_7B, B=1, T=64, K=4, mlp=1),
        # drafting for a batch: Hydra++ heads with four MLP layers
        dict(name="draft_7b_plus_batch4", kind="draft", **_7B, B=4, T=64, K=4, mlp=4),
        # the Hydra++ prefix layer after a step
        dict(name="prefix_7b_batch4", kind="prefix", **_7B, B=4, T=64, ctx=1030),
        # the end of a sampled step: acceptance test over the logits, compaction of 32 layers of cache (the
        # FFN, which takes no part, is small)
        dict(name="tail_7b_batch4", kind="tail", NL=32, H=32, Dh=128, F=256, V=32000, B=4, T=64, ctx=300),
        # the smallest use: the tiny fp32 model, a whole short generation through the loop
        dict(name="generate_tiny_f32", kind="generate", NL=2, H=4, Dh=64, F=688, V=1024, B=1, T=16, ctx=128, K=3, mlp=1, new=16),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _shape(rng):
    if rng.random() < 0.5:
        return dict(rng.choice((_7B, _13B, _33B)))
    H, Dh = rng.choice(((16, 64), (16, 128), (24, 128), (32, 128), (40, 128), (48, 128)))
    d = H * Dh
    return dict(H=H, Dh=Dh, F=128 * max(1, round(d * rng.uniform(2.0, 4.0) / 128)), V=rng.choice((32000, 32016, 32003, rng.randrange(8000, 50000))))


def draw(rng):
    kind = rng.choices(("verify", "prefill", "draft", "prefix", "tail", "generate"), (9, 2, 3, 2, 2, 2))[0]
    if kind == "generate":
        H = rng.choice((2, 4, 8))
        return dict(kind=kind, NL=rng.randint(1, 3), H=H, Dh=64, F=16 * rng.randint(16, 64), V=rng.randrange(500, 4000), B=rng.choice((1, 1, 2, 3)),
                    T=rng.randint(4, 24), ctx=_log(rng, 8, 200), K=4, mlp=rng.randint(1, 2), new=rng.randint(4, 16))
    s = _shape(rng)
    B, T = _log(rng, 1, 16), _log(rng, 1, 128)
    while B * T > 1024:
        B = max(1, B // 2)
    ctx = _log(rng, 16, 4000)
    while B * ctx > 16384:
        ctx = ctx * 2 // 3
    if kind == "verify":
        return dict(kind=kind, NL=rng.randint(1, 2), **s, B=B, T=T, ctx=ctx, logits=rng.randint(0, 1))
    if kind == "prefill":
        return dict(kind=kind, NL=1, **s, B=min(B, 2), ctx=max(16, min(ctx, 1200)), chunk=rng.choice((64, 64, 128, rng.randint(16, 128))))
    T = max(T, 6)
    if kind == "draft":
        return dict(kind=kind, **s, B=min(B, 8), T=T, K=4, mlp=rng.randint(1, 4))
    if kind == "prefix":
        return dict(kind=kind, **s, B=B, T=T, ctx=ctx)
    return dict(kind=kind, NL=rng.randint(2, 32), **dict(s, F=256), B=min(B, 4), T=T, ctx=min(ctx, 1000))


# ---- candidate trees ---------------------------------------------------------------------------------------------
def tree(T, max_depth=4, ranks=10):
    """Parent list of T nodes in breadth-first order, grown greedily by 0.6 * 0.8^depth * 0.5^rank per edge."""
    have, heap = {(): 1.0}, []

    def offer(p):
        if p and p[-1] < ranks:
            w = have[p[:-1]] * 0.6 * 0.8 ** (len(p) - 1) * 0.5 ** p[-1]
            heapq.heappush(heap, (-w, len(p), p, w))

    offer((0,))
    while len(have) < T:
        _, _, p, w = heapq.heappop(heap)
        have[p] = w
        offer(p[:-1] + (p[-1] + 1,))
        if len(p) < max_depth:
            offer(p + (0,))
    order = sorted(have, key=lambda p: (len(p), p))
    at = {p: i for i, p in enumerate(order)}
    return [-1] + [at[p[:-1]] for p in order[1:]]


def depths(parent):
    dep = [0] * len(parent)
    for n in range(1, len(parent)):
        dep[n] = dep[parent[n]] + 1
    return dep


def ancestors(parent):
    T = len(parent)
    m = torch.zeros(T, T, dtype=torch.bool)
    for n in range(T):
        if n:
            m[n] = m[parent[n]]
        m[n, n] = True
    return m


# ---- inputs ------------------------------------------------------------------------------------------------------
def _gen(seed, what):
    return torch.Generator(device=DEV).manual_seed((int(seed) * 1000003 + zlib.crc32(what.encode())) & 0x7FFFFFFFFFFFFFFF)


def _rand(seed, what, shape, std=1.0):
    return torch.randn(shape, generator=_gen(seed, what), device=DEV) * std


def _tokens(seed, what, shape, V):
    return torch.randint(0, V, shape, generator=_gen(seed, what), device=DEV).to(torch.int32)


def weight(case, seed, name):
    """One weight of the model, by the names that Session asks for."""
    d, F, V = case["H"] * case["Dh"], case["F"], case["V"]
    dt = torch.float32 if case["kind"] == "generate" else torch.bfloat16
    leaf = name.split(".")[-1]
    if leaf.endswith("norm"):
        return (1.0 + _rand(seed, name, (d,), 0.1)).to(dt)
    if leaf in ("lm_head", "wout"):
        u = torch.rand(V, generator=_gen(seed, name + "/scale"), device=DEV).clamp_min(1e-5)
        return (_rand(seed, name, (V, d), STD) * u.rsqrt()[:, None]).to(dt)
    if leaf[0] == "b" and leaf[1:].isdigit():
        return _rand(seed, name, (d,), STD).to(dt)
    shape = {"embed": (V, d), "w_gate": (F, d), "w_up": (F, d), "w_down": (d, F)}.get(leaf, (d, d))
    if leaf == "w1":
        shape = (d, (int(name.split(".")[1]) + 1) * d)
    return _rand(seed, name, shape, STD).to(dt)


def lengths(case, seed):
    """Cached tokens of each row: requests of a batch are at different points, the longest at ctx."""
    B, ctx = case["B"], case["ctx"]
    cut = torch.randint(0, max(1, ctx // 4), (B,), generator=torch.Generator().manual_seed(int(seed) & 0x7FFFFFFF))
    cut[0] = 0
    return [ctx - int(c) for c in cut]


def _kv_plain(case, seed, layer, n):
    """K and V of n cached tokens of every row, of values that 16 bits hold."""
    return _rand(seed, "kv/%d" % layer, (case["B"], n, 2, case["H"], case["Dh"])).half().float()


def _shape_of(case):
    return SimpleNamespace(d=case["H"] * case["Dh"], NL=case.get("NL", 1), H=case["H"], Dh=case["Dh"], F=case["F"], V=case["V"],
                           dtype="f32" if case["kind"] == "generate" else "bf16", K=case.get("K", 0), mlp_layers=case.get("mlp", 1),
                           rms_eps=EPS, rope_theta=THETA, include_root_embedding=1, medusa=0, prefix=1 if case["kind"] == "prefix" else 0)


def _chunks(case):
    out, left = [], case["ctx"]
    while left > 0:
        out.append(min(case["chunk"], left))
        left -= out[-1]
    return out


def prepare(case, seed):
    kind, B = case["kind"], case["B"]
    parent = tree(case.get("T", 1))
    sess = Session(_shape_of(case), parent, B, case.get("ctx", 0) + case.get("new", 0) * 8, lambda name: weight(case, seed, name), device=DEV,
                   prefill_chunk=case.get("chunk", 64), page_perm_seed=int(seed) & 0x7FFFFFFF,
                   want_logits=bool(case.get("logits", 0)) or kind == "generate")
    st = {"case": case, "sess": sess}
    o = sess.out()
    V = case["V"]
    if kind in ("verify", "tail"):
        for l in range(case["NL"]):
            sess.main.kv_write(B, l, sess.kv, 0, case["ctx"], _kv_plain(case, seed, l, case["ctx"]))
        sess.seq_len.copy_(torch.tensor(lengths(case, seed), dtype=torch.int32))
        sess.host_len = case["ctx"]
    if kind == "verify":
        o.tree_tokens.copy_(_tokens(seed, "tokens", (B, case["T"]), V))
    elif kind == "prefill":
        st["prompt"] = _tokens(seed, "prompt", (B, case["ctx"]), V)
        for n in _chunks(case):
            sess.ctx("chain%d" % n)
    elif kind == "draft":
        sess.h_last.copy_(_rand(seed, "h", tuple(sess.h_last.shape)))
        sess.root.copy_(_tokens(seed, "root", (B,), V))
    elif kind == "prefix":
        o.hidden.copy_(_rand(seed, "h", tuple(o.hidden.shape)))
        n_acc, path = _paths(case, seed)
        o.n_acc.copy_(n_acc)
        o.path.copy_(path)
        sess.prefix_ctx(path.shape[1]).kv_write(B, 0, sess.pkv, 0, case["ctx"], _kv_plain(case, seed, 0, case["ctx"]))
        st["len"] = torch.tensor(lengths(case, seed), dtype=torch.int32, device=DEV)
        sess.host_len = case["ctx"]
    elif kind == "tail":
        o.hidden.copy_(_rand(seed, "h", tuple(o.hidden.shape)))
        st["logits"], toks = _tail_inputs(case, seed)
        o.tree_tokens.copy_(toks)
        o.logits = st["logits"]
        st["u"] = torch.rand(B, generator=_gen(seed, "u"), device=DEV)
        st["len"] = sess.seq_len.clone()
    elif kind == "generate":
        st["prompt"] = _tokens(seed, "prompt", (B, case["ctx"]), V)
        for n in {min(64, case["ctx"]), case["ctx"] % 64} - {0}:
            sess.ctx("chain%d" % n)
    return st


def _paths(case, seed):
    """Accepted paths of a step: per row a root path of the tree, of random length."""
    parent = tree(case["T"])
    P = max(depths(parent)) + 1
    g = torch.Generator().manual_seed(int(seed) & 0x7FFFFFFF)
    n_acc, path = [], torch.full((case["B"], P), -1, dtype=torch.int32)
    for b in range(case["B"]):
        n = int(torch.randint(0, case["T"], (1,), generator=g))
        p = []
        while n >= 0:
            p.append(n)
            n = parent[n]
        n_acc.append(len(p))
        path[b, :len(p)] = torch.tensor(p[::-1], dtype=torch.int32)
    return torch.tensor(n_acc, dtype=torch.int32), path


def _tail_inputs(case, seed):
    """Peaked logits and a tree whose candidates are the likely tokens of their parents."""
    B, T, V = case["B"], case["T"], case["V"]
    parent = tree(T)
    lg = _rand(seed, "logits", (B, T, V), 2.0)
    top = _tokens(seed, "top", (B, T, 10), V).long()
    lg.scatter_add_(2, top, torch.linspace(16.0, 12.0, 10, device=DEV).expand(B, T, 10).contiguous())
    best = lg.topk(10, dim=2).indices.to(torch.int32)
    toks = _tokens(seed, "root", (B, T), V)
    rank = {}
    for n in range(1, T):
        r = rank[parent[n]] = rank.get(parent[n], -1) + 1
        toks[:, n] = best[:, parent[n], r]
    return lg, toks


TYPICAL = (1.0, 0.09, 0.3)       # tau, eps, alpha


def _many(case):
    """Enough rows that the 2-norm of their margins says something: a margin is the difference of two logits, and a
    single one can be small against the roundings of both."""
    return case["B"] * case["T"] >= 64


# ---- one pass ----------------------------------------------------------------------------------------------------
def run(st):
    case, sess = st["case"], st["sess"]
    kind, o = case["kind"], sess.out()
    if kind == "verify":
        sess.verify()
        out = {"hidden": o.hidden, "argmax": o.argmax, "k": sess.k_pages, "v": sess.v_pages}
        if case["logits"]:
            out["logits"] = o.logits
        elif _many(case):
            out["margin"] = o.margin
        return out
    if kind == "prefill":
        sess.reset()
        sess.prefill(st["prompt"])
        last = sess.out("chain%d" % _chunks(case)[-1])
        return {"h_last": sess.h_last, "root": sess.root, "seq_len": sess.seq_len, "hidden": last.hidden, "k": sess.k_pages, "v": sess.v_pages}
    if kind == "draft":
        sess.draft()
        return {"tokens": o.tree_tokens}
    if kind == "prefix":
        sess.pseq_len.copy_(st["len"])          # the state of this step again: the call advances it
        sess.prefix_attention()
        return {"h_last": sess.h_last, "seq_len": sess.pseq_len, "k": sess.pk_pages, "v": sess.pv_pages}
    if kind == "tail":
        sess.seq_len.copy_(st["len"])           # as above
        sess.accept_typical(*TYPICAL, st["u"])
        sess.compact()
        sess.host_len = case["ctx"]
        return {"n_acc": o.n_acc, "path": o.path, "next_root": o.next_root, "last_node": o.last_node, "kv_index": o.kv_index,
                "seq_len": sess.seq_len, "h_last": sess.h_last, "root": sess.root, "k": sess.k_pages, "v": sess.v_pages}
    sess.reset()
    sess.prefill(st["prompt"])
    toks, _ = sess.generate(case["new"])
    return {"tokens": torch.tensor(toks), "h_last": sess.h_last, "seq_len": sess.seq_len, "tree": o.tree_tokens, "hidden": o.hidden, "logits": o.logits}


# ---- what a pass cannot do without ------------------------------------------------------------------------------
def work(case):
    kind, d, F, V, B = case["kind"], case["H"] * case["Dh"], case["F"], case["V"], case["B"]
    e = 4 if kind == "generate" else 2
    layer, NL, T = 4 * d * d + 3 * d * F, case.get("NL", 1), case.get("T", 1)

    def forward(rows, keys, lm, logits):
        """rows in all, keys: cached tokens that all requests read in all, lm: rows that need the LM head."""
        by = e * (NL * layer + (d * V if lm else 0)) + NL * 2 * d * e * (keys + rows) + rows * d * (e + 4) + (rows * V * 4 if logits else 0)
        fl = 2.0 * rows * NL * layer + 2.0 * lm * d * V + 4.0 * (rows / B) * (keys + rows) * d * NL
        return by, fl

    if kind == "verify":
        keys = sum(lengths(case, 0))
        by, fl = forward(B * T, keys, B * T, case["logits"])
    elif kind == "prefill":
        by = fl = 0.0
        for i, n in enumerate(_chunks(case)):
            b1, f1 = forward(B * n, B * i * case["chunk"], B, 0)
            by, fl = by + b1, fl + f1
    elif kind == "draft":
        dep = depths(tree(T))
        parent = tree(T)
        by = fl = 0.0
        for i in range(1, max(dep) + 1):
            rows = B * len({parent[n] for n in range(T) if dep[n] == i})
            w = (i + 1) * d * d + (case["mlp"] - 1) * d * d + d * V
            by, fl = by + 2.0 * w, fl + 2.0 * rows * w
    elif kind == "prefix":
        n = sum(int(x) for x in _paths(case, 0)[0])
        by, fl = forward(n, sum(lengths(case, 0)), 0, 0)
    elif kind == "tail":
        by, fl = B * T * V * 4.0 + B * 4 * d * 2 * 2 * NL, 4.0 * B * T * V
    else:
        by, fl = forward(B * case["ctx"], 0, B, 0)
        b1, f1 = forward(B * T, B * case["ctx"], B * T, 0)
        w = sum((i + 1) * d * d + (case["mlp"] - 1) * d * d + d * V for i in range(1, case["K"] + 1))
        by, fl = by + case["new"] * (b1 + 4.0 * w), fl + case["new"] * (f1 + 2.0 * B * 4 * w)
    return {"bytes": float(by), "flops": float(fl)}


def tolerance(case):
    kind = case["kind"]
    if kind == "tail":
        return "exact"                                   # whole numbers, and copies of values
    if kind == "generate":
        return {"rel": 2e-5, "max": 2e-4, "differ": 0.005}     # fp32 sums in another order
    # 16-bit GEMM inputs and cache, fp32 sums: the roundings of one layer travel through the ones behind it.  Measured
    # against 64 bits: 1.3e-3 to 1.9e-3 with up to 8 layers, 3.6e-3 with 32 (2-norm).  "max": single logits of rows with a
    # large scale, whose value can be small against their own roundings.
    return {"rel": 7e-3 if case.get("NL", 1) <= 8 else 1.4e-2, "max": 0.25, "differ": 0.01}


# ---- the same in 64 bits ----------------------------------------------------------------------------------------
def _norm(x, g):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * g


def _rope(x, pos):
    half = x.shape[-1] // 2
    a = pos.double()[:, None, None] * THETA ** (-torch.arange(half, device=DEV).double() / half)
    c, s = torch.cos(a), torch.sin(a)
    return torch.cat([x[..., :half] * c - x[..., half:] * s, x[..., half:] * c + x[..., :half] * s], -1)


def _layer64(w, x, pos, caches, masks, H, Dh):
    """One decoder layer over rows x [R, d] of several requests; caches: (K, V) [keys, H, Dh] of each request's prefix, masks:
    [rows of the request, its own rows] of each.  Returns the rows and each request's own (K, V)."""
    R, d = x.shape
    h = _norm(x, w("attn_norm"))
    q, k, v = (torch.mm(h, w(n).t()).view(R, H, Dh) for n in ("wq", "wk", "wv"))
    q, k = _rope(q, pos), _rope(k, pos)
    out, own, at = [], [], 0
    for (K0, V0), m in zip(caches, masks):
        n = m.shape[0]
        kk, vv = torch.cat([K0, k[at:at + n]]), torch.cat([V0, v[at:at + n]])
        s = torch.bmm(q[at:at + n].transpose(0, 1).contiguous(), kk.permute(1, 2, 0).contiguous()) / math.sqrt(Dh)
        s[:, :, K0.shape[0]:].masked_fill_(~m, -math.inf)
        out.append(torch.bmm(torch.softmax(s, -1), vv.transpose(0, 1).contiguous()).transpose(0, 1).reshape(n, d))
        own.append((k[at:at + n], v[at:at + n]))
        at += n
    x = x + torch.mm(torch.cat(out), w("wo").t())
    h = _norm(x, w("ffn_norm"))
    g = torch.mm(h, w("w_gate").t())
    return x + torch.mm(g * torch.sigmoid(g) * torch.mm(h, w("w_up").t()), w("w_down").t()), own


def _no_cache(case):
    z = torch.zeros(0, case["H"], case["Dh"], dtype=torch.float64, device=DEV)
    return z, z


def _heads64(w, case, i, h, path_emb):
    """Logits of head i for the nodes whose path embeddings [n, i, d] are given."""
    n = path_emb.shape[0]
    u = torch.cat([h.expand(n, -1), path_emb.reshape(n, -1)], 1)
    z = torch.mm(u, w("heads.%d.w1" % i).t()) + w("heads.%d.b1" % i)
    z = z * torch.sigmoid(z)
    for j in range(2, case["mlp"] + 1):
        y = torch.mm(z, w("heads.%d.w%d" % (i, j)).t()) + w("heads.%d.b%d" % (i, j))
        z = z + y * torch.sigmoid(y)
    return torch.mm(z, w("heads.%d.wout" % i).t())


def _draft64(w, case, parent, h, root):
    T, dep = len(parent), depths(parent)
    toks = [int(root)] + [0] * (T - 1)
    emb = w("embed")
    for i in range(1, max(dep) + 1):
        nodes = sorted({parent[n] for n in range(T) if dep[n] == i})
        paths = []
        for n in nodes:
            p = []
            while n >= 0:
                p.append(toks[n])
                n = parent[n]
            paths.append(p[::-1])
        lg = _heads64(w, case, i, h[None], emb[torch.tensor(paths, device=DEV)])
        for n, row in zip(nodes, lg):
            kids = [c for c in range(T) if parent[c] == n]
            for c, t in zip(kids, row.topk(len(kids)).indices.tolist()):
                toks[c] = t
    return toks


def _top2(lg):
    t = lg.topk(2, dim=-1)
    return t.indices[..., 0].to(torch.int32), t.values[..., 0] - t.values[..., 1]


def exact(case, seed):
    kind, B, H, Dh, V = case["kind"], case["B"], case["H"], case["Dh"], case["V"]
    kept = {}

    def w(name):
        if name in kept:
            return kept[name]
        t = weight(case, seed, name).double()
        if kind == "generate" or (kind == "draft" and name == "embed"):
            kept[name] = t
        return t

    def layer(l):
        return lambda n: w("layers.%d.%s" % (l, n))

    if kind == "tail":
        return None                                      # copies and whole numbers
    if kind == "draft":
        parent = tree(case["T"])
        h, root = _rand(seed, "h", (B, H * Dh)).double(), _tokens(seed, "root", (B,), V)
        return {"tokens": torch.tensor([_draft64(w, case, parent, h[b], root[b]) for b in range(B)], dtype=torch.int32)}
    if kind == "verify":
        T, lens, parent = case["T"], lengths(case, seed), tree(case["T"])
        toks = _tokens(seed, "tokens", (B, T), V).long()
        pos = torch.cat([torch.tensor(depths(parent), device=DEV) + n for n in lens])
        masks = [ancestors(parent).to(DEV)] * B
        x = w("embed")[toks.reshape(-1)]
        for l in range(case["NL"]):
            kv = _kv_plain(case, seed, l, case["ctx"])
            x, _ = _layer64(layer(l), x, pos, [(kv[b, :lens[b], 0].double(), kv[b, :lens[b], 1].double()) for b in range(B)], masks, H, Dh)
        h = _norm(x, w("final_norm"))
        lg = torch.mm(h, w("lm_head").t())
        am, mg = _top2(lg)
        out = {"hidden": h.view(B, T, -1), "argmax": am.view(B, T), "k": None, "v": None}
        if case["logits"]:
            out["logits"] = lg.view(B, T, V)
        elif _many(case):
            out["margin"] = mg.view(B, T)
        return out
    if kind == "prefix":
        n_acc, path = _paths(case, seed)
        lens = lengths(case, seed)
        hid = _rand(seed, "h", (B, case["T"], H * Dh)).double()
        kv = _kv_plain(case, seed, 0, case["ctx"])
        x = torch.cat([hid[b, path[b, :n_acc[b]].long().to(DEV)] for b in range(B)])
        pos = torch.cat([torch.arange(int(n_acc[b]), device=DEV) + lens[b] for b in range(B)])
        masks = [torch.ones(int(n), int(n), dtype=torch.bool, device=DEV).tril() for n in n_acc]
        x, _ = _layer64(lambda n: w("prefix." + n), x, pos, [(kv[b, :lens[b], 0].double(), kv[b, :lens[b], 1].double()) for b in range(B)], masks, H, Dh)
        last = torch.cumsum(n_acc, 0).long() - 1
        return {"h_last": x[last.to(DEV)], "seq_len": (torch.tensor(lens) + n_acc).to(torch.int32), "k": None, "v": None}

    # a prompt from the empty cache; with generate the decoding steps behind it
    toks = _tokens(seed, "prompt", (B, case["ctx"]), V).long()
    n = case["ctx"]
    x = w("embed")[toks.reshape(-1)]
    caches = []
    for l in range(case["NL"]):
        x, own = _layer64(layer(l), x, torch.arange(n, device=DEV).repeat(B), [_no_cache(case)] * B,
                          [torch.ones(n, n, dtype=torch.bool, device=DEV).tril()] * B, H, Dh)
        caches.append(own)
    hid = _norm(x, w("final_norm")).view(B, n, -1)
    h = hid[:, -1]
    root = torch.mm(h, w("lm_head").t()).argmax(-1)
    if kind == "prefill":
        return {"h_last": h, "root": root.to(torch.int32), "seq_len": torch.full((B,), n, dtype=torch.int32),
                "hidden": hid[:, n - _chunks(case)[-1]:], "k": None, "v": None}
    parent = tree(case["T"])
    T, dep, mask = case["T"], torch.tensor(depths(parent), device=DEV), ancestors(parent).to(DEV)
    said, lens, h, root = [[] for _ in range(B)], [n] * B, [h[b] for b in range(B)], [int(r) for r in root]
    last = [None] * B
    while min(len(s) for s in said) < case["new"]:
        for b in range(B):
            tt = _draft64(w, case, parent, h[b], root[b])
            x = w("embed")[torch.tensor(tt, device=DEV)]
            own = []
            for l in range(case["NL"]):
                x, kv = _layer64(layer(l), x, dep + lens[b], [caches[l][b]], [mask], H, Dh)
                own.append(kv[0])
            hh = _norm(x, w("final_norm"))
            lg = torch.mm(hh, w("lm_head").t())
            am, cur, path = lg.argmax(-1).tolist(), 0, [0]
            while True:
                nxt = [c for c in range(T) if parent[c] == cur and tt[c] == am[cur]]
                if not nxt:
                    break
                cur = nxt[0]
                path.append(cur)
            for l in range(case["NL"]):
                K0, V0 = caches[l][b]
                caches[l][b] = (torch.cat([K0, own[l][0][path]]), torch.cat([V0, own[l][1][path]]))
            said[b] += [tt[p] for p in path]
            lens[b], h[b], root[b], last[b] = lens[b] + len(path), hh[cur], am[cur], (tt, hh, lg)
    return {"tokens": torch.tensor([s[:case["new"]] for s in said]), "h_last": torch.stack(h), "seq_len": torch.tensor(lens, dtype=torch.int32),
            "tree": torch.tensor([t[0] for t in last], dtype=torch.int32), "hidden": torch.stack([t[1] for t in last]),
            "logits": torch.stack([t[2] for t in last])}
