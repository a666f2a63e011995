"""fp32 family: draft and verification where the products carry norm, rotary embedding, activation and bias with them.  Sizes at
the edges of the 16 x 16 tiles, of the 256-long sweep over K, of an FFN width that no vector load fits, and of the one-kernel
top-k (256 ids to a wave, 16 waves)."""
import numpy as np
import pytest
import torch

from oracle import hydra_oracle as O
from synth import random_tree, uniform_tokens
from helpers import make_weights, oracle_model, small_shape
from gpu_util import gpu_session, load_oracle_cache, max_rel, to_np

pytestmark = pytest.mark.gpu
TOL = 1e-4                      # the bar of the fp32 family


@pytest.mark.parametrize("H,Dh,F,V,T,B,lens,mlp,medusa", [
    (1, 64, 16, 255, 5, 1, (0,), 1, 0),
    (1, 128, 15, 256, 17, 1, (16,), 2, 0),
    (2, 64, 270, 257, 16, 2, (31, 5), 3, 0),
    (5, 64, 17, 1025, 33, 1, (70,), 1, 1),
    (3, 128, 1003, 4096, 7, 3, (1, 40, 15), 2, 0),
    (4, 64, 688, 4097, 16, 1, (100,), 1, 0),
    (2, 64, 64, 1000, 34, 1, (9,), 1, 0),       # up to 32 children
])
def test_draft_and_verify(H, Dh, F, V, T, B, lens, mlp, medusa):
    parent = [-1] + [0] * 32 + [1] if T == 34 else random_tree(T, 3, 11)
    tree = O.Tree(parent)
    cfg = small_shape(d=H * Dh, NL=2, H=H, Dh=Dh, F=F, V=V, K=3, mlp_layers=mlp, T=T, medusa=medusa)
    W = make_weights(cfg, std=0.05)
    m = oracle_model(cfg, W)
    Lmax = max(lens)
    sess = gpu_session(cfg, parent, B, Lmax + 16, W, page_perm_seed=2, want_logits=True)
    rng = np.random.default_rng(V)
    f32 = lambda a: a.astype(np.float32).astype(np.float64)
    caches = []
    for b in range(B):
        c = O.FlatCache(m, Lmax + T)
        c.K[:, :lens[b]], c.V[:, :lens[b]] = f32(rng.standard_normal(c.K[:, :lens[b]].shape)), f32(rng.standard_normal(c.V[:, :lens[b]].shape))
        caches.append(c)
    load_oracle_cache(sess, caches, Lmax)
    sess.seq_len.copy_(torch.tensor(lens, dtype=torch.int32)); sess.host_len = Lmax
    h = f32(rng.standard_normal((B, cfg.d)))
    roots = [int(t) for t in uniform_tokens(1, 7, B, V)]
    sess.h_last.copy_(torch.tensor(h)); sess.root.copy_(torch.tensor(roots, dtype=torch.int32))
    print("case", H, Dh, F, V, T, B, flush=True)
    sess.draft()
    torch.cuda.synchronize()
    o = sess.out()
    for b in range(B):
        got = o.tree_tokens[b].cpu().tolist()
        assert got[0] == roots[b]
        _, lg = O.draft_tree(m, tree, h[b], roots[b], forced_tokens=got)
        for n, logits in lg.items():
            kids, ref = [got[c] for c in tree.children[n]], O.top_k_ids(logits, len(tree.children[n]))
            if kids != ref:                                  # only where the oracle's values are as close as the bar
                tol = TOL * np.max(np.abs(logits))
                assert len(set(kids)) == len(kids) and np.all(np.abs(logits[kids] - logits[ref]) <= tol), (b, n)
    toks = np.stack([uniform_tokens(5, 50 + b, T, V).numpy() for b in range(B)])
    o.tree_tokens.copy_(torch.tensor(toks, dtype=torch.int32))
    sess.verify()
    torch.cuda.synchronize()
    assert sess.main.read_flags() == 0
    kv = torch.zeros(B, T, 2, H, Dh, device="cuda:0")
    for b in range(B):
        hid, logits, _ = O.tree_verify(m, caches[b], lens[b], tree, toks[b].tolist())
        assert max_rel(to_np(o.hidden[b]), hid) <= TOL and max_rel(to_np(o.logits[b]), logits) <= TOL
        assert o.argmax[b].cpu().tolist() == o.logits[b].argmax(-1).cpu().tolist()
        for l in range(cfg.NL):
            sess.main.kv_read(B, l, sess.kv, lens[b], T, kv)
            got = to_np(kv[b])
            assert max_rel(got[:, 0].reshape(T, -1), caches[b].K[l, lens[b]:lens[b] + T].reshape(T, -1)) <= TOL
            assert max_rel(got[:, 1].reshape(T, -1), caches[b].V[l, lens[b]:lens[b] + T].reshape(T, -1)) <= TOL


@pytest.mark.parametrize("V,most", [(2, 20), (64, 20), (300, 32), (1024, 1), (3000, 32), (4097, 32), (5000, 12), (5000, 2), (32768, 32)])
def test_topk_of_equal_logits_takes_the_lowest_ids(V, most):
    """All weights of the vocabulary projection are zero: every logit is equal and the children are ids 0, 1, 2, ..."""
    k = min(V, most)
    cfg = small_shape(d=64, NL=1, H=1, Dh=64, F=16, V=V, K=1, T=k + 1)
    W = make_weights(cfg)
    W["heads.1.wout"] = torch.zeros_like(W["heads.1.wout"])
    sess = gpu_session(cfg, [-1] + [0] * k, 1, 16, W)
    sess.h_last.normal_()
    sess.draft()
    torch.cuda.synchronize()
    assert sess.out().tree_tokens[0, 1:].cpu().tolist() == list(range(k))
