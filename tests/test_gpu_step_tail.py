"""Edges of the kernels at the end of a step: compaction of long paths (more than one batch of 64 entries, more than one
group of eight copies, the identity), typical acceptance on rows longer than the workgroup's registers and of lengths that
rule out 16-byte loads."""
import numpy as np
import pytest
import torch

from oracle import hydra_oracle as O
from synth import random_tree
from helpers import make_weights, small_shape
from gpu_util import gpu_session

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("Dh,H", [(64, 6), (128, 1)])
def test_compaction_of_long_paths(dtype, Dh, H):
    """Copies are exact: every slot below the new length holds what its source held, every other slot is untouched."""
    T, B, NL, L0 = 128, 5, 2, [0, 7, 16, 33, 5]
    cfg = small_shape(d=H * Dh, NL=NL, H=H, Dh=Dh, F=256, V=300, K=0, T=T).with_(dtype=dtype)
    sess = gpu_session(cfg, [-1] + list(range(T - 1)), B, 40, make_weights(cfg), page_perm_seed=3)
    rng = np.random.default_rng(Dh + H)
    n = max(L0) + T
    before = []
    for l in range(NL):
        t = torch.tensor(rng.standard_normal((B, n, 2, H, Dh)), dtype=torch.float32, device="cuda:0").half().float().contiguous()
        sess.main.kv_write(B, l, sess.kv, 0, n, t)
        before.append(t)
    paths = [list(range(T)),                                          # the identity: nothing moves
             list(range(0, T, 2)),                                    # 63 moves
             [0, 1, 2] + sorted(rng.choice(np.arange(3, T), 90, replace=False).tolist()),      # two batches of 64 entries
             [T - 1],                                                 # one move from the far end
             list(range(1, T))]                                       # every slot moves down by one: source of one is destination of the next
    o = sess.out()
    o.path.fill_(-1)
    for b, p in enumerate(paths):
        o.path[b, :len(p)] = torch.tensor(p, dtype=torch.int32)
    o.n_acc.copy_(torch.tensor([len(p) for p in paths], dtype=torch.int32))
    o.last_node.copy_(torch.tensor([p[-1] for p in paths], dtype=torch.int32))
    o.hidden.normal_()
    sess.seq_len.copy_(torch.tensor(L0, dtype=torch.int32))
    sess.compact()
    torch.cuda.synchronize()
    assert sess.main.read_flags() == 0
    for l in range(NL):
        after = torch.empty_like(before[l])
        sess.main.kv_read(B, l, sess.kv, 0, n, after)
        for b, p in enumerate(paths):
            want = before[l][b].clone()
            want[L0[b]:L0[b] + len(p)] = before[l][b][[L0[b] + x for x in p]]
            assert torch.equal(after[b], want), (l, b)
    for b, p in enumerate(paths):
        assert int(sess.seq_len[b]) == L0[b] + len(p)
        assert torch.equal(sess.h_last[b], o.hidden[b, p[-1]])
        want = [(int(sess.page_table[b, (L0[b] + j) // 16]), (L0[b] + j) % 16) for j in range(len(p))] + [(-1, -1)] * (T - len(p))
        assert o.kv_index[b].tolist() == [list(x) for x in want]


@pytest.mark.parametrize("V", [2, 4095, 4096, 4100, 32768, 32772, 40001, 70000])
def test_typical_acceptance_at_the_edges_of_a_piece(V):
    """V = 32768 fills the workgroup's registers exactly; 4096 and 4100 end a stripe; 40001 takes 4-byte loads over two pieces.
    Tokens at and around the last entry carry mass, u goes up to the largest float below 1."""
    parent = random_tree(20, 3, 5)
    tree, B = O.Tree(parent), 6
    cfg = small_shape(d=128, NL=1, H=2, Dh=64, F=176, V=V, K=0, T=20)
    sess = gpu_session(cfg, parent, B, 32, make_weights(cfg), want_logits=True)
    rng = np.random.default_rng(V)
    logits = rng.standard_normal((B, tree.T, V)).astype(np.float32)
    tok = rng.integers(0, V, size=(B, tree.T))
    for b in range(B):
        for c in range(1, tree.T):
            logits[b, tree.parent[c], tok[b, c]] += float(rng.choice([0.0, 9.0, 14.0]))
        logits[b, :, V - 1] += 9.0
        logits[b, :, 0] += 7.0
    logits[0, :, V // 2:] = -np.inf                                    # no mass behind the middle
    u = np.array([0.99999994, 0.99999994, 0.0, 0.5, 0.25, 0.9], dtype=np.float32)
    o = sess.out()
    o.tree_tokens.copy_(torch.tensor(tok, dtype=torch.int32)); o.logits.copy_(torch.tensor(logits))
    compared = 0
    for uu in (None, u):
        ud = None if uu is None else torch.tensor(uu, device="cuda:0")
        sess.main.accept_typical(B, sess.ws, o.tree_tokens, o.logits, 0.8, 0.1, 0.3, ud, o.n_acc, o.path, o.next_root, o.last_node)
        torch.cuda.synchronize()
        for b in range(B):
            lg = logits[b].astype(np.float64)
            p = {n: O.tempered_probs(lg[n], 0.8) for n in {tree.parent[c] for c in range(1, tree.T)}}
            def ent(q): return float(-np.sum(q[q > 0] * np.log(q[q > 0])))
            th = {n: min(0.1, 0.3 * np.exp(-ent(q))) for n, q in p.items()}
            if any(abs(p[tree.parent[c]][tok[b, c]] - th[tree.parent[c]]) <= 1e-4 * th[tree.parent[c]] for c in range(1, tree.T)):
                continue                                               # float32 may decide a candidate at its threshold either way
            good = [True] + [False] * (tree.T - 1)
            for c in range(1, tree.T):
                good[c] = good[tree.parent[c]] and p[tree.parent[c]][tok[b, c]] > th[tree.parent[c]]
            last = max((n for n in range(tree.T) if good[n]), key=lambda n: (tree.depth[n], -n))
            assert int(o.last_node[b]) == last and int(o.n_acc[b]) == tree.depth[last] + 1
            assert o.path[b].tolist() == tree.path(last) + [-1] * (tree.max_depth - tree.depth[last])
            got, q = int(o.next_root[b]), O.tempered_probs(lg[last], 0.8)
            compared += 1
            if uu is None:
                assert got == int(np.argmax(lg[last]))
                continue
            cdf = np.cumsum(q)                                          # fp32 sums of V terms: within 1e-5 of the 64-bit distribution
            assert q[got] > 0 and (cdf[got] - q[got]) - 1e-5 <= float(uu[b]) <= cdf[got] + 1e-5, (b, got)
    assert compared >= B


@pytest.mark.parametrize("V,distinct", [(40, 1), (1500, 1), (1500, 7), (5000, 300), (32768, 2)])
def test_draft_ties_take_the_lowest_ids(V, distinct):
    """Rows of the vocabulary projection repeat, so whole groups of logits are equal bit for bit: more entries at the bound
    than a wave has lanes, fewer, and all of them.  Order: value descending, then id ascending."""
    parent = [-1] + [0] * 32 + [1] * 10 + [2] * 3
    cfg = small_shape(d=128, NL=1, H=2, Dh=64, F=176, V=V, K=2, T=len(parent))
    W = make_weights(cfg)
    g = torch.Generator().manual_seed(V + distinct)
    for i in (1, 2):
        W[f"heads.{i}.wout"] = W[f"heads.{i}.wout"][:distinct][torch.randint(0, distinct, (V,), generator=g)].contiguous()
    sess = gpu_session(cfg, parent, 2, 32, W)
    sess.h_last.normal_()
    sess.root.copy_(torch.tensor([3, V - 1], dtype=torch.int32))
    sess.draft()
    torch.cuda.synchronize()
    toks = sess.out().tree_tokens.cpu()
    for b in range(2):
        for n, kids in ((0, range(1, 33)), (1, range(33, 43)), (2, range(43, 46))):
            i, path = (1, [0]) if n == 0 else (2, [0, n])
            u = torch.cat([sess.h_last[b].cpu()] + [W["embed"][int(toks[b, p])] for p in path]).double()
            z = W[f"heads.{i}.w1"].double() @ u + W[f"heads.{i}.b1"].double()
            lg = W[f"heads.{i}.wout"].double() @ (z * torch.sigmoid(z))
            got = [int(toks[b, c]) for c in kids]
            want = lg[torch.tensor(got)]
            best = torch.sort(lg, descending=True).values[:len(got)]
            assert torch.allclose(want, best, rtol=0, atol=2e-5 * float(lg.abs().max()))      # fp32 sums against 64 bits
            for a, c in zip(got, got[1:]):                            # equal rows have equal logits: ids ascend, none is skipped
                assert (W[f"heads.{i}.wout"][a] != W[f"heads.{i}.wout"][c]).any() or a < c
            for t in got:
                same = (W[f"heads.{i}.wout"] == W[f"heads.{i}.wout"][t]).all(1).nonzero().flatten().tolist()
                assert all(x in got for x in same if x < t)
