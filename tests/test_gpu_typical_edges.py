"""Typical acceptance at the edges of what its arguments may be, against the oracle: infinite temperature,
uniform numbers outside [0, 1), rows that start and end anywhere."""
import numpy as np
import pytest
import torch

from oracle import hydra_oracle as O
from synth import random_tree
from helpers import make_weights, small_shape
from gpu_util import gpu_session

pytestmark = pytest.mark.gpu


def _session(parent, B, V):
    cfg = small_shape(d=128, NL=1, H=2, Dh=64, F=176, V=V, K=0, T=len(parent))
    return gpu_session(cfg, parent, B, 32, make_weights(cfg), want_logits=True)


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("V", [2, 7, 1000, 1003, 32000, 32768, 40001])
def test_infinite_temperature_is_the_uniform_distribution(V, static):
    """Every token has probability 1 / V and the entropy is log V: with alpha < 1 every candidate passes, with alpha > 1 (and
    eps out of the way) none does, and the next root is floor(u V).  u = (k + 1/2) / V keeps away from the steps; sums of V
    ones are exact in fp32."""
    parent = random_tree(20, 3, 5)
    tree, B = O.Tree(parent), 3
    sess = _session(parent, B, V)
    rng = np.random.default_rng(V)
    logits = rng.standard_normal((B, tree.T, V)).astype(np.float32)
    tok = rng.integers(0, V, size=(B, tree.T))
    k = np.array([0, V // 2, V - 1])
    u = ((k + 0.5) / V).astype(np.float32)
    o = sess.out()
    o.tree_tokens.copy_(torch.tensor(tok, dtype=torch.int32)); o.logits.copy_(torch.tensor(logits))
    ud = torch.tensor(u, device="cuda:0")
    for alpha in (0.5, 1.5):
        out = (o.n_acc, o.path, o.next_root, o.last_node)
        if static:
            sess.main.accept_typical_static(B, o.tree_tokens, o.logits, float("inf"), 2.0, alpha, ud, *out)
        else:
            sess.main.accept_typical(B, sess.ws, o.tree_tokens, o.logits, float("inf"), 2.0, alpha, ud, *out)
        torch.cuda.synchronize()
        for b in range(B):
            n_acc, path, nxt, last = O.accept_typical(tree, tok[b], logits[b].astype(np.float64), float("inf"), 2.0, alpha, float(u[b]))
            assert nxt == k[b] and (n_acc > 1) == (alpha < 1)
            assert int(o.n_acc[b]) == n_acc and int(o.last_node[b]) == last and int(o.next_root[b]) == nxt
            assert o.path[b, :n_acc].tolist() == path


@pytest.mark.parametrize("V", [7, 5000, 32003, 40000])
def test_numbers_outside_the_unit_interval_give_the_last_token(V):
    """u outside [0, 1) is the caller's mistake and has no answer of its own: the call ends at the last token, whichever
    side u lies on."""
    us = [-0.5, -1e-30, 1.0, 7.0, float("inf"), float("-inf"), float("nan")]
    sess = _session([-1], len(us), V)
    o = sess.out()
    o.logits.normal_()
    o.tree_tokens.zero_()
    sess.main.accept_typical(len(us), sess.ws, o.tree_tokens, o.logits, 0.7, 0.1, 0.3, torch.tensor(us, device="cuda:0"), o.n_acc, o.path,
                             o.next_root, o.last_node)
    torch.cuda.synchronize()
    assert o.next_root.tolist() == [V - 1] * len(us)


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("V", [3, 5, 4094, 4097, 4099, 32767, 32769, 36866, 65539])
def test_rows_that_start_and_end_anywhere(V, shift):
    """The last group of four entries cut by V in every way, at the end of a stripe (4096) and of a piece (32768), rows and the
    logits pointer off 16-byte alignment, and a temperature at which most entries have no mass at all: whatever u, the token
    drawn has mass and lies where the 64-bit distribution puts u, to within the rounding of fp32 sums (1e-5)."""
    B, T, tau = 8, 2, 0.02
    sess = _session([-1, 0], B, V)
    rng = np.random.default_rng(V)
    logits = (rng.standard_normal((B, T, V)) * 0.5).astype(np.float32)
    logits[:, :, -1] = logits.max(axis=-1) - 0.02                     # the last entry and the first one carry mass
    logits[:, :, 0] = logits[:, :, 1:].max(axis=-1) - 0.01
    logits[1, :, 1:-1] = -np.inf
    tok = rng.integers(0, V, size=(B, T))
    tok[:, 1] = np.where(np.arange(B) % 2, logits[:, 0].argmax(-1), tok[:, 1])
    flat = torch.empty(B * T * V + 1, device="cuda:0")
    lg = flat[shift:shift + B * T * V].view(B, T, V)
    lg.copy_(torch.tensor(logits))
    u = np.array([0.0, 0.5, 0.99999994, 0.1, 0.3, 0.6, 0.9, 1e-7], dtype=np.float32)
    o = sess.out()
    o.tree_tokens.copy_(torch.tensor(tok, dtype=torch.int32))
    for ud in (torch.tensor(u, device="cuda:0"), None):
        sess.main.accept_typical(B, sess.ws, o.tree_tokens, lg, tau, 0.05, 0.3, ud, o.n_acc, o.path, o.next_root, o.last_node)
        torch.cuda.synchronize()
        for b in range(B):
            n_acc, path, _, last = O.accept_typical(O.Tree([-1, 0]), tok[b], logits[b].astype(np.float64), tau, 0.05, 0.3, None)
            assert int(o.n_acc[b]) == n_acc and int(o.last_node[b]) == last
            got = int(o.next_root[b])
            if ud is None:
                assert got == int(logits[b, last].argmax())
                continue
            p = O.tempered_probs(logits[b, last].astype(np.float64), tau)
            cdf = np.cumsum(p)
            assert p[got] > 0 and (cdf[got] - p[got]) - 1e-5 <= float(u[b]) <= cdf[got] + 1e-5, (b, got)
