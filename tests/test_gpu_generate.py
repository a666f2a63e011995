"""Session.generate enqueues a step of an fp32 model before the one in front of it is read back, where it is needed either way:
the same tokens, states and number of steps as reading every step back, also where the cache has no room for the upper bound."""
import numpy as np
import pytest
import torch

from synth import uniform_tokens
from helpers import make_weights, small_shape
from gpu_util import gpu_session

pytestmark = pytest.mark.gpu


def _one_by_one(sess, n_new, max_steps):
    out, accs = [[] for _ in range(sess.B)], []
    while min(map(len, out)) < n_new and (max_steps is None or len(accs) < max_steps):
        sess.step()
        o = sess.out()
        na = o.n_acc.tolist()
        for b in range(sess.B):
            out[b] += [int(o.tree_tokens[b, n]) for n in o.path[b, :na[b]].tolist()]
        accs.append(na)
        sess.sync_len()
    return [t[:n_new] for t in out], accs


@pytest.mark.parametrize("n_new,max_steps,room", [(1, None, 64), (9, None, 64), (24, None, 0), (24, 3, 64), (0, None, 64)])
def test_generate_reads_back_late(n_new, max_steps, room):
    # heads that repeat the embedding of the last token and a base model that is all but the identity: drafts are often accepted
    cfg = small_shape(d=128, NL=1, H=2, Dh=64, F=64, V=64, K=3, T=7)
    W = make_weights(cfg, std=0.02)
    W["embed"] = torch.eye(64, 128)
    W["lm_head"] = torch.eye(64, 128)
    for i in (1, 2, 3):
        w1 = torch.zeros_like(W[f"heads.{i}.w1"])
        w1[:, i * 128:(i + 1) * 128] = torch.eye(128) * 4
        W[f"heads.{i}.w1"], W[f"heads.{i}.wout"] = w1, torch.eye(64, 128)
    parent = [-1, 0, 0, 1, 1, 3, 4]
    prompt = torch.stack([uniform_tokens(3, b, 21, 64) for b in range(2)]).to(torch.int32)
    # room: cached tokens beyond what the text and the last step's tree need
    need = 21 + n_new + 3 + room - 16 + 1
    runs = []
    for late in (True, False):
        sess = gpu_session(cfg, parent, 2, need, W, prefill_chunk=7)
        sess.prefill(prompt)
        toks, accs = sess.generate(n_new, max_steps=max_steps) if late else _one_by_one(sess, n_new, max_steps)
        torch.cuda.synchronize()
        assert sess.main.read_flags() == 0
        runs.append((toks, accs, sess.seq_len.tolist(), sess.root.tolist(), sess.host_len))
        h = sess.h_last.cpu().numpy()
        runs[-1] += (h.tobytes(),)
    assert runs[0] == runs[1]
    if n_new == 24 and max_steps is None:
        assert np.max(runs[0][1]) > 1, "no step accepted a draft: the lengths never differed from their lower bound"
