"""Top-k of the draft heads on chosen logits: the head's output is silu(1) in dimension 0 and nothing else, so a logit is silu(1) times
the first column of the vocabulary projection, and the children follow the order of that column exactly.  One kernel up to 4096 ids, chunks
of 1024 and a merge with 8, 4 and 2 lanes to a chunk beyond, a scan past 32768; the largest logits anywhere, in one wave's ids, or one to a wave."""
import pytest
import torch

from helpers import make_weights, small_shape
from gpu_util import gpu_session

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,k", [(33, 32), (300, 3), (700, 32), (1500, 32), (4096, 17), (4097, 32), (5000, 24), (8192, 32), (8193, 7), (16385, 32),
                                 (20000, 12), (32768, 32), (32769, 5)])
def test_children_follow_the_logits(V, k):
    cfg = small_shape(d=64, NL=1, H=1, Dh=64, F=16, V=V, K=1, T=k + 1)
    W = make_weights(cfg)
    W["heads.1.w1"], W["heads.1.b1"] = torch.zeros_like(W["heads.1.w1"]), torch.zeros_like(W["heads.1.b1"])
    W["heads.1.b1"][0] = 1.0
    for i, name in enumerate(("anywhere", "one wave", "one to a wave")):
        best = torch.randperm(V, generator=torch.Generator().manual_seed(V + i))            # ids, largest logit first
        if name != "anywhere":
            first = torch.arange(V) if name == "one wave" else torch.cat([torch.arange(j, V, 256) for j in range(min(256, V))])
            first = first[(V // 2 if name == "one wave" else 0):][:k]
            best = torch.cat([first, best[~torch.isin(best, first)]])
        column = torch.empty(V)
        column[best] = 3.0 - 5.0 * torch.arange(V) / V                                      # distinct, of both signs
        W["heads.1.wout"] = torch.zeros_like(W["heads.1.wout"])
        W["heads.1.wout"][:, 0] = column
        sess = gpu_session(cfg, [-1] + [0] * k, 2, 16, W)
        sess.h_last.normal_()
        print("case", V, k, name, flush=True)
        sess.draft()
        torch.cuda.synchronize()
        assert sess.main.read_flags() == 0
        for b in range(2):
            assert sess.out().tree_tokens[b, 1:].cpu().tolist() == best[:k].tolist(), name
