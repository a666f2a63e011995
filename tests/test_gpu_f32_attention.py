"""fp32 tree attention where its four waves take the 64-key chunks in turn: more than one chunk per wave, chunks that end
with the keys, and chunks without a single finite score."""
import numpy as np
import pytest
import torch

from oracle import hydra_oracle as O
from synth import random_tree
from helpers import make_weights, small_shape
from gpu_util import gpu_session, max_rel, to_np

pytestmark = pytest.mark.gpu


def _attention(Dh, L, parent, edit=lambda keys, vals: None):
    H, B, T = 2, 2, len(parent)
    cfg = small_shape(d=H * Dh, NL=1, H=H, Dh=Dh, F=64, V=64, K=0, T=T)
    sess = gpu_session(cfg, parent, B, L + T, make_weights(cfg), page_perm_seed=5)
    rng = np.random.default_rng(L + Dh)
    q = rng.standard_normal((B, T, H, Dh)) * 2
    keys, vals = rng.standard_normal((B, L + T, H, Dh)) * 2, rng.standard_normal((B, L + T, H, Dh))
    edit(keys, vals)
    sess.main.kv_write(B, 0, sess.kv, 0, L + T, torch.tensor(np.stack([keys, vals], axis=2), dtype=torch.float32, device="cuda:0").contiguous())
    sess.seq_len.fill_(L)
    out = torch.zeros(B, T, H, Dh, dtype=torch.float32, device="cuda:0")
    sess.main.tree_attention(B, 0, sess.ws, torch.tensor(q, dtype=torch.float32, device="cuda:0").contiguous(), sess.seq_len, sess.kv, out)
    torch.cuda.synchronize()
    assert sess.main.read_flags() == 0
    return to_np(out), q, keys, vals


@pytest.mark.parametrize("Dh", [64, 128])
@pytest.mark.parametrize("L", [191, 192, 255, 256, 257, 449, 640])
def test_more_chunks_than_waves(Dh, L):
    """Parity bar of the fp32 family (1e-4 relative) against the oracle."""
    tree = O.Tree(random_tree(20, 3, 4))
    got, q, keys, vals = _attention(Dh, L, tree.parent)
    for b in range(2):
        for h in range(2):
            assert max_rel(got[b, :, h], O.tree_attention(q[b, :, h], keys[b, :, h], vals[b, :, h], L, tree)) <= 1e-4


@pytest.mark.parametrize("chunk", [1, 2, 3, 4])
def test_a_chunk_of_nan_keys_is_not_left_out(chunk):
    """The cached keys of one 64-key chunk of row 1, head 0 are NaN: every query sees them, so its result is not a number.
    Row 0 and head 1 keep theirs."""
    def edit(keys, vals):
        keys[1, 64 * chunk:64 * chunk + 64, 0] = np.nan
    got, *_ = _attention(64, 330, [-1, 0, 0, 1], edit)
    assert np.isnan(got[1, :, 0]).all()
    assert np.isfinite(got[0]).all() and np.isfinite(got[1, :, 1]).all()


def test_masked_nan_keys_are_not_read():
    """K and V of a tree node are NaN: only the node itself and its descendants see them."""
    parent, L = [-1, 0, 0, 1, 2], 70
    def edit(keys, vals):
        keys[:, L + 1], vals[:, L + 1] = np.nan, np.nan
    got, *_ = _attention(64, L, parent, edit)
    assert np.isnan(got[:, [1, 3]]).all() and np.isfinite(got[:, [0, 2, 4]]).all()
