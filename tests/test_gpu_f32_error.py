"""fp32 family: products that hold two features per lane (q|k|v with the rotary embedding, gate with up) lose no more to rounding
than the ones that hold one.

The LM head has the weights of wv here and reads the same rows with the same gain, since wo and w_down are zero: cached V (two
features per lane) and logits (one) are the same products.  The expected error, as the mean square of the roundings on a product's way
(a sum of n terms is rounded by n^(1/2) of a term's size) at K = 2048: 1072 for 16 chains of K / 256 products and a tree over them, which
is what one feature per lane has, and for a chain over K / 256 sums of eight pairs; 1600 for eight chains over all of K, an error
1.2 times as large (1.09 at 512).  Both figures are root mean squares over 128 rows x K values, whose own spread is below 0.01."""
import pytest
import torch

from helpers import make_weights, small_shape
from gpu_util import gpu_session

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,Dh", [(4, 128), (8, 128), (16, 128)])
def test_products_of_two_features_per_lane(H, Dh):
    d, T = H * Dh, 128
    cfg = small_shape(d=d, NL=1, H=H, Dh=Dh, F=16, V=d, K=0, T=T)
    W = make_weights(cfg, std=1.0)
    W["layers.0.wo"], W["layers.0.w_down"] = torch.zeros_like(W["layers.0.wo"]), torch.zeros_like(W["layers.0.w_down"])
    W["lm_head"], W["final_norm"] = W["layers.0.wv"], W["layers.0.attn_norm"]
    sess = gpu_session(cfg, [-1] + list(range(T - 1)), 1, 16, W, want_logits=True)
    o = sess.out()
    toks = torch.randint(0, d, (1, T), generator=torch.Generator().manual_seed(4))
    o.tree_tokens.copy_(toks)
    sess.verify()
    kv = torch.zeros(1, T, 2, H, Dh, device="cuda:0")
    sess.main.kv_read(1, 0, sess.kv, 0, T, kv)
    torch.cuda.synchronize()
    assert sess.main.read_flags() == 0
    x = W["embed"][toks[0]].double()
    ref = (x / torch.sqrt((x * x).mean(-1, keepdim=True) + cfg.rms_eps) * W["final_norm"].double()) @ W["lm_head"].double().T

    def error(got):
        return float((got.cpu().double().reshape(T, d) - ref).norm() / ref.norm())

    two, one = error(kv[0, :, 1]), error(o.logits[0])
    print(f"d = {d}: two features per lane {two:.3e}, one {one:.3e}", flush=True)
    assert two <= 1.06 * one
