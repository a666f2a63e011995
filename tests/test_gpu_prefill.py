"""Reading a prompt: chunks that end behind the decoder layers leave the same cache, state and (for every chunk length) the
outputs of that length's last chunk as chunks that are computed whole."""
import pytest
import torch

from synth import uniform_tokens
from helpers import make_weights, small_shape
from gpu_util import gpu_session
from paper_2402_05109_amd import binding as hb

pytestmark = pytest.mark.gpu


def _whole(sess, prompts):
    """Every chunk through tree_verify_forward."""
    B, L = prompts.shape
    prompts = prompts.to("cuda:0", torch.int32)
    for pos in range(0, L, sess.prefill_chunk):
        n = min(sess.prefill_chunk, L - pos)
        c = sess.ctx(f"chain{n}")
        o = sess.out(f"chain{n}")
        o.tree_tokens.copy_(prompts[:, pos:pos + n])
        sess.kv.seq_len_hint = sess.host_len
        c.tree_verify_forward(B, sess.ws, o.tree_tokens, sess.seq_len, sess.kv, o.hidden, o.argmax, o.margin, o.logits)
        o.n_acc.fill_(n)
        o.path.copy_(torch.arange(n, dtype=torch.int32).expand(B, n))
        o.last_node.fill_(n - 1)
        o.next_root.copy_(o.argmax[:, n - 1])
        c.kv_compact(B, o.n_acc, o.path, o.next_root, o.last_node, o.hidden, sess.kv, sess.seq_len, sess.h_last, sess.root, o.kv_index)
        sess.host_len += n


FIELDS = ("tree_tokens", "hidden", "argmax", "margin", "logits", "n_acc", "path", "next_root", "last_node", "kv_index")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("NL,L,chunk,B", [(1, 40, 16, 2), (3, 96, 32, 1), (2, 7, 16, 2), (2, 17, 16, 1), (2, 300, 72, 2)])
def test_prefill_equals_whole_chunks(dtype, NL, L, chunk, B):
    cfg = small_shape(d=256, NL=NL, H=2, Dh=128, F=384, V=1000, K=0, T=3, dtype=dtype)
    W = make_weights(cfg)
    prompts = torch.stack([uniform_tokens(9, b, L, cfg.V) for b in range(B)])
    got = []
    for fn in (lambda s: s.prefill(prompts), lambda s: _whole(s, prompts)):
        sess = gpu_session(cfg, [-1, 0, 1], B, L + 8, W, prefill_chunk=chunk, page_perm_seed=4, want_logits=True)
        fn(sess)
        fn(sess) if L == 17 else None                # a second text behind the first
        torch.cuda.synchronize()
        assert sess.main.read_flags() == 0
        outs = [sess.k_pages, sess.v_pages, sess.seq_len, sess.h_last, sess.root]
        for n in sorted({min(chunk, L - p) for p in range(0, L, chunk)}):
            outs += [getattr(sess.out(f"chain{n}"), f) for f in FIELDS]
        got.append([t.clone() for t in outs] + [torch.tensor(sess.host_len)])
    assert all(torch.equal(a, b) for a, b in zip(*got))


def test_a_prompt_that_does_not_fit_leaves_the_chunks_in_front_of_it_whole():
    cfg = small_shape(d=256, NL=2, H=2, Dh=128, F=384, V=1000, K=0, T=3, dtype="bf16")
    W = make_weights(cfg)
    prompts = uniform_tokens(9, 0, 100, cfg.V).reshape(1, -1)
    got = []
    for fn in (lambda s: s.prefill(prompts), lambda s: _whole(s, prompts)):
        sess = gpu_session(cfg, [-1, 0, 1], 1, 40, W, prefill_chunk=16)
        with pytest.raises(hb.HydraError) as e:
            fn(sess)
        assert e.value.code == hb.E_CAPACITY
        torch.cuda.synchronize()
        o = sess.out("chain16")
        got.append([t.clone() for t in (sess.k_pages, sess.v_pages, sess.seq_len, sess.h_last, sess.root, o.hidden, o.argmax)])
    assert all(torch.equal(a, b) for a, b in zip(*got))


@pytest.mark.parametrize("NL,L,chunk,B", [(2, 75, 16, 2), (3, 200, 64, 1)])
def test_prefill_equals_whole_chunks_with_the_layer_kernel(NL, L, chunk, B, monkeypatch):
    """HYDRA_LAYER_KERNEL=1: chunks that end early take the persistent kernel where whole ones do (up to 64 rows behind cached tokens)."""
    monkeypatch.setenv("HYDRA_LAYER_KERNEL", "1")
    cfg = small_shape(d=256, NL=NL, H=2, Dh=128, F=384, V=1000, K=0, T=3, dtype="bf16")
    W = make_weights(cfg, std=0.05)
    prompts = torch.stack([uniform_tokens(9, b, L, cfg.V) for b in range(B)])
    got = []
    for fn in (lambda s: s.prefill(prompts), lambda s: _whole(s, prompts)):
        sess = gpu_session(cfg, [-1, 0, 1], B, L + 8, W, prefill_chunk=chunk, page_perm_seed=4)
        assert sess.ctx(f"chain{chunk}").layer_kernel_info(B)[0] == 1
        fn(sess)
        torch.cuda.synchronize()
        assert sess.main.read_flags() == 0
        got.append([t.clone() for t in (sess.k_pages, sess.v_pages, sess.seq_len, sess.h_last, sess.root)])
    assert all(torch.equal(a, b) for a, b in zip(*got))


def test_a_prompt_that_is_broken_off_leaves_a_state_that_belongs_together():
    """An exception in front of the third chunk, behind two that end early: seq_len, h_last and root are those behind the text before, and
    reading the prompt again gives what it gives without the interruption."""
    cfg = small_shape(d=256, NL=2, H=2, Dh=128, F=384, V=1000, K=0, T=3, dtype="bf16")
    W = make_weights(cfg)
    first, second = (uniform_tokens(9, i, n, cfg.V).reshape(1, -1) for i, n in ((0, 20), (1, 90)))
    sessions = [gpu_session(cfg, [-1, 0, 1], 1, 128, W, prefill_chunk=16) for _ in range(2)]
    for s in sessions:
        s.prefill(first)
    s = sessions[0]
    state = [t.clone() for t in (s.seq_len, s.h_last, s.root)]
    c, done = s.ctx("chain16"), []
    early = c.hydra_prefill_chunk

    def broken(*a):
        if len(done) == 2:
            raise KeyboardInterrupt
        done.append(early(*a))

    c.hydra_prefill_chunk = broken
    with pytest.raises(KeyboardInterrupt):
        s.prefill(second)
    del c.hydra_prefill_chunk
    torch.cuda.synchronize()
    assert len(done) == 2 and s.host_len == 20
    assert all(torch.equal(a, b) for a, b in zip(state, (s.seq_len, s.h_last, s.root)))
    for s in sessions:
        s.prefill(second)
    torch.cuda.synchronize()
    a, b = sessions
    assert all(torch.equal(x, y) for x, y in zip((a.k_pages, a.v_pages, a.seq_len, a.h_last, a.root), (b.k_pages, b.v_pages, b.seq_len, b.h_last, b.root)))
    assert a.main.read_flags() == 0 and a.host_len == b.host_len == 110
