"""fp32 GEMM and attention at the edges of their tiles: ragged sizes, operands without 16-byte rows, every head size
the kernels are built for and ones between, non-finite values behind the causal mask."""
import numpy as np
import pytest
import torch

from oracle import gpt_layer as L
from paper_2104_04473_amd import binding as B
from paper_2104_04473_amd import synth
from gpu_util import assert_close, np64, randn, rel_l2, stream, sync

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [B.GEMM_NN, B.GEMM_NT, B.GEMM_TN])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (33, 65, 30), (31, 32, 33), (64, 96, 1024), (130, 70, 257), (1030, 1090, 100),
                                   (1025, 1024, 36), (40, 24, 0),
                                   # tiles of 16 x 16: one and four requests of a wave's k-chunks and one more, ragged
                                   # everywhere, the most tiles and one more column of them
                                   (17, 15, 257), (33, 50, 1024), (31, 16, 1056), (250, 509, 1300), (256, 512, 288), (256, 513, 288),
                                   # thin outputs and long k ranges of 257 to 512 such tiles
                                   (1, 8190, 300), (65, 1613, 300), (64, 2046, 300), (70, 1600, 4100)])
def test_gemm_fp32(mode, M, N, K):
    a, b, bias = randn((M, K), B.F32, 1), randn((K, N), B.F32, 2), randn((N,), B.F32, 3)
    A = a.t().contiguous() if mode == B.GEMM_TN else a
    Bm = b.t().contiguous() if mode == B.GEMM_NT else b
    if K == 0:
        A = Bm = torch.zeros(16, device="cuda")
    want = a.double() @ b.double() + bias.double()
    c = torch.full((M, N), 9.0, device="cuda")
    for acc in (0, 1):   # overwritten, then added to
        B.check(B.ptdp_gemm(B.F32, mode, A.data_ptr(), Bm.data_ptr(), c.data_ptr(), bias.data_ptr(), M, N, K, 1, acc, None, 0,
                            stream()), "gemm")
        sync()
        # K products of size about 1 in fp32: error below 2^-24 * K, doubled for the second pass
        assert float((c.double() - (1 + acc) * want).abs().max()) <= 2.0 ** -21 * (K + 8)


def forward_backward(qkv, dctx, s, b, heads, dh, mask=None):
    ctx, lse = torch.zeros_like(dctx), torch.zeros((b, heads, s), device="cuda")
    dqkv, delta = torch.zeros_like(qkv), torch.zeros((b, heads, s), device="cuda")
    if mask is None:
        B.check(B.ptdp_attn_fwd(B.F32, qkv.data_ptr(), ctx.data_ptr(), lse.data_ptr(), s, b, heads, dh, stream()), "fwd")
        B.check(B.ptdp_attn_bwd(B.F32, qkv.data_ptr(), ctx.data_ptr(), lse.data_ptr(), dctx.data_ptr(), dqkv.data_ptr(),
                                delta.data_ptr(), s, b, heads, dh, stream()), "bwd")
    else:
        B.check(B.ptdp_attn_masked_fwd(B.F32, qkv.data_ptr(), mask.data_ptr(), ctx.data_ptr(), lse.data_ptr(), s, b, heads, dh,
                                       stream()), "fwd")
        B.check(B.ptdp_attn_masked_bwd(B.F32, qkv.data_ptr(), mask.data_ptr(), ctx.data_ptr(), lse.data_ptr(), dctx.data_ptr(),
                                       dqkv.data_ptr(), delta.data_ptr(), s, b, heads, dh, stream()), "bwd")
    sync()
    return ctx, lse, dqkv


@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("s,b,heads,dh", [(1, 1, 2, 8), (15, 2, 1, 24), (17, 1, 3, 40), (64, 2, 2, 64), (65, 1, 2, 96),
                                          (129, 1, 1, 128), (96, 2, 1, 160), (83, 1, 1, 200), (50, 1, 2, 256),
                                          # more than four tiles: workgroups of eight waves, in one launch and in two
                                          (81, 1, 3, 32), (130, 1, 2, 64), (200, 2, 2, 72), (260, 1, 16, 64), (257, 1, 9, 40)])
def test_attention_fp32(s, b, heads, dh, masked):
    hp = heads * dh
    qkv, dctx = randn((s, b, 3 * hp), B.F32, 1), randn((s, b, hp), B.F32, 2)
    mask = None
    if masked:
        m = (np.random.default_rng(3).random((b, s, s)) < 0.4).astype(np.uint8)
        m[0, s // 2] = 1   # a query without a visible key
        mask = m
    ctx, lse, dqkv = forward_backward(qkv, dctx, s, b, heads, dh, torch.from_numpy(mask).cuda() if masked else None)
    cfg = L.LayerConfig(h=hp, a=heads, t=1, s=s, b=b, causal=not masked)
    wctx, probs, wlse = L.attention_core(np64(qkv), cfg, mask) if masked else L.attention_core(np64(qkv), cfg)
    want = L.attention_core_backward(np64(dctx), np64(qkv), probs, cfg, mask) if masked else \
        L.attention_core_backward(np64(dctx), np64(qkv), probs, cfg)
    assert_close(np64(ctx), wctx, B.F32, "ctx", 0.1)
    assert np.allclose(np64(lse), wlse, rtol=1e-6, atol=1e-4)
    got = np64(dqkv)
    for name, lo in (("dq", 0), ("dk", hp), ("dv", 2 * hp)):
        if np.abs(want[..., lo:lo + hp]).max() > 1e-9:   # (one query: its softmax is constant, dq and dk are zero)
            # a query without a visible key has a log-sum-exp near -10^4, stored in fp32 to 2^-11: its probabilities (1/s
            # each) are off by that much, which only dv sees; the stated tolerance holds
            assert_close(got[..., lo:lo + hp], want[..., lo:lo + hp], B.F32, name, 1.0 if masked and name == "dv" else 0.1)


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("s,heads,dh,many", [(17, 8, 32, 70), (33, 8, 64, 14), (16, 4, 96, 70), (49, 4, 128, 12), (31, 2, 160, 40)])
def test_attention_fp32_backward_in_one_and_in_two_launches(s, heads, dh, many, causal):
    """Few workgroups run dQ and dK/dV in one launch, in which dK/dV computes the queries' delta itself; more run them one after
    the other.  A sample's gradients have the same bits alone and among `many` (280 to 680 and more workgroups)."""
    hp = heads * dh
    qkv, dctx = randn((s, many, 3 * hp), B.F32, 1), randn((s, many, hp), B.F32, 2)
    mask = None if causal else torch.from_numpy((np.random.default_rng(3).random((many, s, s)) < 0.3).astype(np.uint8)).cuda()
    _, _, all_of_them = forward_backward(qkv, dctx, s, many, heads, dh, mask)
    for j in (0, many // 2, many - 1):
        one = mask[j:j + 1].clone() if mask is not None else None
        _, _, alone = forward_backward(qkv[:, j:j + 1].contiguous(), dctx[:, j:j + 1].contiguous(), s, 1, heads, dh, one)
        assert torch.equal(alone, all_of_them[:, j:j + 1]), j


# s > 64: eight partial sums per row, by eight waves in workgroups of few, by four that make two each in those of many; heads beyond 96
# (backward) and 128 (forward) have four sums either way
@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("s,heads,dh,many", [(65, 2, 24, 60), (81, 4, 64, 40), (128, 3, 96, 30), (130, 2, 40, 33), (257, 1, 64, 35), (300, 2, 32, 20),
                                             (97, 2, 128, 24), (70, 1, 160, 60), (67, 1, 200, 60)])
def test_attention_fp32_sample_alone_and_among_many(s, heads, dh, many, causal):
    """A sample's output, lse and gradients have the same bits alone and among `many`."""
    hp = heads * dh
    qkv, dctx = randn((s, many, 3 * hp), B.F32, 1), randn((s, many, hp), B.F32, 2)
    mask = None if causal else torch.from_numpy((np.random.default_rng(3).random((many, s, s)) < 0.3).astype(np.uint8)).cuda()
    ctx, lse, grads = forward_backward(qkv, dctx, s, many, heads, dh, mask)
    for j in (0, many // 2, many - 1):
        one = mask[j:j + 1].clone() if mask is not None else None
        c, l, g = forward_backward(qkv[:, j:j + 1].contiguous(), dctx[:, j:j + 1].contiguous(), s, 1, heads, dh, one)
        assert torch.equal(c, ctx[:, j:j + 1]) and torch.equal(l, lse[j:j + 1]) and torch.equal(g, grads[:, j:j + 1]), j


# weight gradients in tiles of 16, of 32, of both sizes, of 32 with eight waves each, of 32 and 64
@pytest.mark.parametrize("h,a,t,s,b", [(96, 3, 1, 300, 1), (64, 2, 1, 37, 3), (256, 8, 8, 300, 1), (256, 4, 1, 128, 2), (512, 8, 1, 65, 1)])
def test_weight_gradients_fp32_together_and_one_by_one(h, a, t, s, b):
    """A layer's four weight gradients run in shared launches: every bit is that of a call of its own with the same operands."""
    hp, fp, T = h // t, 4 * h // t, s * b
    cfg = B.make_cfg(h=h, a=a, t=t, s=s, b=b, dtype=B.F32, p_hidden=0.1, seed=5)
    P, G = synth.layer_params(h, a, t, B.F32, seed=1, device="cuda"), synth.zero_grads(h, a, t, "cuda")
    ch = B.Chunk(cfg, 1, 0)
    ch.bind(0, P, G)
    x, dy = synth.activations(s, b, h, B.F32, 2, "cuda"), synth.activations(s, b, h, B.F32, 3, "cuda")
    y, dx = torch.empty_like(x), torch.empty_like(x)
    stash = torch.empty(ch.stash_bytes(), dtype=torch.uint8, device="cuda")
    ws = torch.empty(ch.workspace_bytes(), dtype=torch.uint8, device="cuda")
    for g in G.values():
        g.fill_(0.25)   # += : the old value counts
    B.check(ch.forward(0, x.data_ptr(), y.data_ptr(), stash.data_ptr(), ws.data_ptr()), "forward")
    B.check(ch.backward(0, dy.data_ptr(), dx.data_ptr(), stash.data_ptr(), ws.data_ptr()), "backward")
    sync()
    at, wat = B.stash_offsets(cfg), B.workspace_offsets(cfg)
    for name, A, Bm, M, N in (("w_2", stash[at["G"]:], ws[wat["DMO"]:], fp, h), ("w_1", stash[at["U2"]:], ws[wat["DZ"]:], h, fp),
                              ("w_qkv", stash[at["U"]:], ws[wat["DQKV"]:], h, 3 * hp), ("w_o", stash[at["CTX"]:], ws[wat["DO"]:], hp, h)):
        want = torch.full((M, N), 0.25, device="cuda")
        B.check(B.ptdp_gemm(B.F32, B.GEMM_TN, A.data_ptr(), Bm.data_ptr(), want.data_ptr(), None, M, N, T, 1, 1, None, 0, stream()), name)
        sync()
        assert torch.equal(G[name].view(M, N), want), name


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_attention_fp32_future_tokens_stay_hidden(bad):
    """Undefined or infinite values in a later token's K, V, Q or output gradient change no bit of an earlier token's output
    (K, V) and of a later key's gradients (Q, dctx), also inside a tile on the diagonal."""
    s, b, heads, dh, at = 50, 1, 2, 24, 21
    hp = heads * dh
    qkv, dctx = randn((s, b, 3 * hp), B.F32, 1), randn((s, b, hp), B.F32, 2)
    ctx, _, dqkv = forward_backward(qkv, dctx, s, b, heads, dh)
    q2 = qkv.clone()
    q2[at:, :, hp:] = bad
    ctx2, _, dqkv2 = forward_backward(q2, dctx, s, b, heads, dh)
    assert torch.equal(ctx[:at], ctx2[:at])
    assert torch.equal(dqkv[:at, :, :hp], dqkv2[:at, :, :hp])
    assert not bool(torch.isfinite(ctx2[at:]).any())   # the tokens that see such a value do not lose it
    d3 = dctx.clone()
    d3[:at] = bad
    _, _, dqkv3 = forward_backward(qkv, d3, s, b, heads, dh)
    assert torch.equal(dqkv[at:, :, hp:], dqkv3[at:, :, hp:])


@pytest.mark.parametrize("causal", [True, False])
def test_attention_fp32_scores_of_minus_infinity(causal):
    """A score of -inf has probability zero, also where it is the only one (causal: query 16 and key 16) or all of those (16 keys,
    no mask) that a wave sees in its first tile; the key in front of them is finite for every query."""
    s, b, heads, dh = 40, 1, 2, 24
    hp = heads * dh
    qkv = randn((s, b, 3 * hp), B.F32, 1)
    qkv[..., 0:hp:dh] = qkv[..., 0:hp:dh].abs() + 0.1            # first element of every query positive
    qkv[16:17 if causal else 32, :, hp:2 * hp:dh] = -float("inf")    # first element of those keys
    ctx, lse = torch.zeros((s, b, hp), device="cuda"), torch.zeros((b, heads, s), device="cuda")
    if causal:
        B.check(B.ptdp_attn_fwd(B.F32, qkv.data_ptr(), ctx.data_ptr(), lse.data_ptr(), s, b, heads, dh, stream()), "fwd")
    else:
        B.check(B.ptdp_attn_masked_fwd(B.F32, qkv.data_ptr(), None, ctx.data_ptr(), lse.data_ptr(), s, b, heads, dh, stream()), "fwd")
    sync()
    cfg = L.LayerConfig(h=hp, a=heads, t=1, s=s, b=b, causal=causal)
    wctx, _, wlse = L.attention_core(np64(qkv), cfg)
    assert np.isfinite(wctx).all()
    assert_close(np64(ctx), wctx, B.F32, "ctx", 0.1)
    assert np.allclose(np64(lse), wlse, rtol=1e-6, atol=1e-4)


@pytest.mark.parametrize("dh", [64, 160, 256])
def test_attention_fp32_error_does_not_grow_with_head_size(dh):
    """The dot products over dh are summed as a tree: an error of about sqrt(log2(dh)) roundings of 2^-24 each, where a chain of dh
    additions has sqrt(dh / 2).  What follows (softmax, sums over the tokens) adds about as much again: 2.2e-7 for the
    output and 4.2e-7 for the gradients hold a tree at any head size, a chain of 256 gives 3.4e-7 and 5.5e-7."""
    s, b, heads = 128, 1, 2
    hp = heads * dh
    qkv, dctx = randn((s, b, 3 * hp), B.F32, 1), randn((s, b, hp), B.F32, 2)
    ctx, _, dqkv = forward_backward(qkv, dctx, s, b, heads, dh)
    cfg = L.LayerConfig(h=hp, a=heads, t=1, s=s, b=b)
    wctx, probs, _ = L.attention_core(np64(qkv), cfg)
    want, got = L.attention_core_backward(np64(dctx), np64(qkv), probs, cfg), np64(dqkv)
    err = [rel_l2(np64(ctx), wctx)] + [rel_l2(got[..., i * hp:(i + 1) * hp], want[..., i * hp:(i + 1) * hp]) for i in range(3)]
    assert err[0] <= 2.2e-7 and max(err[1:]) <= 4.2e-7, err
