"""General-mask attention (section 4.2's fused softmax with a general mask) through the C ABI against
the oracle: the attention op alone and a whole layer with cfg.causal = 0."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import gpt_layer as L
from paper_2104_04473_amd import binding as B
from gpu_util import LayerRig, assert_close, np64, oracle_cfg, params_np, randn, stream, sync, tdt

pytestmark = pytest.mark.gpu


def make_mask(b, s, seed, frac=0.3, empty_rows=()):
    rng = np.random.default_rng(seed)
    m = (rng.random((b, s, s)) < frac).astype(np.uint8)
    for j in range(b):
        np.fill_diagonal(m[j], 0)
    for (j, q) in empty_rows:
        m[j, q, :] = 1
    return m


CASES = [  # dtype, s, b, heads, dh, masked?, empty rows
    (B.F32, 50, 2, 2, 32, True, [(1, 7)]),
    (B.F32, 33, 1, 1, 64, False, []),
    (B.BF16, 128, 2, 2, 64, True, [(0, 5), (1, 127)]),
    (B.BF16, 333, 1, 2, 160, True, [(0, 300)]),
    (B.BF16, 200, 2, 3, 128, True, []),
    (B.BF16, 130, 1, 2, 96, False, []),
    (B.BF16, 64, 1, 1, 32, True, []),
    (B.BF16, 257, 1, 1, 128, True, [(0, 256)]),
    # 528 and 540 blocks of 64 rows
    (B.BF16, 130, 6, 30, 64, True, [(2, 129)]),
    (B.BF16, 140, 4, 44, 160, True, []),
    (B.BF16, 130, 6, 30, 96, True, [(3, 64)]),
    (B.BF16, 200, 5, 27, 128, True, [(4, 199)]),
    (B.BF16, 257, 3, 36, 128, False, []),
    # heads of 96 and 128 in both forms of the dK/dV kernel, two pairs
    (B.BF16, 257, 1, 2, 96, True, [(0, 256)]),
    (B.BF16, 300, 2, 3, 128, False, []),
]


@pytest.mark.parametrize("dtype,s,b,heads,dh,masked,empty", CASES)
def test_masked_attention_forward_backward(dtype, s, b, heads, dh, masked, empty):
    hp = heads * dh
    qkv = randn((s, b, 3 * hp), dtype, 1)
    mask = make_mask(b, s, 2, empty_rows=empty) if masked else None
    mask_d = torch.from_numpy(mask).cuda() if masked else None
    mp = mask_d.data_ptr() if masked else None
    ctx = torch.zeros((s, b, hp), dtype=tdt(dtype), device="cuda")
    lse = torch.zeros((b, heads, s), device="cuda")
    B.check(B.ptdp_attn_masked_fwd(dtype, qkv.data_ptr(), mp, ctx.data_ptr(), lse.data_ptr(), s, b, heads, dh, stream()),
            "attn_masked_fwd")
    sync()
    cfg = L.LayerConfig(h=hp, a=heads, t=1, s=s, b=b, causal=False)
    wctx, probs, wlse = L.attention_core(np64(qkv), cfg, mask)
    assert_close(np64(ctx), wctx, dtype, "ctx")
    assert np.allclose(np64(lse), wlse, rtol=0, atol=3e-2 if dtype == B.BF16 else 1e-3)
    for (j, q) in empty:        # a query that sees no key averages V
        assert_close(np64(ctx)[q, j], np64(qkv)[:, j, 2 * hp:].mean(axis=0), dtype, "empty row")
    dctx = randn((s, b, hp), dtype, 7)
    dqkv = torch.zeros_like(qkv)
    delta = torch.zeros((b, heads, s), device="cuda")
    B.check(B.ptdp_attn_masked_bwd(dtype, qkv.data_ptr(), mp, ctx.data_ptr(), lse.data_ptr(), dctx.data_ptr(),
                                   dqkv.data_ptr(), delta.data_ptr(), s, b, heads, dh, stream()), "attn_masked_bwd")
    sync()
    want = L.attention_core_backward(np64(dctx), np64(qkv), probs, cfg, mask)
    got = np64(dqkv)
    for name, lo in (("dq", 0), ("dk", hp), ("dv", 2 * hp)):
        assert_close(got[..., lo:lo + hp], want[..., lo:lo + hp], dtype, name)
    for (j, q) in empty:
        assert np.all(got[q, j, :hp] == 0.0)      # no gradient reaches the query of an empty row


# Mask rows that travel whole (s a multiple of 4: tiles inside the row), word by word (the last tile) and byte by byte (any other
# s), in the forms of the kernels for few and many workgroups.
@pytest.mark.parametrize("s,b,heads,dh", [(196, 1, 3, 64), (132, 2, 3, 160), (132, 8, 43, 32), (131, 8, 43, 32), (192, 4, 65, 128),
                                          (256, 2, 35, 96), (130, 5, 53, 96), (132, 5, 53, 64), (132, 4, 43, 32), (133, 3, 90, 64),
                                          # the forms that the lists above leave out, rows of whole words
                                          (68, 1, 1, 32), (68, 5, 103, 32), (452, 5, 13, 32), (68, 1, 257, 64), (68, 5, 103, 64), (452, 5, 13, 64),
                                          (36, 1, 1, 96), (68, 1, 1, 96), (36, 5, 103, 96), (68, 13, 31, 96), (388, 5, 8, 96), (36, 1, 1, 128),
                                          (36, 5, 103, 128), (388, 5, 8, 128), (36, 10, 103, 160),
                                          # and of single bytes
                                          (33, 1, 1, 32), (327, 1, 3, 32), (65, 1, 257, 32), (33, 5, 103, 32), (65, 5, 103, 32), (33, 1, 1, 64),
                                          (327, 1, 3, 64), (65, 5, 103, 64), (327, 1, 3, 96), (65, 13, 31, 96), (327, 1, 3, 128),
                                          (33, 5, 103, 128), (65, 1, 257, 128), (65, 13, 31, 128), (33, 10, 103, 160),
                                          # dQ and dK/dV side by side, and with some more heads one after the other
                                          (388, 1, 3, 128), (388, 1, 3, 160), (68, 1, 80, 96), (68, 1, 80, 160), (68, 1, 200, 32), (68, 1, 150, 64),
                                          (65, 1, 3, 128), (65, 1, 3, 160), (65, 1, 80, 96), (65, 1, 80, 128), (65, 1, 80, 160), (65, 1, 200, 32),
                                          (65, 1, 150, 64)])
def test_masked_attention_forms(s, b, heads, dh):
    test_masked_attention_forward_backward(B.BF16, s, b, heads, dh, True, [(0, s - 1)])


# No mask at all, in every form.
@pytest.mark.parametrize("s,b,heads,dh", [(33, 1, 1, 32), (65, 1, 1, 32), (33, 5, 103, 32), (65, 1, 257, 32), (65, 5, 103, 32), (449, 5, 13, 32),
                                          (33, 1, 1, 64), (65, 1, 1, 64), (33, 5, 103, 64), (65, 1, 257, 64), (65, 5, 103, 64), (449, 5, 13, 64),
                                          (33, 1, 1, 96), (65, 3, 43, 96), (33, 5, 103, 96), (65, 13, 31, 96), (389, 5, 8, 96),
                                          (33, 1, 1, 128), (33, 5, 103, 128), (65, 13, 31, 128), (389, 5, 8, 128),
                                          (33, 1, 1, 160), (33, 10, 103, 160),
                                          # as above
                                          (389, 1, 3, 160), (65, 1, 200, 160), (65, 1, 200, 32), (65, 1, 150, 64), (65, 1, 80, 96)])
def test_unmasked_attention_forms(s, b, heads, dh):
    test_masked_attention_forward_backward(B.BF16, s, b, heads, dh, False, [])


def test_upper_triangular_mask_equals_the_causal_kernels():
    s, b, heads, dh = 192, 1, 2, 128
    hp = heads * dh
    qkv = randn((s, b, 3 * hp), B.BF16, 3)
    mask = torch.from_numpy(np.triu(np.ones((b, s, s), dtype=np.uint8), 1)).cuda()
    outs = []
    for general in (False, True):
        ctx = torch.zeros((s, b, hp), dtype=torch.bfloat16, device="cuda"); lse = torch.zeros((b, heads, s), device="cuda")
        if general:
            B.check(B.ptdp_attn_masked_fwd(B.BF16, qkv.data_ptr(), mask.data_ptr(), ctx.data_ptr(), lse.data_ptr(), s, b,
                                           heads, dh, stream()), "masked")
        else:
            B.check(B.ptdp_attn_fwd(B.BF16, qkv.data_ptr(), ctx.data_ptr(), lse.data_ptr(), s, b, heads, dh, stream()), "causal")
        sync()
        outs.append((ctx, lse))
    assert_close(np64(outs[1][0]), np64(outs[0][0]), B.BF16, "ctx", 0.05)
    assert np.allclose(np64(outs[1][1]), np64(outs[0][1]), atol=1e-4)


@pytest.mark.parametrize("dtype", [B.F32, B.BF16])
def test_layer_with_general_mask(dtype):
    cfg = B.make_cfg(h=256, a=4, t=2, s=72, b=2, dtype=dtype, p_hidden=0.1, seed=2, causal=0)
    rig = LayerRig(cfg, 2, first_layer=1, seed=30)
    mask = make_mask(cfg.b, cfg.s, 5, empty_rows=[(1, 3)])
    mask_d = torch.from_numpy(mask).cuda()
    assert B.ptdp_chunk_set_mask(rig.chunk.handle, mask_d.data_ptr() + 1) == B.E_INVALID_ARG     # alignment
    B.check(B.ptdp_chunk_set_mask(rig.chunk.handle, mask_d.data_ptr()), "set_mask")
    shape = (cfg.s, cfg.b, cfg.h)
    x = randn(shape, dtype, 1); dy = randn(shape, dtype, 2)
    y = torch.empty_like(x); dx = torch.empty_like(x)
    B.check(rig.chunk.forward(3, x.data_ptr(), y.data_ptr(), rig.stash.data_ptr(), rig.ws.data_ptr()), "fwd")
    B.check(rig.chunk.backward(3, dy.data_ptr(), dx.data_ptr(), rig.stash.data_ptr(), rig.ws.data_ptr()), "bwd")
    sync()
    ocfg = oracle_cfg(cfg)
    ocfg.causal = False
    Ps = [params_np(P) for P in rig.params]
    cur = np64(x); caches = []
    for l, P in enumerate(Ps):
        cur, c = L.layer_forward(cur, P, ocfg, 1 + l, 3, mask=mask)
        caches.append(c)
    assert_close(np64(y), cur, dtype, "y")
    wdx, wg = L.chunk_backward(np64(dy), Ps, ocfg, caches)
    assert_close(np64(dx), wdx, dtype, "dx")
    for l in range(2):
        for k in B.PARAM_NAMES:
            assert_close(np64(rig.grads[l][k]), wg[l][k], dtype, "layer %d grad %s" % (l, k))
    # a causal chunk refuses a mask
    crig = LayerRig(B.make_cfg(h=256, a=4, t=1, s=8, b=1, dtype=dtype), 1)
    assert B.ptdp_chunk_set_mask(crig.chunk.handle, mask_d.data_ptr()) == B.E_INVALID_ARG
