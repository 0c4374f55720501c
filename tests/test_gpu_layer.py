"""GPU parity of whole layers, chunks and the schedule runner against the oracle (C ABI)."""
import ctypes as C

import numpy as np
import pytest
import torch

from oracle import gpt_layer as L
from oracle import schedule as S
from paper_2104_04473_amd import binding as B
from gpu_util import LayerRig, assert_close, dev_bytes, np64, oracle_cfg, params_np, randn, stream, sync, tdt

pytestmark = pytest.mark.gpu


def check_layer(cfg, n_layers=1, first_layer=0, microbatches=(0,), factor=1.0):
    rig = LayerRig(cfg, n_layers, first_layer)
    ocfg = oracle_cfg(cfg)
    Ps = [params_np(P) for P in rig.params]
    want_grads = [None] * n_layers
    errs = {}
    for mb in microbatches:
        x = randn((cfg.s, cfg.b, cfg.h), cfg.dtype, 1000 + mb)
        dy = randn((cfg.s, cfg.b, cfg.h), cfg.dtype, 2000 + mb)
        y = torch.empty_like(x); dx = torch.empty_like(x)
        B.check(rig.chunk.forward(mb, x.data_ptr(), y.data_ptr(), rig.stash.data_ptr(), rig.ws.data_ptr()), "forward")
        B.check(rig.chunk.backward(mb, dy.data_ptr(), dx.data_ptr(), rig.stash.data_ptr(), rig.ws.data_ptr()), "backward")
        sync()
        wy, caches = L.chunk_forward(np64(x), Ps, ocfg, first_layer, mb)
        wdx, grads = L.chunk_backward(np64(dy), Ps, ocfg, caches)
        errs["y"] = assert_close(np64(y), wy, cfg.dtype, "y (mb %d)" % mb, factor)
        errs["dx"] = assert_close(np64(dx), wdx, cfg.dtype, "dx (mb %d)" % mb, factor)
        # stashed intermediates of the last layer (what the backward pass consumed)
        T = cfg.s * cfg.b
        last = n_layers - 1
        for name, key, shape in (("U", "u", (cfg.s, cfg.b, cfg.h)), ("QKV", "qkv", (cfg.s, cfg.b, 3 * cfg.h // cfg.t)),
                                 ("CTX", "ctx", (cfg.s, cfg.b, cfg.h // cfg.t)), ("X1", "x1", (cfg.s, cfg.b, cfg.h)),
                                 ("G", "g", (cfg.s, cfg.b, 4 * cfg.h // cfg.t))):
            assert_close(np64(rig.field(last, name, shape)), caches[last][key], cfg.dtype, "stash " + name, factor)
        assert_close(np64(rig.field(last, "LSE", (cfg.b, cfg.a // cfg.t, cfg.s), torch.float32)), caches[last]["lse"],
                     cfg.dtype, "lse", factor)
        for i in range(n_layers):
            want_grads[i] = grads[i] if want_grads[i] is None else {k: want_grads[i][k] + grads[i][k] for k in grads[i]}
    for i in range(n_layers):
        for name in B.PARAM_NAMES:
            errs[name] = assert_close(np64(rig.grads[i][name]), want_grads[i][name], cfg.dtype,
                                      "grad %s layer %d" % (name, i), factor)
    return errs


def test_config1_fp32_layer():
    """1 GPT layer fp32, h=256, a=4, s=128, b=2, t=1, dropout 0.1 seed 0: forward + backward."""
    cfg = B.make_cfg(h=256, a=4, t=1, s=128, b=2, dtype=B.F32, p_hidden=0.1, seed=0)
    errs = check_layer(cfg)
    print({k: "%.2e" % v for k, v in errs.items()})


@pytest.mark.parametrize("kw", [
    dict(h=256, a=4, t=1, s=72, b=3, dtype=B.F32, p_hidden=0.25, seed=5, gelu_mode=B.GELU_TANH),
    dict(h=512, a=8, t=2, s=96, b=2, dtype=B.F32, p_hidden=0.0, seed=1),
    dict(h=512, a=8, t=1, s=200, b=2, dtype=B.BF16, p_hidden=0.1, seed=2),
    dict(h=1024, a=8, t=2, s=136, b=1, dtype=B.BF16, p_hidden=0.1, seed=3),
    dict(h=1280, a=8, t=4, s=264, b=2, dtype=B.BF16, p_hidden=0.1, seed=4),          # dh = 160
])
def test_layer_variants(kw):
    check_layer(B.make_cfg(**kw))


# LayerNorm backward with the attention half's dropout in the same pass: 1, 2 and 4 waves per row with one and two vectors a lane, rows
# that do not fill the last block's groups
@pytest.mark.parametrize("kw", [
    dict(h=512, a=8, t=1, s=301, b=7, dtype=B.BF16, p_hidden=0.1, seed=6),           # one wave, one vector
    dict(h=1024, a=8, t=4, s=301, b=7, dtype=B.BF16, p_hidden=0.1, seed=7),          # one wave, two
    dict(h=256, a=4, t=1, s=301, b=7, dtype=B.F32, p_hidden=0.1, seed=8),
    dict(h=512, a=8, t=4, s=301, b=7, dtype=B.F32, p_hidden=0.1, seed=9),
    dict(h=512, a=8, t=1, s=259, b=4, dtype=B.BF16, p_hidden=0.1, seed=10),          # two waves, one vector
    dict(h=2048, a=16, t=8, s=259, b=4, dtype=B.BF16, p_hidden=0.1, seed=11),        # two waves, two vectors
    dict(h=2304, a=24, t=8, s=259, b=4, dtype=B.BF16, p_hidden=0.1, seed=12),        # four waves
])
def test_layer_rows_shared_by_few_waves(kw):
    check_layer(B.make_cfg(**kw))


# one row, rows and columns that leave a block's last lanes empty, 1, 2, 4 and 8 waves a row; 504 and 528 workgroups of sums (the second: two launches)
@pytest.mark.parametrize("h,a,t,s,b,dtype", [
    (64, 2, 1, 1, 1, B.F32), (96, 3, 1, 37, 1, B.F32), (256, 4, 1, 129, 1, B.F32), (512, 4, 1, 33, 8, B.F32), (512, 8, 1, 301, 7, B.F32),
    (256, 8, 1, 1, 1, B.BF16), (160, 1, 1, 65, 1, B.BF16), (1024, 16, 2, 301, 7, B.BF16), (2048, 16, 8, 259, 4, B.BF16), (2304, 24, 8, 259, 4, B.BF16),
    (12288, 96, 96, 17, 2, B.BF16), (1024, 16, 1, 383, 7, B.BF16), (1024, 16, 1, 401, 7, B.BF16),
])
def test_qkv_bias_sums_beside_layernorm_backward(h, a, t, s, b, dtype):
    """The QKV bias gradient's sums share a launch with the first LayerNorm's backward where they are few: every bit is that of
    LayerNorm backward and of column sums in calls of their own with the same operands."""
    cfg = B.make_cfg(h=h, a=a, t=t, s=s, b=b, dtype=dtype, p_hidden=0.1, seed=5)
    rig, T, w = LayerRig(cfg), s * b, 3 * h // t
    x, dy = randn((s, b, h), dtype, 1), randn((s, b, h), dtype, 2)
    y, dx, dx2 = torch.empty_like(x), torch.empty_like(x), torch.empty_like(x)
    for g in rig.grads[0].values():
        g.fill_(0.25)   # += : the old value counts
    B.check(rig.chunk.forward(0, x.data_ptr(), y.data_ptr(), rig.stash.data_ptr(), rig.ws.data_ptr()), "forward")
    B.check(rig.chunk.backward(0, dy.data_ptr(), dx.data_ptr(), rig.stash.data_ptr(), rig.ws.data_ptr()), "backward")
    at = {k: rig.ws.data_ptr() + v for k, v in B.workspace_offsets(cfg).items()}
    st = {k: rig.stash.data_ptr() + v for k, v in rig.offsets.items()}
    gain, bias = torch.full((h,), 0.25, device="cuda"), torch.full((h,), 0.25, device="cuda")
    scratch = dev_bytes(max(B.ptdp_layernorm_bwd_scratch_bytes(T, h), B.ptdp_colsum_scratch_bytes(T, w)))
    B.check(B.ptdp_layernorm_bwd(dtype, at["DU"], st["X"], rig.params[0]["ln1_g"].data_ptr(), st["MU1"], st["RSTD1"], at["DX1"],
                                 dx2.data_ptr(), gain.data_ptr(), bias.data_ptr(), scratch.data_ptr(), T, h, stream()), "layernorm")
    sums, out = torch.full((w,), 0.25, device="cuda"), torch.empty((T, w), dtype=tdt(dtype), device="cuda")
    B.check(B.ptdp_bias_dropout_add_bwd(dtype, at["DQKV"], out.data_ptr(), sums.data_ptr(), scratch.data_ptr(), T, w, 0.0, 0, 0, 0, 0, stream()), "sums")
    sync()
    G = rig.grads[0]
    assert torch.equal(dx, dx2) and torch.equal(G["ln1_g"], gain) and torch.equal(G["ln1_b"], bias)
    assert torch.equal(G["b_qkv"], sums)


# workgroups of 2, 4 and 8 waves, fewer parts than waves and more, columns that leave a block's last lanes empty; 256 x 256 tiles (a launch of their own)
@pytest.mark.parametrize("h,a,t,s,b,dtype", [
    (64, 2, 1, 1, 1, B.F32), (96, 3, 1, 37, 1, B.F32), (256, 4, 1, 128, 2, B.F32), (512, 8, 1, 301, 7, B.F32),
    (256, 8, 1, 1, 1, B.BF16), (160, 1, 1, 65, 1, B.BF16), (512, 8, 1, 333, 2, B.BF16), (1024, 16, 2, 301, 7, B.BF16), (2048, 16, 2, 1024, 1, B.BF16),
    (4096, 32, 1, 512, 2, B.BF16),
])
def test_column_sums_beside_weight_gradients(h, a, t, s, b, dtype):
    """Column sums are finished in the launch of the weight gradients where its tiles are small: the bits of a call of their own."""
    cfg = B.make_cfg(h=h, a=a, t=t, s=s, b=b, dtype=dtype, p_hidden=0.1, seed=7)
    rig, T = LayerRig(cfg, first_layer=3), s * b
    x, dy = randn((s, b, h), dtype, 1), randn((s, b, h), dtype, 2)
    y, dx, out = torch.empty_like(x), torch.empty_like(x), torch.empty_like(x)
    for g in rig.grads[0].values():
        g.fill_(0.25)   # += : the old value counts
    B.check(rig.chunk.forward(1, x.data_ptr(), y.data_ptr(), rig.stash.data_ptr(), rig.ws.data_ptr()), "forward")
    B.check(rig.chunk.backward(1, dy.data_ptr(), dx.data_ptr(), rig.stash.data_ptr(), rig.ws.data_ptr()), "backward")
    scratch = dev_bytes(B.ptdp_colsum_scratch_bytes(T, h))
    at = {k: rig.ws.data_ptr() + v for k, v in B.workspace_offsets(cfg).items()}
    for name, site, grad in (("b_2", 1, dy.data_ptr()), ("b_o", 0, at["DX1"])):
        sums = torch.full((h,), 0.25, device="cuda")
        B.check(B.ptdp_bias_dropout_add_bwd(dtype, grad, out.data_ptr(), sums.data_ptr(), scratch.data_ptr(), T, h, 0.1, 7, 3, site, 1, stream()), name)
        sync()
        if name == "b_2":
            assert torch.equal(rig.grads[0][name], sums)
        else:   # its rows are summed in another order, by the workgroups of LayerNorm backward: fp32 sums of T terms each
            assert_close(np64(rig.grads[0][name]), np64(sums), B.F32, name)


def test_chunk_of_layers_and_gradient_accumulation():
    cfg = B.make_cfg(h=256, a=4, t=1, s=40, b=2, dtype=B.F32, p_hidden=0.1, seed=9)
    check_layer(cfg, n_layers=3, first_layer=4, microbatches=(0, 3))
    cfg = B.make_cfg(h=512, a=4, t=2, s=136, b=1, dtype=B.BF16, p_hidden=0.1, seed=9)
    check_layer(cfg, n_layers=2, first_layer=2, microbatches=(1, 2))


def test_layer_is_deterministic():
    cfg = B.make_cfg(h=512, a=4, t=1, s=136, b=2, dtype=B.BF16, p_hidden=0.1, seed=1)
    outs = []
    for _ in range(2):
        rig = LayerRig(cfg)
        x = randn((cfg.s, cfg.b, cfg.h), cfg.dtype, 1); dy = randn((cfg.s, cfg.b, cfg.h), cfg.dtype, 2)
        y = torch.empty_like(x); dx = torch.empty_like(x)
        B.check(rig.chunk.forward(0, x.data_ptr(), y.data_ptr(), rig.stash.data_ptr(), rig.ws.data_ptr()), "f")
        B.check(rig.chunk.backward(0, dy.data_ptr(), dx.data_ptr(), rig.stash.data_ptr(), rig.ws.data_ptr()), "b")
        sync()
        outs.append((y.clone(), dx.clone(), {k: v.clone() for k, v in rig.grads[0].items()}))
    assert torch.equal(outs[0][0], outs[1][0]) and torch.equal(outs[0][1], outs[1][1])
    for k in outs[0][2]:
        assert torch.equal(outs[0][2][k], outs[1][2][k]), k


def test_schedule_run_interleaved():
    """One device's interleaved order (p=4, v=2, m=4, rank 1) on tiny chunks: every (chunk, microbatch)
    result is bit-identical to running it alone, gradients are the sum over microbatches, and the
    stash pool never needs more slots than the order's peak."""
    p, v, m, rank = 4, 2, 4, 1
    cfg = B.make_cfg(h=256, a=4, t=1, s=24, b=2, dtype=B.BF16, p_hidden=0.1, seed=4)
    rigs = [LayerRig(cfg, 2, first_layer=2 * (c * p + rank), seed=50 + 10 * c) for c in range(v)]
    steps = B.schedule_build(p, v, m, rank)
    peak = B.ptdp_schedule_peak_inflight(p, v, m, rank)
    slot_bytes = rigs[0].chunk.stash_bytes()
    pool = dev_bytes(slot_bytes * peak)
    shape = (cfg.s, cfg.b, cfg.h)
    xin = [randn(shape, cfg.dtype, 300 + i) for i in range(v * m)]
    dout = [randn(shape, cfg.dtype, 400 + i) for i in range(v * m)]
    yout = [torch.empty_like(xin[0]) for _ in range(v * m)]
    din = [torch.empty_like(xin[0]) for _ in range(v * m)]
    arr = lambda ts: (C.c_void_p * len(ts))(*[t.data_ptr() for t in ts])
    handles = (C.c_void_p * v)(*[r.chunk.handle for r in rigs])
    args = (handles, v, m, steps, len(steps), arr(xin), arr(yout), arr(dout), arr(din))
    assert B.ptdp_schedule_run(*args, pool.data_ptr(), slot_bytes, peak - 1, rigs[0].ws.data_ptr(), stream()) == B.E_TOO_SMALL
    B.check(B.ptdp_schedule_run(*args, pool.data_ptr(), slot_bytes, peak, rigs[0].ws.data_ptr(), stream()), "run")
    sync()
    sched_grads = [[{k: g.clone() for k, g in G.items()} for G in r.grads] for r in rigs]
    # the same work, one (chunk, microbatch) at a time, in plain order
    for r in rigs:
        for G in r.grads:
            for g in G.values():
                g.zero_()
    for c in range(v):
        for mb in range(m):
            y = torch.empty_like(xin[0]); dx = torch.empty_like(xin[0])
            i = c * m + mb
            B.check(rigs[c].chunk.forward(mb, xin[i].data_ptr(), y.data_ptr(), rigs[c].stash.data_ptr(), rigs[c].ws.data_ptr()), "f")
            B.check(rigs[c].chunk.backward(mb, dout[i].data_ptr(), dx.data_ptr(), rigs[c].stash.data_ptr(), rigs[c].ws.data_ptr()), "b")
            sync()
            assert torch.equal(y, yout[i]) and torch.equal(dx, din[i])
    # gradient sums: same addends, but the schedule adds them in a different microbatch order
    for c in range(v):
        for l in range(2):
            for k in B.PARAM_NAMES:
                assert_close(np64(sched_grads[c][l][k]), np64(rigs[c].grads[l][k]), B.F32, "grad " + k, 0.1)
    # and against the oracle for one pair
    ocfg = oracle_cfg(cfg)
    Ps = [params_np(P) for P in rigs[1].params]
    wy, _ = L.chunk_forward(np64(xin[1 * m + 2]), Ps, ocfg, 2 * (1 * p + rank), 2)
    assert_close(np64(yout[1 * m + 2]), wy, cfg.dtype, "y of (chunk 1, microbatch 2)")


def test_chunk_forward_backward_replays_from_a_hip_graph():
    """The library allocates nothing, clears nothing with memsets and never synchronises, so a step can be
    captured into a HIP graph.  Every replay (with eager work and synchronisations in between) must give the
    bits of the eager step, including the += into the gradient buffers."""
    cfg = B.make_cfg(h=256, a=4, t=1, s=64, b=2, dtype=B.BF16, p_hidden=0.1, seed=6)
    rig = LayerRig(cfg, 2, first_layer=0, seed=90)
    shape = (cfg.s, cfg.b, cfg.h)
    x = randn(shape, cfg.dtype, 1); dy = randn(shape, cfg.dtype, 2)
    y = torch.empty_like(x); dx = torch.empty_like(x)

    def step():
        B.check(rig.chunk.forward(1, x.data_ptr(), y.data_ptr(), rig.stash.data_ptr(), rig.ws.data_ptr()), "fwd")
        B.check(rig.chunk.backward(1, dy.data_ptr(), dx.data_ptr(), rig.stash.data_ptr(), rig.ws.data_ptr()), "bwd")

    step()                      # eager reference (also sets the kernels' one-time attributes before capture)
    sync()
    y_ref, dx_ref = y.clone(), dx.clone()
    g1 = [{k: v.clone() for k, v in G.items()} for G in rig.grads]       # gradients after one step
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()                  # captured on the capture stream (torch's current stream inside the context)
    sync()
    for G in rig.grads:
        for v in G.values():
            v.zero_()
    for replay in range(1, 4):
        y.zero_(); dx.zero_()
        graph.replay()
        sync()
        assert torch.equal(y, y_ref) and torch.equal(dx, dx_ref), "replay %d" % replay
        scratch = randn(shape, cfg.dtype, 10 + replay) * 2.0            # unrelated eager work between replays
        sync()
        del scratch
        if replay == 1:
            for l in range(2):
                for k in B.PARAM_NAMES:
                    assert torch.equal(rig.grads[l][k], g1[l][k]), (l, k)
    # three replays accumulated three times the same addend, in the order an eager loop would
    for G in rig.grads:
        for v in G.values():
            v.zero_()
    for _ in range(3):
        step()
    sync()
    eager3 = [{k: v.clone() for k, v in G.items()} for G in rig.grads]
    for G in rig.grads:
        for v in G.values():
            v.zero_()
    for _ in range(3):
        graph.replay()
    sync()
    for l in range(2):
        for k in B.PARAM_NAMES:
            assert torch.equal(rig.grads[l][k], eager3[l][k]), (l, k)


# The LayerNorms that run in the launch of the residual sum in front of them (inside a layer, and across two layers of a chunk)
# give the bits of the op by itself on the stored row.  Widths: one, two, four and eight vectors per thread, the last ones partly used.
@pytest.mark.parametrize("dtype,h,a,t", [(B.F32, 256, 4, 1), (B.F32, 2176, 34, 2), (B.BF16, 256, 4, 1), (B.BF16, 4608, 48, 8),
                                         (B.BF16, 12288, 96, 8), (B.BF16, 25600, 160, 8)])
def test_layernorm_behind_a_residual_sum(dtype, h, a, t):
    s, b, n = 5, 1, 2
    cfg = B.make_cfg(h=h, a=a, t=t, s=s, b=b, dtype=dtype, p_hidden=0.1, seed=3)
    rig = LayerRig(cfg, n)
    x, y = randn((s, b, h), dtype, 4), torch.empty((s, b, h), dtype=tdt(dtype), device="cuda")
    B.check(rig.chunk.forward(0, x.data_ptr(), y.data_ptr(), rig.stash.data_ptr(), rig.ws.data_ptr()), "forward")
    sync()
    for l in range(n):
        for src, dst, mean, rstd, norm in (("X", "U", "MU1", "RSTD1", "ln1"), ("X1", "U2", "MU2", "RSTD2", "ln2")):
            row, P = rig.field(l, src, (s, b, h)), rig.params[l]
            u, mu, rs = torch.empty_like(row), torch.empty(s * b, device="cuda"), torch.empty(s * b, device="cuda")
            B.check(B.ptdp_layernorm_fwd(dtype, row.data_ptr(), P[norm + "_g"].data_ptr(), P[norm + "_b"].data_ptr(), u.data_ptr(),
                                         mu.data_ptr(), rs.data_ptr(), None, s * b, h, cfg.ln_eps, stream()), "layernorm_fwd")
            sync()
            assert torch.equal(u, rig.field(l, dst, (s, b, h)))
            assert torch.equal(mu, rig.field(l, mean, (s * b,), torch.float32))
            assert torch.equal(rs, rig.field(l, rstd, (s * b,), torch.float32))


# every small form of both products, rows and columns that fill no tile, tanh; 256 x 192, 256 x 256 and fp32's 64 x 64 tiles (kernels of their own);
# 16 x 16 tiles (the gradient's in a kernel of its own)
@pytest.mark.parametrize("h,a,t,s,b,dtype,gelu,tile", [
    (512, 8, 1, 25, 8, B.BF16, B.GELU_TANH, (64, 64, 2)), (320, 2, 2, 200, 1, B.BF16, B.GELU_ERF, (128, 64, 1)),
    (1536, 12, 1, 200, 1, B.BF16, B.GELU_ERF, (128, 64, 2)), (320, 2, 1, 400, 5, B.BF16, B.GELU_TANH, (128, 128, 1)),
    (512, 8, 1, 400, 5, B.BF16, B.GELU_ERF, (128, 128, 2)), (768, 12, 1, 400, 10, B.BF16, B.GELU_ERF, (256, 192, 1)),
    (1024, 16, 1, 400, 10, B.BF16, B.GELU_ERF, (256, 256, 1)),
    (64, 2, 1, 37, 1, B.F32, B.GELU_ERF, None), (256, 4, 1, 128, 2, B.F32, B.GELU_TANH, None), (384, 6, 1, 100, 1, B.F32, B.GELU_ERF, None),
    (384, 6, 1, 66, 1, B.F32, B.GELU_ERF, None), (384, 6, 1, 66, 1, B.F32, B.GELU_TANH, None),
    (512, 8, 1, 301, 7, B.F32, B.GELU_ERF, None),
])
def test_gelu_in_the_products_beside_it(h, a, t, s, b, dtype, gelu, tile):
    """GeLU and its derivative in the output stage of the products next to them: the bits of a product and a GeLU in calls of their
    own; the bias gradient's sums take the rows in another order."""
    cfg = B.make_cfg(h=h, a=a, t=t, s=s, b=b, dtype=dtype, p_hidden=0.1, seed=5, gelu_mode=gelu)
    rig, T, f = LayerRig(cfg), s * b, 4 * h // t
    if tile:
        got = [C.c_int() for _ in range(3)]
        for mode in (0, 1):
            B.check(B.ptdp_gemm_form(mode, T, f, h, 0, 0, 0, B.ptdp_gemm_workspace_bytes(), *[C.byref(x) for x in got]), "form")
            assert tuple(x.value for x in got) == tile
    x, dy = randn((s, b, h), dtype, 1), randn((s, b, h), dtype, 2)
    y, dx = torch.empty_like(x), torch.empty_like(x)
    rig.grads[0]["b_1"].fill_(0.25)
    B.check(rig.chunk.forward(0, x.data_ptr(), y.data_ptr(), rig.stash.data_ptr(), rig.ws.data_ptr()), "forward")
    B.check(rig.chunk.backward(0, dy.data_ptr(), dx.data_ptr(), rig.stash.data_ptr(), rig.ws.data_ptr()), "backward")
    P, at = rig.params[0], {k: rig.ws.data_ptr() + v for k, v in B.workspace_offsets(cfg).items()}
    Z, G = rig.field(0, "Z", (T, f)), rig.field(0, "G", (T, f))
    z, g, dz = (torch.empty((T, f), dtype=tdt(dtype), device="cuda") for _ in range(3))
    db, scratch = torch.full((f,), 0.25, device="cuda"), dev_bytes(B.ptdp_colsum_scratch_bytes(T, f))
    n = B.ptdp_gemm_workspace_bytes() if dtype == B.BF16 else 0
    ws = dev_bytes(n)
    gemm = lambda mode, A, W, out: B.check(B.ptdp_gemm(dtype, mode, A, W.data_ptr(), out.data_ptr(), None, T, f, h, 0, 0, ws.data_ptr(), n, stream()), "gemm")
    gemm(0, rig.field(0, "U2", (T, h)).data_ptr(), P["w_1"], z)
    B.check(B.ptdp_bias_gelu_fwd(dtype, gelu, z.data_ptr(), P["b_1"].data_ptr(), g.data_ptr(), T, f, stream()), "gelu")
    gemm(1, at["DMO"], P["w_2"], dz)
    B.check(B.ptdp_bias_gelu_bwd(dtype, gelu, dz.data_ptr(), Z.data_ptr(), P["b_1"].data_ptr(), dz.data_ptr(), db.data_ptr(), scratch.data_ptr(), T, f,
                                 stream()), "gelu backward")
    sync()
    off = B.workspace_offsets(cfg)["DZ"]
    got_dz = rig.ws[off:off + dz.numel() * dz.element_size()].view(dz.dtype).view(T, f)
    assert torch.equal(Z, z) and torch.equal(G, g) and torch.equal(got_dz, dz)
    # two fp32 sums of T terms in different orders: relative to the sum of the terms' sizes, below T * 2^-24 (here far below)
    lim = T * 2.0 ** -24 * (got_dz.double().abs().sum(0) + 0.25)
    assert ((rig.grads[0]["b_1"].double() - db.double()).abs() <= lim).all()


# every small form, rows that fill no tile, no dropout; 256 x 256 tiles and fp32 (a kernel of its own)
@pytest.mark.parametrize("h,a,t,s,b,dtype,p,tile", [
    (768, 12, 1, 41, 8, B.BF16, 0.1, (64, 64, 2)), (64, 2, 1, 8, 1, B.BF16, 0.1, (128, 64, 1)), (96, 3, 1, 8, 5, B.BF16, 0.0, (128, 64, 1)),
    (512, 8, 1, 1500, 2, B.BF16, 0.1, (128, 64, 2)), (1536, 12, 4, 1500, 2, B.BF16, 0.25, (128, 128, 1)), (768, 12, 2, 600, 5, B.BF16, 0.1, (128, 128, 2)),
    (2048, 16, 1, 1000, 2, B.BF16, 0.1, (256, 256, 1)), (128, 2, 1, 37, 1, B.F32, 0.1, None),
])
def test_residual_sum_in_the_last_product(h, a, t, s, b, dtype, p, tile):
    """The last layer's residual sum in the output stage of its second MLP product: the bits of a product and a sum in calls of their own."""
    cfg = B.make_cfg(h=h, a=a, t=t, s=s, b=b, dtype=dtype, p_hidden=p, seed=9)
    rig, T, f = LayerRig(cfg, n_layers=2, first_layer=4), s * b, 4 * h // t
    n = B.ptdp_gemm_workspace_bytes() if dtype == B.BF16 else 0
    if tile:
        got = [C.c_int() for _ in range(3)]
        B.check(B.ptdp_gemm_form(0, T, h, f, 0, 0, 0, n, *[C.byref(x) for x in got]), "form")
        assert tuple(x.value for x in got) == tile
    x, y = randn((s, b, h), dtype, 1), torch.empty((s, b, h), dtype=tdt(dtype), device="cuda")
    B.check(rig.chunk.forward(2, x.data_ptr(), y.data_ptr(), rig.stash.data_ptr(), rig.ws.data_ptr()), "forward")
    o, want, ws, P = torch.empty_like(y), torch.empty_like(y), dev_bytes(n), rig.params[1]
    B.check(B.ptdp_gemm(dtype, 0, rig.field(1, "G", (T, f)).data_ptr(), P["w_2"].data_ptr(), o.data_ptr(), None, T, h, f, 0, 0, ws.data_ptr(), n, stream()), "gemm")
    B.check(B.ptdp_bias_dropout_add_fwd(dtype, o.data_ptr(), P["b_2"].data_ptr(), rig.field(1, "X1", (T, h)).data_ptr(), want.data_ptr(), T, h, p, 9, 5, 1, 2,
                                        stream()), "sum")
    sync()
    assert torch.equal(y, want)


def launches(rig, x):
    """Launches per family of one forward and one backward."""
    y, dx = torch.empty_like(x), torch.empty_like(x)
    B.ptdp_prof_enable(1)
    try:
        B.check(rig.chunk.forward(0, x.data_ptr(), y.data_ptr(), rig.stash.data_ptr(), rig.ws.data_ptr()), "forward")
        B.check(rig.chunk.backward(0, y.data_ptr(), dx.data_ptr(), rig.stash.data_ptr(), rig.ws.data_ptr()), "backward")
        sync()
        return {k: v[2] for k, v in B.prof_collect().items()}
    finally:
        B.ptdp_prof_enable(0)


# 32 x 32 tiles next to the MLP's GeLU, 16 x 16 (the gradient a kernel of its own), 64 x 64 (both)
@pytest.mark.parametrize("h,a,s,b,own", [(64, 2, 37, 1, (0, 0)), (256, 4, 128, 2, (0, 0)), (384, 6, 66, 1, (0, 1)), (256, 4, 341, 3, (1, 1)),
                                         (640, 10, 348, 4, (1, 1))])
def test_fp32_gelu_is_a_kernel_of_its_own_beside_large_tiles(h, a, s, b, own):
    cfg = B.make_cfg(h=h, a=a, t=1, s=s, b=b, dtype=B.F32, p_hidden=0.1, seed=3)
    n = launches(LayerRig(cfg), randn((s, b, h), B.F32, 1))
    assert (n["bias_gelu_fwd"], n["bias_gelu_bwd"]) == own


# weight gradients that 256 x 256 tiles compute faster, but not with the launch for the column sums that follows them; and (the last) with it
@pytest.mark.parametrize("h,a,t,s,b,own", [(1024, 16, 1, 512, 4, False), (2624, 82, 2, 169, 2, False), (11520, 72, 8, 291, 2, False), (2304, 18, 1, 877, 2, True)])
def test_column_sums_need_no_launch_where_the_forms_are_close(h, a, t, s, b, own):
    cfg = B.make_cfg(h=h, a=a, t=t, s=s, b=b, dtype=B.BF16, p_hidden=0.1, seed=3)
    n = launches(LayerRig(cfg), randn((s, b, h), B.BF16, 1))
    assert (n["colsum"] > 0) == own and n["gemm_tn"] == 1
