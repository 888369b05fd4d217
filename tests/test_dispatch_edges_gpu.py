"""GPU parity at the edges of the kernels' size rules (tile remainders, split
ranges, staging limits): small blocks and steps against the fp64 oracle,
metric and bars as in test_parity_gpu.py."""
import numpy as np
import pytest
import torch

import synth
from oracle import dit_oracle as O
from tests.test_parity_gpu import TOL, _gpu, block_case, check, f64

pytestmark = pytest.mark.gpu


def _cfg(dtype, hidden, dh, **kw):
    kw.setdefault("mlp_hidden", 256)
    return synth.CONFIGS["c1"].with_(dtype=dtype, hidden=hidden, heads=hidden // dh, head_dim=dh, cond="given",
                                     n_blocks=1, **kw)


# adaLN: odd numbers of 128-byte weight lines split over the four waves
# (hidden 64: one or two lines for four waves), one and several passes of 16
# samples, the bf16 switch between SiLU computed by the workgroups (matrices x
# samples <= 4) and read back, fp32 samples beyond one 64 KB staging pass
# (15 x 1156 floats), joint blocks (two matrices).
ADA = [("bf16", 64, 64, 1, 0), ("bf16", 192, 64, 4, 0), ("bf16", 192, 64, 5, 0), ("bf16", 320, 64, 2, 3),
       ("bf16", 576, 72, 16, 0), ("bf16", 576, 72, 17, 0), ("bf16", 256, 128, 40, 0), ("f32", 64, 64, 1, 0),
       ("f32", 192, 64, 5, 2), ("f32", 1152, 72, 15, 0), ("f32", 576, 72, 33, 0)]


@pytest.mark.parametrize("dtype,hidden,dh,batch,tt", ADA)
def test_adaln_edges(dtype, hidden, dh, batch, tt):
    block_case(_cfg(dtype, hidden, dh, batch=batch, tokens=2, text_tokens=tt))


def test_cond_of_four_byte_alignment():
    """cond need only be 4-byte aligned: the same bits from a shifted copy."""
    g = _gpu()
    for dtype in ("bf16", "f32"):
        cfg = _cfg(dtype, 192, 64, batch=3, tokens=4)
        db, inp = g.DeviceBlock(cfg, synth.block_weights(cfg, 0)), synth.inputs(cfg)
        import paper_2605_25550_amd as dm
        ws = dm.alloc_workspace(db.shape, dm.DIT_WS_BLOCK)
        outs = []
        for shift in (0, 1):
            buf = torch.zeros(cfg.batch * cfg.hidden + 1, device="cuda")
            c = buf[shift:shift + cfg.batch * cfg.hidden].view(cfg.batch, cfg.hidden)
            c.copy_(g.dev(inp["cond"]))
            x = g.dev(inp["x"])
            dm.block_forward(db.shape, db.struct, x, c, ws)
            torch.cuda.synchronize()
            outs.append(x.cpu())
        assert torch.equal(*outs)


# fp32 GEMM tiles (32 x 32, 64 x 64, 96 x 64, 96 x 48, and 96 x 64 in k-ranges
# with the residual reduction), fewer k-slices than k-groups (hidden 64), odd
# slice counts per k-group, ragged rows, two problems of different row counts;
# attention with waves that own no keys, partial 16-query and 32-key groups,
# and 32 queries per workgroup (from 512 such workgroups on).
F32 = [(64, 64, 1, 1, 0), (64, 64, 3, 15, 0), (192, 64, 2, 17, 5), (576, 72, 1, 33, 0), (576, 72, 2, 97, 3),
       (256, 128, 2, 127, 0), (256, 128, 1, 130, 31), (1152, 72, 2, 333, 0), (576, 72, 2, 333, 77),
       (576, 72, 2, 1030, 0), (1152, 72, 1, 1030, 0), (1024, 128, 2, 1100, 0), (1024, 64, 1, 1041, 0)]


@pytest.mark.parametrize("hidden,dh,batch,t,tt", F32)
def test_f32_edges(hidden, dh, batch, t, tt):
    # fp32 sums of up to 4 hidden products: sqrt(4608) 2^-24 = 4e-6 of the
    # largest term for each of two chained products, and the softmax between
    cfg = _cfg("f32", hidden, dh, batch=batch, tokens=t, text_tokens=tt, mlp_hidden=4 * hidden)
    g = _gpu()
    w, inp = synth.block_weights(cfg, 0), synth.inputs(cfg)
    x, c, xt = inp["x"], inp["cond"], inp.get("x_txt")
    y, yt = g.run_block(cfg, w, x, c, xt)
    if tt:
        ry, ryt = O.joint_block(x, xt, c, f64(w["img"]), f64(w["txt"]), cfg.heads, cfg.ln_eps)
        check("txt", yt, ryt, xt, 2e-5)
    else:
        ry = O.dit_block(x, c, f64(w["img"]), cfg.heads, cfg.ln_eps)
    check("img", y, ry, x, 2e-5)


# Conditioning: one and several groups of four samples, more samples than one
# staging pass holds (16 for the features; 64 KB of hidden states: 42 at hidden
# 384, 4 at 4096), both register sizes of the output layer's rows (hidden up
# to 1280 and above), a last group of 256 columns that is not full.
@pytest.mark.parametrize("dtype,hidden,dh,batch", [("bf16", 64, 64, 1), ("bf16", 1152, 72, 5), ("bf16", 384, 64, 45),
                                                   ("bf16", 1344, 64, 17), ("bf16", 4096, 128, 6), ("f32", 1280, 64, 13),
                                                   ("f32", 1152, 72, 33)])
def test_cond_embed_edges(dtype, hidden, dh, batch):
    import paper_2605_25550_amd as dm
    g = _gpu()
    cfg = synth.CONFIGS["c1"].with_(dtype=dtype, hidden=hidden, heads=hidden // dh, head_dim=dh, batch=batch, tokens=1,
                                    n_blocks=1, n_classes=30, mlp_hidden=64)
    sw = {k: v for k, v in synth.step_weights(cfg).items()}
    t = np.linspace(0.0, 999.0, batch).astype(np.float32)
    y = (np.arange(batch) * 7 % 30).astype(np.int32)
    shape = dm.shape_of(cfg)
    w = {k: g.dev(sw[k], dm.weight_dtype(shape)) for k in ("w_t1", "b_t1", "w_t2", "b_t2", "class_table")}
    out = torch.full((batch, hidden), float("nan"), device="cuda")
    dm.cond_embed(shape, g.dev(t), g.dev(y, torch.int32), w, out, dm.alloc_workspace(shape, dm.DIT_WS_COND))
    torch.cuda.synchronize()
    ref = O.class_conditioning(t.astype(np.float64), y, **f64({k: sw[k] for k in w}))
    # fp32 arithmetic for both weight types: two chained sums of up to 4096 products
    check("cond", g.host(out), ref, None, 4e-6)


# An infinite hidden value in the last columns of a row: the lanes past the
# row's end, which re-read them, must not add 0 x inf = NaN.  One sample and
# several (the two layouts of the output layer), rows that end inside, at and a
# whole group of columns before the end of the registers' range.
@pytest.mark.parametrize("dtype,hidden,dh,batch", [("bf16", 64, 64, 1), ("bf16", 1152, 72, 1), ("bf16", 1152, 72, 3),
                                                   ("f32", 1280, 64, 2), ("f32", 1344, 64, 1), ("f32", 1344, 64, 13),
                                                   ("bf16", 2048, 128, 8), ("bf16", 3072, 128, 5)])
def test_cond_embed_infinite_hidden_value(dtype, hidden, dh, batch):
    import paper_2605_25550_amd as dm
    g = _gpu()
    cfg = synth.CONFIGS["c1"].with_(dtype=dtype, hidden=hidden, heads=hidden // dh, head_dim=dh, batch=batch, tokens=1,
                                    n_blocks=1, n_classes=30, mlp_hidden=64)
    sw = synth.step_weights(cfg)
    sw["b_t1"][-2] = np.inf  # SiLU(inf) = inf
    sw["w_t2"][:, -2] = np.where(np.arange(hidden) % 2, 0.5, -0.25)
    shape = dm.shape_of(cfg)
    w = {k: g.dev(sw[k], dm.weight_dtype(shape)) for k in ("w_t1", "b_t1", "w_t2", "b_t2", "class_table")}
    t, y = g.dev(np.linspace(0.0, 999.0, batch)), torch.zeros(batch, dtype=torch.int32, device="cuda")
    out = torch.zeros((batch, hidden), device="cuda")
    dm.cond_embed(shape, t, y, w, out, dm.alloc_workspace(shape, dm.DIT_WS_COND))
    want = np.broadcast_to(np.where(np.arange(hidden) % 2, np.inf, -np.inf), (batch, hidden))
    assert np.array_equal(g.host(out), want)


# Small grids (one round of 64 x 32, 64 x 64, 64 x 96 or 64 x 128 tiles, k-ranges
# with the residual reduction): hidden 64 (fewer k-slices than k-groups),
# ragged rows, tiles that straddle samples, q/k padding of head_dim 72, v^T
# columns of samples that start off a four-key group, joint streams, one
# 256-row round and the first grid past it.
SMALL_GRID = [(64, 64, 1, 1, 0), (64, 64, 2, 67, 5), (192, 64, 3, 21, 0), (576, 72, 3, 85, 0), (576, 72, 2, 63, 9),
              (1152, 72, 1, 64, 0), (1152, 72, 1, 256, 0), (1152, 72, 1, 333, 0), (1152, 72, 2, 257, 0),
              (1152, 72, 3, 333, 0), (768, 64, 2, 130, 30), (256, 128, 5, 50, 0), (384, 64, 1, 700, 0)]


@pytest.mark.parametrize("hidden,dh,batch,t,tt", SMALL_GRID)
def test_small_grid_edges(hidden, dh, batch, t, tt):
    block_case(_cfg("bf16", hidden, dh, batch=batch, tokens=t, text_tokens=tt, mlp_hidden=4 * hidden))


# Steps whose residual GEMMs are split: their reductions do the LayerNorms that
# follow, the next block's and the final one after fc2 (hidden 192 and 576: one
# 4-column group per thread, 1152: two, 2304: three of four) and, where it is
# split too (hidden 2560), the one after the output projection.  `lns` of the
# five LayerNorms of two blocks and the final layer remain launches of their own.
@pytest.mark.parametrize("dtype,hidden,dh,mlp,batch,t,lns", [
    ("bf16", 192, 64, 3072, 1, 40, 3), ("bf16", 576, 72, 2304, 3, 85, 3), ("bf16", 1152, 72, 4608, 1, 200, 3),
    ("bf16", 1152, 72, 4608, 2, 77, 3), ("bf16", 2304, 72, 9216, 1, 65, 3), ("bf16", 2560, 128, 2560, 1, 17, 1),
    ("f32", 576, 72, 2304, 1, 33, 3), ("f32", 1152, 72, 4608, 2, 333, 3)])
def test_step_with_split_residuals(dtype, hidden, dh, mlp, batch, t, lns):
    import paper_2605_25550_amd as dm
    g = _gpu()
    cfg = _cfg(dtype, hidden, dh, batch=batch, tokens=t, mlp_hidden=mlp).with_(n_blocks=2, grid=None)
    sw, blocks, inp = synth.step_weights(cfg), [synth.block_weights(cfg, l) for l in range(2)], synth.inputs(cfg)
    ds = g.DeviceStep(cfg, blocks, sw)
    dm.timing_enable("ln_mod", 16)
    out, _ = ds.run(inp["patches"], inp["cond"])
    launches = dm.timing_read()[1]
    dm.timing_disable()
    assert launches == lns
    from tests.test_parity_gpu import step_ref
    ref, _ = step_ref(cfg, sw, blocks, inp, None, inp["cond"])
    check("step", out, ref, None, TOL[dtype])


# bf16 attention by grid and length: keys split over the waves (waves without
# keys, partial query blocks and key tiles, the mask inside a 16-key group,
# several tiles per wave), the four-wave kernel just past that grid, and the
# pipelined one from 64 items on.
ATT = [(64, 64, 1, 1, 0), (256, 128, 1, 31, 0), (576, 72, 1, 65, 0), (576, 72, 1, 129, 0), (576, 72, 2, 203, 6),
       (256, 64, 1, 257, 0), (256, 128, 1, 641, 0), (576, 72, 1, 1030, 0), (192, 64, 1, 2049, 0),
       (1024, 128, 5, 200, 0), (1024, 64, 9, 70, 0), (1152, 72, 3, 300, 0), (1024, 64, 4, 385, 0),
       (1024, 128, 4, 390, 25), (1152, 72, 5, 400, 0)]


@pytest.mark.parametrize("hidden,dh,batch,t,tt", ATT)
def test_attention_dispatch_edges(hidden, dh, batch, t, tt):
    block_case(_cfg("bf16", hidden, dh, batch=batch, tokens=t, text_tokens=tt))


# Patch embedding: channels in whole 16s on the matrix cores (one 16-channel
# step, a partial and several 64-channel passes, ragged rows, position table or
# none), other channel counts and misaligned latents on the other kernels.
@pytest.mark.parametrize("dtype,hidden,dh,batch,grid,p,shift", [
    ("bf16", 64, 64, 1, (1, 1), 16, 0), ("bf16", 192, 64, 3, (5, 7), 48, 0), ("f32", 128, 64, 2, (9, 15), 80, 0),
    ("bf16", 128, 128, 1, (8, 17), 256, 0), ("bf16", 192, 64, 2, (5, 9), 64, 1), ("f32", 64, 64, 1, (3, 11), 16, 1),
    ("bf16", 64, 64, 1, (6, 6), 20, 0), ("bf16", 64, 64, 2, (4, 4), 7, 0), ("bf16", 256, 64, 1, None, 64, 0)])
def test_patch_embed_edges(dtype, hidden, dh, batch, grid, p, shift):
    import paper_2605_25550_amd as dm
    g = _gpu()
    t = grid[0] * grid[1] if grid else 33
    cfg = _cfg(dtype, hidden, dh, batch=batch, tokens=t, mlp_hidden=64).with_(grid=grid, patch_in=p, patch_out=4)
    sw, blocks, inp = synth.step_weights(cfg), [synth.block_weights(cfg, 0)], synth.inputs(cfg)
    pos = O.pos_embed_2d(*grid, hidden) if grid else None
    ds = g.DeviceStep(cfg, blocks, sw)
    buf = torch.zeros(batch * t * p + 1, device="cuda")  # latents need only 4-byte alignment
    z = buf[shift:shift + batch * t * p].view(batch, t, p)
    z.copy_(g.dev(inp["patches"]))
    out = torch.empty((batch, t, 4), device="cuda")
    dm.step_forward(ds.shape, ds.table, z, g.dev(inp["cond"]), out, ds.ws)
    torch.cuda.synchronize()
    from tests.test_parity_gpu import step_ref
    ref, _ = step_ref(cfg, sw, blocks, inp, pos, inp["cond"])
    check("step", g.host(out), ref, None, TOL[dtype])


# fc2 as 256 x 128 tiles in S k-ranges over the whole problem: both streams of a
# joint block (in three ranges beside fc1's text stream in two, the tail
# schedule; in two), and one stream.  The reductions' bytes show the ranges.
@pytest.mark.parametrize("hidden,dh,f,batch,t,tt,S,tail", [(768, 64, 6144, 2, 1000, 512, 3, 2),
                                                           (1536, 64, 6144, 2, 1000, 77, 2, 0),
                                                           (1536, 128, 6144, 1, 2100, 0, 2, 0)])
def test_whole_split_edges(hidden, dh, f, batch, t, tt, S, tail):
    import paper_2605_25550_amd as dm
    dm.timing_enable("other", 16)
    block_case(_cfg("bf16", hidden, dh, batch=batch, tokens=t, text_tokens=tt, mlp_hidden=f))
    _, launches, _, nbytes = dm.timing_read()
    dm.timing_disable()
    # SiLU(c) is computed by adaLN's workgroups: the reductions are all there is
    assert launches == (2 if tt else 1) + (1 if tail else 0)
    want = sum(batch * n * hidden * (4 * S + 8) + 2 * hidden for n in (t, tt) if n)
    assert nbytes == want + (batch * tt * f * (4 * tail + 2) + 2 * f if tail else 0)


# Keys split over the waves: a wave whose only key scores -inf against every
# query (the product overflows fp32) adds nothing to the others' results.
# Tokens are Walsh patterns, which LayerNorm keeps (mean 0, variance 1): the
# last one meets the only non-zero row of W_k, the others are orthogonal to it.
@pytest.mark.parametrize("dtype,t", [("bf16", 65), ("f32", 33)])
def test_attention_wave_of_overflowed_scores(dtype, t):
    cfg = _cfg(dtype, 64, 64, batch=1, tokens=t).with_(ln_eps=1e-20)  # 1 + eps is 1 in 64 bits: exact patterns
    walsh = np.array([[(-1.0) ** bin(i & j).count("1") for i in range(64)] for j in range(64)], dtype=np.float32)
    w, inp = synth.block_weights(cfg, 0), synth.inputs(cfg)
    img = w["img"]
    img["w_ada"][:] = 0
    img["b_ada"][:] = 0
    img["b_ada"][2 * 64:3 * 64] = 1  # attention gate; the MLP's stays 0
    img["w_qkv"][:128] = 0
    img["b_qkv"][:128] = 0
    img["b_qkv"][0] = 2.0 ** 66
    img["w_qkv"][64] = walsh[1] * 2.0 ** 63
    x = walsh[2 + np.arange(t) % 62][None].copy()
    x[0, -1] = -walsh[1]
    y, _ = _gpu().run_block(cfg, w, x, inp["cond"], None)
    ref = O.dit_block(x, inp["cond"], f64(img), cfg.heads, cfg.ln_eps)
    check("img", y, ref, x, TOL[dtype])
