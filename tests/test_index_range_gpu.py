"""GPU parity at the upper end of the index ranges (operands whose byte offsets
pass 2^32, grids beyond 65536 blocks of rows) against the fp64 oracle, on the
rows and weights that lie there.  Metric and fp32 bar as in
test_dispatch_edges_gpu.py."""
import numpy as np
import pytest
import torch

import synth
from oracle import dit_oracle as O
from tests.test_parity_gpu import _gpu, check, f64

pytestmark = pytest.mark.gpu


def _cfg(**kw):
    return synth.CONFIGS["c1"].with_(dtype="f32", hidden=64, heads=1, head_dim=64, cond="given", n_blocks=1, **kw)


def test_f32_rows_past_four_gib():
    """fc2's operand has 262400 rows of 16 KB; the last four samples (rows from
    2^32 bytes on) must come out as when they are run alone."""
    import paper_2605_25550_amd as dm
    cfg = _cfg(batch=4100, tokens=64, mlp_hidden=4096)
    assert (cfg.batch - 4) * cfg.tokens * cfg.mlp_hidden * 4 == 1 << 32
    g = _gpu()
    w = synth.block_weights(cfg, 0)
    db = g.DeviceBlock(cfg, w)
    rng = np.random.default_rng(5)
    x = rng.standard_normal((cfg.batch, cfg.tokens, cfg.hidden), dtype=np.float32)
    c = rng.standard_normal((cfg.batch, cfg.hidden), dtype=np.float32)
    xd = g.dev(x)
    dm.block_forward(db.shape, db.struct, xd, g.dev(c), dm.alloc_workspace(db.shape, dm.DIT_WS_BLOCK))
    y = g.host(xd[-5:])
    ref = O.dit_block(x[-5:], c[-5:], f64(w["img"]), cfg.heads, cfg.ln_eps)
    check("img", y, ref, x[-5:], 2e-5)


def test_f32_weights_past_four_gib():
    """MLP matrices of 4.06 GiB of which only the last 320 hidden columns
    are not zero: fc1's weight rows for them lie past 2^32 bytes, as does fc2's
    last row; the oracle has those columns as its whole MLP."""
    import paper_2605_25550_amd as dm
    F, D, live = 17043584, 64, 320
    assert (F - live) * D * 4 >= 1 << 32 and (D - 1) * F * 4 >= 1 << 32
    cfg = _cfg(batch=1, tokens=2, mlp_hidden=live)
    g = _gpu()
    w, inp = synth.block_weights(cfg, 0), synth.inputs(cfg)
    db = g.DeviceBlock(cfg, w)
    big = {"w_fc1": torch.zeros(F, D, device="cuda"), "b_fc1": torch.zeros(F, device="cuda"),
           "w_fc2": torch.zeros(D, F, device="cuda")}
    for k in ("w_fc1", "b_fc1"):
        big[k][-live:] = db.img[k]
    big["w_fc2"][:, -live:] = db.img["w_fc2"]
    img = dict(db.img, **big)
    shape = dm.shape_of(cfg.with_(mlp_hidden=F))
    x = g.dev(inp["x"])
    dm.block_forward(shape, dm.block_struct(img, None, db.dt), x, g.dev(inp["cond"]),
                     dm.alloc_workspace(shape, dm.DIT_WS_BLOCK))
    ref = O.dit_block(inp["x"], inp["cond"], f64(w["img"]), cfg.heads, cfg.ln_eps)
    check("img", g.host(x), ref, inp["x"], 2e-5)


def test_patch_embed_of_nine_million_rows():
    """16 channels, more than 65536 blocks of 128 rows: the last sample of a step
    against the oracle."""
    import paper_2605_25550_amd as dm
    from tests.test_parity_gpu import TOL, step_ref
    cfg = _cfg(batch=8200, tokens=1024, mlp_hidden=64).with_(dtype="bf16", grid=None, patch_in=16, patch_out=4)
    assert cfg.batch * cfg.tokens > 65536 * 128
    g = _gpu()
    sw, blocks, inp = synth.step_weights(cfg), [synth.block_weights(cfg, 0)], synth.inputs(cfg.with_(batch=1))
    ds = g.DeviceStep(cfg, blocks, sw)
    z = torch.zeros(cfg.batch, cfg.tokens, 16, device="cuda")
    c = torch.zeros(cfg.batch, cfg.hidden, device="cuda")
    z[-1], c[-1] = g.dev(inp["patches"])[0], g.dev(inp["cond"])[0]
    out = torch.empty(cfg.batch, cfg.tokens, 4, device="cuda")
    dm.step_forward(ds.shape, ds.table, z, c, out, ds.ws)
    ref, _ = step_ref(cfg, sw, blocks, inp, None, inp["cond"])
    check("step", g.host(out[-1:]), ref, None, TOL["bf16"])
