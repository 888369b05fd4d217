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
# samples <= 16) and read back, fp32 samples beyond one 64 KB staging pass
# (15 x 1156 floats), joint blocks (two matrices).
ADA = [("bf16", 64, 64, 1, 0), ("bf16", 192, 64, 3, 0), ("bf16", 192, 64, 8, 2), ("bf16", 320, 64, 9, 3),
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
