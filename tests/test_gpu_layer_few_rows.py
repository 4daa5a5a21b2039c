"""Encoder layer forward (bf16, d = 64 and 128) on both sides of the lines between the kernels for few rows -- one of Q, K, V per
workgroup, eight waves per layer tail -- and those for many."""
import numpy as np
import pytest
import torch

import oracle
from paper_2505_01068_amd import binding as B, synth
from tests.gpu_util import assert_close, to_dev, TOL

pytestmark = pytest.mark.gpu


def forward(g, p, d_ff, H, live):
    x = to_dev(g["x"], "bf16")
    shape = B.make_shape(x.shape[0], g["seg_len"], x.shape[2], H, live, g["scale"], "bf16")
    ws = torch.empty(B.gsit_layer_sizes(shape, d_ff), dtype=torch.uint8, device="cuda")
    y = torch.empty_like(x)
    B.gsit_layer_fwd(shape, d_ff, x, {k: to_dev(v, "bf16") for k, v in p.items()}, y=y, workspace=ws)
    torch.cuda.synchronize()
    return y


# hidden widths that end in half a 128-column chunk, in the first one already, and whole ones; rows off the 64- and 128-row tiles
@pytest.mark.parametrize("d,H,d_ff", [(128, 8, 64), (128, 8, 192), (128, 16, 512), (64, 8, 64), (64, 8, 192)])
@pytest.mark.parametrize("seg", [(1, 2, 1), (30, 67, 40)])
def test_few_rows(d, H, d_ff, seg):
    print(f"[case] few rows d={d} d_ff={d_ff} seg={seg}", flush=True)
    g = synth.attention_inputs(2, seg, d, H, "bf16", "none", seed=3, with_dy=False)
    p = synth.layer_params(d, d_ff, 3, 0, dtype="bf16")
    y = forward(g, p, d_ff, H, oracle.IM_IFM_FORWARD)
    ref = oracle.gsit_layer_forward(g["x"], p, seg, oracle.IM_IFM_FORWARD, H, g["scale"])
    assert_close(y, ref, TOL["bf16"], f"d={d} d_ff={d_ff}")


# 8 samples (816 rows) are few; on 256 CUs the layer tail's line is at 16384 rows (20.1 copies), the projection's at 8192 (10.04).
# The samples' results differ by the order of fp32 sums and by bf16 roundings behind them.
@pytest.mark.parametrize("d,H,repeat", [(128, 8, 19), (128, 8, 21), (64, 8, 7), (64, 8, 21)])
def test_both_sides_agree(d, H, repeat):
    print(f"[case] both sides d={d} repeat={repeat}", flush=True)
    seg, d_ff = (20, 50, 32), 4 * d
    g = synth.attention_inputs(8, seg, d, H, "bf16", "none", seed=5, with_dy=False)
    p = synth.layer_params(d, d_ff, 5, 0, dtype="bf16")
    few = forward(g, p, d_ff, H, oracle.IM_IEM)
    many = forward(dict(g, x=np.tile(g["x"], (repeat, 1, 1))), p, d_ff, H,
                   oracle.IM_IEM).view(repeat, 8, sum(seg), d)
    for i in (0, repeat - 1):
        assert_close(many[i], few.float().cpu().numpy(), TOL["bf16"], f"copy {i}")
