"""bf16 GEMMs with 64- and 128-row tiles and an asynchronous operand ring (mfma_gemm.hip), through the encoder layer's
training step: every epilogue (bias, score scale, residual, GELU with its pre-activation, GELU'), both weight layouts, the
contraction split over three weights, at the edges of the tiles and of the 64-deep k-tiles."""
import pytest
import torch

import oracle
from paper_2505_01068_amd import binding as B, synth
from tests.gpu_util import TOL, assert_close, to_dev
from tests.test_gpu_layer_backward import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,H,d_ff,batch,seg", [
    (64, 8, 256, 1, (1, 2, 1)),           # 4 rows, one k-tile
    (192, 3, 192, 1, (20, 30, 13)),       # 63 rows; a 128-column tile meets two of the three weights
    (192, 3, 200, 1, (20, 30, 15)),       # 65 rows; 200 columns, and a contraction of 200 that the ring does not take
    (320, 5, 128, 1, (40, 50, 39)),       # 129 rows
    (256, 4, 1024, 2, (70, 33, 25)),      # 256 rows
    (128, 2, 4096, 1, (512, 700, 325)),   # 1537 rows x 32 column tiles: 128-row tiles, the last with one row
    (256, 4, 1056, 1, (20, 30, 15)),      # contractions that end in half a k-tile: 16 and a half,
    (192, 3, 96, 2, (70, 33, 26)),        # one and a half,
    (288, 32, 160, 1, (40, 50, 39)),      # and the GELU product's four and a half
])
def test_layer_training_step(d, H, d_ff, batch, seg):
    print(f"[case] ring GEMM d={d} d_ff={d_ff} rows={batch * sum(seg)}", flush=True)
    g = synth.attention_inputs(batch, seg, d, H, "bf16", "valid_len", seed=901)
    p = synth.layer_params(d, d_ff, 901, 0, dtype="bf16")
    check(g, p, oracle.IM_IFM_FORWARD, "bf16", d_ff, f"ring/d={d}/f={d_ff}/rows={batch * sum(seg)}")


@pytest.mark.parametrize("batch", [170, 171])   # 25 500 and 25 650 rows x 2 column tiles: 128-row tiles, the last with 28 / 50 rows
def test_half_k_tile_of_128_row_tiles(batch):
    d, H, d_ff, seg = 256, 4, 1056, (50, 50, 50)
    print(f"[case] ring GEMM, half a k-tile, rows={batch * sum(seg)}", flush=True)
    g = synth.attention_inputs(batch, seg, d, H, "bf16", "none", seed=911, with_dy=False)
    p = synth.layer_params(d, d_ff, 911, 0, dtype="bf16")
    shape = B.make_shape(batch, seg, d, H, oracle.IM_IFM_FORWARD, g["scale"], "bf16")
    ws = torch.empty(B.gsit_layer_sizes(shape, d_ff), dtype=torch.uint8, device="cuda")
    y = B.gsit_layer_fwd(shape, d_ff, to_dev(g["x"], "bf16"), {k: to_dev(v, "bf16") for k, v in p.items()}, workspace=ws)
    some = [0, 84, batch - 2, batch - 1]
    ref = oracle.gsit_layer_forward(g["x"][some], p, seg, oracle.IM_IFM_FORWARD, H, g["scale"])
    assert_close(y[some], ref, TOL["bf16"], "y")
