"""LayerNorm forward and backward in 16-byte pieces with the gain and bias gradients summed beside it, through the encoder
layer's training step: lanes per row 8 to 64 with and without idle ones, rows around the 64-row blocks."""
import pytest

import oracle
from paper_2505_01068_amd import synth
from tests.test_gpu_layer_backward import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,H", [("fp32", 8, 2), ("fp32", 36, 4), ("fp32", 64, 8), ("fp32", 132, 12), ("fp32", 256, 16),
                                       ("bf16", 40, 8), ("bf16", 128, 2), ("bf16", 192, 3), ("bf16", 512, 8)])
@pytest.mark.parametrize("seg", [(1, 1, 1), (20, 30, 13), (20, 30, 14), (60, 50, 19)])   # 3, 63, 64 and 129 rows
def test_layer_training_step(dtype, d, H, seg):
    print(f"[case] LayerNorm {dtype} d={d} rows={sum(seg)}", flush=True)
    g = synth.attention_inputs(1, seg, d, H, dtype, "none", seed=941)
    p = synth.layer_params(d, 2 * d, 941, 0, dtype=dtype)
    check(g, p, oracle.IM_IFM_FORWARD, dtype, 2 * d, f"layernorm/{dtype}/d={d}/rows={sum(seg)}")
