"""bf16 matrix-core attention at head dimension 64 on both sides of the line between 128-row tiles and 64-row tiles whose stages
are split between two waves, and where the workgroups are dealt out evenly, and tile edges at all head dimensions: against the
fp64 oracle, forward and backward."""
import pytest

import oracle
from paper_2505_01068_amd import synth
from tests.gpu_util import Problem

pytestmark = pytest.mark.gpu


# 4 tiles of 128 rows x 4 heads per sample: 384 workgroups at 24 samples, the last split size on 256 CUs; 400 at 25; 21 samples of
# 3 heads and 23 of 4 give (sample, head) pairs that do not divide over the 8 XCDs
@pytest.mark.parametrize("batch", [21, 23, 24, 25])
@pytest.mark.parametrize("name,padding", [("ifm_forward", "valid_len"), ("self_only", "key_pad"), ("dense", "none")])
def test_split_line(batch, name, padding):
    print(f"[case] split line batch={batch} {name} {padding}", flush=True)
    H = 3 if batch == 21 else 4
    g = synth.attention_inputs(batch, (130, 33, 65), 64 * H, H, "bf16", padding, seed=batch, bias=True)
    Problem(g, oracle.NAMED_PATTERNS[name]).check(what=f"{name}/{padding}/{batch}")


# one sample, 64 columns: lengths around the 64-row tile, the 32-row blocks of a stage and a stage's second half
@pytest.mark.parametrize("seg", [(63, 64, 65), (1, 32, 33), (96, 97, 31), (129, 160, 2)])
@pytest.mark.parametrize("padding", ["none", "valid_len", "key_pad"])
@pytest.mark.parametrize("H", [1, 4, 8])   # of 64, 16 and 8 columns: 4 and 8 run the sub-head kernels (32- and 64-row tiles)
def test_tile_edges(seg, padding, H):
    print(f"[case] tile edges seg={seg} H={H} {padding}", flush=True)
    g = synth.attention_inputs(1, seg, 64, H, "bf16", padding, seed=sum(seg))
    for name in ("ifm_backward", "self_only"):
        Problem(g, oracle.NAMED_PATTERNS[name]).check(what=f"{name}/{seg}/{padding}")
