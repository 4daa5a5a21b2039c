"""fp32 calls whose rows hold extreme values.  The products of these calls run on the bf16 matrix cores, each operand as three
bf16 parts; the results are what fp32 multiply-adds give (a masked key has weight exactly zero, whatever its row holds)."""
import numpy as np
import pytest

import oracle
from paper_2505_01068_amd import synth
from tests.gpu_util import TOL, Problem, assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dh", [4, 5, 7, 12, 16])
def test_contents_of_masked_keys_do_not_matter(dh):
    # a masked key whose row holds 3e35 (left-over memory).  As a query the row is computed like any other; every other row's
    # y is that of a harmless row.
    print(f"[case] masked keys dh={dh}", flush=True)
    d, H, seg, rows = 3 * dh, 3, (20, 70, 40), [50]
    g = synth.attention_inputs(2, seg, d, H, "fp32", "none", seed=1004, bias=True)
    g["key_pad"] = np.zeros((2, sum(seg)), np.uint8)
    g["key_pad"][:, rows] = 1
    y = []
    for value in (0.0, 3e35):
        pr = Problem(g, oracle.NAMED_PATTERNS["self_only"])
        pr.t["x"][:, rows] = value
        y.append(pr.fwd())
    keep = [i for i in range(sum(seg)) if i not in rows]
    assert_close(y[1][:, keep], y[0][:, keep].double().cpu().numpy(), TOL["fp32"], "y")
