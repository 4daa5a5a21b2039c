"""Small-head attention in fp32 arithmetic on the bf16 matrix cores: every head dimension the kernels are instantiated or
padded for, the edges of the 16-row blocks, 32-row steps and 64-row tiles, and the moving softmax reference."""
import numpy as np
import pytest
import torch

import oracle
from paper_2505_01068_amd import binding as B, synth
from tests.gpu_util import TOL, Problem, assert_close

pytestmark = pytest.mark.gpu


def say(msg):
    print(msg, flush=True)


@pytest.mark.parametrize("dh", range(1, 17))
def test_every_head_dimension(dh):
    # one, two and four k-steps of the score product; one to four row blocks of the transposed operand
    say(f"[case] split attention dh={dh}")
    g = synth.attention_inputs(2, (17, 65, 33), 3 * dh, 3, "fp32", "valid_len", seed=700 + dh, bias=True)
    Problem(g, oracle.NAMED_PATTERNS["self_only"]).check(what=f"split/dh{dh}")


@pytest.mark.parametrize("seg", [(1, 15, 16), (17, 31, 32), (33, 63, 64), (65, 127, 128), (129, 1, 2)])
@pytest.mark.parametrize("padding", ["none", "key_pad"])
def test_block_step_and_tile_edges(seg, padding):
    say(f"[case] split attention seg={seg} padding={padding}")
    g = synth.attention_inputs(3, seg, 40, 8, "fp32", padding, seed=731)
    for name in ("ifm_forward", "ifm_backward", "dense"):
        Problem(g, oracle.NAMED_PATTERNS[name]).check(what=f"split/{seg}/{name}")


def test_rows_and_samples_without_a_valid_key():
    say("[case] split attention, no valid key")
    g = synth.attention_inputs(3, (20, 70, 40), 40, 8, "fp32", "valid_len", seed=741)
    g["valid_len"][0, :] = 0            # no key at all
    g["valid_len"][1, 1] = 0            # one segment's keys missing
    g["key_pad"] = np.zeros((3, 130), dtype=np.uint8)
    g["key_pad"][2, 20:52] = 1          # the first 32-row step of a segment masked: the reference comes later
    for name in ("ifm_forward", "dense"):
        Problem(g, oracle.NAMED_PATTERNS[name]).check(what=f"split/no-key/{name}")


def test_moving_reference():
    # scores that grow along the keys move the softmax reference in many steps.  |scores| reach 40 in the exponent of 2,
    # where one fp32 rounding of a score is 2.4e-6 of its probability; the bar of 1e-5 of the largest element stays.
    say("[case] split attention, growing scores")
    g = synth.attention_inputs(2, (40, 200, 130), 40, 8, "fp32", "none", seed=751)
    for s0, n in ((0, 40), (40, 200), (240, 130)):
        g["x"][:, s0:s0 + n] *= np.linspace(0.05, 3.0, n, dtype=np.float32)[None, :, None]
    Problem(g, oracle.IM_IFM_FORWARD).check(what="split/growing")


def test_bias_gradients_collect_no_rounding():
    # dbq and dbv add dQ and dV over 19 600 rows.  A rounding to nearest per row is 6e-8 times the square root of the number
    # of rows against a sum that grows the same way: the 2-norm error stays a few 1e-7.  A rounding with one sign grows with
    # the number of rows itself; the bar of 1.4e-6 lies between (measured 4.7e-7 and 2.4e-6 at this shape).
    say("[case] split attention, bias gradients of many rows")
    seg, d, H, batch = (39, 480, 461), 32, 4, 20
    g = synth.attention_inputs(batch, seg, d, H, "fp32", "valid_len", seed=761, bias=True)
    pr = Problem(g, oracle.NAMED_PATTERNS["structure3_a"])
    pr.fwd()
    grads = pr.bwd()
    ref = {"dbq": 0.0, "dbv": 0.0}
    for b0 in range(0, batch, 4):   # the dense oracle walks the batch four elements at a time
        sl = slice(b0, b0 + 4)
        _, cache = oracle.forward(g["x"][sl], g["wq"], g["wk"], g["wv"], g["wo"], seg, pr.lm, H, g["scale"], bq=g["bq"], bk=g["bk"],
                                  bv=g["bv"], bo=g["bo"], valid_len=g["valid_len"][sl], return_cache=True)
        part = oracle.backward(cache, g["dy"][sl])
        for k in ref:
            ref[k] = ref[k] + part[k]
    for k, r in ref.items():
        err = np.linalg.norm(grads[k].double().cpu().numpy() - r) / np.linalg.norm(r)
        say(f"    {k} {err:.1e}")
        assert err < 1.4e-6, (k, err)


def test_bias_gradients_collect_no_rounding_in_short_segments():
    # segments of at most 32 rows: one step of the dV product per key, so that only other keys' steps can turn the rounding
    # around.  fp32 multiply-adds give 2.4e-7 in the mean over inputs, a rounding with one sign 3.2e-7: over the 24 inputs of
    # 64 columns the mean scatters by 2 per cent, and 2.8e-7 lies between.
    say("[case] split attention, bias gradients of short segments")
    seg, d, H, batch, total = (10, 30, 25), 64, 8, 200, 0.0
    for seed in range(24):
        g = synth.attention_inputs(batch, seg, d, H, "fp32", "valid_len", seed=1800 + seed, bias=True)
        pr = Problem(g, oracle.NAMED_PATTERNS["structure2_b"])
        pr.fwd()
        _, cache = pr.oracle_fwd(cache=True)
        ref = oracle.backward(cache, g["dy"])["dbv"]
        total += (np.linalg.norm(pr.bwd()["dbv"].double().cpu().numpy() - ref) / np.linalg.norm(ref)) ** 2
    err = (total / 24) ** 0.5
    say(f"    dbv {err:.2e}")
    assert err < 2.8e-7, err


def test_zero_scores_before_the_first_large_one():
    # Leading zero rows without a mask and without a key bias: the first 32 keys of every segment give exactly zero scores, of
    # either sign of zero.  They enter the sum with weight one and must be rescaled when the large scores behind them arrive.
    say("[case] split attention, leading zero keys")
    g = synth.attention_inputs(2, (80, 100, 70), 40, 8, "fp32", "none", seed=771)
    for s0 in (0, 80, 180):
        g["x"][:, s0:s0 + 32] = 0
        g["x"][:, s0 + 32:s0 + 70] *= 3
    for name in ("ifm_forward", "ifm_backward", "dense"):
        Problem(g, oracle.NAMED_PATTERNS[name]).check(what=f"split/zero-keys/{name}")


def test_more_pairs_than_one_grid_holds():
    # 65 535 x 257 (batch element, head) pairs are 2^32 threads and more; the last batch elements in the last launch
    say("[case] split attention, 16.8 million pairs")
    batch, few, d, seg = 65535, 5, 257, (1, 1, 1)
    g = synth.attention_inputs(few, seg, d, d, "fp32", "none", seed=781, with_dy=False)
    w = {k: torch.from_numpy(g[k]).cuda() for k in ("wq", "wk", "wv", "wo")}
    x = torch.from_numpy(g["x"]).cuda()
    out = []
    for n in (few, batch):
        xs = x.repeat(n // few, 1, 1)
        shape = B.make_shape(n, seg, d, d, oracle.IM_IFM_FORWARD, g["scale"], "fp32")
        ws = torch.empty(B.im_attention_sizes(shape)[1], dtype=torch.uint8, device="cuda")
        out.append(B.im_attention_fwd(shape, xs, **w, workspace=ws))
    torch.cuda.synchronize()
    assert_close(out[0], oracle.forward(g["x"], *(g[k] for k in ("wq", "wk", "wv", "wo")), seg, oracle.IM_IFM_FORWARD, d, g["scale"]),
                 TOL["fp32"], "y")
    assert torch.equal(out[1].view(batch // few, few, 3, d), out[0].expand(batch // few, few, 3, d))
