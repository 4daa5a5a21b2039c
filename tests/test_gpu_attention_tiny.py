"""fp32 inference of the smallest calls (one launch, projections included) and of those just beyond its lines, against the fp64
oracle at the fp32 bar."""
import numpy as np
import pytest
import torch

import oracle
from paper_2505_01068_amd import binding as B, synth
from tests.gpu_util import PackedProblem, Problem, assert_close, TOL

pytestmark = pytest.mark.gpu


# keys of a query segment: 40 and 41 (one launch, three), one row per segment, ragged 8-row tiles; widths 32 and 33, odd head
# dimensions, head dimensions 1 and 16
@pytest.mark.parametrize("seg,d,H", [((1, 1, 1), 4, 1), ((8, 8, 8), 32, 4), ((7, 24, 9), 30, 5), ((10, 30, 10), 32, 2), ((10, 30, 11), 32, 2),
                                     ((9, 17, 14), 32, 32), ((9, 10, 11), 33, 3), ((40,), 32, 8), ((41,), 32, 8), ((5, 6, 7, 8), 26, 2)])
@pytest.mark.parametrize("padding", ["none", "valid_len", "key_pad"])
def test_tiny_inference(seg, d, H, padding):
    print(f"[case] tiny seg={seg} d={d} H={H} {padding}", flush=True)
    n = len(seg)
    for bias in (False, True):
        g = synth.attention_inputs(3, seg, d, H, "fp32", padding, seed=d + n, bias=bias)
        for lm in ((1 << (n * n)) - 1, sum(1 << (i * n + (i + 1) % n) for i in range(n)), 1 << (n * n - 1)):   # the last: dead query segments
            p = Problem(g, lm)
            y = p.fwd(save=False)
            torch.cuda.synchronize()
            assert_close(y, p.oracle_fwd(), TOL["fp32"], f"{seg} {d} {H} {padding} {lm:#x}")


def test_tiny_packed():
    print("[case] tiny packed", flush=True)
    seg, lengths = (10, 20, 17), [[10, 3, 17], [1, 20, 5], [4, 0, 9]]
    g = synth.attention_inputs(3, seg, 32, 4, "fp32", "none", seed=9, bias=True)
    p = PackedProblem(g, oracle.IM_IFM_FORWARD, lengths)
    y = p.fwd(save=False)
    torch.cuda.synchronize()
    ref = oracle.forward(g["x"], g["wq"], g["wk"], g["wv"], g["wo"], seg, oracle.IM_IFM_FORWARD, 4, g["scale"], bq=g["bq"], bk=g["bk"],
                         bv=g["bv"], bo=g["bo"], valid_len=np.asarray(lengths))
    assert_close(y, synth.pack_rows(ref, p.lengths, seg), TOL["fp32"], "packed")


def test_tiny_output_over_input_and_large_scores():
    # y = x takes the three launches, whose last one alone writes y; scores around 300 and a masked key's left-over contents
    print("[case] tiny in place, large scores", flush=True)
    g = synth.attention_inputs(2, (8, 9, 10), 32, 4, "fp32", "key_pad", seed=4, bias=True)
    g["wq"] = g["wq"] * 30.0
    p = Problem(g, oracle.IM_DENSE)
    y = p.fwd(save=False)
    x = p.t["x"].clone()
    B.im_attention_fwd(p.shape, x, *(p.t[n] for n in ("wq", "wk", "wv", "wo", "bq", "bk", "bv", "bo")), p.t["valid_len"], p.t["key_pad"], y=x,
                       saved=None, workspace=p.ws)
    torch.cuda.synchronize()
    ref = p.oracle_fwd()
    assert_close(y, ref, 1e-4, "large scores")   # a score of 300 carries 300 * 2^-24 * sqrt(32) = 1e-4 into the exponent
    assert_close(x, ref, 1e-4, "in place")
    h = dict(g, x=np.where(g["key_pad"][:, :, None] != 0, np.float32(3e30), g["x"]))
    z = Problem(h, oracle.IM_DENSE).fwd(save=False)
    torch.cuda.synchronize()
    valid = torch.from_numpy(g["key_pad"] == 0).cuda()
    assert torch.equal(z[valid], y[valid])


@pytest.mark.parametrize("name", ["wq", "wk", "wv", "wo"])
@pytest.mark.parametrize("d,H", [(4, 1), (26, 2), (30, 5), (32, 4)])
def test_tiny_infinite_weights(d, H, name):
    # An infinite element in a weight's last row makes the same infinities and NaN as in the three launches (which a call with
    # saved takes), at widths that fill the kernel's 32 columns and at others.
    print(f"[case] tiny infinity in {name} d={d}", flush=True)
    g = synth.attention_inputs(2, (8, 9, 10), d, H, "fp32", "none", seed=6, bias=True)
    g["x"][:, :, d - 1] = np.abs(g["x"][:, :, d - 1]) + np.float32(0.1)   # infinities of one sign
    g[name] = g[name].copy()
    g[name][d - 1, d // 2] = np.inf
    p = Problem(g, oracle.IM_IFM_FORWARD)
    y, z = p.fwd(save=False), p.fwd(save=True)
    torch.cuda.synchronize()
    for kind in (torch.isnan, torch.isposinf, torch.isneginf):
        assert torch.equal(kind(y), kind(z)), kind.__name__
    fin = z.isfinite()
    if name in ("wv", "wo"):
        assert not z.isnan().all() and z.isinf().any()
    if fin.any():
        assert (y[fin] - z[fin]).abs().max() <= TOL["fp32"] * z[fin].abs().max()
