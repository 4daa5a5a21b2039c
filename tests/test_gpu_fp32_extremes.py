"""fp32 calls whose rows hold extreme values.  The products of these calls run on the bf16 matrix cores, each operand as three
bf16 parts, which infinities and values beyond bf16's largest do not have; the results are what fp32 multiply-adds give (an
infinity stays one; a masked key has weight exactly zero, whatever its row holds)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2505_01068_amd import synth
from tests.gpu_util import TOL, PackedProblem, Problem, assert_close

pytestmark = pytest.mark.gpu
TOP = 3.4e38   # finite in fp32, rounds to infinity in bf16


def same(got, want, what):
    """NaN, +inf and -inf where `want` (fp32, CPU) has them; elsewhere within the fp32 bar."""
    got, want = got.cpu(), want.float()
    assert torch.equal(got.isnan(), want.isnan()), what
    assert torch.equal(got.isposinf(), want.isposinf()) and torch.equal(got.isneginf(), want.isneginf()), what
    fin = want.isfinite()
    assert (got[fin] - want[fin]).abs().max() <= TOL["fp32"] * want[fin].abs().max(), what


@pytest.mark.parametrize("d,H", [(40, 8), (33, 3), (32, 2)])
def test_infinities_in_weights_and_upstream_gradients(d, H):
    # y = O Wo + bo, dWo = O^T dy, dbo = sum of dy rows: an infinite element of Wo or dy makes infinities of one sign per
    # element of O, everything else stays finite.  dV, hence dbv, is infinite for the heads' columns that the row's keys feed.
    print(f"[case] infinities d={d}", flush=True)
    g = synth.attention_inputs(2, (20, 70, 40), d, H, "fp32", "none", seed=1001, bias=True)
    ref_y, cache = oracle.forward(g["x"], g["wq"], g["wk"], g["wv"], g["wo"], g["seg_len"], oracle.IM_IFM_FORWARD, H, g["scale"],
                                  bq=g["bq"], bk=g["bk"], bv=g["bv"], bo=g["bo"], return_cache=True)
    o = torch.from_numpy(np.ascontiguousarray(cache["o"])).reshape(-1, d)
    pr = Problem(g, oracle.IM_IFM_FORWARD)
    pr.t["wo"][3, 5] = float("inf")
    wo = pr.t["wo"].cpu().double()
    same(pr.fwd().reshape(-1, d), (o @ torch.nan_to_num(wo, posinf=0.0)) + torch.from_numpy(g["bo"]).double()
         + torch.where(torch.arange(d) == 5, o[:, 3:4] * float("inf"), torch.zeros(())), "y")
    pr = Problem(g, oracle.IM_IFM_FORWARD)
    pr.fwd()
    dy = torch.from_numpy(g["dy"]).double().reshape(-1, d)
    dy[90, 7], dy[11, 2] = float("-inf"), TOP
    pr.t["dy"].copy_(dy.float().reshape(pr.t["dy"].shape))
    grads = pr.bwd()
    fin = dy.clone()
    fin[90, 7] = 0
    want = o.t() @ fin
    want[:, 7] = -o[90] * float("inf")
    same(grads["dwo"], want, "dwo")
    want_b = fin.sum(0)
    want_b[7] = float("-inf")
    same(grads["dbo"], want_b, "dbo")
    assert grads["dbv"].isinf().all()   # row 90 attends every key of its key segment with a positive weight


@pytest.mark.parametrize("d,H", [(40, 8), (32, 2), (16, 16)])
def test_finite_values_beyond_the_bf16_range(d, H):
    # one element of x at the end of the fp32 range, weights small enough that every result is finite
    print(f"[case] huge operands d={d}", flush=True)
    g = synth.attention_inputs(2, (20, 70, 40), d, H, "fp32", "none", seed=1002, bias=True)
    g["x"][1, 30, 3] = TOP
    for n in ("wq", "wk", "wv"):
        g[n] = (g[n] * np.float32(2e-38)).astype(np.float32)
    g["dy"] = (g["dy"] * np.float32(1e-3)).astype(np.float32)
    pr = Problem(g, oracle.NAMED_PATTERNS["self_only"])
    y_ref, cache = pr.oracle_fwd(cache=True)
    y = pr.fwd()
    grads = pr.bwd()
    ref = oracle.backward(cache, g["dy"])
    assert_close(y, y_ref, TOL["fp32"], "y")
    for n in ("dwv", "dwo", "dbv", "dbo"):   # (dWq and dWk multiply the rounding of a small dQ, dK by 3.4e38)
        assert_close(grads[n], ref[n], TOL["fp32"], n)
    for n in ("dwq", "dwk", "dx"):
        assert grads[n].isfinite().all(), n


@pytest.mark.parametrize("dh", [5, 8, 16])
@pytest.mark.parametrize("size", [1e3, 1e5, 1e17])
def test_scores_far_apart(dh, size):
    # scores of 1e6, 1e10 and 1e34: a row attends one key.  exp2(score - lse) of that key is one, not the difference of two
    # roundings of the score; dWq and dWk, rounding noise times such keys, are finite.
    print(f"[case] scores far apart dh={dh} size={size}", flush=True)
    d, H = 4 * dh, 4
    g = synth.attention_inputs(2, (40, 100, 30), d, H, "fp32", "valid_len", seed=1005)
    for w in ("wq", "wk"):
        g[w] = (g[w] * np.float32(size)).astype(np.float32)
    pr = Problem(g, oracle.IM_IFM_FORWARD)
    y_ref, cache = pr.oracle_fwd(cache=True)
    close = lambda got, ref, what: assert_close(got, ref, 5e-3, what)  # noqa: E731  (near ties: weights of single rows)
    close(pr.fwd(), y_ref, "y")
    grads, ref = pr.bwd(), oracle.backward(cache, g["dy"])
    for name in ("dwo", "dwv"):
        close(grads[name], ref[name], name)
    assert all(grads[n].isfinite().all() for n in ("dwq", "dwk"))


@pytest.mark.parametrize("size", [3, 10, 30])
def test_probabilities_of_the_backward_are_those_of_the_forward(size):
    # scores around 30, 300 and 3000 (in the exponent of 2).  A score s has an error of 2^-24 s from its own rounding, and so
    # have single probabilities; but a row's probabilities sum to one, and where one key takes the row its weight is exactly
    # one.  dWv over many rows is good to the rounding of lse: 1.6e-8 x 30 .. 3000, with the 4e-7 of an ordinary call
    # (measured 7e-7, 3.0e-6 and 8e-6).  Two roundings of the score that differ: 1.2e-6, 1.1e-5, 9.5e-5.
    print(f"[case] large scores size={size}", flush=True)
    g = synth.attention_inputs(8, (50, 200, 150), 40, 8, "fp32", "valid_len", seed=1006)
    for w in ("wq", "wk"):
        g[w] = (g[w] * np.float32(size)).astype(np.float32)
    pr = Problem(g, oracle.IM_IFM_FORWARD)
    pr.fwd()
    _, cache = pr.oracle_fwd(cache=True)
    ref = oracle.backward(cache, g["dy"])["dwv"]
    err = np.linalg.norm(pr.bwd()["dwv"].double().cpu().numpy() - ref) / np.linalg.norm(ref)
    print(f"    {err:.1e}")
    assert err <= {3: 1.0e-6, 10: 5e-6, 30: 2e-5}[size], err


def test_scores_of_minus_infinity():
    # head dimension 1: keys of -3.4e38 (beyond bf16's largest value) times a query overflow to -inf, a weight of zero
    print("[case] scores of minus infinity", flush=True)
    n, seg, d = 1, (70, 70, 33), 4
    g = synth.attention_inputs(n, seg, d, d, "fp32", "none", seed=1003)
    g["x"] = (1.5 + np.random.default_rng(3).random(g["x"].shape)).astype(np.float32)
    g["x"][:, 5::9, 1] = -1.7e38                    # the key feature: K = 2 x_1
    g["x"][:, 5::9, 0] = 2.0
    for w, c, v in (("wq", 0, 1.0), ("wk", 1, 2.0), ("wv", 2, np.linspace(0.5, 1.5, d))):
        g[w] = np.zeros((d, d), np.float32)
        g[w][c] = v
    g["dy"] = (g["dy"] * np.float32(1e-3)).astype(np.float32)
    pr = Problem(g, oracle.NAMED_PATTERNS["self_only"])
    y_ref, cache = pr.oracle_fwd(cache=True)        # fp64: the scores are -1e39, their weights zero
    assert_close(pr.fwd(), y_ref, TOL["fp32"], "y")
    grads, ref = pr.bwd(), oracle.backward(cache, g["dy"])
    for name in ("dwo", "dwv"):
        assert_close(grads[name], ref[name], TOL["fp32"], name)


@pytest.mark.parametrize("dh", [4, 5, 7, 12, 16])
@pytest.mark.parametrize("rows", [(50,), (4, 50, 111)])
def test_contents_of_masked_keys_do_not_matter(dh, rows):
    # masked keys whose rows hold 3e35 (left-over memory); with several, the rows attend one another's products of 1e70.  As a
    # query a masked row is computed like any other; every other row's y and dx, and what the rows give as keys (dV = dK = 0:
    # dWv, dbv, dbk), are those of harmless rows.
    print(f"[case] masked keys dh={dh} rows={rows}", flush=True)
    d, H, seg, rows = 3 * dh, 3, (20, 70, 40), list(rows)
    g = synth.attention_inputs(2, seg, d, H, "fp32", "none", seed=1004, bias=True)
    g["key_pad"] = np.zeros((2, sum(seg)), np.uint8)
    g["key_pad"][:, rows] = 1
    out = []
    for value in (0.0, 3e35):
        pr = Problem(g, oracle.NAMED_PATTERNS["self_only"])
        pr.t["x"][:, rows] = value
        pr.t["dy"][:, rows] = 0     # as queries the rows have no part in any gradient
        y = pr.fwd()
        out.append((y, pr.bwd()))
    keep = [i for i in range(sum(seg)) if i not in rows]
    (y0, g0), (y1, g1) = out
    assert_close(y1[:, keep], y0[:, keep].double().cpu().numpy(), TOL["fp32"], "y")
    assert_close(g1["dx"][:, keep], g0["dx"][:, keep].double().cpu().numpy(), TOL["fp32"], "dx")
    for n in ("dwv", "dbv", "dbk"):
        scale = g0["dwv" if n == "dwv" else "dbv"].abs().max().item()
        assert_close(g1[n], g0[n].double().cpu().numpy(), TOL["fp32"], n, scale)


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("form", ["packed", "valid_len"])
def test_contents_of_masked_keys_in_other_forms(dtype, form):
    # the same for packed rows and for valid lengths beside key_pad (the masked keys' tiles end at other rows), and for bf16
    # tensors whose heads (dimension 5) the small-head kernels serve.  A masked row of 3e35 as a query has scores of 1e70: its
    # own y and every sum over queries that it enters are left out.
    print(f"[case] masked keys {form} {dtype}", flush=True)
    seg, rows = (20, 70, 40), [3, 22, 60, 95]
    g = synth.attention_inputs(2, seg, 40, 8, dtype, "none", seed=1007)
    lengths = np.array([[17, 70, 12], [20, 45, 40]], np.int32)
    g["key_pad"] = np.zeros((2, sum(seg)), np.uint8)
    g["key_pad"][:, rows] = 1
    g["dy"][:, rows] = 0
    inside = np.concatenate([np.arange(n)[None] < lengths[:, i:i + 1] for i, n in enumerate(seg)], axis=1)
    g["x"][~inside], g["dy"][~inside] = 0, 0
    if form == "valid_len":
        g["valid_len"] = lengths
    keep = inside.copy()
    keep[:, rows] = False
    y = []
    for value in (0.0, 3e35):
        g["x"][:, rows] = np.where(inside[:, rows, None], np.float32(value), 0)
        pr = PackedProblem(g, oracle.NAMED_PATTERNS["self_only"], lengths) if form == "packed" else Problem(g, oracle.NAMED_PATTERNS["self_only"])
        out, grads = pr.fwd(), pr.bwd()
        at = torch.from_numpy(keep[inside] if form == "packed" else keep).cuda()
        y.append((out[at], grads["dx"][at], grads["dwv"]))
    for a, b, what in zip(y[1], y[0], ("y", "dx", "dwv")):
        assert_close(a, b.double().cpu().numpy(), TOL[dtype], what)


@pytest.mark.parametrize("d,H", [(40, 8), (33, 3), (32, 2)])
def test_rows_of_nan(d, H):
    # rows of x beyond the valid lengths hold NaN: as keys they are not read, as queries they give NaN, and every other row is
    # bit for bit what it is without them.  The lengths split waves' 16 rows and the products' 32-row blocks, and leave some
    # of both whole.
    print(f"[case] rows of NaN d={d}", flush=True)
    seg, lengths = (20, 70, 40), np.array([[17, 70, 12], [20, 9, 40]], np.int32)
    g = synth.attention_inputs(2, seg, d, H, "fp32", "none", seed=1008, bias=True)
    g["valid_len"] = lengths
    pad = torch.from_numpy(np.concatenate([np.arange(n)[None] >= lengths[:, i:i + 1] for i, n in enumerate(seg)], axis=1))
    y = []
    for value in (0.0, float("nan")):
        pr = Problem(g, oracle.IM_IFM_FORWARD)
        pr.t["x"][pad.cuda()] = value
        y.append(pr.fwd().cpu())
    assert torch.equal(y[1][~pad], y[0][~pad])
    assert y[0].isfinite().all() and y[1][pad].isnan().all()
