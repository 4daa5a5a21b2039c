"""bf16 matrix-core attention: scores far from 0, exactness of a probability of 1, and rows whose scores outgrow the reference that the
forward took from their first block."""
import numpy as np
import pytest
import torch

import oracle
from paper_2505_01068_amd import synth
from tests.gpu_util import PackedProblem, Problem, assert_close, rows_outgrowing_the_first_block, TOL

pytestmark = pytest.mark.gpu

# t reads v, v reads v, a reads a: no row of t is a key
LIVE = (1 << 1) | (1 << 4) | (1 << 8)


def padded_rows(g, seg):
    """[B, T_m]: the rows that are masked as keys."""
    n, T = g["x"].shape[:2]
    if g["key_pad"] is not None:
        return g["key_pad"] != 0
    if g["valid_len"] is None:
        return np.zeros((n, T), bool)
    pos = np.concatenate([np.arange(k) for k in seg])
    return pos[None, :] >= np.asarray(g["valid_len"])[:, np.repeat(np.arange(len(seg)), seg)]


def shifted(d, H, seg, padding, shift_bits, left=0.0):
    """Every score of query row r of t is off by shift_bits[r] in the exponent of 2, by the first channel of each head: 8 in
    every valid key, the shift in the query.  Softmax does not see it; 2^s overflows or vanishes.  left: what the masked keys' rows
    hold there, so that their scores lie elsewhere than those that the row's sum is made of."""
    g = synth.attention_inputs(2, seg, d, H, "bf16", padding, seed=31)
    dh = d // H
    eye = np.eye(d, dtype=np.float32)
    g["wq"], g["wk"] = eye, eye
    x = g["x"].copy()
    x[:, :, ::dh] = np.where(padded_rows(g, seg), np.float32(left), np.float32(8.0))[:, :, None]
    a = np.zeros(seg[0], np.float32)
    a[:len(shift_bits)] = np.asarray(shift_bits, np.float32) / (8.0 * g["scale"] * np.log2(np.e))
    x[:, :seg[0], ::dh] = np.asarray(torch.from_numpy(a).to(torch.bfloat16).float())[None, :, None]
    g["x"] = x
    return g


@pytest.mark.parametrize("padding,left", [("none", 0.0), ("valid_len", 0.0), ("valid_len", 96.0), ("key_pad", 0.0), ("key_pad", -96.0)])
@pytest.mark.parametrize("d,H,seg", [(64, 8, (70, 150, 33)), (64, 4, (33, 97, 20)), (192, 24, (65, 64, 65)), (128, 2, (140, 200, 50))])
def test_shifted_rows(d, H, seg, padding, left):
    n = seg[0]
    bits = [0.0] * n
    for r, v in ((1, 180.0), (2, -180.0), (5, 110.0), (6, -95.0), (n - 1, 300.0), (n // 2, -300.0)):
        bits[r] = v
    print(f"[case] shifted rows d={d} H={H} seg={seg} {padding} {left}", flush=True)
    g = shifted(d, H, seg, padding, bits, left)
    p = Problem(g, LIVE)
    y = p.fwd(save=True).clone()
    grads = p.bwd()
    torch.cuda.synchronize()
    y_ref, cache = p.oracle_fwd(cache=True)
    ref = oracle.backward(cache, g["dy"])
    assert_close(y, y_ref, TOL["bf16"], "y")
    # dV, dO and P from the saved log-sum-exp; the first channels of dQ and dK are differences of large numbers here
    for name in ("dwv", "dwo"):
        assert_close(grads[name], ref[name], TOL["bf16"], name)
    for name in ("dx", "dwq", "dwk"):
        assert torch.isfinite(grads[name]).all(), name
    assert torch.equal(p.fwd(save=False), y)
    q = Problem(shifted(d, H, seg, padding, [0.0] * n, left), LIVE)
    y0 = q.fwd(save=False)
    torch.cuda.synchronize()
    same = np.ones(sum(seg), bool)
    same[[r for r in range(n) if bits[r] != 0.0]] = False
    same = torch.from_numpy(same).cuda()
    assert torch.equal(y[:, same], y0[:, same])


@pytest.mark.parametrize("left", [0, 5, 37, 64, 99])
@pytest.mark.parametrize("d,H", [(64, 8), (64, 4), (128, 2)])
def test_one_valid_key_is_exact(d, H, left):
    """With one valid key a row's probability is 1, in the backward too: V, dO and x are whole numbers, so are y and the gradients
    of wv and wo, and dQ and dK vanish.  A reference other than the row's maximum leaves the probability off by a bf16 rounding."""
    print(f"[case] one key d={d} H={H} key {left}", flush=True)
    seg, n = (9, 100, 4), 6
    g = synth.attention_inputs(n, seg, d, H, "bf16", "none", seed=17)
    rng = np.random.default_rng(5)
    g["wv"] = g["wo"] = np.eye(d, dtype=np.float32)
    g["x"] = rng.integers(-4, 5, g["x"].shape).astype(np.float32)
    g["dy"] = rng.integers(-4, 5, g["dy"].shape).astype(np.float32)
    kp = np.ones((n, sum(seg)), np.uint8)
    kp[:, seg[0] + left] = 0
    g["key_pad"] = kp
    p = Problem(g, 1 << 1)   # t reads v
    y = p.fwd(save=True)
    grads = p.bwd()
    torch.cuda.synchronize()
    y_ref, cache = p.oracle_fwd(cache=True)
    ref = oracle.backward(cache, g["dy"])
    whole = lambda t: t.float().cpu().numpy().astype(np.float64)  # noqa: E731
    for b in ("bv", "bo"):
        assert g.get(b) is None
    assert np.array_equal(whole(y), np.rint(y_ref))
    for name in ("dwv", "dwo"):
        assert np.array_equal(whole(grads[name]), np.rint(ref[name])), name
    for name in ("dwq", "dwk"):
        assert not grads[name].any(), name


@pytest.mark.parametrize("d,H,seg,n", [(64, 8, (70, 90, 40), 3), (64, 4, (33, 64, 65), 3), (128, 2, (140, 90, 50), 3), (128, 2, (140, 90, 50), 100)])
def test_first_segment_without_valid_keys(d, H, seg, n):
    """The first live segment of a row has no valid key, and its K and V rows are infinite: they are multiplied by nothing.
    (3 and 100 samples: 64- and 128-row tiles at head dimension 64.)"""
    print(f"[case] empty first segment d={d} H={H} seg={seg} n={n}", flush=True)
    g = synth.attention_inputs(n, seg, d, H, "bf16", "none", seed=23)
    vl = np.tile(np.array(seg, np.int32), (n, 1))
    vl[:, 1] = 0
    vl[1, 2] = 0              # no key at all
    vl[2, 1], vl[2, 2] = 10, 0
    vl[3:, 2] = np.arange(n - 3) % (seg[2] + 1)
    g["valid_len"] = vl
    x = g["x"].copy()
    v_rows = (np.arange(sum(seg)) >= seg[0]) & (np.arange(sum(seg)) < seg[0] + seg[1])
    x[:, :, 0] = 0.0
    x[np.ix_(vl[:, 1] == 0, v_rows, [0])] = 2.0 ** 127
    g["x"] = x
    for name, v in (("wq", 0.0), ("wk", 4.0), ("wv", 4.0)):
        w = g[name].copy()
        w[0, :] = v
        g[name] = w
    p = Problem(g, (1 << 1) | (1 << 2))   # t reads v and a
    y = p.fwd(save=True)
    grads = p.bwd()
    torch.cuda.synchronize()
    y_ref, cache = p.oracle_fwd(cache=True)
    ref = oracle.backward(cache, g["dy"])
    assert_close(y, y_ref, TOL["bf16"], "y")
    for name in ("dx", "dwq", "dwk", "dwv", "dwo"):
        assert_close(grads[name], ref[name], TOL["bf16"], name)


@pytest.mark.parametrize("d,H", [(64, 8), (64, 4), (128, 2)])
def test_masked_samples_take_one_pass(d, H):
    """Keys that are all masked give zeros, and the call takes no longer than with valid keys: their tiles are streamed once
    (2.0 to 3.0 times as long where rows with a sum of 0 asked for a second pass)."""
    print(f"[case] all keys masked d={d} H={H}", flush=True)
    g = synth.attention_inputs(16, (64, 2048), d, H, "bf16", "none", seed=3, with_dy=False)
    times = []
    for masked in (0, 1):
        p = Problem(dict(g, key_pad=np.full(g["x"].shape[:2], masked, np.uint8)), 1 << 3)   # v reads v
        p.fwd()
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(9)]
        ev[0].record()
        for e in ev[1:]:
            y = p.fwd()
            e.record()
        torch.cuda.synchronize()
        times.append(min(a.elapsed_time(b) for a, b in zip(ev, ev[1:])))
        assert torch.isfinite(y).all() and (not masked or not y.any())
    print(f"    {times[0] * 1e3:.1f} us, masked {times[1] * 1e3:.1f} us", flush=True)
    assert times[1] < 1.2 * times[0]


# rows of t: how far their scores rise from one 32-key block of v to the next, and at its third block alone, in the exponent of 2
GROWTH = {1: (30, 0), 2: (15, 0), 5: (-30, 0), 6: (0, 60), 9: (130, 0), -1: (30, -100)}


def growing(n, d, H, seg, padding, rows):
    g = synth.attention_inputs(n, seg, d, H, "bf16", padding if padding != "packed" else "none", seed=37)
    dh = d // H
    g["wq"] = g["wk"] = np.eye(d, dtype=np.float32)
    block = np.concatenate([np.arange(k) for k in seg]) // 32
    x = g["x"].copy()
    x[:, :, ::dh] = block[None, :, None]
    x[:, :, 1::dh] = (block == 2)[None, :, None]
    x[:, :seg[0], ::dh] = x[:, :seg[0], 1::dh] = 0.0
    for r, (rise, bump) in rows.items():
        x[:, r % seg[0], ::dh] = rise / (g["scale"] * np.log2(np.e))
        x[:, r % seg[0], 1::dh] = bump / (g["scale"] * np.log2(np.e))
    g["x"] = synth.to_bf16_grid(np.where(padded_rows(g, seg)[:, :, None], np.float32(0), x))
    return g


# 64- and 128-row tiles at head dimension 64 (2 and 70 samples), tiles of half the height (the 50 rows of t that read 500 keys)
@pytest.mark.parametrize("padding", ["none", "valid_len", "key_pad", "packed"])
@pytest.mark.parametrize("d,H,seg,n", [(64, 8, (70, 150, 33), 2), (64, 4, (33, 97, 20), 2), (128, 2, (140, 200, 50), 2),
                                       (128, 2, (140, 200, 50), 70), (64, 8, (50, 500, 375), 2), (64, 4, (50, 500, 375), 2)])
def test_scores_that_outgrow_the_first_block(d, H, seg, n, padding):
    """Rows with scores more than 2^24 above their first block's maximum, some beyond 2^100 and 2^128, move their reference; the other
    rows of their wave keep every bit."""
    print(f"[case] growing scores d={d} H={H} seg={seg} n={n} {padding}", flush=True)
    live = (1 << 1) | (1 << 5) | (1 << 8)   # t reads v, v reads a, a reads a: no row of t is a key
    lengths = [[s if b % 2 == 0 else s - s // 4 for s in seg] for b in range(n)]
    make = lambda rows: (PackedProblem(growing(n, d, H, seg, padding, rows), live, lengths) if padding == "packed"  # noqa: E731
                         else Problem(growing(n, d, H, seg, padding, rows), live))
    p = make(GROWTH)
    y = p.fwd(save=True).clone()
    grads = p.bwd()
    torch.cuda.synchronize()
    g = p.g
    pack = (lambda a: synth.pack_rows(a, p.lengths, seg)) if padding == "packed" else (lambda a: a)
    y_ref, cache = oracle.forward(g["x"], g["wq"], g["wk"], g["wv"], g["wo"], seg, live, H, g["scale"], key_pad=g["key_pad"],
                                  valid_len=p.lengths if padding == "packed" else g["valid_len"], return_cache=True)
    moving = rows_outgrowing_the_first_block(p, cache)
    for r in (1, 2, 6, 9):
        assert moving[0, :, r].all() and not moving[:, :, 5].any()
    dy = g["dy"] if padding != "packed" else synth.unpack_rows(pack(g["dy"]), p.lengths, seg)
    ref = oracle.backward(cache, dy)
    assert_close(y, pack(y_ref), TOL["bf16"], "y")
    for name in ("dwv", "dwo"):
        assert_close(grads[name], ref[name], TOL["bf16"], name)
    for name in ("dx", "dwq", "dwk"):
        assert torch.isfinite(grads[name]).all(), name
    assert torch.equal(p.fwd(save=False), y)
    y0 = make({}).fwd(save=False)
    torch.cuda.synchronize()
    same = np.ones((n, sum(seg)), bool)
    same[:, [r % seg[0] for r in GROWTH]] = False
    same = torch.from_numpy(pack(same)).cuda()
    assert torch.equal(y[same], y0[same])
