"""bf16 weight and bias gradients of a whole backward pass in one launch (wgrad_ring.hip): both tile sizes, products whose
sides are not whole tiles, and numbers of rows around the 64-row stages and the row ranges."""
import pytest
import torch

import oracle
from paper_2505_01068_amd import binding as B, synth
from tests.gpu_util import TOL, assert_close, grad_scale, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,H,d_ff,batch,seg", [
    (64, 8, 256, 1, (1, 1, 1)),          # one stage, 3 rows
    (64, 4, 8, 1, (20, 30, 13)),         # 63 rows; a product with a side of 8
    (64, 8, 200, 1, (20, 30, 14)),       # 64 rows; 200 = 3 tiles of 64 and 8 columns
    (64, 8, 264, 1, (20, 30, 15)),       # 65 rows; tiles of 128
    (128, 2, 136, 2, (70, 33, 26)),      # 258 rows
    (192, 3, 72, 1, (100, 90, 129)),     # 319 rows = two ranges, the second not whole
    (64, 8, 256, 5, (40, 200, 101)),     # 1705 rows: many ranges
])
def test_layer_weight_gradients(d, H, d_ff, batch, seg):
    print(f"[case] bf16 weight gradients d={d} d_ff={d_ff} rows={batch * sum(seg)}", flush=True)
    g = synth.attention_inputs(batch, seg, d, H, "bf16", "none", seed=921)
    p = synth.layer_params(d, d_ff, 921, 0, dtype="bf16")
    lm = oracle.IM_IFM_FORWARD
    shape = B.make_shape(batch, seg, d, H, lm, g["scale"], "bf16")
    sb, wb = B.gsit_layer_train_sizes(shape, d_ff)
    saved, ws = (torch.empty(n, dtype=torch.uint8, device="cuda") for n in (sb, wb))
    ws.fill_(0xff)   # NaNs: nothing that was not written may reach a sum
    x, dy, pd = to_dev(g["x"], "bf16"), to_dev(g["dy"], "bf16"), {k: to_dev(v, "bf16") for k, v in p.items()}
    B.gsit_layer_fwd_train(shape, d_ff, x, pd, saved, workspace=ws)
    grads = {k: torch.empty(v.shape, dtype=torch.float32, device="cuda") for k, v in pd.items()}
    dx = B.gsit_layer_bwd(shape, d_ff, x, pd, saved, dy, grads, workspace=ws)
    torch.cuda.synchronize()
    ref = oracle.gsit_layer_backward(g["x"], p, g["dy"], seg, lm, H, g["scale"])
    floor = 2.0 ** -8 * max(float(abs(v).max()) for k, v in ref.items() if k != "attn_dk")
    dk_sum = abs(ref["attn_dk"]).sum(axis=(0, 1)).max()
    assert_close(dx, ref["dx"], TOL["bf16"], "dx")
    for n, v in grads.items():
        assert_close(v, ref["d" + n], TOL["bf16"], "d" + n, grad_scale(n, ref["d" + n], floor, dk_sum))
    # the column sums of dy are sums of exact values: fp32 rounding only, at most one unit per addition
    want = to_dev(g["dy"], "bf16").double().sum(dim=(0, 1))
    bound = 2.0 ** -23 * batch * sum(seg) * to_dev(g["dy"], "bf16").double().abs().sum(dim=(0, 1))
    assert ((grads["b2"].double() - want).abs() <= bound).all()
    # a gradient's bits do not depend on which others are asked for
    for names in (("w1",), ("b1", "bq"), ("wk", "bo", "w2")):
        some = {k: torch.full_like(grads[k], float("nan")) for k in names}
        B.gsit_layer_bwd(shape, d_ff, x, pd, saved, dy, some, workspace=ws)
        for k in names:
            assert torch.equal(some[k], grads[k]), k


@pytest.mark.parametrize("batch", [8750, 4501])   # 183 and 94 stages per range: two runs of 80 and a rest, one and a rest
def test_ranges_of_more_than_80_stages(batch):
    # Every segment one row that attends itself and Wv = I: O = x exactly, so dWo = x^T dy and dbo have exact references.
    # A sum of 80 stages is rounded 320 times, by a few tenths of 2^-23 of its size: 5e-7 (measured 4.3e-7).
    d, H, seg = 1024, 16, (1,) * 8
    print(f"[case] bf16 weight gradients, tall d={d} rows={8 * batch}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(931)
    x, dy = (torch.randn(batch, 8, d, device="cuda", generator=gen).bfloat16() for _ in range(2))
    w = {k: (torch.randn(d, d, device="cuda", generator=gen) / 32).bfloat16() for k in ("wq", "wk", "wo")}
    w["wv"] = torch.eye(d, device="cuda").bfloat16()
    shape = B.make_shape(batch, seg, d, H, sum(1 << (9 * i) for i in range(8)), 0.125, "bf16")
    saved, ws = (torch.empty(n, dtype=torch.uint8, device="cuda") for n in B.im_attention_sizes(shape))
    B.im_attention_fwd(shape, x, **w, saved=saved, workspace=ws)
    dwo, dbo = torch.empty(d, d, device="cuda"), torch.empty(d, device="cuda")
    B.im_attention_bwd(shape, x, **w, saved=saved, dy=dy, dx=torch.empty_like(x), dwq=None, dwk=None, dwv=None, dwo=dwo, dbo=dbo,
                       workspace=ws)
    a, g = x.view(-1, d).double(), dy.view(-1, d).double()
    for got, ref, bar in ((dwo, a.t() @ g, 6e-7), (dbo, g.sum(0), 3e-7)):
        err = ((got - ref).norm() / ref.norm()).item()
        print(f"    {err:.1e}")
        assert err < bar, err
