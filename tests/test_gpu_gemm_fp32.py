"""fp32 GEMMs on the bf16 matrix cores (gemm_split.hip), through the encoder layer: every product of a layer forward
(three-buffer QKV with biases, residual, GELU) at the edges of the 64 x 64 tiles, of the 16-deep k-steps and of the chunk
sizes, with widths that are and are not multiples of 8."""
import pytest
import torch

import oracle
from paper_2505_01068_amd import binding as B, synth
from tests.gpu_util import TOL, assert_close, grad_scale, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,H,d_ff", [(8, 1, 24), (16, 2, 40), (40, 8, 160), (48, 6, 192), (64, 8, 256), (80, 8, 320),
                                      (96, 6, 96), (20, 4, 52), (33, 3, 70), (42, 7, 161)])
@pytest.mark.parametrize("batch,seg", [(1, (1, 3, 2)), (3, (5, 9, 7)), (2, (13, 40, 12))])   # 6, 63 and 130 rows
def test_layer_products(d, H, d_ff, batch, seg):
    print(f"[case] fp32 GEMM d={d} d_ff={d_ff} rows={batch * sum(seg)}", flush=True)
    g = synth.attention_inputs(batch, seg, d, H, "fp32", "none", seed=801, with_dy=False)
    p = synth.layer_params(d, d_ff, 801, 0, dtype="fp32")
    lm = oracle.NAMED_PATTERNS["self_only"]
    shape = B.make_shape(batch, seg, d, H, lm, g["scale"], "fp32")
    ws = torch.empty(B.gsit_layer_sizes(shape, d_ff), dtype=torch.uint8, device="cuda")
    y = B.gsit_layer_fwd(shape, d_ff, to_dev(g["x"], "fp32"), {k: to_dev(v, "fp32") for k, v in p.items()}, workspace=ws)
    torch.cuda.synchronize()
    assert_close(y, oracle.gsit_layer_forward(g["x"], p, seg, lm, H, g["scale"]), TOL["fp32"], f"layer d={d} d_ff={d_ff}")


@pytest.mark.parametrize("d,H,d_ff", [(8, 1, 24), (40, 8, 160), (64, 8, 256), (33, 3, 70), (42, 7, 161)])
@pytest.mark.parametrize("batch,seg", [(1, (1, 3, 2)), (3, (11, 9, 13)), (5, (40, 31, 30))])   # 6, 99 and 505 rows
def test_layer_weight_gradients(d, H, d_ff, batch, seg):
    # 32-row workgroups with whole, partial and single 16-row steps; blocks and quads that end inside a row
    print(f"[case] fp32 weight gradients d={d} d_ff={d_ff} rows={batch * sum(seg)}", flush=True)
    g = synth.attention_inputs(batch, seg, d, H, "fp32", "none", seed=811)
    p = synth.layer_params(d, d_ff, 811, 0, dtype="fp32")
    lm = oracle.IM_IFM_FORWARD
    shape = B.make_shape(batch, seg, d, H, lm, g["scale"], "fp32")
    sb, wb = B.gsit_layer_train_sizes(shape, d_ff)
    saved, ws = (torch.empty(n, dtype=torch.uint8, device="cuda") for n in (sb, wb))
    x, dy, pd = to_dev(g["x"], "fp32"), to_dev(g["dy"], "fp32"), {k: to_dev(v, "fp32") for k, v in p.items()}
    B.gsit_layer_fwd_train(shape, d_ff, x, pd, saved, workspace=ws)
    grads = {k: torch.empty(v.shape, dtype=torch.float32, device="cuda") for k, v in pd.items()}
    dx = B.gsit_layer_bwd(shape, d_ff, x, pd, saved, dy, grads, workspace=ws)
    torch.cuda.synchronize()
    ref = oracle.gsit_layer_backward(g["x"], p, g["dy"], seg, lm, H, g["scale"])
    floor = 2.0 ** -23 * max(float(abs(v).max()) for k, v in ref.items() if k != "attn_dk")
    dk_sum = abs(ref["attn_dk"]).sum(axis=(0, 1)).max()
    assert_close(dx, ref["dx"], TOL["fp32"], "dx")
    for n, v in grads.items():
        assert_close(v, ref["d" + n], TOL["fp32"], "d" + n, grad_scale(n, ref["d" + n], floor, dk_sum))
    # a gradient's bits do not depend on which others are asked for
    for want in (("w1",), ("b1", "bq"), ("wk", "bo", "w2")):
        some = {k: torch.full_like(grads[k], float("nan")) for k in want}
        B.gsit_layer_bwd(shape, d_ff, x, pd, saved, dy, some, workspace=ws)
        for k in want:
            assert torch.equal(some[k], grads[k]), k


def test_weight_gradient_over_a_million_rows():
    # dWo = O^T dy over 1 048 560 rows, each row of O good to 2e-7.  A partial sum of n rows is a random walk that is rounded
    # once per 16 rows, by up to a few tenths of 2^-23 of its size: 2^-24 sqrt(n / 16), 4.2e-7 measured with ranges of 4 688
    # rows; 2.9e-7 with fp32 multiply-adds in ranges of 1 024.
    print("[case] fp32 weight gradient over 1 048 560 rows", flush=True)
    batch, seg, d, H = 65535, (5, 5, 6), 8, 2
    gen = torch.Generator(device="cuda").manual_seed(821)
    x, dy = (torch.randn(batch, 16, d, device="cuda", generator=gen) for _ in range(2))
    w = {k: torch.randn(d, d, device="cuda", generator=gen) * 0.4 for k in ("wq", "wk", "wv", "wo")}
    shape = B.make_shape(batch, seg, d, H, oracle.IM_IFM_FORWARD, 0.5, "fp32")
    saved, ws = (torch.empty(n, dtype=torch.uint8, device="cuda") for n in B.im_attention_sizes(shape))
    B.im_attention_fwd(shape, x, **w, saved=saved, workspace=ws)
    dwo, dx = torch.empty(d, d, device="cuda"), torch.empty_like(x)
    B.im_attention_bwd(shape, x, **w, saved=saved, dy=dy, dx=dx, dwq=None, dwk=None, dwv=None, dwo=dwo, workspace=ws)
    q, k, v = ((x.double() @ w[n].double()).view(batch, 16, H, d // H).transpose(1, 2).contiguous() for n in ("wq", "wk", "wv"))
    segment = torch.tensor([0] * 5 + [1] * 5 + [2] * 6, device="cuda")
    live = torch.tensor([[(oracle.IM_IFM_FORWARD >> (3 * i + j)) & 1 for j in range(3)] for i in range(3)], device="cuda")
    p = (0.5 * (q @ k.transpose(2, 3).contiguous())).masked_fill(live[segment][:, segment] == 0, float("-inf")).softmax(-1)
    o = (p @ v).transpose(1, 2).reshape(-1, d)
    ref = o.t() @ dy.double().view(-1, d)
    err = ((dwo - ref).norm() / ref.norm()).item()
    print(f"    {err:.2e}")
    assert err < 3.4e-7, err
