"""Per-channel sums of the backward kernels: what a term is, how far the sum
may round, and that rows which are no pixel add nothing to it (GPU)."""
import numpy as np
import pytest
import torch

from helpers import dev, f32dev
from paper_1807_01702_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_1807_01702_amd import bnr
    return bnr


def f32(t):
    return t.detach().float().cpu().numpy()


@pytest.mark.parametrize("k", [1, 3])
@pytest.mark.parametrize("ci,co", [(64, 32), (128, 24), (32, 64)])
def test_dgamma_of_one_pixel_is_dy_times_xhat(B, k, ci, co):
    """One pixel, so dgamma is its only term: dy times xhat, xhat rounded to
    float32 first, bit for bit."""
    x = dev(synth.normal(3, "x", (1, 1, 1, ci), bf16=True), True)
    g = dev(synth.normal(3, "g", (1, 1, 1, co), bf16=True), True)
    w = dev(synth.conv_weight(3, "w", k, ci, co, True), True)
    p = synth.bn_params(3, "bn", ci)
    mean, rstd = synth.normal(3, "m", (ci,)) * np.float32(0.1), np.float32(1.0) + np.abs(synth.normal(3, "r", (ci,)))
    bn = B.BN(f32dev(p["gamma"]), f32dev(p["beta"]), 1e-5, f32dev(mean), torch.ones(ci, device="cuda"), f32dev(rstd))
    dy = torch.empty_like(x)
    dgamma, dbeta = torch.empty(ci, device="cuda"), torch.empty(ci, device="cuda")
    B.bnr_bwd_data(B.desc_for(x, g, k, 1, 1, 1), x, bn, w, B.grad_dense(g), dgamma, dbeta, dy)
    torch.cuda.synchronize()
    d, xv = f32(dy).reshape(ci), f32(x).reshape(ci)
    assert np.count_nonzero(d) > ci // 8
    np.testing.assert_array_equal(f32(dbeta), d)
    np.testing.assert_array_equal(f32(dgamma), d * ((xv - f32(bn.mean)) * f32(bn.rstd)))


@pytest.mark.parametrize("n,h,w,ci,co", [(2, 5, 5, 64, 32), (1, 3, 7, 32, 24), (3, 9, 4, 128, 32)])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("src", ["z", "x"])
def test_stored_z_backward_keeps_a_channels_infinity_to_itself(B, n, h, w, ci, co, value, src):
    """The 3x3 data gradient on the stored z reads something for the rows of
    its padded grid that are no pixel, and adds 0 times it: an infinite or NaN
    value of channel 0 may reach dgamma of channel 0 only (src x: the vectors
    that hold a gamma = 0 channel read x instead)."""
    x = dev(synth.normal(4, "x", (n, h, w, ci), bf16=True), True)
    g = dev(synth.normal(4, "g", (n, h, w, co), bf16=True), True)
    wt = dev(synth.conv_weight(4, "w", 3, ci, co, True), True)
    p = synth.bn_params(4, "bn", ci)
    gam = f32dev(p["gamma"])
    if src == "x":
        gam[1::8] = 0.0
    bn = B.BN(gam, f32dev(p["beta"]), 1e-5, torch.zeros(ci, device="cuda"), torch.ones(ci, device="cuda"),
              torch.ones(ci, device="cuda"))
    z = torch.relu(x.float() * gam + bn.beta).to(torch.bfloat16)
    out = []
    for v in (1.0, value):
        (z if src == "z" else x)[0, 0, 0, 0] = v
        dw = torch.empty((3, 3, ci, co), device="cuda")
        dg, db = torch.empty(ci, device="cuda"), torch.empty(ci, device="cuda")
        B.bnr_bwd_fused_o2(B.desc_for(x, g, 3, n, h, w), x, bn, z, wt, B.grad_dense(g), dw, dg, db, torch.empty_like(x))
        torch.cuda.synchronize()
        out.append((f32(dg), f32(db)))
    for clean, got in zip(*out):
        np.testing.assert_array_equal(got[1:], clean[1:])


@pytest.mark.parametrize("k,n,h,w,ci,co", [(1, 1, 5, 7, 8, 12), (1, 3, 9, 11, 40, 68), (3, 2, 6, 7, 20, 36)])
def test_stored_z_backward_float32_rows_past_the_tensor(B, k, n, h, w, ci, co):
    """The last tile's rows past the tensor add nothing: an infinite z of the
    first pixel makes its channel's dgamma infinite (that pixel's own term),
    not NaN, and touches no other channel."""
    x, g = dev(synth.normal(4, "x", (n, h, w, ci)), False), dev(synth.normal(4, "g", (n, h, w, co)), False)
    wt = dev(synth.conv_weight(4, "w", k, ci, co, False), False)
    p = synth.bn_params(4, "bn", ci)
    bn = B.BN(f32dev(p["gamma"]), f32dev(p["beta"]), 1e-5, torch.zeros(ci, device="cuda"),
              torch.ones(ci, device="cuda"), torch.ones(ci, device="cuda"))
    z = torch.relu(x * bn.gamma + bn.beta)
    out = []
    for v in (1.0, float("inf")):
        z[0, 0, 0, 0] = v
        dw = torch.empty((k, k, ci, co), device="cuda")
        dg, db = torch.empty(ci, device="cuda"), torch.empty(ci, device="cuda")
        B.bnr_bwd_fused_o2(B.desc_for(x, g, k, n, h, w), x, bn, z, wt, B.grad_dense(g), dw, dg, db, torch.empty_like(x))
        torch.cuda.synchronize()
        out.append(f32(dg))
    assert np.isinf(out[1][0]), out[1][0]
    np.testing.assert_array_equal(out[1][1:], out[0][1:])


def _sum_errors(dgamma, dbeta, dy, x, bn):
    """2-norm over the channels of the errors of both sums against float64 sums
    of the stored dy, over the 2-norm of the sums of their terms' magnitudes."""
    c = x.shape[-1]
    d = dy.reshape(-1, c).double()
    t = d * ((x.reshape(-1, c).double() - bn.mean.double()) * bn.rstd.double())
    return (float((dgamma.double() - t.sum(0)).norm() / t.abs().sum(0).norm()),
            float((dbeta.double() - d.sum(0)).norm() / d.abs().sum(0).norm()))


def _bn_of(B, x, seed):
    c = x.shape[-1]
    p, xd = synth.bn_params(seed, "bn", c), x.reshape(-1, c).double()
    mean = xd.mean(0)
    var = (xd - mean).square().mean(0)
    return B.BN(f32dev(p["gamma"]), f32dev(p["beta"]), 1e-5, mean.float(), var.float(), torch.rsqrt(var + 1e-5).float())


def test_pooled_gradient_sums_round_no_further(B):
    """dgamma of a pooled gradient, error over the sum of its terms' magnitudes
    (512 channels): 1.53e-9 (a window's pixels, then pairs of threads); the
    general kernels, pixel by pixel, have 1.58e-9, sums in chains 1.85e-9."""
    n, h, w, ci, co = 32, 28, 28, 512, 256
    x = dev(synth.normal(6, "x", (n, h, w, ci), bf16=True), True)
    g = dev(synth.normal(6, "g", (n, h // 2, w // 2, co), bf16=True), True)
    wt = dev(synth.conv_weight(6, "w", 1, ci, co, True), True)
    bn = _bn_of(B, x, 6)
    dy, dg, db = torch.empty_like(x), torch.empty(ci, device="cuda"), torch.empty(ci, device="cuda")
    B.bnr_bwd_data(B.conv_desc(n, h, w, ci, co, 1, ci, co, B.dtype_code(x)), x, bn, wt, B.grad_avgpool2(g), dg, db, dy)
    e = _sum_errors(dg, db, dy, x, bn)
    assert e[0] <= 1.65e-9 and e[1] <= 5.2e-10, e
# (bounds: between what the kernel has, 5.7e-10 to 6.8e-10, and the float32
# chains of single pixels and of columns, 9.7e-10 to 1.2e-9; the kernel that
# scanned every window has 6.8e-10 to 9.4e-10)
@pytest.mark.parametrize("bf16,n,h,w,c,bound", [
    (True, 20, 95, 95, 64, 8.0e-10),
    (True, 60, 50, 50, 64, 9.0e-10),
    (False, 20, 95, 95, 64, 6.7e-10),
    (False, 60, 50, 50, 64, 7.4e-10),
])
def test_maxpool_backward_sums_round_no_further(B, bf16, n, h, w, c, bound):
    ho, wo = (h - 1) // 2 + 1, (w - 1) // 2 + 1
    x, g = dev(synth.normal(6, "x", (n, h, w, c), bf16=bf16), bf16), dev(synth.normal(6, "g", (n, ho, wo, c), bf16=bf16), bf16)
    bn = _bn_of(B, x, 6)
    dy, dg, db = torch.empty_like(x), torch.empty(c, device="cuda"), torch.empty(c, device="cuda")
    B.bnr_maxpool_bn_bwd(x, bn, g, dy, n, h, w, dg, db)
    e = _sum_errors(dg, db, dy, x, bn)
    assert e[0] <= bound and e[1] <= (2.4e-10 if bf16 else 5.5e-10), e
