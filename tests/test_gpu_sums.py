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
