"""Edges of the kernels' tiles and dispatch rules, against the CPU oracle (GPU).

Each case runs one BN-ReLU-CONV layer forward (with the statistics of its
output) and backward (dense gradient, and the deferred gradient of the BN
after it) at a size where a tile, a remainder or a rule of the dispatch turns,
and compares every output with the fp64 oracle on the same inputs.  Tolerances
are those of the parity tests (helpers.RTOL: max |gpu - ref| / max |ref|); the
per-channel sums are bounded by the sum of their terms' magnitudes, and
elements whose ReLU decision lies within rounding of 0 are excluded.
"""
import numpy as np
import pytest
import torch

from helpers import RTOL, assert_close, bf16_round, dev, f32dev, host, relu_ambiguous
from oracle import prims as P
from paper_1807_01702_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_1807_01702_amd import bnr
    return bnr


def _wide(t):
    """t as a view whose pixel stride makes it span more than 2^31 bytes (what lies between is never written)."""
    m, c = t.numel() // t.shape[-1], t.shape[-1]
    vec = 16 // t.element_size()
    ldc = ((1 << 31) // (t.element_size() * (m - 1)) // vec + 1) * vec
    v = torch.empty((m - 1) * ldc + c, dtype=t.dtype, device=t.device).as_strided((m, c), (ldc, 1))
    v.copy_(t.reshape(m, c))
    shape, stride = t.shape[:-1], [ldc]
    for s in reversed(shape[1:]):
        stride.insert(0, stride[0] * s)
    return v.as_strided(t.shape, (*stride, 1))


def _layer(B, bf16, k, n, h, w, ci, co, seed=11, pad_in=0, pad_out=0, wide=False):
    """Runs the layer both ways on views of wider buffers (wide: an input that
    spans more than 2^31 bytes); returns nothing, asserts."""
    rnd = bf16_round if bf16 else (lambda a: np.asarray(a, np.float64))
    rtol, m = RTOL[bf16], n * h * w
    xf = synth.normal(seed, "x", (n, h, w, ci + pad_in), bf16=bf16)
    wt = synth.conv_weight(seed, "w", k, ci, co, bf16)
    p1, p2 = synth.bn_params(seed, "bn1", ci), synth.bn_params(seed, "bn2", co)
    x64 = xf[..., :ci].astype(np.float64)
    y1, mu, var, rstd = P.bn_fwd(x64.reshape(m, ci), p1["gamma"], p1["beta"], 1e-5)
    z = rnd(P.relu_fwd(y1).reshape(n, h, w, ci))
    out_r = rnd(P.conv_fwd(z, wt.astype(np.float64)))
    x = dev(xf, bf16)[..., :ci]
    if wide:
        x = _wide(x)
    wd = dev(wt, bf16)
    buf = torch.full((n, h, w, co + pad_out), 7.0, dtype=x.dtype, device=x.device)
    out = buf[..., :co]
    bn1 = B.BN(f32dev(p1["gamma"]), f32dev(p1["beta"]), 1e-5, f32dev(mu), f32dev(var), f32dev(rstd))
    bn2 = B.BN(f32dev(p2["gamma"]), f32dev(p2["beta"]), 1e-5)
    desc = B.desc_for(x, out, k, n, h, w)
    B.workspace(B.bnr_workspace_size(desc), x.device)
    B._ws_cache[(x.device, 0)].fill_(255)                   # NaN: nothing may read what the call did not write
    B.bnr_bn_relu_conv_fwd(desc, x, bn1, wd, out, bn2)
    torch.cuda.synchronize()
    assert_close("out", host(out), out_r, rtol)
    assert bool((buf[..., co:] == 7.0).all()), "the forward wrote past its channels"
    o64 = host(out).reshape(m, co)
    mo, vo, ro = P.bn_stats(o64, 1e-5)
    # one-sweep statistics from float32 partial sums: E[x^2] - E[x]^2 carries the rounding of its terms,
    # a few 2^-24 of mean^2 + var, whatever is left of them (two pixels can differ by 1/30 of their mean)
    if m > 1:
        assert np.all(np.abs(host(bn2.mean) - mo) <= 1e-4 * np.sqrt(vo) + 4 * 2.0 ** -24 * np.abs(mo)), "out mean"
        assert np.all(np.abs(host(bn2.var) - vo) <= 1e-4 * vo + 8 * 2.0 ** -24 * (mo * mo + vo)), "out var"

    # backward: dense gradient, then the deferred gradient of a BN reading out
    gf = synth.normal(seed, "g", (n, h, w, co), bf16=bf16)
    gd = dev(gf, bf16)
    dgn, dbn = f32dev(synth.normal(seed, "dgn", (co,))), f32dev(synth.normal(seed, "dbn", (co,)))
    bn2.mean.copy_(f32dev(mo)), bn2.rstd.copy_(f32dev(np.minimum(ro, 10.0)))
    mo32, ro32 = host(bn2.mean), host(bn2.rstd)
    xh_o = (o64 - mo32) * ro32
    k2 = p2["gamma"] * ro32
    g2 = rnd((k2 * (gf.reshape(m, co) - host(dbn) / m - xh_o * host(dgn) / m)).reshape(n, h, w, co))
    for name, src, g in (("dense", B.grad_dense(gd), gf.astype(np.float64)),
                         ("deferred", B.grad_bn(gd, out, bn2, dgn, dbn), g2)):
        dw = torch.empty(tuple(wt.shape), dtype=torch.float32, device=x.device)
        dga, dbe = (torch.empty(ci, dtype=torch.float32, device=x.device) for _ in range(2))
        dy = torch.empty((n, h, w, ci), dtype=x.dtype, device=x.device)
        B._ws_cache[(x.device, 0)].fill_(255)
        B.bnr_bwd_fused(desc, x, bn1, wd, src, dw, dga, dbe, dy)
        torch.cuda.synchronize()
        dz = P.conv_dgrad(g, wt.astype(np.float64), (h, w)).reshape(m, ci)
        dyr = P.relu_bwd(dz, y1)
        amb = relu_ambiguous(y1, bf16)
        assert_close(name + " dy", host(dy).reshape(m, ci), dyr, rtol, exclude=amb, max_excluded_frac=1e-2)
        assert_close(name + " dW", host(dw), P.conv_wgrad(z, g, k), rtol)
        # the sums are of the dy that was stored
        d64, xh = host(dy).reshape(m, ci), (x64.reshape(m, ci) - host(bn1.mean)) * host(bn1.rstd)
        for s, got, t in (("dbeta", dbe, d64), ("dgamma", dga, d64 * xh)):
            bound = 1e-5 * np.abs(t).sum(0) + 1e-6
            assert np.all(np.abs(host(got) - t.sum(0)) <= bound), name + " " + s


@pytest.mark.parametrize("n,h,w,ci,co", [
    (2, 1, 1, 32, 32),          # one pixel: every row a wrap of the padded grid
    (9, 2, 1, 8, 136),          # output channels past the persistent kernel (row-tile kernel)
    (3, 3, 5, 96, 24),          # three 32-channel K slices (a zero fourth one), a ragged N slice
    (5, 2, 3, 72, 32),          # K slices cut at 8 channels
    (1, 61, 61, 64, 64),        # widest rows: the longest window of the input ring
    (2, 7, 61, 32, 128),        # the same with four N slices
    (3, 37, 2, 128, 8),         # narrow rows: many rows of the padded grid in a tile
    (4, 13, 9, 48, 40),         # two K and two N slices, ragged
    (2, 9, 30, 24, 96),         # one K slice, a ragged fourth N slice
    (40, 14, 14, 128, 32),      # one-tile ranges that cross images
    (1, 300, 2, 32, 64),        # tall images
    (76, 32, 8, 40, 24),        # two 64-row tiles per workgroup, the second one short
    (60, 30, 26, 16, 16),       # two 128-row tiles
    (90, 24, 20, 40, 8),        # four 64-row tiles: the pipelined loop
    (40, 56, 40, 8, 8),         # three 128-row tiles: the pipelined loop
])
def test_conv3x3_tiles_bf16(B, n, h, w, ci, co):
    _layer(B, True, 3, n, h, w, ci, co, pad_in=8, pad_out=8)


@pytest.mark.parametrize("n,h,w,ci,co", [
    (90, 24, 20, 40, 8),        # four 64-row tiles a workgroup, two K slices
    (40, 56, 40, 8, 8),         # three 128-row tiles
    (60, 22, 40, 128, 32),      # four 64-row tiles, four K slices (forward), four N slices (data gradient)
    (64, 22, 30, 64, 64),       # three 64-row tiles, two slices each
])
def test_conv3x3_long_ranges_equal_short_ones(B, n, h, w, ci, co):
    """Every form of the bf16 3x3 CONV gives each image of a batch (ranges of
    many tiles: the pipelined loop) bit for bit what it gives the image alone
    (ranges of one or two tiles, without the loop)."""
    x = dev(synth.normal(7, "x", (n, h, w, ci + 8), bf16=True), True)[..., :ci]
    g = dev(synth.normal(7, "g", (n, h, w, co + 8), bf16=True), True)[..., :co]
    xo = dev(synth.normal(7, "xo", (n, h, w, co), bf16=True), True)
    old = dev(synth.normal(7, "old", (n, h, w, ci), bf16=True), True)
    wt = dev(synth.conv_weight(7, "w", 3, ci, co, True), True)
    p1 = synth.bn_params(7, "bn", ci)
    gam = f32dev(p1["gamma"])
    gam[ci // 2] = 0.0                                      # its vector reads x in the z form
    mk = lambda v, c: torch.full((c,), v, device="cuda")
    bn = lambda: B.BN(gam, f32dev(p1["beta"]), 1e-5, mk(0.05, ci), mk(1.0, ci), mk(1.1, ci))
    bo = B.BN(mk(1.0, co), mk(0.0, co), 1e-5, mk(0.1, co), mk(1.0, co), mk(0.9, co))
    al, be = f32dev(synth.normal(7, "al", (co,)) * 0.1), f32dev(synth.normal(7, "be", (co,)) * 0.1)

    def forms(sl):
        xs, gs, xos, olds = x[sl], g[sl], xo[sl], old[sl].clone()
        nn = xs.shape[0]
        desc = B.desc_for(xs, gs, 3, nn, h, w)
        new = lambda c: torch.empty((nn, h, w, c), dtype=x.dtype, device="cuda")
        f32 = lambda c: torch.empty(c, device="cuda")
        o = {}
        yd = new(co + 8)                                    # (the descriptor's output stride)
        o["plain"] = yd[..., :co]
        B.bnr_conv_fwd(desc, xs, wt, o["plain"])
        o["bn"] = new(co + 8)[..., :co]
        B.bnr_bn_relu_conv_fwd(desc, xs, bn(), wt, o["bn"])
        o["bn stats"] = new(co + 8)[..., :co]
        B.bnr_bn_relu_conv_fwd(desc, xs, bn(), wt, o["bn stats"], B.BN.stats_only(co, x.device))
        o["saved z"], o["z out"], o["z stats"] = new(ci), new(co + 8)[..., :co], new(co + 8)[..., :co]
        B.bnr_bn_relu_conv_fwd_o2(desc, xs, bn(), wt, o["z out"], o["saved z"])
        B.bnr_bn_relu_conv_fwd_o2(desc, xs, bn(), wt, o["z stats"], o["saved z"], B.BN.stats_only(co, x.device))
        dense, split = B.grad_dense(gs), B.grad_split(gs, xos, bo, al, be)
        for name, src in (("dense", dense), ("split", split)):
            o[name + " dy"], o[name + " z dy"], o[name + " dx"], o[name + " dx add"] = new(ci), new(ci), new(ci), olds.clone()
            B.bnr_bwd_data(desc, xs, bn(), wt, src, f32(ci), f32(ci), o[name + " dy"])
            B.bnr_bwd_fused_o2(desc, xs, bn(), o["saved z"], wt, src, torch.empty((3, 3, ci, co), device="cuda"), f32(ci),
                               f32(ci), o[name + " z dy"])
            B.bnr_bwd_data(desc, xs, None, wt, src, dx=o[name + " dx"])
            B.bnr_bwd_data(desc, xs, None, wt, src, dx=o[name + " dx add"], dx_accumulate=True)
        y = torch.relu(xs.float() - 0.1).to(x.dtype).contiguous()
        o["relu mask"] = new(ci)
        B.bnr_reference_path(B.MODE_RCF, True, desc, xs, bn(), wt, y, g=gs, dy=o["relu mask"],
                             dw=torch.empty((3, 3, ci, co), device="cuda"), dgamma=f32(ci), dbeta=f32(ci), dx=new(ci))
        torch.cuda.synchronize()
        return o

    whole = forms(slice(0, n))
    for i in (0, 1, n // 3, n // 2, n - 2, n - 1):
        for name, t in forms(slice(i, i + 1)).items():
            assert torch.equal(whole[name][i], t[0]), "%s, image %d" % (name, i)


# The kernels with 32-bit offsets leave operands of 2 GiB and more to the general
# ones; a wide pixel stride reaches those with little work.
@pytest.mark.parametrize("bf16,k,n,h,w,ci,co", [
    (False, 1, 3, 7, 9, 36, 20),
    (False, 1, 2, 9, 11, 140, 68),
    (False, 3, 2, 5, 6, 12, 20),
    (False, 3, 3, 7, 6, 40, 72),
    (True, 1, 2, 9, 11, 64, 40),
    (True, 1, 1, 9, 13, 264, 72),
    (True, 3, 2, 6, 7, 96, 24),         # three K slices
    (True, 3, 3, 5, 6, 128, 32),
    (True, 3, 2, 9, 7, 40, 136),
])
def test_layer_on_an_input_past_2_gib(B, bf16, k, n, h, w, ci, co):
    _layer(B, bf16, k, n, h, w, ci, co, pad_out=8, wide=True)


@pytest.mark.parametrize("bf16,ci,co", [(False, 36, 20), (False, 72, 68), (True, 64, 40), (True, 264, 72)])
def test_forms_on_an_input_past_2_gib(B, bf16, ci, co):
    """The 1x1 CONV's other forms give on an input past 2 GiB what they give on
    the same values close together."""
    n, h, w, rtol = 2, 6, 10, RTOL[bf16]
    x = dev(synth.normal(8, "x", (n, h, w, ci), bf16=bf16), bf16)
    ident = dev(synth.normal(8, "id", (n, h, w, ci), bf16=bf16), bf16)
    g, gp = (dev(synth.normal(8, s, (n, h // d, w // d, co), bf16=bf16), bf16) for s, d in (("g", 1), ("gp", 2)))
    wt = dev(synth.conv_weight(8, "w", 1, ci, co, bf16), bf16)
    p1 = synth.bn_params(8, "bn", ci)
    gam = f32dev(p1["gamma"])
    gam[ci // 2] = 0.0                                      # its vector reads x in the z form
    bn = lambda: B.BN(gam, f32dev(p1["beta"]), 1e-5, f32dev(np.full(ci, 0.05)), f32dev(np.ones(ci)), f32dev(np.full(ci, 1.1)))

    def run(xv):
        new = lambda c, d=1: torch.empty((n, h // d, w // d, c), dtype=x.dtype, device="cuda")
        o, f32 = {}, lambda *s: torch.empty(s, device="cuda")
        desc = B.desc_for(xv, g, 1, n, h, w)
        o["pooled"], st = new(co, 2), B.BN.stats_only(co, x.device)
        B.bnr_bn_relu_conv_pool_fwd(desc, xv, bn(), wt, o["pooled"], st)
        o["pooled mean"], o["pooled var"] = st.mean, st.var
        o["r"], o["sum out"] = new(ci), new(co)
        B.bnr_bn_add_relu_conv_fwd(desc, xv, bn(), ident, o["r"], wt, o["sum out"], B.BN.stats_only(co, x.device))
        o["z"], o["z out"] = new(ci), new(co)
        B.bnr_bn_relu_conv_fwd_o2(desc, xv, bn(), wt, o["z out"], o["z"], B.BN.stats_only(co, x.device))
        for name, src in (("dense", B.grad_dense(g)), ("pooled gradient", B.grad_avgpool2(gp))):
            dw = o[name + " dw"] = f32(1, 1, ci, co)
            for form in ("dy", "z dy", "split", "split add", "dx", "dx add"):
                y = o[name + " " + form] = torch.full((n, h, w, ci), 0.5, dtype=x.dtype, device="cuda")
                dg, db, al, be = (torch.full((ci,), 0.5, device="cuda") for _ in range(4))
                if form == "dy":
                    B.bnr_bwd_fused(desc, xv, bn(), wt, src, dw, dg, db, y)
                elif form == "z dy":
                    B.bnr_bwd_fused_o2(desc, xv, bn(), o["z"], wt, src, f32(1, 1, ci, co), dg, db, y)
                elif form.startswith("split"):
                    B.bnr_bwd_fused_split(desc, xv, bn(), wt, src, f32(1, 1, ci, co), dg, db, y, al, be, accumulate=form == "split add")
                    o[name + " " + form + " alpha"], o[name + " " + form + " betap"] = al, be
                else:
                    B.bnr_bwd_fused(desc, xv, None, wt, src, f32(1, 1, ci, co), dx=y, dx_accumulate=form == "dx add")
                if not form.startswith("dx"):
                    o[name + " " + form + " dgamma"], o[name + " " + form + " dbeta"] = dg, db
        torch.cuda.synchronize()
        return o

    near, far = run(x), run(_wide(x))
    for name in near:
        assert_close(name, host(far[name]), host(near[name]), rtol)


@pytest.mark.parametrize("k,n,h,w,ci,co", [
    (1, 1, 1, 1, 4, 4),         # one pixel, one vector
    (1, 3, 7, 9, 36, 20),       # K and N cut inside a 16-channel product, a short last tile
    (1, 2, 8, 8, 64, 64),       # whole tiles
    (1, 5, 13, 5, 300, 68),     # ten K chunks (the last of 12 channels), two column tiles of 64
    (1, 1, 33, 2, 8, 132),      # one chunk, three column tiles
    (1, 40, 16, 15, 160, 128),  # weight gradient: several 32-pixel chunks per split
    (1, 2, 9, 7, 832, 36),      # thirteen K chunks
    (1, 1, 5, 5, 1100, 12),     # more coefficients than leave room for four workgroups
    (1, 40, 8, 51, 64, 112),    # weight gradient: half the splits (two chunks each)
    (3, 12, 24, 29, 232, 40),   # weight gradient: eight column tiles, whole rounds of splits
    (3, 2, 1, 1, 4, 8),         # one pixel: the centre tap only
    (3, 1, 5, 62, 32, 32),      # widest rows: the longest halo, one row per weight-gradient chunk
    (3, 3, 7, 6, 20, 36),       # ragged channels, eight rows of positions in a chunk
    (3, 9, 14, 14, 128, 32),    # chunks that end inside an image
    (3, 2, 3, 2, 40, 100),      # two column tiles; images lower than a chunk
])
def test_conv_f32_tiles(B, k, n, h, w, ci, co):
    _layer(B, False, k, n, h, w, ci, co, pad_in=4, pad_out=8)


def test_conv3x3_nan_and_inf_stay_local(B):
    """A NaN input is dropped by the ReLU (max(NaN, 0) = 0), an infinite one
    reaches exactly the 3x3 outputs that read it; padding rows of the input
    ring are zeros whatever their neighbours hold."""
    n, h, w, ci, co = 2, 9, 9, 64, 32
    x = torch.zeros((n, h, w, ci), dtype=torch.bfloat16, device="cuda")
    x[0, 0, 8, 3] = float("nan")
    x[1, 4, 0, 5] = float("inf")
    ones, zeros = torch.ones(ci, device="cuda"), torch.zeros(ci, device="cuda")
    bn = B.BN(ones.clone(), zeros.clone(), 1e-5, zeros.clone(), ones.clone(), ones.clone())
    wt = torch.ones((3, 3, ci, co), dtype=torch.bfloat16, device="cuda")
    out = torch.empty((n, h, w, co), dtype=torch.bfloat16, device="cuda")
    B.bnr_bn_relu_conv_fwd(B.desc_for(x, out, 3, n, h, w), x, bn, wt, out)
    torch.cuda.synchronize()
    want = torch.zeros((n, h, w))
    want[1, 3:6, 0:2] = float("inf")
    got = out.float().cpu()
    assert bool((got == want[..., None]).all())


@pytest.mark.parametrize("bf16,n,h,w,c", [
    (True, 1, 1, 1, 8),         # one pixel, one vector
    (False, 1, 2, 3, 4),
    (True, 2, 5, 128, 64),      # widest rows: every thread a window column
    (False, 2, 4, 127, 64),     # the same with an odd last column, float32 vectors
    (True, 60, 35, 9, 16),      # chunks of two row pairs
    (False, 150, 35, 6, 8),     # chunks of three
    (True, 1100, 5, 4, 8),      # more images than places: whole images as chunks
    (True, 33, 6, 66, 64),      # workgroups of five waves
    (True, 115, 18, 5, 32),     # chunks of two, the last of an image one pair
    (True, 2500, 5, 4, 8),      # more images than workgroups: several chunks each
    (False, 300, 21, 30, 64),   # more images than places: images split
    (True, 70, 9, 128, 64),     # the widest workgroups, one on a CU
])
def test_maxpool_bwd_chunks(B, bf16, n, h, w, c):
    """Small whole numbers (many ties) and whole-number gradients: every sum is
    exact, so the result equals the oracle's."""
    rng = np.random.default_rng(5)
    x = rng.integers(-3, 4, size=(n, h, w, c)).astype(np.float64)
    ho, wo = (h - 1) // 2 + 1, (w - 1) // 2 + 1
    gy = rng.integers(-8, 9, size=(n, ho, wo, c)).astype(np.float64)
    xd, gd = dev(x, bf16), dev(gy, bf16)
    dz = torch.full((n, h, w, c), 9.0, dtype=xd.dtype, device=xd.device)
    B.bnr_maxpool_bn_bwd(xd, None, gd, dz, n, h, w)
    torch.cuda.synchronize()
    ref = P.maxpool_bwd(x, gy, 3, 2, 1)
    np.testing.assert_array_equal(host(dz), ref)
    # with a BN of unit scale and an offset that no input cancels, the mask is exact too
    ones, zeros = torch.ones(c, device="cuda"), torch.zeros(c, device="cuda")
    bn = B.BN(ones.clone(), torch.full((c,), 0.5, device="cuda"), 1e-5, zeros.clone(), ones.clone(), ones.clone())
    dg, db = torch.empty(c, device="cuda"), torch.empty(c, device="cuda")
    B.bnr_maxpool_bn_bwd(xd, bn, gd, dz, n, h, w, dg, db)
    torch.cuda.synchronize()
    refy = P.maxpool_bwd(P.relu_fwd(x + 0.5), gy, 3, 2, 1) * (x + 0.5 > 0)
    np.testing.assert_array_equal(host(dz), refy)
    np.testing.assert_allclose(host(db), refy.reshape(-1, c).sum(0), rtol=0, atol=1e-6 * np.abs(refy).sum() / c + 1e-6)
    np.testing.assert_allclose(host(dg), (refy * x).reshape(-1, c).sum(0), rtol=0, atol=4e-6 * np.abs(refy).sum() / c + 1e-6)


@pytest.mark.parametrize("bf16", [True, False])
def test_maxpool_bwd_rows_past_2_gib(B, bf16):
    """An input view whose image rows span more than 2^31 bytes (64-bit offsets in a row)."""
    h, w, c = 3, 2, 8
    ldc = (1 << 31) // (2 if bf16 else 4)
    rng = np.random.default_rng(5)
    x = rng.integers(-3, 4, size=(1, h, w, c)).astype(np.float64)
    gy = rng.integers(-8, 9, size=(1, 2, 1, c)).astype(np.float64)
    buf = torch.empty((h * w - 1) * ldc + c, dtype=torch.bfloat16 if bf16 else torch.float32, device="cuda")
    xd = buf.as_strided((1, h, w, c), (h * w * ldc, w * ldc, ldc, 1))
    xd.copy_(dev(x, bf16))
    dz = torch.full((1, h, w, c), 9.0, dtype=xd.dtype, device="cuda")
    B.bnr_maxpool_bn_bwd(xd, None, dev(gy, bf16), dz, 1, h, w)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(host(dz), P.maxpool_bwd(x, gy, 3, 2, 1))


@pytest.mark.parametrize("n,h,w,c_in", [(1, 1, 1, 3), (3, 9, 255, 3), (2, 256, 256, 4), (700, 5, 6, 1), (3, 11, 64, 3),
                                        (3, 11, 65, 3)])
def test_stem_wgrad_items(B, n, h, w, c_in):
    """Weight gradient of the first CONV at the ends of its staging slots: one
    output pixel, the widest image (all slots), an odd last row, more items
    than workgroups, the widest image of the kernel with few slots and one more.  Whole numbers: exact in bf16 and in float32 sums."""
    rng = np.random.default_rng(6)
    ho, wo = (h - 1) // 2 + 1, (w - 1) // 2 + 1
    img = np.zeros((n, h, w, 4))
    img[..., :c_in] = rng.integers(-2, 3, size=(n, h, w, c_in))
    g = rng.integers(-2, 3, size=(n, ho, wo, 64)).astype(np.float64)
    dw = torch.empty((7, 7, c_in, 64), dtype=torch.float32, device="cuda")
    B.bnr_stem_wgrad(dev(img, True), c_in, B.grad_dense(dev(g, True)), dw)
    torch.cuda.synchronize()
    ip = np.pad(img[..., :c_in], ((0, 0), (3, 4), (3, 4), (0, 0)))
    ref = np.empty((7, 7, c_in, 64))
    for a in range(7):
        for b in range(7):
            ref[a, b] = ip[:, a:a + 2 * ho:2, b:b + 2 * wo:2].reshape(-1, c_in).T @ g.reshape(-1, 64)
    np.testing.assert_array_equal(host(dw), ref)


@pytest.mark.parametrize("n,h,w,ci,co", [
    (1, 2, 2, 8, 8),            # one window, one vector
    (1, 6, 10, 136, 72),        # a short window tile, two column tiles, two K chunks (the last of 8 channels)
    (3, 14, 14, 264, 264),      # N and K past the persistent kernel, ragged
    (8, 32, 32, 32, 64),        # whole 32-window tiles, one K chunk
    (64, 46, 46, 256, 40),      # 64-window tiles, the last one short
])
def test_pooled_gradient_forms(B, n, h, w, ci, co):
    """The 1x1 data gradient of a pooled gradient runs over windows: every form
    of its epilogue against the oracle, and its sums against the general kernels'
    on the gradient written out per pixel (g / 4 is exact)."""
    rtol, m = RTOL[True], n * h * w
    x = dev(synth.normal(5, "x", (n, h, w, ci + 8), bf16=True), True)[..., :ci]
    gp = dev(synth.normal(5, "g", (n, h // 2, w // 2, co + 8), bf16=True), True)[..., :co]
    wd = dev(synth.conv_weight(5, "w", 1, ci, co, True), True)
    up = (gp * 0.25).repeat_interleave(2, 1).repeat_interleave(2, 2).contiguous()
    p1 = synth.bn_params(5, "bn1", ci)
    gam = f32dev(p1["gamma"])
    gam[ci // 2] = 0.0                                      # its vector reads x in the z form
    bn = B.BN(gam, f32dev(p1["beta"]), 1e-5, x.reshape(-1, ci).float().mean(0).contiguous(),
              torch.ones(ci, device="cuda"), torch.full((ci,), 1.25, device="cuda"))
    z = torch.relu((x.float() - bn.mean) * bn.rstd * bn.gamma + bn.beta).to(torch.bfloat16).contiguous()
    desc = B.desc_for(x, up, 1, n, h, w)
    # the oracle's tensors
    x64, w64 = host(x), host(wd)
    k64 = host(bn.rstd) * host(gam)
    y64 = (x64 - host(bn.mean)) * k64 + host(bn.beta)
    g64 = P.avgpool2_bwd(host(gp), (h, w))
    dz = P.conv_dgrad(g64, w64, (h, w))
    dy = P.relu_bwd(dz, y64)
    amb = relu_ambiguous(y64, True)
    want = dict(bn=dy, z=dy, split=k64 * dy, split_acc=3.0 + k64 * dy, store=dz, store_acc=3.0 + dz)
    dw_bn, dw_x = P.conv_wgrad(bf16_round(P.relu_fwd(y64)), g64, 1), P.conv_wgrad(x64, g64, 1)

    def run(src, form):
        o = dict(dw=torch.empty(tuple(wd.shape), device="cuda"))
        o.update({k: torch.full((ci,), 0.5, device="cuda") for k in ("dgamma", "dbeta", "alpha", "betap")})
        y = torch.full((n, h, w, ci + 8), 3.0, dtype=x.dtype, device="cuda")
        B.workspace(B.bnr_workspace_size(desc), x.device)
        B._ws_cache[(x.device, 0)].fill_(255)
        if form == "bn":
            o["y"] = torch.empty((n, h, w, ci), dtype=x.dtype, device="cuda")
            B.bnr_bwd_fused(desc, x, bn, wd, src, o["dw"], o["dgamma"], o["dbeta"], o["y"])
        elif form == "z":
            o["y"] = torch.empty((n, h, w, ci), dtype=x.dtype, device="cuda")
            B.bnr_bwd_fused_o2(desc, x, bn, z, wd, src, o["dw"], o["dgamma"], o["dbeta"], o["y"])
        elif form.startswith("split"):
            B.bnr_bwd_fused_split(desc, x, bn, wd, src, o["dw"], o["dgamma"], o["dbeta"], y[..., :ci], o["alpha"],
                                  o["betap"], accumulate=form == "split_acc")
            o["y"] = y[..., :ci]
        else:
            B.bnr_bwd_fused(desc, x, None, wd, src, o["dw"], dx=y[..., :ci], dx_accumulate=form == "store_acc")
            o["y"] = y[..., :ci]
        torch.cuda.synchronize()
        assert bool((y[..., ci:] == 3.0).all()), form + " wrote past its channels"
        return o

    for form in ("bn", "z", "split", "split_acc", "store", "store_acc"):
        got, ref = run(B.grad_avgpool2(gp), form), run(B.grad_dense(up), form)
        assert_close(form + " y", host(got["y"]), want[form], rtol, exclude=None if form.startswith("store") else amb)
        assert_close(form + " dw", host(got["dw"]), dw_x if form.startswith("store") else dw_bn, rtol)
        if form in ("bn", "z"):                             # the sums are of the dy that was stored
            d = host(got["y"]).reshape(m, ci)
            xh = (host(x).reshape(m, ci) - host(bn.mean)) * host(bn.rstd)
            assert np.all(np.abs(host(got["dbeta"]) - d.sum(0)) <= 1e-5 * np.abs(d).sum(0) + 1e-6)
            if form == "z":                                 # xhat from z: the general kernel's, from the same z
                assert_close("z dgamma", host(got["dgamma"]), host(ref["dgamma"]), 1e-5)
            else:
                assert np.all(np.abs(host(got["dgamma"]) - (d * xh).sum(0)) <= 1e-5 * np.abs(d * xh).sum(0) + 1e-6)
        else:
            for k in ("dgamma", "dbeta", "alpha", "betap"):
                assert_close(form + " " + k, host(got[k]), host(ref[k]), rtol)
