"""GPU parity where the choice of kernel or tile turns on the size of the grid or on the
channel count: eight-wave tiles on grids that fill rounds of the GPU; small grids whose waves split the reduction (32 x 32, 32 x 64 and 64 x 64
tiles), 8-multiple channel counts on the halo and direct-to-LDS kernels, 128-row halo tiles
of 64 to 95 columns, weight-gradient patches and channel chunks that pass the image or the
channels, and short pixel splits.  Against the fp64 oracle, rel_inf <= 2e-2 (bf16 outputs and
gradients) and the statistics' own bound."""
import numpy as np
import pytest

import oracle
from oracle import ConvShape
from parity import Inputs, assert_close, assert_stats, f64
from paper_2609_10632_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if torch.cuda.is_available():
    from paper_2609_10632_amd import blocks
    from paper_2609_10632_amd import numbat as nb

EPS = 1e-3
# n, h, w, ci, co, k, s
CASES = [
    # reduction-splitting forward: 32 x 32 tiles (a ragged row and column tile; a reduction that
    # ends mid-step; 1x1; stride 2), 32 x 64, 64 x 64
    (1, 20, 20, 576, 72, 3, 1), (1, 9, 7, 120, 40, 3, 1), (2, 5, 5, 1152, 64, 1, 1), (1, 13, 17, 136, 48, 3, 2),
    (3, 28, 28, 200, 136, 3, 1), (5, 28, 28, 264, 136, 3, 1),
    # ... data gradient: 32 x 32 tiles at stride 1 (the plain case and c_out that ends a
    # chunk early) and over four stride phases, 64 x 64 over four phases
    (1, 12, 10, 40, 288, 3, 1), (1, 11, 11, 24, 136, 3, 1), (1, 13, 17, 40, 272, 3, 2), (1, 34, 30, 264, 576, 3, 2),
    # 8-multiple channel counts: halo (one chunk and a tail, 8 channels, 128-row tiles of 70
    # columns, two-dimensional tiles), direct-to-LDS (1x1, stride 2, more than 32768 rows)
    (2, 30, 30, 24, 72, 3, 1), (2, 12, 62, 8, 16, 3, 1), (1, 21, 70, 40, 56, 3, 1), (1, 64, 96, 24, 40, 3, 1),
    (2, 35, 35, 104, 80, 1, 1), (2, 31, 29, 24, 40, 3, 2), (4, 190, 190, 88, 24, 3, 2), (2, 140, 130, 24, 56, 1, 1), (2, 19, 17, 56, 88, 1, 1),
    # two halo tiles of 64 columns for 80 channels
    (2, 33, 41, 64, 80, 3, 1),
    # patch-staged weight gradient past the image and the channels: 52 x 52 on 20 x 4, 13 x 37,
    # 72 of 96 and 40 of 64 rows; 1x1 chunks of which the last ends early
    (2, 52, 52, 64, 80, 3, 1), (2, 31, 45, 88, 72, 3, 1), (3, 18, 31, 144, 40, 3, 1), (2, 9, 31, 280, 48, 1, 1),
    # the general weight gradient on splits of 4 steps
    (2, 32, 32, 16, 32, 3, 1), (1, 60, 61, 16, 24, 3, 2),
    # eight-wave halo tiles of 256 rows, forward or data gradient: up to 63 columns, 64 to 95, and
    # two-dimensional; a last chunk of 8 or 16 channels, a ragged last row tile
    (9, 40, 41, 48, 288, 3, 1), (9, 40, 41, 288, 40, 3, 1), (3, 70, 71, 40, 288, 3, 1), (3, 70, 71, 288, 48, 3, 1),
    (8, 160, 160, 16, 64, 3, 1),
    # eight-wave direct-to-LDS tiles: 256 x 192, 256 x 128 (1x1 and stride 2) and 128 x 128
    (5, 57, 57, 264, 576, 1, 1), (5, 60, 60, 576, 40, 1, 1), (5, 75, 75, 256, 248, 1, 1), (10, 95, 94, 40, 248, 3, 2),
    (3, 37, 37, 72, 576, 1, 1), (2, 50, 58, 640, 48, 1, 1),
    # 80 columns as one tile of 96 (as two of 64 above)
    (12, 40, 40, 40, 80, 3, 1),
    # short reductions into many rows on tiles of 96 and 128 columns
    (1, 190, 190, 16, 168, 1, 1), (1, 190, 190, 104, 24, 1, 1),
]
IDS = ["n{}h{}w{}ci{}co{}k{}s{}".format(*c) for c in CASES]


@pytest.mark.parametrize("i", range(len(CASES)), ids=IDS)
def test_conv_passes(i):
    """Forward with statistics, data gradient (plain and accumulated) and weight gradient (plain
    and accumulated) on channel slices of wider tensors, whose other channels stay as they were."""
    n, h, w, ci, co, k, st = CASES[i]
    s = ConvShape(n, h, w, ci, co, k, k, st, st, k // 2, k // 2)
    ip = Inputs(140, i)
    xp, yp = ci + 16, co + 8
    xb, dyb = ip.normal((n, h, w, xp), synth.T_X), ip.normal((*s.y_shape[:3], yp), synth.T_DY)
    d0, wb = ip.normal((n, h, w, xp), synth.T_RES), ip.weight(co, k, ci)
    blk = blocks.ConvBlock(n, h, w, ci, co, k, st, x_pixel_stride=xp, y_pixel_stride=yp)
    ws = blocks.workspace(blk.ws_bytes())
    x, dy, wt = blocks.dev_bf16(xb)[..., 16:], blocks.dev_bf16(dyb)[..., 8:], blocks.dev_bf16(wb)
    y = torch.full((*s.y_shape[:3], yp), 7.0, dtype=torch.bfloat16, device="cuda")
    stats = torch.empty(2 * co, device="cuda")
    dx, dxa = torch.full((n, h, w, xp), 7.0, dtype=torch.bfloat16, device="cuda"), blocks.dev_bf16(d0)
    dw = torch.full(s.w_shape, float("nan"), device="cuda")
    nb.numbat_conv_fwd(blk.prob, x, wt, y[..., 8:], stats, ws)
    nb.numbat_conv_bwd_data(blk.prob, dy, wt, dx[..., 16:], False, ws)
    nb.numbat_conv_bwd_data(blk.prob, dy, wt, dxa[..., 16:], True, ws)
    nb.numbat_conv_bwd_weight(blk.prob, x, dy, dw, False, ws)
    dwa = dw.clone()
    nb.numbat_conv_bwd_weight(blk.prob, x, dy, dwa, True, ws)
    torch.cuda.synchronize()
    x64, dy64, w64 = f64(xb[..., 16:]), f64(dyb[..., 8:]), f64(wb)
    yref = oracle.conv_fwd(x64, w64, s)
    got = blocks.host_f64(y)
    assert_close(got[..., 8:], yref, "y")
    assert np.all(got[..., :8] == 7.0)
    mref, vref = oracle.bn_stats(yref)
    sg = blocks.host_f64(stats)
    assert_stats(sg[:co], sg[co:], mref, vref, EPS, "batch statistics")
    dxref = oracle.conv_dgrad(dy64, w64, s)
    got = blocks.host_f64(dx)
    assert_close(got[..., 16:], dxref, "dx")
    assert np.all(got[..., :16] == 7.0)
    got = blocks.host_f64(dxa)
    assert_close(got[..., 16:], dxref + f64(d0[..., 16:]), "dx accumulated")
    assert np.array_equal(got[..., :16], f64(d0[..., :16]))
    dwref = oracle.conv_wgrad(x64, dy64, s)
    # fp32 sums: the weight gradient's own error is far below the bf16 bound
    assert_close(blocks.host_f64(dw), dwref, "dw", 1e-5)
    assert_close(blocks.host_f64(dwa), 2 * dwref, "dw accumulated", 1e-5)


# split tiles and a halo tile; eight-wave halo tiles, linear (two widths) and two-dimensional;
# 256 x 192, 256 x 128 and 128 x 128 direct-to-LDS tiles
INFER = [0, 1, 4, 5, 10] + [CASES.index(c) for c in ((9, 40, 41, 48, 288, 3, 1), (3, 70, 71, 40, 288, 3, 1),
                                                     (8, 160, 160, 16, 64, 3, 1), (5, 57, 57, 264, 576, 1, 1),
                                                     (5, 75, 75, 256, 248, 1, 1), (3, 37, 37, 72, 576, 1, 1))]


@pytest.mark.parametrize("i", INFER, ids=[IDS[i] for i in INFER])
def test_inference_outputs(i):
    """The bias and the evaluation-mode BN + SiLU output stages on those tiles."""
    n, h, w, ci, co, k, st = CASES[i]
    s = ConvShape(n, h, w, ci, co, k, k, st, st, k // 2, k // 2)
    ip = Inputs(141, i)
    xb, wb = ip.normal(s.x_shape, synth.T_X), ip.weight(co, k, ci)
    f = lambda a: a.astype(np.float64)
    bias, g = ip.f32_normal((co,), synth.T_RES, 0.0, 0.5), ip.f32_uniform((co,), synth.T_GAMMA, 0.5, 1.5)
    b, m, v = (ip.f32_normal((co,), synth.T_BETA, 0.0, 0.1), ip.f32_normal((co,), synth.T_MEAN, 0.0, 0.2),
               ip.f32_uniform((co,), synth.T_VAR, 0.3, 2.0))
    p = nb.conv_problem(n, h, w, ci, co, k, stride=st)
    x, wt = blocks.dev_bf16(xb), blocks.dev_bf16(wb)
    y1 = torch.empty(s.y_shape, dtype=torch.bfloat16, device="cuda")
    y2 = torch.empty_like(y1)
    nb.numbat_conv_fwd_bias(p, x, wt, blocks.dev_f32(bias), y1)
    nb.numbat_conv_bn_silu_infer(p, x, wt, *(blocks.dev_f32(t) for t in (g, b, m, v)), EPS, y2)
    torch.cuda.synchronize()
    yref = oracle.conv_fwd(f64(xb), f64(wb), s)
    assert_close(blocks.host_f64(y1), yref + f(bias), "conv + bias")
    assert_close(blocks.host_f64(y2), oracle.bn_silu_eval(yref, f(m), f(v), f(g), f(b), EPS), "conv + eval BN + SiLU")


# rows, channels: at most five partials a thread (the apply adds them itself) and just past
# it; one partial; more channels than threads
@pytest.mark.parametrize("m,c", [(65536, 32), (65537, 32), (300, 8), (784, 288), (785, 288), (16, 2048), (50, 264),
                                 (20480, 32), (20481, 32), (320, 256), (321, 256), (500, 200)])
def test_bn_backward_folds_few_partials(m, c):
    ip = Inputs(142, c)
    yb, gb = ip.normal((m, c), synth.T_Y, 0.3, 2.0), ip.normal((m, c), synth.T_G)
    gamma, beta = ip.f32_uniform((c,), synth.T_GAMMA, 0.5, 1.5), ip.f32_normal((c,), synth.T_BETA, 0.0, 0.3)
    mean, var = oracle.bn_stats(f64(yb))
    mean32, rstd32 = mean.astype(np.float32), (1 / np.sqrt(var + EPS)).astype(np.float32)
    p = nb.bn_problem(m, c, EPS)
    dy = torch.empty((m, c), dtype=torch.bfloat16, device="cuda")
    dgamma, dbeta = torch.empty(c, device="cuda"), torch.empty(c, device="cuda")
    ws = blocks.workspace(nb.numbat_workspace_size(nb.OP_BN_SILU_BWD, p))
    dev = [blocks.dev_f32(t) for t in (mean32, rstd32, gamma, beta)]
    nb.numbat_bn_silu_bwd(p, blocks.dev_bf16(gb), blocks.dev_bf16(yb), *dev, dy, dgamma, dbeta, None, ws=ws)
    torch.cuda.synchronize()
    ref = oracle.bn_silu_bwd(f64(gb), f64(yb), mean, var, gamma.astype(np.float64), beta.astype(np.float64), EPS)
    for got, want, name in zip((dy, dgamma, dbeta), ref, ("dy", "dgamma", "dbeta")):
        assert_close(blocks.host_f64(got), want, name)


@pytest.mark.parametrize("shape", [(1, 20, 20, 288, 288), (1, 12, 10, 48, 288), (9, 40, 41, 288, 48),
                                   (3, 70, 71, 288, 48), (8, 160, 160, 64, 48)])
def test_backward_prologue_equals_the_two_calls(shape):
    """numbat_conv_bwd_data_bn_silu_prologue where the data gradient's waves split the reduction
    or run on eight-wave halo tiles: dx (accumulated) and dy equal numbat_bn_silu_bwd followed by
    numbat_conv_bwd_data bit for bit."""
    n, h, w, ci, co = shape
    ip = Inputs(143, ci)
    blk = blocks.ConvBlock(n, h, w, ci, co, 3, 1)
    g, y = blocks.dev_bf16(ip.normal((n, h, w, co + 8), synth.T_G)), blocks.dev_bf16(ip.normal((n, h, w, co), synth.T_Y))
    wt, x0 = blocks.dev_bf16(ip.weight(co, 3, ci)), blocks.dev_bf16(ip.normal((n, h, w, ci), synth.T_RES))
    mean, rstd, gamma, beta = (blocks.dev_f32(ip.f32_uniform((co,), t, 0.5, 1.5)) for t in
                               (synth.T_MEAN, synth.T_VAR, synth.T_GAMMA, synth.T_BETA))
    ws = blocks.workspace(blk.ws_bytes())
    dy, dy2 = torch.empty_like(y), torch.empty_like(y)
    dx, dx2 = x0.clone(), x0.clone()
    dgamma, dbeta = torch.empty(co, device="cuda"), torch.empty(co, device="cuda")
    bn = blk.bn(a_pixel_stride=co + 8)
    nb.numbat_bn_silu_bwd(bn, g, y, mean, rstd, gamma, beta, dy, dgamma, dbeta, None, ws=ws)
    nb.numbat_conv_bwd_data(blk.prob, dy, wt, dx, True, ws)
    nb.numbat_conv_bwd_data_bn_silu_prologue(blk.prob, g, y, mean, rstd, gamma, beta, dgamma, dbeta, wt, dx2, dy2, True,
                                             g_pixel_stride=co + 8)
    torch.cuda.synchronize()
    assert torch.equal(dy.view(torch.int16), dy2.view(torch.int16))
    assert torch.equal(dx.view(torch.int16), dx2.view(torch.int16))


@pytest.mark.parametrize("shape", [(9, 40, 41, 48, 288), (3, 70, 71, 48, 288), (8, 160, 160, 48, 64)])
def test_forward_prologue_equals_the_two_calls(shape):
    """numbat_conv_fwd_bn_silu_prologue on eight-wave halo tiles: y and the batch statistics equal
    numbat_bn_silu_fwd followed by numbat_conv_fwd bit for bit."""
    n, h, w, ci, co = shape
    ip = Inputs(144, ci)
    blk = blocks.ConvBlock(n, h, w, ci, co, 3, 1)
    y0, wt = blocks.dev_bf16(ip.normal((n, h, w, ci), synth.T_Y)), blocks.dev_bf16(ip.weight(co, 3, ci))
    stats0 = blocks.dev_f32(ip.f32_uniform((2 * ci,), synth.T_VAR, 0.3, 2.0))
    gamma = blocks.dev_f32(ip.f32_uniform((ci,), synth.T_GAMMA, 0.5, 1.5))
    beta = blocks.dev_f32(ip.f32_normal((ci,), synth.T_BETA, 0.0, 0.3))
    ws = blocks.workspace(max(blk.ws_bytes(), 256))
    a, sm, sr = torch.empty_like(y0), torch.empty(ci, device="cuda"), torch.empty(ci, device="cuda")
    y = [torch.empty((n, h, w, co), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    st = [torch.empty(2 * co, device="cuda") for _ in range(2)]
    nb.numbat_bn_silu_fwd(nb.bn_problem(n * h * w, ci, EPS), y0, stats0, gamma, beta, None, a, sm, sr, ws=ws)
    nb.numbat_conv_fwd(blk.prob, a, wt, y[0], st[0], ws)
    nb.numbat_conv_fwd_bn_silu_prologue(blk.prob, y0, stats0, gamma, beta, EPS, wt, y[1], st[1], ws)
    torch.cuda.synchronize()
    assert torch.equal(y[0].view(torch.int16), y[1].view(torch.int16))
    assert torch.equal(st[0].view(torch.int32), st[1].view(torch.int32))


# patches that pass the image's last row: 20 x 4, 8 x 16 (96-row tiles and a chunk that ends early;
# 48-channel chunks; all but one row outside), 20 x 8; sizes whose patches' slices would pass it,
# and the last column, on the general kernel
@pytest.mark.parametrize("shape", [(2, 52, 52, 64, 80), (2, 45, 48, 88, 96), (3, 22, 32, 144, 40), (5, 41, 16, 32, 64),
                                   (2, 30, 40, 32, 64), (2, 31, 45, 88, 72), (3, 18, 31, 144, 40), (9, 19, 7, 32, 64),
                                   # (grids that fill the patch-staged kernel's block slots: 8 x 16, on
                                   # 96 rows and on 48-channel chunks, and 20 x 8)
                                   (4, 45, 48, 96, 192), (9, 22, 32, 144, 64), (12, 58, 24, 64, 64)])
def test_weight_gradient_keeps_infinities_to_their_taps(shape):
    """An infinity in the input's last row and a NaN in its last column reach the gradients of the
    taps that pair them with an output pixel, and no other."""
    n, h, w, ci, co = shape
    s = ConvShape(n, h, w, ci, co, 3, 3, 1, 1, 1, 1)
    ip = Inputs(145, ci)
    xb, dyb = ip.normal(s.x_shape, synth.T_X), ip.normal(s.y_shape, synth.T_DY)
    xb[0, h - 1, w // 2, 1], xb[n - 1, h // 2, w - 1, 9], xb[n - 1, h - 1, w - 1, ci - 1] = 0x7f80, 0x7fc0, 0xff80
    blk = blocks.ConvBlock(n, h, w, ci, co, 3, 1)
    dw = torch.empty(s.w_shape, device="cuda")
    nb.numbat_conv_bwd_weight(blk.prob, blocks.dev_bf16(xb), blocks.dev_bf16(dyb), dw, False, blocks.workspace(blk.ws_bytes()))
    torch.cuda.synchronize()
    got = blocks.host_f64(dw)
    # (the infinite input pixels' products by hand: the oracle's padding is not asked about them)
    x64, dy64 = f64(xb), f64(dyb)
    bad = ~np.isfinite(x64)
    want = oracle.conv_wgrad(np.where(bad, 0.0, x64), dy64, s)
    hit = np.zeros(s.w_shape, bool)
    for img, i, j, c in np.argwhere(bad):
        for r in range(3):
            for q in range(3):
                if 0 <= i + 1 - r < h and 0 <= j + 1 - q < w:
                    hit[:, r, q, c] = True
    assert hit.any() and not hit.all()
    assert not np.isfinite(got[hit]).any()
    assert np.isfinite(got[~hit]).all()
    assert_close(np.where(hit, 0.0, got), np.where(hit, 0.0, want), "dw", 1e-5)
