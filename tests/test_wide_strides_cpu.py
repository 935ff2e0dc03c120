"""Which kernel takes a problem whose strides reach the limits of 31-bit byte offsets, without a
GPU: every check has passed when the launch itself reports that there is no device, so a
refusal by a launcher ("invalid argument") or a launch that should not be made shows in the
status text.  Nothing is launched."""
import pytest

from paper_2609_10632_amd import numbat as nb

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.skipif(torch.cuda.is_available(), reason="launches would run: the pointers are not memory")

FAKE = 1 << 20
BIG = 1 << 50  # bytes: no workspace check refuses


def device_error(fn, *a, **k):
    """The detail text of a call that reaches a launch."""
    with pytest.raises(nb.NumbatError) as ei:
        fn(*a, **k)
    assert ei.value.status == nb.ERR_DEVICE, ei.value
    text = nb.numbat_last_error()
    assert "invalid argument" not in text, text
    return text


def fwd(p):
    return device_error(nb.numbat_conv_fwd, p, FAKE, FAKE, FAKE)


def bwd_data(p):
    return device_error(nb.numbat_conv_bwd_data, p, FAKE, FAKE, FAKE, False, FAKE, ws_bytes=BIG)


# small grids with long reductions (one image, or the few tiles of a strided layer) whose images
# span over a gigabyte: n, h, w, ci, co, k, s, x stride, y stride
SPANS = [(1, 20, 20, 288, 288, 3, 1, 1300000, 1300000), (1, 360, 360, 4160, 32, 5, 4, 0, 0),
         (1, 512, 512, 2304, 64, 5, 4, 0, 0), (1, 64, 64, 32, 128, 3, 1, 0, 131072),
         (2, 20, 20, 288, 288, 3, 1, 1300000, 1300000)]


@pytest.mark.parametrize("c", SPANS, ids=lambda c: "x".join(map(str, c)))
def test_spans_of_two_images_past_31_bits(c):
    n, h, w, ci, co, k, s, xp, yp = c
    p = nb.conv_problem(n, h, w, ci, co, k, stride=s, x_pixel_stride=xp, y_pixel_stride=yp)
    assert fwd(p).startswith("conv forward launch")
    bwd_data(p)


@pytest.mark.parametrize("c", [(1, 20, 20, 288, 288, 1300000), (1, 64, 64, 32, 128, 131072)])
def test_backward_prologue_without_a_workspace(c):
    """The entry has no workspace, so it must not come to a data gradient that re-lays its weights
    out in one: on these problems the halo kernel forms dy."""
    n, h, w, ci, co, yp = c
    p = nb.conv_problem(n, h, w, ci, co, 3, y_pixel_stride=yp)
    assert nb.numbat_workspace_size(nb.OP_CONV_BWD_DATA_BN_SILU, p) == 0
    assert device_error(nb.numbat_conv_bwd_data_bn_silu_prologue, p, *([FAKE] * 11)).startswith("data-gradient launch")
    # the halo kernel is the data gradient's own too
    assert bwd_data(p).startswith("data-gradient launch")


@pytest.mark.parametrize("n,h,w,ci,co,last", [(1, 20, 20, 288, 48, 169), (1, 16, 70, 96, 64, 269), (1, 8, 96, 64, 48, 897)])
def test_prologues_up_to_the_halo_of_their_tile(n, h, w, ci, co, last):
    """The prologue entries have no other kernel to fall back on: they take every pixel stride with
    which the last halo pixel of their own tile is within 31-bit byte offsets, and refuse the
    first that is not (`last`: that pixel, from the tile's first)."""
    fits = (0x7ffffff0 - 64) // (2 * last) // 8 * 8
    for stride in (fits - 8, fits + 8):
        ok = stride < fits
        p = nb.conv_problem(n, h, w, ci, co, 3, y_pixel_stride=stride)
        q = nb.conv_problem(n, h, w, co, ci, 3, x_pixel_stride=stride)
        bwd = (nb.numbat_conv_bwd_data_bn_silu_prologue, p, *([FAKE] * 11))
        fwd = (nb.numbat_conv_fwd_bn_silu_prologue, q, FAKE, FAKE, FAKE, FAKE, 1e-3, FAKE, FAKE)
        # (the incoming gradient's own pixel stride)
        g = (nb.numbat_conv_bwd_data_bn_silu_prologue, nb.conv_problem(n, h, w, ci, co, 3), *([FAKE] * 11))
        for (fn, *args), kw in ((bwd, {}), (fwd, {}), (g, {"g_pixel_stride": stride})):
            if ok:
                device_error(fn, *args, **kw)
            else:
                with pytest.raises(nb.NumbatError) as ei:
                    fn(*args, **kw)
                assert ei.value.status == nb.ERR_UNSUPPORTED, ei.value
