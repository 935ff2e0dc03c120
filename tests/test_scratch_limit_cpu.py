"""Problems whose statistics partials fill the static scratch of numbat_conv_fwd_noalloc (8 MiB,
header included) with 256-row tiles stay within it, whichever kernel their channel count
takes (workspace sizes need no GPU)."""
import pytest

from paper_2609_10632_amd import numbat as nb

SCRATCH = 8 << 20


# n, h, w, ci, co, k, s: channel counts that are no multiple of 16, or below 32, on images the
# halo kernel takes, on 1x1 and on strided layers; 256-row partials just under the scratch
@pytest.mark.parametrize("c", [(400, 60, 60, 24, 184, 3, 1), (400, 60, 60, 40, 184, 1, 1), (400, 119, 119, 16, 184, 3, 2),
                               (160, 95, 94, 8, 184, 3, 1)])
def test_partials_fit_the_static_scratch(c):
    n, h, w, ci, co, k, s = c
    p = nb.conv_problem(n, h, w, ci, co, k, stride=s)
    ho, wo = nb.numbat_conv_output_shape(p)
    rows = -(-n * ho * wo // 256)
    assert rows * co * 8 + 512 <= SCRATCH  # what 256-row tiles need
    assert nb.numbat_workspace_size(nb.OP_CONV_FWD, p) <= SCRATCH


# 256-row partials past the scratch too: nothing is gained on other tiles, so such a problem keeps the
# 128-row tiles of the kernel it would take without the limit
@pytest.mark.parametrize("c", [(400, 60, 60, 40, 400, 1, 1), (400, 60, 60, 24, 400, 1, 1)])
def test_partials_past_the_static_scratch(c):
    n, h, w, ci, co, k, s = c
    p = nb.conv_problem(n, h, w, ci, co, k, stride=s)
    assert -(-n * h * w // 256) * co * 8 > SCRATCH
    assert nb.numbat_workspace_size(nb.OP_CONV_FWD, p) >= -(-n * h * w // 128) * co * 8
