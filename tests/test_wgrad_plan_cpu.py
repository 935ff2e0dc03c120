"""How the weight gradient splits its pixels, from the workspace sizes (no GPU needed): a split
costs fp32 partials of the whole gradient, a grid that is too small leaves the GPU idle."""
import pytest

from paper_2609_10632_amd import numbat as nb


def splits(n, h, w, ci, co, k, s):
    """Splits of the problem's partials (0 for a gradient written directly)."""
    b = nb.numbat_workspace_size(nb.OP_CONV_BWD_WEIGHT, nb.conv_problem(n, h, w, ci, co, k, stride=s))
    return b // (co * k * k * ci * 4)


@pytest.mark.parametrize("c", [(1, 25, 25, 352, 608, 3, 1), (9, 15, 15, 280, 600, 3, 2), (13, 9, 9, 288, 320, 3, 1),
                               (1, 28, 28, 560, 144, 3, 1)])
def test_few_pixels_into_large_gradients_stay_whole(c):
    """Ten steps of work are not worth partials of millions of elements."""
    assert splits(*c) == 0


@pytest.mark.parametrize("c", [(2, 32, 32, 16, 32, 3, 1), (1, 100, 98, 88, 128, 3, 2), (8, 14, 14, 592, 144, 3, 1)])
def test_few_pixels_into_small_gradients_are_split(c):
    assert splits(*c) >= 2


def test_patches_past_the_image_need_a_full_grid():
    """Patches past the last row on 88 tiles, of one split each, would leave most CUs idle: the
    general kernel splits its pixels.  A padded 1x1 layer of six steps stays whole."""
    assert splits(7, 242, 8, 704, 216, 3, 1) >= 2
    assert splits(1, 19, 19, 528, 576, 1, 1) == 0
