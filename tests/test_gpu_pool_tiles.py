"""The max pool's LDS tiles (and the kernel without them) at their edges: several row bands and
column tiles with remainders, vector groups that end early, and elements that never win (NaN, -inf) or tie (signed zeros).
Values and positions bit for bit against the oracle, gradients within rel_inf 2e-2."""
import numpy as np
import pytest

from oracle import pool
from parity import Inputs, assert_close, f64
from paper_2609_10632_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if torch.cuda.is_available():
    from paper_2609_10632_amd import blocks
    from paper_2609_10632_amd import numbat as nb


@pytest.mark.parametrize("shape", [(1, 11, 40, 40), (2, 5, 41, 8), (1, 6, 75, 24), (3, 1, 1, 72), (1, 16, 33, 56),
                                   # column tiles, forward and both; the first size past whole rows
                                   (2, 7, 52, 64), (9, 41, 52, 256), (2, 6, 41, 64), (3, 9, 21, 24), (3, 9, 20, 24)])
def test_tiles(shape):
    n, h, w, c = shape
    ip = Inputs(150, c)
    xb, dyb, d0 = (ip.normal(shape, t) for t in (synth.T_X, synth.T_DY, synth.T_RES))
    p = nb.pool_problem(n, h, w, c)
    y = torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    idx = torch.full(shape, 255, dtype=torch.uint8, device="cuda")
    dx = blocks.dev_bf16(d0)
    nb.numbat_maxpool5_fwd(p, blocks.dev_bf16(xb), y, idx)
    nb.numbat_maxpool5_bwd(p, blocks.dev_bf16(dyb), idx, dx, True)
    torch.cuda.synchronize()
    yref, iref = pool.maxpool_fwd(f64(xb))
    assert np.array_equal(blocks.host_f64(y), yref)
    assert np.array_equal(idx.cpu().numpy().astype(np.int64), iref)
    assert_close(blocks.host_f64(dx), pool.maxpool_bwd(f64(dyb), iref) + f64(d0), "dx accumulated")


def test_more_tiles_than_a_launch_holds():
    """8.4M tiles of these images would be 2^32 threads, past which a launch wraps unreported: every
    image's result is that of a small batch, which the tests above check."""
    base, reps = 4096, 2053
    shape = (base, 1, 24, 8)
    g = torch.Generator(device="cuda").manual_seed(5)
    x, dy = (torch.randn(shape, device="cuda", generator=g).to(torch.bfloat16) for _ in range(2))

    def run(x, dy):
        p = nb.pool_problem(*x.shape)
        y, dx, idx = torch.empty_like(x), torch.empty_like(x), torch.empty(x.shape, dtype=torch.uint8, device="cuda")
        nb.numbat_maxpool5_fwd(p, x, y, idx)
        nb.numbat_maxpool5_bwd(p, dy, idx, dx, False)
        return y, idx, dx

    want, got = run(x, dy), run(x.repeat(reps, 1, 1, 1), dy.repeat(reps, 1, 1, 1))
    for w, v in zip(want, got):
        assert bool((v.view(reps, *shape) == w).all())


def test_elements_that_never_win():
    """A window's first maximum over strict comparisons from -inf: NaN and -inf never replace it
    (a window of nothing else gives -inf at position 0), an equal zero of the other sign neither."""
    n, h, w, c = 1, 9, 12, 8
    x = np.random.default_rng(3).choice([np.nan, -np.inf, -1.0, -0.0, 0.0], size=(n, h, w, c), p=[.4, .3, .1, .1, .1])
    x[:, :, :6, 0] = np.nan
    x[:, 4:, :, 1] = -np.inf
    xt = torch.from_numpy(x).to(torch.bfloat16).cuda()
    y, idx = torch.empty_like(xt), torch.empty(x.shape, dtype=torch.uint8, device="cuda")
    nb.numbat_maxpool5_fwd(nb.pool_problem(n, h, w, c), xt, y, idx)
    torch.cuda.synchronize()
    y, idx = y.float().cpu().numpy(), idx.cpu().numpy()
    for p in range(h):
        for q in range(w):
            for ch in range(c):
                best, at = -np.inf, 0
                for t in range(25):
                    i, j = p + t // 5 - 2, q + t % 5 - 2
                    if 0 <= i < h and 0 <= j < w and x[0, i, j, ch] > best:
                        best, at = x[0, i, j, ch], t
                assert float(y[0, p, q, ch]) == best and int(idx[0, p, q, ch]) == at
                if best == 0:
                    assert np.signbit(float(y[0, p, q, ch])) == np.signbit(best)
