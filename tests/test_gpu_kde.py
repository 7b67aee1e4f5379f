"""The sample application (Sec. VI-A), per-pixel sums of Gaussian kernels,
on the GPU against the FP64 oracle: with expf and __expf against the exact
Gaussian; through a table of exp(-u^2/2) on [0, 8] (the paper's interval)
against the oracle evaluating the same table, and against the exact
Gaussian within three times the table's L-infinity error (a product of three
kernel values, each at most 1)."""

import numpy as np
import pytest
import torch

import oracle as O
import workloads as W
from tests.gpu_util import device, library, say

pytestmark = pytest.mark.gpu

SIGMA = (6.0, 6.0, 6.0)


def _run(P, dev, H, W_, T, r, table_N):
    f_h, h_h = W.kde_frames(H, W_, T, seed=4)
    f, h = torch.from_numpy(f_h).to(dev), torch.from_numpy(h_h).to(dev)
    exact = O.kde_likelihood(f_h, h_h, r, SIGMA)
    t = P.pwl_build(O.GAUSSIAN, (1.0, 1.0), 0.0, 8.0, table_N, O.OPTIMAL, O.PROJ)
    d = P.pwl_table_download(t)
    X, v = d["knots"].astype(np.float64), d["values"].astype(np.float64)
    via_table = O.kde_likelihood(f_h, h_h, r, SIGMA, g=lambda u: O.evaluate(X, v, np.abs(u)))
    linf = O.linf_error(O.GAUSSIAN, (1.0, 1.0), X, v)
    out = {}
    for mode in (P.KDE_TABLE, P.KDE_EXPF, P.KDE_FAST_EXPF):
        out[mode] = P.pwl_kde(t, mode, f, h, r, SIGMA).cpu().numpy().astype(np.float64)
    e_exp = np.max(np.abs(out[P.KDE_EXPF] - exact))
    e_fast = np.max(np.abs(out[P.KDE_FAST_EXPF] - exact))
    e_tab = np.max(np.abs(out[P.KDE_TABLE] - via_table))
    e_tab_exact = np.max(np.abs(out[P.KDE_TABLE] - exact))
    say("  %dx%d T=%d r=%d: expf %.2e, __expf %.2e, table vs oracle table %.2e, table vs exact %.2e "
        "(table L-inf %.2e)" % (H, W_, T, r, e_exp, e_fast, e_tab, e_tab_exact, linf))
    assert e_exp <= 1e-6
    assert e_fast <= 1e-5
    assert e_tab <= 1e-6
    assert e_tab_exact <= 3.0 * linf + 1e-6
    t.free()


def test_kde_small_frame():
    import paper_1510_02975_amd as P
    library()
    _run(P, device(), 37, 53, 3, 2, 256)


def test_kde_cif_frame():
    import paper_1510_02975_amd as P
    library()
    c = W.KDE_CIF
    _run(P, device(), c["H"], c["W"], c["T"], c["radius"], 1024)


def test_kde_expf_modes_need_no_table():
    import paper_1510_02975_amd as P
    library()
    dev = device()
    f_h, h_h = W.kde_frames(9, 11, 2, seed=5)
    f, h = torch.from_numpy(f_h).to(dev), torch.from_numpy(h_h).to(dev)
    y = P.pwl_kde(None, P.KDE_EXPF, f, h, 1, SIGMA).cpu().numpy()
    assert np.max(np.abs(y - O.kde_likelihood(f_h, h_h, 1, SIGMA))) <= 1e-6
    with pytest.raises(P.PWLError):
        P.pwl_kde(None, P.KDE_TABLE, f, h, 1, SIGMA)


@pytest.mark.parametrize("H,W_,T,r", [
    (7, 3, 1, 2),          # narrower than a thread's pixels, window wider than the image
    (5, 66, 2, 0),         # one tap per frame
    (9, 129, 3, 1),
    (21, 65, 4, 3),        # frames split over four waves
    (11, 70, 5, 4),        # a radius without a body of its own
    (6, 131, 6, 33 - 1),   # the largest radius
    (8209, 1, 2, 1),       # frames split over two waves
    (16391, 5, 2, 2),      # one wave per tile
], ids=lambda v: str(v))
def test_kde_tile_edges(H, W_, T, r):
    """Images that end inside a tile, a wave or a thread's four pixels, every
    split of the frames over waves and every body by radius, against the
    oracle: through the table within 1e-6 of the oracle on the same table
    (each kernel value rounds to FP32, the sum is FP64), expf alike."""
    import paper_1510_02975_amd as P
    library()
    dev = device()
    f_h, h_h = W.kde_frames(max(H, 12), max(W_, 12), T, seed=6)
    f_h, h_h = np.ascontiguousarray(f_h[:H, :W_]), np.ascontiguousarray(h_h[:, :H, :W_])
    f_h[0, 0], h_h[:, H // 2, 0] = (0, 255, 0, 255), (255, 0, 255, 255)   # the largest differences
    f, h = torch.from_numpy(f_h).to(dev), torch.from_numpy(h_h).to(dev)
    sigma = (6.0, 9.5, 31.0)
    t = P.pwl_build(O.GAUSSIAN, (1.0, 1.0), -8.0, 8.0, 200, O.OPTIMAL, O.PROJ)
    d = P.pwl_table_download(t)
    X, v = d["knots"].astype(np.float64), d["values"].astype(np.float64)
    say("  kde %dx%d T=%d r=%d" % (H, W_, T, r))
    for mode, g in ((P.KDE_TABLE, lambda u: O.evaluate(X, v, u)), (P.KDE_EXPF, None)):
        ref = O.kde_likelihood(f_h, h_h, r, sigma, g=g) if g else O.kde_likelihood(f_h, h_h, r, sigma)
        got = P.pwl_kde(t, mode, f, h, r, sigma).cpu().numpy()
        assert np.max(np.abs(got - ref)) <= 1e-6
    t.free()


def _against_oracle(P, dev, H, W_, T, r):
    f_h, h_h = W.kde_frames(max(H, 12), max(W_, 12), T, seed=6)
    f_h, h_h = np.ascontiguousarray(f_h[:H, :W_]), np.ascontiguousarray(h_h[:, :H, :W_])
    f_h[0, 0], h_h[:, H // 2, 0] = (0, 255, 0, 255), (255, 0, 255, 255)
    say("  kde %dx%d T=%d r=%d" % (H, W_, T, r))
    sigma = (6.0, 9.5, 31.0)
    got = P.pwl_kde(None, P.KDE_EXPF, torch.from_numpy(f_h).to(dev), torch.from_numpy(h_h).to(dev), r, sigma)
    assert np.max(np.abs(got.cpu().numpy() - O.kde_likelihood(f_h, h_h, r, sigma))) <= 1e-6


@pytest.mark.parametrize("T,r", [(1, 0), (1, 1), (1, 3), (1, 4), (1, 20), (2, 3), (3, 2), (5, 2)])
@pytest.mark.parametrize("W_", [1, 2, 4, 5, 8, 9, 16, 17, 32, 33, 61, 64, 65, 100, 131])
def test_kde_widths(W_, T, r):
    """Every width of a wave's tile, with its edges, and window rows split
    over the waves of a workgroup at any row, one frame's rows too."""
    import paper_1510_02975_amd as P
    library()
    _against_oracle(P, device(), 37, W_, T, r)


@pytest.mark.parametrize("waves_per_cu,T,r", [(6, 2, 3), (9, 2, 3), (6, 3, 1), (9, 3, 1), (6, 1, 3), (9, 1, 3), (9, 2, 4)])
def test_kde_splits_of_large_images(waves_per_cu, T, r):
    """Images of enough tiles (64 rows of one pixel each) for two waves per
    tile (up to 8 tiles per compute unit at these few taps) or one."""
    import paper_1510_02975_amd as P
    library()
    dev = device()
    cus = torch.cuda.get_device_properties(dev).multi_processor_count
    _against_oracle(P, dev, 64 * cus * waves_per_cu - 7, 1, T, r)
