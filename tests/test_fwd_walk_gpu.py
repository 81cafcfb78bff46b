"""The ray-per-thread forward projections (ray_walk) against the FP64 oracle: the planes inside the grid and those at
its faces, lists small enough for several lanes to share a ray and the first that are not, grids without inner
planes, and one whose columns lie too far apart for the walk's 24-bit products.

Tolerance: a ray sums at most 160 samples of one sign (longer ones, 10^6 samples along axis 2 of the grid with far
columns, are not compared), each with a dozen float32 roundings and a TOF weight within
5e-7 of the largest: 160 * 2^-24 = 1e-5 at the very worst."""
import numpy as np
import pytest
import torch

import oracle
from helpers import f32, random_rays, rel_l2, tofd

pytestmark = pytest.mark.gpu

TOL = 1e-5
GRIDS = {
    "odd": ((37, 41, 29), (4.0, 3.5, 5.0)),
    "tall": ((9, 12, 150), (6.0, 6.0, 2.0)),
    "one_slice": ((40, 33, 1), (4.0, 4.0, 5.0)),
    "one_column": ((50, 1, 8), (4.0, 40.0, 5.0)),
    "two": ((2, 2, 2), (40.0, 30.0, 30.0)),
    "far_columns": ((2, 2, 4_194_400), (300.0, 300.0, 1e-4)),
}


def _case(name, n, seed):
    dim, vox = GRIDS[name]
    rng = np.random.default_rng(seed)
    h = [f32(v) for v in vox]
    o = [f32(-(d - 1) / 2 * v) for d, v in zip(dim, vox)]
    xs, xe = random_rays(rng, n, o, h, dim, inside_frac=0.1)
    if n > 4:
        xs[0], xe[1] = np.nan, np.inf
        xe[2] = xs[2]
        xs[3], xe[3] = (o[0], -500.0, o[2]), (o[0], 500.0, o[2])  # along an axis, through voxel centres
        xs[4], xe[4] = (-500.0, o[1], -o[2]), (500.0, o[1], -o[2])  # the grid's last slice
    img = rng.random(dim, dtype=np.float32)
    return dim, vox, o, h, xs, xe, rng.integers(-2, 31, n).astype(np.int16), img


@pytest.mark.parametrize("name", list(GRIDS))
@pytest.mark.parametrize("n", [1, 67, 20_011, 140_003])
def test_walk(gpu, name, n):
    if name == "far_columns" and n > 67:
        pytest.skip("a 67 MB image; its branch does not depend on n")
    dim, vox, o, h, xs, xe, bins, img = _case(name, n, 11)
    dev = torch.device("cuda")
    t = lambda a: torch.from_numpy(a).to(dev)  # noqa: E731
    G = gpu.ImageGeom(dim, vox)
    order = np.random.default_rng(1).permutation(n).astype(np.int32)
    want = oracle.fwd(xs, xe, o, h, dim, img)
    for od in (None, t(order)):
        assert rel_l2(gpu.fwd(t(xs), t(xe), G, t(img), order=od).cpu().numpy(), want) <= TOL
    for tof in (tofd(28.0, 24.8, 3.0, 29), tofd(28.0, 3.0, 3.0, 29)):  # the polynomial, the erf
        T = gpu.TofParams(tof["bin_width"], tof["sigma"], tof["n_sigmas"], tof["n_bins"])
        got = gpu.fwd_tof_lm(t(xs), t(xe), t(bins), G, T, t(img), order=t(order)).cpu().numpy()
        want = oracle.fwd_tof_lm(xs, xe, o, h, dim, tof, bins, img)
        few = oracle.count_samples(xs, xe, o, h, dim, tof, bins, per_ray=True)[1] <= 160
        assert rel_l2(got[few], want[few]) <= TOL


@pytest.mark.parametrize("name", ["odd", "tall", "one_slice", "one_column", "two"])
@pytest.mark.parametrize("n_img", [2, 3, 4, 5, 9, 10])
def test_batch_interleaved(gpu, name, n_img):
    """Images interleaved two, four and eight at a time: each image's projection is pp_fwd_tof_lm's, bit for bit."""
    n = 5003
    dim, vox, _, _, xs, xe, bins, _ = _case(name, n, 12)
    dev = torch.device("cuda")
    t = lambda a: torch.from_numpy(a).to(dev)  # noqa: E731
    G = gpu.ImageGeom(dim, vox)
    imgs = torch.rand((n_img, *dim), generator=torch.Generator().manual_seed(1)).to(dev)
    order = t(np.random.default_rng(2).permutation(n).astype(np.int32))
    lib = gpu.load()
    for T in (gpu.TofParams(28.0, 24.8, 3.0, 29), gpu.TofParams(28.0, 3.0, 3.0, 29)):
        assert lib.pp_fwd_tof_lm_batch_workspace_bytes(n, G.c(), T.c(n), n_img) > 0
        assert lib.pp_fwd_tof_lm_batch_workspace_bytes(n, G.c(), T.c(n), 1) == 0
        got = gpu.fwd_tof_lm_batch(t(xs), t(xe), t(bins), G, T, imgs, order)
        for b in range(n_img):
            assert torch.equal(got[b], gpu.fwd_tof_lm(t(xs), t(xe), t(bins), G, T, imgs[b].contiguous(), order)), b


@pytest.mark.parametrize("n", [20_011, 140_003])
def test_infinite_voxel(gpu, n):
    """A ray through an infinite voxel is infinite, not a NaN, and no other ray is touched."""
    dim, vox, o, h, xs, xe, bins, img = _case("odd", n, 13)
    img[18, 20, 14] = np.inf
    keep = np.isfinite(xs).all(1) & np.isfinite(xe).all(1) & (np.abs(xe - xs) > 1e-3).all(1)  # no exact weights of 0
    xs, xe, bins = xs[keep], xe[keep], bins[keep]
    dev = torch.device("cuda")
    t = lambda a: torch.from_numpy(a).to(dev)  # noqa: E731
    want = oracle.fwd(xs, xe, o, h, dim, img)
    got = gpu.fwd(t(xs), t(xe), gpu.ImageGeom(dim, vox), t(img)).cpu().numpy()
    assert np.isinf(want).any() and not np.isnan(got).any() and np.array_equal(np.isinf(got), np.isinf(want))
    imgs = t(np.stack([img, np.ones_like(img)]))
    T = gpu.TofParams(28.0, 24.8, 3.0, 29)
    got = gpu.fwd_tof_lm_batch(t(xs), t(xe), t(bins), gpu.ImageGeom(dim, vox), T, imgs).cpu().numpy()
    want = oracle.fwd_tof_lm(xs, xe, o, h, dim, tofd(28.0, 24.8, 3.0, 29), bins, img)
    assert np.isinf(got[0][np.isinf(want) & ~np.isnan(got[0])]).all() and np.isfinite(got[1]).all()
    assert not np.isfinite(got[0][np.isinf(want)]).any()  # a plane at the window's end may weigh the voxel by 0: NaN
