"""The projections of ray lists through line sheets (runs of rays on one transaxial line) against the FP64 oracle: run lengths around the wave and workgroup sizes and the shortest run that gets a sheet, single rays and rays
along axis 2 between them, both directions of a ray, odd grids, bin counts around the blocks of eight that a row is
written in, and TOF kernels with one to five bin edges on a side, with and without a fit.

Tolerance: a projection sums up to some 200 samples of a dozen float32 roundings each, mostly of one sign; the TOF
weights are within 3.4e-7 of a largest weight of 0.4 to 1: 5e-6 in relative L2.  A back projection's sheets keep at
least 8 bits of every value and carry the remainders: 1e-4, the bar of the other back projections."""
import numpy as np
import pytest
import torch
from scipy.ndimage import binary_dilation

import oracle
from helpers import f32, random_rays, rel_l2, tofd

pytestmark = pytest.mark.gpu

TOL, BACK_TOL = 5e-6, 1e-4
GRIDS = {"flat": ((40, 37, 1), (5.0, 5.5, 9.0)), "odd": ((61, 75, 33), (3.1, 2.7, 2.5)), "tall": ((30, 30, 130), (6.0, 6.0, 1.2))}


def _rays(name, runs, seed):
    """Runs of rays on random transaxial lines, ends at random heights, some reversed; after every run a few rays of
    their own, one of them along axis 2."""
    dim, vox = GRIDS[name]
    rng = np.random.default_rng(seed)
    h = [f32(v) for v in vox]
    o = [f32(-(d - 1) / 2 * v) for d, v in zip(dim, vox)]
    half = 0.5 * np.asarray(dim) * np.asarray(vox)
    xs, xe = [], []
    for i, n in enumerate(runs):
        a, off = rng.uniform(0.0, np.pi), rng.uniform(-0.9, 0.9) * min(half[0], half[1])
        d, nrm = np.array([np.cos(a), np.sin(a)]), np.array([-np.sin(a), np.cos(a)])
        reach = 1.6 * max(half[0], half[1])
        z = rng.uniform(-1.3, 1.3, (n, 2)) * half[2]
        s = np.column_stack([np.tile(off * nrm - reach * d, (n, 1)), z[:, 0]])
        e = np.column_stack([np.tile(off * nrm + reach * d, (n, 1)), z[:, 1]])
        xs.append(e if i % 3 == 2 else s)
        xe.append(s if i % 3 == 2 else e)
        r = random_rays(rng, 3, o, h, dim, inside_frac=0.4)
        r[0][1], r[1][1] = (1.0, 2.0, -3 * half[2]), (1.5, 2.5, 3 * half[2])
        if i % 4 == 1:
            r[0][2] = np.nan
        xs.append(r[0])
        xe.append(r[1])
    img = rng.uniform(0.0, 2.0, dim).astype(np.float32)
    img[: dim[0] // 3] = 0.0  # a part that contributes nothing
    return dim, vox, o, h, np.concatenate(xs).astype(np.float32), np.concatenate(xe).astype(np.float32), img


RUNS = {"short": [1, 2, 31, 62, 63], "edges": [64, 65, 97, 127, 128, 129, 200], "long": [510, 700, 513, 2204, 3000]}


@pytest.mark.parametrize("name", list(GRIDS))
@pytest.mark.parametrize("runs", list(RUNS))
def test_nontof(gpu, name, runs):
    dim, vox, o, h, xs, xe, img = _rays(name, RUNS[runs] * (40 if runs == "long" else 9), 3)
    dev = torch.device("cuda")
    got = gpu.fwd(torch.from_numpy(xs).to(dev), torch.from_numpy(xe).to(dev), gpu.ImageGeom(dim, vox),
                  torch.from_numpy(img).to(dev)).cpu().numpy()
    assert rel_l2(got, oracle.fwd(xs, xe, o, h, dim, img)) <= TOL


# bin width, sigma, n_sigmas, bins: 1, 2, 3, 4, 5 edges on a side; 6 and a very narrow Gaussian (no fit)
TOFS = [(90.0, 24.8, 3.0, 9), (40.0, 24.8, 3.0, 8), (28.0, 24.8, 3.0, 29), (20.0, 24.8, 3.0, 41), (15.0, 24.8, 3.0, 1),
        (15.0, 24.8, 3.0, 67), (12.5, 24.8, 3.0, 17), (28.0, 1.0, 3.0, 16), (3.0, 4.0, 2.0, 7), (24.8, 24.8, 2.0, 10)]


@pytest.mark.parametrize("tof", TOFS, ids=lambda t: "-".join(str(v) for v in t))
@pytest.mark.parametrize("runs", ["edges", "long"])
def test_tof(gpu, tof, runs):
    dim, vox, o, h, xs, xe, img = _rays("odd", RUNS[runs] * 2, 4)
    dev = torch.device("cuda")
    t = tofd(*tof, center_offset=3.0)
    T = gpu.TofParams(*tof, center_offset=3.0)
    got = gpu.fwd_tof_sino(torch.from_numpy(xs).to(dev), torch.from_numpy(xe).to(dev), gpu.ImageGeom(dim, vox), T,
                           torch.from_numpy(img).to(dev)).cpu().numpy()
    assert rel_l2(got, oracle.fwd_tof_sino(xs, xe, o, h, dim, t, img)) <= TOL


@pytest.mark.parametrize("name", ["flat", "tall"])
def test_tof_grids(gpu, name):
    dim, vox, o, h, xs, xe, img = _rays(name, RUNS["short"] + RUNS["edges"] + RUNS["long"], 5)
    dev = torch.device("cuda")
    t = tofd(28.0, 24.8, 3.0, 29)
    got = gpu.fwd_tof_sino(torch.from_numpy(xs).to(dev), torch.from_numpy(xe).to(dev), gpu.ImageGeom(dim, vox),
                           gpu.TofParams(28.0, 24.8, 3.0, 29), torch.from_numpy(img).to(dev)).cpu().numpy()
    assert rel_l2(got, oracle.fwd_tof_sino(xs, xe, o, h, dim, t, img)) <= TOL


def _large(name, n, seed):
    """At least n rays: long runs, with short ones and strays among them, and a stretch of short runs only."""
    runs = RUNS["long"] * max(1, n // 7000) + RUNS["edges"] * 60 + RUNS["short"] * 200
    dim, vox, o, h, xs, xe, img = _rays(name, runs, seed)
    assert xs.shape[0] >= n
    rng = np.random.default_rng(seed)
    y = rng.normal(1.0, 0.6, xs.shape[0]) * 10.0 ** rng.integers(-2, 3, xs.shape[0])
    y[rng.random(xs.shape[0]) < 0.1] = 0.0
    return dim, vox, o, h, xs, xe, img, y.astype(np.float32)


@pytest.mark.parametrize("name", ["flat", "odd"])
def test_large_lists(gpu, name):
    """Lists long enough for the non-TOF line kernels, which small ones do not reach."""
    dim, vox, o, h, xs, xe, img, y = _large(name, 5_800_000, 6)
    dev = torch.device("cuda")
    t = lambda a: torch.from_numpy(a).to(dev)  # noqa: E731
    G = gpu.ImageGeom(dim, vox)
    got = gpu.fwd(t(xs), t(xe), G, t(img)).cpu().numpy()
    assert rel_l2(got, oracle.fwd(xs, xe, o, h, dim, img)) <= TOL
    got = gpu.back(t(xs), t(xe), G, t(y)).cpu().numpy()
    assert rel_l2(got, oracle.back(xs, xe, o, h, dim, y)) <= BACK_TOL


@pytest.mark.parametrize("tof", [(90.0, 24.8, 3.0, 5), (40.0, 24.8, 3.0, 8), (28.0, 24.8, 3.0, 13), (20.0, 24.8, 3.0, 9),
                                 (15.0, 24.8, 3.0, 9)], ids=lambda t: str(t[0]))
def test_large_tof_back(gpu, tof):
    dim, vox, o, h, xs, xe, _, y = _large("flat", 1_060_000, 7)
    dev = torch.device("cuda")
    t = lambda a: torch.from_numpy(a).to(dev)  # noqa: E731
    rng = np.random.default_rng(8)
    y = (y[:, None] * rng.uniform(-0.2, 1.0, (y.size, tof[3]))).astype(np.float32)
    y[rng.random(y.shape) < 0.3] = 0.0
    T = gpu.TofParams(*tof, center_offset=-4.0)
    got = gpu.back_tof_sino(t(xs), t(xe), gpu.ImageGeom(dim, vox), T, t(y)).cpu().numpy()
    want = oracle.back_tof_sino(xs, xe, o, h, dim, tofd(*tof, center_offset=-4.0), y)
    assert rel_l2(got, want) <= BACK_TOL


def test_large_back_values_not_finite(gpu):
    """A ray with an infinite value reaches its own voxels only."""
    dim, vox, o, h, xs, xe, _, y = _large("flat", 5_800_000, 9)
    dev = torch.device("cuda")
    t = lambda a: torch.from_numpy(a).to(dev)  # noqa: E731
    at = 100_000
    y[at] = np.inf
    got = gpu.back(t(xs), t(xe), gpu.ImageGeom(dim, vox), t(y)).cpu().numpy()
    hit = oracle.back(xs[at:at + 1], xe[at:at + 1], o, h, dim, np.ones(1, np.float32)) != 0
    near = binary_dilation(hit, np.ones((3, 3, 3)))
    assert np.isfinite(got[~near]).all()


@pytest.mark.parametrize("share", [0.04])
def test_small_values_beside_large(gpu, share):
    """A few rays of a wave with 1e-9 of their line's values: the half of the grid that only they cross."""
    dim, vox, o, h, xs, xe, _, _ = _large("odd", 1_060_000, 10)
    dev = torch.device("cuda")
    t = lambda a: torch.from_numpy(a).to(dev)  # noqa: E731
    rng = np.random.default_rng(11)
    z = o[2] + h[2] * (dim[2] - 1) / 2
    up = (xs[:, 2] > z + h[2]) & (xe[:, 2] > z + h[2])
    down = (xs[:, 2] < z - h[2]) & (xe[:, 2] < z - h[2])
    y = rng.uniform(0.5, 1.5, (xs.shape[0], 13)).astype(np.float32)
    y *= np.where(up & (rng.random(xs.shape[0]) < share), np.float32(1e-9), down.astype(np.float32))[:, None]
    tof = (28.0, 24.8, 3.0, 13)
    got = gpu.back_tof_sino(t(xs), t(xe), gpu.ImageGeom(dim, vox), gpu.TofParams(*tof), t(y)).cpu().numpy()
    want = oracle.back_tof_sino(xs, xe, o, h, dim, tofd(*tof), y)
    first = (dim[2] + 1) // 2 + 1
    assert want[:, :, first:].any() and rel_l2(got[:, :, first:], want[:, :, first:]) <= BACK_TOL
    assert rel_l2(got, want) <= BACK_TOL
