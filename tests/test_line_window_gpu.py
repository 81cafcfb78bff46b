"""The TOF sinogram projections through line sheets where the wave's window of bins could go wrong, against the FP64
oracle: rays in both directions on one line, infinite voxels, bins beyond the truncation.

Lists long enough for the line kernels (512 rays a line, more than 2^20 rays).  Tolerances as in test_lines_gpu.py: a
projection sums few samples of a dozen float32 roundings each, 5e-6 in relative L2; a back projection 1e-4."""
import numpy as np
import pytest
import torch

import oracle
from helpers import f32, rel_l2, tofd

pytestmark = pytest.mark.gpu

TOL, BACK_TOL = 5e-6, 1e-4
LINES, RAYS = 2100, 512


def _grid(dim, vox):
    return [f32(-(d - 1) / 2 * v) for d, v in zip(dim, vox)], [f32(v) for v in vox]


def _both_ways(name, seed):
    """LINES lines of RAYS rays each that share U0 and dU bit for bit in either direction: along axis 0 through a grid of
    four planes, or at 45 degrees across a grid's corner (coordinates that are exact in float32).  Every chord is
    shorter than half a bin of 28 mm."""
    rng = np.random.default_rng(seed)
    if name == "slab":
        dim, vox = (4, 40, 33), (3.5, 4.0, 2.5)
        y = rng.integers(-300, 301, LINES) * 0.25
        a = np.column_stack([np.full(LINES, -60.0), y])
        b = np.column_stack([np.full(LINES, 60.0), y])
    else:
        dim, vox = (24, 24, 33), (4.0, 4.0, 2.5)
        c, m = rng.integers(80, 92, LINES) * 1.0, 48.0 - rng.integers(0, 32, LINES) * 0.25
        a = np.column_stack([m - 64.0, m - c - 64.0])
        b = np.column_stack([m + 64.0, m - c + 64.0])
    a, b = a.repeat(RAYS, 0), b.repeat(RAYS, 0)
    z = rng.uniform(-1.1, 1.1, (a.shape[0], 2)) * 0.5 * dim[2] * vox[2]
    xs, xe = np.column_stack([a, z[:, 0]]), np.column_stack([b, z[:, 1]])
    turn = rng.random(xs.shape[0]) < 0.5
    xs[turn], xe[turn] = xe[turn].copy(), xs[turn].copy()
    return dim, vox, xs.astype(np.float32), xe.astype(np.float32), rng


@pytest.mark.parametrize("name", ["slab", "corner"])
@pytest.mark.parametrize("offset", [-16.8, -2.0, 0.0, 13.0, 16.8])
def test_both_directions_of_a_line(gpu, name, offset):
    dim, vox, xs, xe, rng = _both_ways(name, 21)
    o, h = _grid(dim, vox)
    tof = (28.0, 24.8, 3.0, 9)
    T, t64, G = gpu.TofParams(*tof, center_offset=offset), tofd(*tof, center_offset=offset), gpu.ImageGeom(dim, vox)
    dev = torch.device("cuda")
    t = lambda a: torch.from_numpy(a).to(dev)  # noqa: E731
    img = rng.uniform(0.5, 2.0, dim).astype(np.float32)
    got = gpu.fwd_tof_sino(t(xs), t(xe), G, T, t(img)).cpu().numpy()
    assert rel_l2(got, oracle.fwd_tof_sino(xs, xe, o, h, dim, t64, img)) <= TOL
    y = rng.uniform(0.0, 2.0, (xs.shape[0], tof[3])).astype(np.float32)
    got = gpu.back_tof_sino(t(xs), t(xe), G, T, t(y)).cpu().numpy()
    assert rel_l2(got, oracle.back_tof_sino(xs, xe, o, h, dim, t64, y)) <= BACK_TOL


def _lines(dim, vox, seed, lines=LINES):
    """Random lines of RAYS rays each, all of a line in one direction, heights at random."""
    rng = np.random.default_rng(seed)
    half = 0.5 * np.asarray(dim) * np.asarray(vox)
    a, off = rng.uniform(0.0, 2.0 * np.pi, lines), rng.uniform(-0.8, 0.8, lines) * min(half[0], half[1])
    d, nrm = np.column_stack([np.cos(a), np.sin(a)]), np.column_stack([-np.sin(a), np.cos(a)])
    mid, reach = off[:, None] * nrm, 1.6 * max(half[0], half[1]) * d
    ends = [e.astype(np.float32).repeat(RAYS, 0) for e in (mid - reach, mid + reach)]
    z = rng.uniform(-0.9, 0.9, (lines * RAYS, 2)) * half[2]
    return [np.column_stack([e, z[:, i]]).astype(np.float32) for i, e in enumerate(ends)], rng


@pytest.mark.parametrize("lines", [LINES, 7])
def test_infinite_voxel(gpu, lines):
    """A ray's bins that the infinite voxel reaches are infinite, no value is a NaN, and the others are as without it,
    through line sheets and (the short list) by gathers."""
    dim, vox, tof = (37, 41, 15), (4.0, 3.5, 5.0), (28.0, 24.8, 3.0, 13)
    (xs, xe), rng = _lines(dim, vox, 22, lines)
    o, h = _grid(dim, vox)
    dev = torch.device("cuda")
    t = lambda a: torch.from_numpy(a).to(dev)  # noqa: E731
    img = rng.uniform(0.5, 2.0, dim).astype(np.float32)
    at = (18, 20, 7)
    img[at] = 0.0
    one = np.zeros(dim, np.float32)
    one[at] = 1.0
    want = oracle.fwd_tof_sino(xs, xe, o, h, dim, tofd(*tof), img)
    reached = oracle.fwd_tof_sino(xs, xe, o, h, dim, tofd(*tof), one)
    clear = oracle.fwd_tof_sino(xs, xe, o, h, dim, tofd(28.0, 24.8, 3.0001, 13), one) == 0.0
    img[at] = np.inf
    got = gpu.fwd_tof_sino(t(xs), t(xe), gpu.ImageGeom(dim, vox), gpu.TofParams(*tof), t(img)).cpu().numpy()
    assert (reached > 1e-5).any() and not np.isnan(got).any()
    assert np.isinf(got[reached > 1e-5]).all() and np.isfinite(got[clear]).all()
    assert rel_l2(got[clear], want[clear]) <= TOL


def test_infinite_voxel_nontof(gpu):
    """The same without TOF, a list long enough for its line kernel: rays that the voxel reaches are infinite, no other."""
    dim, vox = (19, 17, 9), (4.0, 3.5, 5.0)
    (xs, xe), rng = _lines(dim, vox, 23, 11_400)
    o, h = _grid(dim, vox)
    dev = torch.device("cuda")
    t = lambda a: torch.from_numpy(a).to(dev)  # noqa: E731
    img = rng.uniform(0.5, 2.0, dim).astype(np.float32)
    img[9, 8, 4] = np.inf
    one = np.where(np.isinf(img), np.float32(1.0), np.float32(0.0))
    reached = oracle.fwd(xs, xe, o, h, dim, one)
    got = gpu.fwd(t(xs), t(xe), gpu.ImageGeom(dim, vox), t(img)).cpu().numpy()
    assert (reached > 1e-5).any() and not np.isnan(got).any()
    assert np.isinf(got[reached > 1e-5]).all() and np.isfinite(got[reached == 0.0]).all()


# truncations just above and just below an edge of a bin (3.08 and 4.96 bins), and the one of 58.5 mm FWHM in 28 mm bins
@pytest.mark.parametrize("tof", [(12.0, 29.0 / 2.355, 3.0, 31), (15.0, 24.8, 3.0, 17), (28.0, 58.5 / 2.355, 3.0, 29)],
                         ids=lambda t: str(t[0]))
@pytest.mark.parametrize("lines", [600, 7])
def test_bins_beyond_the_truncation(gpu, tof, lines):
    """Of an image without negative voxels no bin is negative, and bins that no sample's truncated Gaussian reaches (nor
    one truncated 1e-4 further out) are exactly 0."""
    dim, vox = (37, 41, 15), (4.0, 3.5, 5.0)
    (xs, xe), rng = _lines(dim, vox, 24, lines)
    o, h = _grid(dim, vox)
    dev = torch.device("cuda")
    t = lambda a: torch.from_numpy(a).to(dev)  # noqa: E731
    img = rng.uniform(0.5, 2.0, dim).astype(np.float32)
    img[:, 12:] = 0.0
    got = gpu.fwd_tof_sino(t(xs), t(xe), gpu.ImageGeom(dim, vox), gpu.TofParams(*tof), t(img)).cpu().numpy()
    out = oracle.fwd_tof_sino(xs, xe, o, h, dim, tofd(tof[0], tof[1], tof[2] * 1.0001, tof[3]), img) == 0.0
    assert out.any() and got[out].any() == False  # noqa: E712
    assert got.min() >= 0.0
    assert rel_l2(got, oracle.fwd_tof_sino(xs, xe, o, h, dim, tofd(*tof), img)) <= TOL
