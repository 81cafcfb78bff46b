"""The rules by which ray lists without an order reach the line kernels: grids at the limit of the LDS, and lists that the
back projection splits between its kernels group by group.

Tolerances as in test_lines_gpu.py (a ray sums at most ten samples here)."""
import numpy as np
import pytest
import torch

import oracle
from helpers import f32, rel_l2, tofd

pytestmark = pytest.mark.gpu

TOL, BACK_TOL = 5e-6, 1e-4


@pytest.mark.parametrize("planes,axis", [(6802, 0), (6803, 1), (6826, 0)])
def test_flat_grids_at_the_lds_limit(gpu, planes, axis):
    """One slice: the sheet (3 words a plane) and its planes' records (3) fit a CU together up to 6802 planes; each alone
    fits half of it up to 6826."""
    dim = (planes, 5, 1) if axis == 0 else (5, planes, 1)
    vox = (2.0, 2.0, 3.0)
    rng = np.random.default_rng(41)
    o, h = [f32(-(d - 1) / 2 * v) for d, v in zip(dim, vox)], [f32(v) for v in vox]
    lines, rays = 11_400, 512
    x = rng.uniform(-0.5, 0.5, lines) * (planes - 12) * 2.0
    ends = [np.column_stack([x - 8.0, rng.uniform(-5.0, 5.0, lines)]), np.column_stack([x + 8.0, rng.uniform(-5.0, 5.0, lines)])]
    ends = [e[:, ::1 if axis == 0 else -1].repeat(rays, 0) for e in ends]
    z = rng.uniform(-2.0, 2.0, (lines * rays, 2))
    xs, xe = (np.column_stack([e, z[:, i]]).astype(np.float32) for i, e in enumerate(ends))
    dev = torch.device("cuda")
    t = lambda a: torch.from_numpy(a).to(dev)  # noqa: E731
    G = gpu.ImageGeom(dim, vox)
    img = rng.uniform(0.5, 2.0, dim).astype(np.float32)
    y = rng.uniform(0.5, 1.5, xs.shape[0]).astype(np.float32)
    assert rel_l2(gpu.fwd(t(xs), t(xe), G, t(img)).cpu().numpy(), oracle.fwd(xs, xe, o, h, dim, img)) <= TOL
    assert rel_l2(gpu.back(t(xs), t(xe), G, t(y)).cpu().numpy(), oracle.back(xs, xe, o, h, dim, y)) <= BACK_TOL
    tof, n = (28.0, 24.8, 3.0, 3), 2100 * rays
    xs, xe, y = xs[:n], xe[:n], rng.uniform(0.5, 1.5, (n, 3)).astype(np.float32)
    T, t64 = gpu.TofParams(*tof), tofd(*tof)
    got = gpu.fwd_tof_sino(t(xs), t(xe), G, T, t(img)).cpu().numpy()
    assert rel_l2(got, oracle.fwd_tof_sino(xs, xe, o, h, dim, t64, img)) <= TOL
    got = gpu.back_tof_sino(t(xs), t(xe), G, T, t(y)).cpu().numpy()
    assert rel_l2(got, oracle.back_tof_sino(xs, xe, o, h, dim, t64, y)) <= BACK_TOL


def _list(runs, order, dim, vox, seed):
    """Rays of random lines, runs[i] on the i-th: heights in the order of a sinogram's ring pairs, at random or sorted."""
    rng = np.random.default_rng(seed)
    runs = np.asarray(runs)
    half = 0.5 * np.asarray(dim) * np.asarray(vox)
    a, off = rng.uniform(0.0, 2.0 * np.pi, runs.size), rng.uniform(-0.8, 0.8, runs.size) * min(half[0], half[1])
    d, nrm = np.column_stack([np.cos(a), np.sin(a)]), np.column_stack([-np.sin(a), np.cos(a)])
    mid, reach = off[:, None] * nrm, 1.6 * max(half[0], half[1]) * d
    n = int(runs.sum())
    if order == "pairs":
        pairs = np.array([(i, j) for i in range(41) for j in range(41) if abs(i - j) <= 15])
        z = (pairs[np.arange(n) % len(pairs)] / 20.0 - 1.0) * 1.1 * half[2]
    else:
        z = rng.uniform(-1.1, 1.1, (n, 2)) * half[2]
        if order == "sorted":
            line = np.arange(runs.size).repeat(runs)
            z = z[np.lexsort((z.sum(1), line))]
    xs, xe = (np.column_stack([e.astype(np.float32).repeat(runs, 0), z[:, i]]).astype(np.float32)
              for i, e in enumerate((mid - reach, mid + reach)))
    return xs, xe, rng


@pytest.mark.parametrize("order", ["pairs", "random", "sorted"])
@pytest.mark.parametrize("crystals", [False, True])
def test_lists_split_between_the_kernels(gpu, order, crystals):
    """Lines around the length that the line kernel takes, strays and short runs between them, a stretch of short runs
    only, the list's end inside a group; as coordinates and as crystal pairs (a table of all end points)."""
    dim, vox = (19, 17, 9), (4.0, 3.5, 5.0)
    runs = ([2204, 1, 600, 3, 545, 560, 90, 512, 7, 7, 480, 1300, 64] * 900 + [5, 130, 40] * 700)[: 12_500]
    xs, xe, rng = _list(runs, order, dim, vox, 42)
    n = xs.shape[0]
    assert n >= 11 << 19 and n % 512
    xs[1000], xe[70_000, 2] = np.nan, np.inf
    o, h = [f32(-(d - 1) / 2 * v) for d, v in zip(dim, vox)], [f32(v) for v in vox]
    y = (rng.uniform(0.5, 1.5, n) * 10.0 ** rng.uniform(-2.0, 1.0, n)).astype(np.float32)
    y[rng.random(n) < 0.1] = 0.0
    dev = torch.device("cuda")
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    G = gpu.ImageGeom(dim, vox)
    if crystals:
        pair = np.column_stack([np.arange(n), np.arange(n) + n]).astype(np.int32)
        pair[2000] = (-1, 5)
        y[2000] = 0.0  # contributes nothing
        img = torch.zeros(dim, device=dev)
        table, dp, dy = t(np.concatenate([xs, xe])), t(pair), t(y)
        from paper_2212_12519_amd._lib import check, ptr, stream_of
        check(gpu.load().pp_back_crystals(ptr(table), 2 * n, ptr(dp), n, G.c(), ptr(img), ptr(dy), None, stream_of(img)))
        got = img.cpu().numpy()
    else:
        got = gpu.back(t(xs), t(xe), G, t(y)).cpu().numpy()
    assert rel_l2(got, oracle.back(xs, xe, o, h, dim, y)) <= BACK_TOL
    if not crystals:
        k = 1_100_000
        tof = (28.0, 24.8, 3.0, 5)
        yt = (y[:k, None] * rng.uniform(0.2, 1.0, (k, 5))).astype(np.float32)
        got = gpu.back_tof_sino(t(xs[:k]), t(xe[:k]), G, gpu.TofParams(*tof), t(yt)).cpu().numpy()
        assert rel_l2(got, oracle.back_tof_sino(xs[:k], xe[:k], o, h, dim, tofd(*tof), yt)) <= BACK_TOL
