"""The tile back projection (pp_back_lm_ws) against the FP64 oracle: grids at the edges of the tiles (one column or
slice more or less than a tile, slices cut in parts, a single tile), rays along every axis, degenerate rays and
TOF bins, every form of the TOF weight, several images, any processing order, and values far apart.

Tolerance: every added value carries at most a dozen float32 roundings (12 * 2^-24 = 7e-7) and a TOF weight within
5e-7 of the largest weight, and a voxel sums at most a few hundred flushed floats: 1e-5 in relative L2."""
import numpy as np
import pytest
import torch
from scipy.ndimage import binary_dilation

import oracle
from helpers import f32, random_rays, rel_l2, tofd

pytestmark = pytest.mark.gpu

TOL = 1e-5
TOF = tofd(28.0, 24.8, 3.0, 29)
GRIDS = {
    "one_tile": ((7, 5, 3), (9.0, 11.0, 7.0)),
    "edge": ((24, 25, 8), (5.0, 4.0, 6.0)),  # 24 columns are a tile of a thin grid
    "edge_less": ((23, 48, 9), (5.0, 4.0, 6.0)),
    "whole_slices": ((31, 29, 71), (4.0, 4.0, 2.0)),
    "cut_slices": ((33, 20, 161), (4.0, 6.0, 1.5)),
    "long": ((130, 17, 40), (1.5, 8.0, 3.0)),
}


def _case(name, n, seed):
    dim, vox = GRIDS[name]
    rng = np.random.default_rng(seed)
    h = [f32(v) for v in vox]
    o = [f32(-(d - 1) / 2 * v) for d, v in zip(dim, vox)]
    xs, xe = random_rays(rng, n, o, h, dim, inside_frac=0.1)
    xs[0], xe[1] = np.nan, np.inf
    xe[2] = xs[2]  # no length
    xs[3] = xe[3] + np.float32(1e4)  # beside the grid
    xs[4], xe[4] = (o[0], -500.0, o[2]), (o[0], 500.0, o[2])  # along an axis, through voxel centres
    bins = rng.integers(-2, 31, n).astype(np.int16)
    return dim, vox, o, h, xs, xe, bins, rng.uniform(0.5, 1.5, n).astype(np.float32)


def _back(gpu, xs, xe, bins, geom, tof, p, n_img=1, order=None):
    from paper_2212_12519_amd import projectors as P

    dev = torch.device("cuda")
    t = lambda a: torch.from_numpy(a).to(dev)  # noqa: E731
    img = torch.zeros((n_img, *geom.dim), device=dev)
    od = None if order is None else t(order)
    n = xs.shape[0]
    assert P._back_lm_tiles(t(xs), t(xe), 0, None, None if bins is None else t(bins), n, geom.c(),
                            None if tof is None else tof.c(n), img, n_img, t(p), od)
    torch.cuda.synchronize()
    return img.cpu().numpy()


@pytest.mark.parametrize("name", list(GRIDS))
@pytest.mark.parametrize("n", [1, 255, 1025, 20_011])
def test_grids_and_counts(gpu, name, n):
    n = max(n, 5)
    dim, vox, o, h, xs, xe, bins, p = _case(name, n, 5)
    geom = gpu.ImageGeom(dim, vox)
    T = gpu.TofParams(TOF["bin_width"], TOF["sigma"], TOF["n_sigmas"], TOF["n_bins"])
    order = np.random.default_rng(1).permutation(n).astype(np.int32)
    got = _back(gpu, xs, xe, None, geom, None, p, order=order)
    assert rel_l2(got, oracle.back(xs, xe, o, h, dim, p)) <= TOL
    got = _back(gpu, xs, xe, bins, geom, T, p)
    assert rel_l2(got, oracle.back_tof_lm(xs, xe, o, h, dim, TOF, bins, p)) <= TOL


@pytest.mark.parametrize("form", ["poly", "erf", "table", "per_ray", "table_offset"])
@pytest.mark.parametrize("n_img", [1, 3, 17])
def test_weights_and_images(gpu, form, n_img):
    n = 3001
    dim, vox, o, h, xs, xe, bins, p = _case("whole_slices", n, 6)
    dev = torch.device("cuda")
    geom = gpu.ImageGeom(dim, vox)
    kw, ref = {}, dict(TOF)
    if form == "erf":  # a kernel the polynomial does not fit
        ref = tofd(28.0, 3.0, 3.0, 29)
    rng = np.random.default_rng(2)
    if form in ("per_ray", "table_offset"):
        off = rng.normal(0.0, 5.0, n).astype(np.float32)
        kw["offset_per_ray"] = torch.from_numpy(off).to(dev)
        ref["offset_per_ray"] = off
    if form == "per_ray":
        sig = (24.8 * rng.uniform(0.8, 1.25, n)).astype(np.float32)
        sig[7], sig[8] = 0.0, np.nan
        kw["sigma_per_ray"] = torch.from_numpy(sig).to(dev)
        ref["sigma_per_ray"] = sig
    T = gpu.TofParams(ref["bin_width"], ref["sigma"], ref["n_sigmas"], ref["n_bins"])
    if form.startswith("table"):
        T = gpu.gaussian_tof_table(T, 0.05)
        ref.update(lut=T.lut.cpu().numpy(), lut_x0=T.lut_x0, lut_dx=T.lut_dx)
    T = gpu.TofParams(T.bin_width, T.sigma, T.n_sigmas, T.n_bins, 0.0, T.lut, T.lut_x0, T.lut_dx, **kw)
    ps = np.stack([p * np.float32(s) for s in np.linspace(0.0, 3.0, n_img + 1)[1:]])
    if n_img > 1:
        ps[1] = 0.0
    got = _back(gpu, xs, xe, bins, geom, T, ps, n_img=n_img)
    want = oracle.back_tof_lm(xs, xe, o, h, dim, ref, bins, p)
    for b in range(n_img):
        scale = float(ps[b, 9] / p[9])
        assert rel_l2(got[b], want * scale) <= TOL if scale else not got[b].any(), b


def test_values_far_apart(gpu):
    """Events 1e-6 and 1e-13 of the largest (the latter go to the image directly), in grids' halves of
    their own, and an infinite one: its voxels only."""
    n = 6000
    dim, vox, o, h, xs, xe, _, p = _case("whole_slices", n, 7)
    xs[:5], xe[:5] = xs[5:10], xe[5:10]
    cls = np.arange(n) % 3
    for c, y in ((0, -40.0), (1, 0.0), (2, 40.0)):  # nearly parallel to axis 0, apart along axis 1
        m = cls == c
        xs[m] = np.stack([np.full(m.sum(), -300.0), np.full(m.sum(), y), xs[m, 2] * 0.2], 1)
        xe[m] = np.stack([np.full(m.sum(), 300.0), np.full(m.sum(), y + 3.0), xe[m, 2] * 0.2], 1)
    p = (p * np.array([1.0, 1e-6, 1e-13])[cls]).astype(np.float32)
    geom = gpu.ImageGeom(dim, vox)
    got = _back(gpu, xs, xe, None, geom, None, p)[0]
    for c in range(3):
        only = oracle.back(xs[cls == c], xe[cls == c], o, h, dim, p[cls == c])
        at = only != 0
        assert at.sum() > 500
        assert rel_l2(got[at], only[at]) <= TOL, c
    p[0] = np.inf
    bad = _back(gpu, xs, xe, None, geom, None, p)[0]
    hit = oracle.back(xs[:1], xe[:1], o, h, dim, np.ones(1, np.float32)) != 0
    near = binary_dilation(hit, np.ones((3, 3, 3)))  # neighbours of weight 0 may take 0 * inf
    assert np.isfinite(bad[~near]).all() and not np.isfinite(bad[hit]).all()


@pytest.mark.parametrize("listmode", [False, True])
def test_tall_grid_rule(gpu, listmode):
    """Grids of more slices than a sheet holds: the tiles also take ray lists without an order, and more events."""
    lib = gpu.load()
    n = 20_011
    dim, vox, o, h, xs, xe, _, p = _case("cut_slices", n, 8)
    geom = gpu.ImageGeom(dim, vox)
    most = 40_000_000 if listmode else 5_700_000
    bytes_of = lambda d, k: lib.pp_back_lm_workspace_bytes(k, gpu.ImageGeom(d, vox).c(), None, int(listmode), 1)  # noqa: E731
    assert bytes_of(dim, most) > 0 and bytes_of(dim, most + 1) == 0
    assert (bytes_of((33, 20, 128), 1000) > 0) == listmode
    assert bytes_of((33, 20, 128), 7_000_001) == 0
    T, G = gpu.TofParams(28.0, 24.8, 3.0, 29).c(), gpu.ImageGeom((33, 20, 128), vox).c()
    for n_img, events in ((1, 10_000_000), (2, 20_000_000)):
        assert (lib.pp_back_lm_workspace_bytes(events, G, T, int(listmode), n_img) > 0) == listmode
        assert lib.pp_back_lm_workspace_bytes(events + 1, G, T, int(listmode), n_img) == 0
    assert bytes_of((2000, 2000, 700), 40_000_000) == 0  # the workspace's own limit
    dev = torch.device("cuda")
    t = lambda a: torch.from_numpy(a).to(dev)  # noqa: E731
    order = t(np.random.default_rng(3).permutation(n).astype(np.int32)) if listmode else None
    img = gpu.back(t(xs), t(xe), geom, t(p), order=order)
    assert rel_l2(img.cpu().numpy(), oracle.back(xs, xe, o, h, dim, p)) <= TOL


@pytest.mark.parametrize("sigma,table", [(24.8, False), (3.0, False), (24.8, True)])
@pytest.mark.parametrize("n,n_sub", [(1, 1), (7, 9), (4001, 3)])
def test_osem_frame_against_slots(gpu, sigma, table, n, n_sub):
    """Every subset of a frame accumulated by tiles and by the fused kernel over the slot table: the float32 forward is
    the same code; 1 / ybar and the sums differ by roundings (TOL)."""
    from paper_2212_12519_amd import osem

    dim, vox, o, h, xs, xe, bins, _ = _case("whole_slices", max(n, 10), 8)
    dev = torch.device("cuda")
    xs, xe, bins = (torch.from_numpy(a[-n:].copy()).to(dev) for a in (xs, xe, bins))
    geom, T = gpu.ImageGeom(dim, vox), gpu.TofParams(28.0, sigma, 3.0, 29)
    if table:
        T = gpu.gaussian_tof_table(T, 0.05)
    a, b, c = osem.prepare_frame(xs, xe, bins, geom, T, n_sub)
    x = torch.rand(dim, device=dev) + 0.1
    sens = torch.ones(dim, device=dev)
    lib = gpu.load()
    for j in range(n_sub):
        acc = [torch.zeros(dim, device=dev) for _ in range(2)]
        for q in range(2):
            tab = osem.SlotTable(1, dev)
            tab.set(0, a, b, c, x, acc[q], sens, n_sub, 1, 0.1)
            tab.host[0].subset = j
            tab.upload()
            if q == 0:
                osem.check(lib.pp_lm_osem_subset_batched(osem.ptr(tab.dev), 1, geom.c(), T.c(), osem.stream_of(x)))
            else:
                nb = lib.pp_lm_osem_frame_workspace_bytes(n, n_sub, geom.c(), T.c())
                ws = torch.empty(nb, dtype=torch.uint8, device=dev)
                osem.check(lib.pp_lm_osem_frame_ws(tab.host[0], geom.c(), T.c(), osem.ptr(ws), nb, osem.stream_of(x)))
            torch.cuda.synchronize()
        want, got = (t.cpu().numpy() for t in acc)
        assert rel_l2(got, want) <= TOL, j
