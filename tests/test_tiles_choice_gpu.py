"""The choice on the device between the tiles and the run/sheet kernel for listmode back projections of many events
(pp_back_lm_ws): the same image either way, and the way that the lines' lengths ask for.

Tolerance: 1e-4, the bar of the back projections (the sheets' fixed point)."""
import numpy as np
import pytest
import torch

import oracle
from helpers import f32, rel_l2, tofd

pytestmark = pytest.mark.gpu

BACK_TOL = 1e-4
DIM, VOX = (20, 20, 6), (12.0, 12.0, 8.0)
HEAD = 21  # the word of the workspace that holds the counted line changes


def _events(lines, n, seed):
    """n events of `lines` random transaxial lines, both directions of a line, ends at random heights, grouped by line."""
    rng = np.random.default_rng(seed)
    half = 0.5 * np.asarray(DIM) * np.asarray(VOX)
    a, off = rng.uniform(0.0, 2.0 * np.pi, lines), rng.uniform(-0.7, 0.7, lines) * half[0]
    d, nrm = np.column_stack([np.cos(a), np.sin(a)]), np.column_stack([-np.sin(a), np.cos(a)])
    at = np.sort(rng.integers(0, lines, n))
    ends = [((off[:, None] * nrm + s * 1.6 * half[0] * d).astype(np.float32))[at] for s in (-1.0, 1.0)]
    z = rng.uniform(-1.1, 1.1, (n, 2)) * half[2]
    xs, xe = (np.column_stack([e, z[:, i]]).astype(np.float32) for i, e in enumerate(ends))
    turn = rng.random(n) < 0.5
    xs[turn], xe[turn] = xe[turn].copy(), xs[turn].copy()
    return xs, xe, rng


@pytest.mark.parametrize("mode", ["nontof", "crystals", "tof", "batch"])
@pytest.mark.parametrize("grouped", [True, False])
def test_choice(gpu, mode, grouped):
    lib = gpu.load()
    n = {"nontof": 3_400_000, "crystals": 3_400_000, "tof": 6_600_000, "batch": 8_000_001}[mode]
    xs, xe, rng = _events(400, n, 71)
    xs[5], xe[6, 0] = np.nan, np.inf
    order = np.arange(n, dtype=np.int32) if grouped else rng.permutation(n).astype(np.int32)
    order[[17, 18]] = (-1, n)  # skipped: the two events there contribute nothing
    skipped = np.setdiff1d(np.arange(n), order)
    o, h = [f32(-(d - 1) / 2 * v) for d, v in zip(DIM, VOX)], [f32(v) for v in VOX]
    p = rng.uniform(0.5, 1.5, n).astype(np.float32)
    want_p = p.copy()
    want_p[skipped] = 0.0
    tof = None if mode in ("nontof", "crystals") else (28.0, 24.8, 3.0, 9)
    bins = None if tof is None else rng.integers(-1, 10, n).astype(np.int16)
    dev = torch.device("cuda")
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev)  # noqa: E731
    G, nb = gpu.ImageGeom(DIM, VOX), 2 if mode == "batch" else 1
    gc, tc = G.c(), None if tof is None else gpu.TofParams(*tof).c(n)
    img = torch.zeros((nb, *DIM), device=dev)
    dp = torch.stack([t(p), 2.0 * t(p)]) if nb == 2 else t(p)
    do, dxs, dxe, db = t(order), t(xs), t(xe), None if bins is None else t(bins)
    pair, nc = None, 0
    if mode == "crystals":
        dxs, dxe, nc = torch.cat([dxs, dxe]), None, 2 * n
        pair = t(np.column_stack([np.arange(n), np.arange(n) + n]).astype(np.int32))
    size = lib.pp_back_lm_workspace_bytes(n, gc, tc, 1, nb)
    assert size > 0
    ws = torch.zeros(size, dtype=torch.uint8, device=dev)
    from paper_2212_12519_amd._lib import check, ptr, stream_of
    check(lib.pp_back_lm_ws(ptr(dxs), ptr(dxe), nc, ptr(pair), ptr(db), n, gc, tc, ptr(img), nb, ptr(dp), ptr(do), ptr(ws), size,
                            stream_of(img)))
    torch.cuda.synchronize()
    head = ws[:88].view(torch.int32).tolist()
    assert (head[HEAD] < 100) == grouped and (head[0] == 0) == grouped  # pieces only where the tiles were taken
    want = oracle.back(xs, xe, o, h, DIM, want_p) if tof is None else oracle.back_tof_lm(xs, xe, o, h, DIM, tofd(*tof), bins, want_p)
    for b in range(nb):
        assert rel_l2(img[b].cpu().numpy(), want * (b + 1)) <= BACK_TOL, b


@pytest.mark.parametrize("n_img", [1, 2, 18])
def test_passes_over_the_events(gpu, n_img):
    """More events than one pass's workspace (4 GiB) holds: several passes, the last one shorter, in one workspace.  Most
    events miss the grid of more than 128 slices, so that only their records take time."""
    lib = gpu.load()
    dim, vox = (40, 36, 140), (6.0, 6.0, 1.5)
    G, T = gpu.ImageGeom(dim, vox), gpu.TofParams(28.0, 24.8, 3.0, 9)
    size = lambda k: lib.pp_back_lm_workspace_bytes(k, G.c(), T.c(), 1, n_img)  # noqa: E731
    one = next(k for k in range(1_000_000, 40_000_000, 500_000) if size(k + 500_000) < size(k))  # the most of one pass
    n = one + 700_001
    assert 0 < size(n) < size(one) <= (4 << 30) + (1 << 20)
    rng = np.random.default_rng(72)
    o, h = [f32(-(d - 1) / 2 * v) for d, v in zip(dim, vox)], [f32(v) for v in vox]
    k = 20_000
    half = 0.5 * np.asarray(dim) * np.asarray(vox)
    xs = rng.uniform(-1.0, 1.0, (k, 3)) * half * [0.4, 0.4, 0.9]
    u = rng.normal(size=(k, 3)) * [1.0, 1.0, 0.2]
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    xs, xe = (xs - 400.0 * u).astype(np.float32), (xs + 400.0 * u).astype(np.float32)
    at = np.sort(rng.choice(n, k, replace=False))
    at[0], at[-1] = 0, n - 1
    bins, p = rng.integers(0, 9, k).astype(np.int16), rng.uniform(0.5, 1.5, k).astype(np.float32)
    dev = torch.device("cuda")
    t = lambda a: torch.from_numpy(a).to(dev)  # noqa: E731
    dxs, dxe = (torch.full((n, 3), v, device=dev) for v in (1e4, 1.1e4))
    dp, db, w = torch.ones((n_img, n), device=dev), torch.zeros(n, dtype=torch.int16, device=dev), t(at)
    dxs[w], dxe[w], db[w] = t(xs), t(xe), t(bins)
    for b in range(n_img):
        dp[b, w] = t(p) * (b + 1)
    img = torch.zeros((n_img, *dim), device=dev)
    from paper_2212_12519_amd._lib import check, ptr, stream_of
    ws = torch.empty(size(n), dtype=torch.uint8, device=dev)
    check(lib.pp_back_lm_ws(ptr(dxs), ptr(dxe), 0, None, ptr(db), n, G.c(), T.c(n), ptr(img), n_img, ptr(dp), None, ptr(ws),
                            ws.numel(), stream_of(img)))
    want = oracle.back_tof_lm(xs, xe, o, h, dim, tofd(28.0, 24.8, 3.0, 9), bins, p)
    for b in range(n_img):
        assert rel_l2(img[b].cpu().numpy(), want * (b + 1)) <= 1e-5, b


def test_without_memory_for_a_workspace(gpu):
    """Where the workspace cannot be had the calls take their way without one, with the same result."""
    xs, xe, rng = _events(400, 300_000, 73)
    n, dev = xs.shape[0], torch.device("cuda")
    o, h = [f32(-(d - 1) / 2 * v) for d, v in zip(DIM, VOX)], [f32(v) for v in VOX]
    p = rng.uniform(0.5, 1.5, n).astype(np.float32)
    t = lambda a: torch.from_numpy(a).to(dev)  # noqa: E731
    G, dxs, dxe, dp = gpu.ImageGeom(DIM, VOX), t(xs), t(xe), t(p)
    order, img = t(rng.permutation(n).astype(np.int32)), torch.zeros(DIM, device=dev)
    need = gpu.load().pp_back_lm_workspace_bytes(n, G.c(), None, 1, 1)
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    assert need > 8 << 20
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (4 << 20)) / total)
    try:
        gpu.pp_back(dxs, dxe, G, img, dp, order)
        peak = torch.cuda.memory_reserved()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert peak < need
    assert rel_l2(img.cpu().numpy(), oracle.back(xs, xe, o, h, DIM, p)) <= BACK_TOL


@pytest.mark.parametrize("mode", ["nontof", "tof", "missing"])
def test_single_event(gpu, mode):
    """One event, one record, nearly all tiles empty; and one that misses the grid, with no piece at all."""
    from paper_2212_12519_amd import projectors as P

    o, h = [f32(-(d - 1) / 2 * v) for d, v in zip(DIM, VOX)], [f32(v) for v in VOX]
    xs, xe = np.array([[-200.0, 13.0, -7.0]], np.float32), np.array([[210.0, -31.0, 9.0]], np.float32)
    if mode == "missing":
        xs, xe = xs + np.float32(1e4), xe + np.float32(1e4)
    p, bins = np.array([1.7], np.float32), np.array([5], np.int16)
    dev = torch.device("cuda")
    t = lambda a: torch.from_numpy(a).to(dev)  # noqa: E731
    G, img = gpu.ImageGeom(DIM, VOX), torch.zeros((1, *DIM), device=dev)
    T = gpu.TofParams(28.0, 24.8, 3.0, 9)
    assert P._back_lm_tiles(t(xs), t(xe), 0, None, t(bins) if mode == "tof" else None, 1, G.c(),
                            T.c(1) if mode == "tof" else None, img, 1, t(p), None)
    want = oracle.back_tof_lm(xs, xe, o, h, DIM, tofd(28.0, 24.8, 3.0, 9), bins, p) if mode == "tof" else oracle.back(xs, xe, o, h, DIM, p)
    got = img[0].cpu().numpy()
    assert rel_l2(got, want) <= 1e-5 and want.any() == (mode != "missing") and got.any() == want.any()
