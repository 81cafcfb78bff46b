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
