"""The rules by which ray lists without an order reach the line kernels: grids at the limit of the LDS.

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
