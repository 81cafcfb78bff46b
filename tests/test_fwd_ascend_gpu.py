"""The non-TOF forward's choices per wave and image (planes in rising order with or without bounds, one or four at a time)
against the FP64 oracle, and that they change no bit: a ray's value does not depend on the rays of its wave.

Tolerance: a ray sums at most 130 samples of one sign with a dozen float32 roundings each: 130 * 2^-24 = 8e-6."""
import numpy as np
import pytest
import torch

import oracle
from helpers import f32, random_rays, rel_l2

pytestmark = pytest.mark.gpu

TOL = 8e-6
GRIDS = {
    "small_image": ((80, 75, 33), (3.0, 3.2, 2.5)),  # fits an XCD's L2
    "large_image": ((130, 126, 70), (2.0, 2.1, 2.0)),  # 4.6 MB
    "thin": ((128, 90, 4), (2.0, 2.0, 3.0)),
    "short": ((33, 39, 50), (5.0, 5.0, 4.0)),  # fewer than 40 planes
}


@pytest.mark.parametrize("name", list(GRIDS))
def test_waves_of_any_rays(gpu, name):
    """Rays inside the grid over their whole chord, steep ones, and rays along its faces, in waves of one kind and mixed."""
    dim, vox = GRIDS[name]
    rng = np.random.default_rng(61)
    o, h = [f32(-(d - 1) / 2 * v) for d, v in zip(dim, vox)], [f32(v) for v in vox]
    half = 0.5 * np.asarray(dim) * np.asarray(vox)
    n = 150_000
    xs, xe = random_rays(rng, n, o, h, dim, inside_frac=0.1)
    third = n // 3
    flat = slice(third, n)  # nearly transaxial: within the slices, or along the first and the last ones
    z = rng.uniform(-0.9, 0.9, n - third) * half[2]
    z[: third // 2] = half[2] * rng.choice([-1.0, 1.0], third // 2) * rng.uniform(0.9, 1.05, third // 2)
    xs[flat, 2], xe[flat, 2] = z, z + rng.uniform(-0.2, 0.2, n - third) * vox[2]
    img = rng.uniform(0.1, 2.0, dim).astype(np.float32)
    dev = torch.device("cuda")
    t = lambda a: torch.from_numpy(a).to(dev)  # noqa: E731
    G, dxs, dxe, dimg = gpu.ImageGeom(dim, vox), t(xs), t(xe), t(img)
    got = gpu.fwd(dxs, dxe, G, dimg)
    assert rel_l2(got.cpu().numpy(), oracle.fwd(xs, xe, o, h, dim, img)) <= TOL
    mixed = t(rng.permutation(n).astype(np.int32))
    assert torch.equal(gpu.fwd(dxs, dxe, G, dimg, order=mixed), got)
