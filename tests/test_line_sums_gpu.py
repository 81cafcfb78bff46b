"""The fixed-point sums of the back projection by a ray per lane (k_back_lines): what a sheet keeps of one line's rays.

A list long enough for the kernel holds one line of rays with values, all others are 0, so that the image is the sheet
itself.  Tolerance: a sheet's unit u is at most 2 S / 2^31 for bounds that sum to S; a value's two shares are rounded to
it, and N values in an entry err by sqrt(N) u / 2 at most in the root mean square.  The entry holds S / n_slices, each
slice taking its part of N = 2 rays / n_slices; the flush adds three float32 roundings (1e-7):
rel <= sqrt(2 rays / n_slices) n_slices / 2^31 + 1e-7."""
import numpy as np
import pytest
import torch

import oracle
from helpers import f32, rel_l2

pytestmark = pytest.mark.gpu

DIM, VOX = (61, 75, 33), (3.1, 2.7, 2.5)
N, GROUP = 5_900_000, 512


def _line(angle, off, rays):
    half = 0.5 * np.asarray(DIM) * np.asarray(VOX)
    d, nrm = np.array([np.cos(angle), np.sin(angle)]), np.array([-np.sin(angle), np.cos(angle)])
    xy = np.array([off * nrm - 1.6 * half[1] * d, off * nrm + 1.6 * half[1] * d], np.float32)
    # ring pairs of 41 rings, the second one fastest, as a sinogram has them
    pairs = np.array([(a, b) for a in range(41) for b in range(41) if abs(a - b) <= 20])
    z = (pairs[np.arange(rays) % len(pairs)] / 20.0 - 1.0) * 0.85 * half[2]
    return [np.column_stack([np.tile(xy[i], (rays, 1)), z[:, i]]).astype(np.float32) for i in range(2)]


@pytest.mark.parametrize("angle", [0.3, 1.8])
@pytest.mark.parametrize("groups,growth", [(1, 1.0), (4, 1.0), (4, 3.0), (4, 0.2), (24, 1.0)])
def test_bits_of_a_line(gpu, angle, groups, growth):
    """One group of rays, and several on one line whose values stay, grow (the fixed point is coarsened, or the sheet
    flushed) or fall."""
    rays = groups * GROUP
    xs, xe = _line(angle, 7.3, rays)
    o, h = [f32(-(d - 1) / 2 * v) for d, v in zip(DIM, VOX)], [f32(v) for v in VOX]
    y = growth ** (np.arange(rays) // GROUP).astype(np.float64)
    y *= np.random.default_rng(32).uniform(0.9, 1.1, rays)
    y = y.astype(np.float32)
    want = oracle.back(xs, xe, o, h, DIM, y)
    dev = torch.device("cuda")
    at = 777 * GROUP
    all_s, all_e = (torch.from_numpy(a[:1]).to(dev).expand(N, 3).clone() for a in (xs, xe))
    p = torch.zeros(N, device=dev)
    for full, part in ((all_s, xs), (all_e, xe), (p, y)):
        full[at:at + rays] = torch.from_numpy(part).to(dev)
    got = gpu.back(all_s, all_e, gpu.ImageGeom(DIM, VOX), p).cpu().numpy()
    assert rel_l2(got, want) <= np.sqrt(2.0 * rays / DIM[2]) * DIM[2] / 2.0**31 + 1e-7
