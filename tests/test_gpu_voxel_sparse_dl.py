"""The voxelised model's gradient for dL/di that is zero in most pixels: the
gather looks at the rectangle of each camera's other pixels only.  One pixel at
a corner, two at opposite corners, the last pixel of the last camera, one in
each camera, none at all; cameras inside, outside and with a matrix that has no
inverse.  Against the oracle to 1e-10, as for the whole images; and the gradient
of a pixel takes less than half the time of the images' (a tenth, measured)."""
import math

import numpy as np
import pytest

from paper_1512_02110_amd import scenes

from ._scene_helpers import look_camera
from .test_gpu_voxel_gather import _cam

pytestmark = pytest.mark.gpu


def _scene():
    n, d = (19, 16, 14), (0.03, 0.05, 0.04)
    L = [a * b for a, b in zip(n, d)]
    rng = np.random.default_rng(12)
    b = rng.uniform(0.0, 3.0, n[0] * n[1] * n[2]) * (rng.random(n[0] * n[1] * n[2]) < 0.6)
    cams = [scenes.upward_camera(0.4 * L[0], 0.6 * L[1], 0.0, 13, 10, 80.0),
            _cam((0.5 * L[0], 0.5 * L[1], 0.0), [[1, 0, 0], [1, 0, 0], [0, 0, 1]], 8.0, 10, 9),
            look_camera((0.5 * L[0], 0.4 * L[1], 0.6 * L[2]), (0.3, 1, 0.2), (0, 0, 1), 70, 65, 110.0),
            look_camera((-0.2 * L[0], 0.5 * L[1], 0.5 * L[2]), (1, 0.1, 0), (0, 0, 1), 12, 9, 80.0)]
    return scenes.Scene(*n, *d, b, cams, 0.9, 0.8, 0.4, 0.3, 1000, 0, "sparse")


@pytest.mark.parametrize("case", ["corner", "corners", "last", "each", "none"])
@pytest.mark.parametrize("n_side", [1, 3])
def test_few_pixels_match_oracle(oracle, case, n_side):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1512_02110_amd import mcrt as M
    print(f"case voxel gradient of few pixels: {case}, n_side {n_side}", flush=True)
    s = _scene()
    first = np.cumsum([0] + [c.n_pix for c in s.cameras])
    dl = np.zeros(s.n_pix_total)
    big = s.cameras[2]
    at = {"corner": [first[0]], "corners": [first[2] + big.width - 1, first[2] + (big.height - 1) * big.width],
          "last": [first[4] - 1], "each": [first[i] + s.cameras[i].n_pix // 2 + 3 for i in range(4)], "none": []}[case]
    dl[at] = np.arange(1, len(at) + 1) - 3.5
    rng = np.random.default_rng(13)
    j = rng.uniform(0.0, 1.0, size=(s.n_cams, s.n_vox)) * (rng.random((s.n_cams, s.n_vox)) < 0.8)
    b = torch.as_tensor(s.beta, device="cuda")
    g = M.mc_voxel_grad(s, b, torch.as_tensor(j, device="cuda"), torch.as_tensor(dl, device="cuda"), n_side).cpu().numpy()
    ref = oracle.voxel_grad(s, j, dl, n_side)
    assert (np.abs(ref).max() > 0) == bool(at)
    assert np.allclose(g, ref, rtol=1e-10, atol=1e-12 * np.abs(ref).max())


def test_a_pixel_costs_less_than_the_images():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1512_02110_amd import mcrt as M
    print("case voxel gradient of one pixel, 4 cameras of 512 x 512", flush=True)
    n, d = 64, 0.02
    b = scenes.threshold_scale(scenes.value_noise(n, n, n, d, d, d, seed=2), 0.55, 50.0)
    s = scenes.Scene(n, n, n, d, d, d, np.ascontiguousarray(b).reshape(-1),
                     scenes.camera_lattice(2, n * d, n * d, 512, 512, 140.0), 0.99, 0.85, math.radians(45.0), 0.0, 1, 0,
                     "pixel")
    beta = torch.as_tensor(s.beta, device="cuda")
    j = (0.02 * (beta > 0)).repeat(s.n_cams).contiguous()
    dense = torch.randn(s.n_pix_total, dtype=torch.float64, device="cuda")
    one = torch.zeros_like(dense)
    one[s.n_pix_total // 2 + 256] = 1.0

    def best(dl):
        ms = []
        for _ in range(12):
            a, e = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            M.mc_voxel_grad(s, beta, j, dl, 2)
            e.record()
            torch.cuda.synchronize()
            ms.append(a.elapsed_time(e))
        return min(ms)
    t_dense, t_one = best(dense), best(one)
    assert t_one < 0.5 * t_dense, (t_one, t_dense)
