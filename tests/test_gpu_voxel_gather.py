"""The voxelised model's gathers against the oracle where their parts meet:
voxels inside and outside the near boxes, footprints of one ray and of the
whole image, cameras inside, outside and looking sideways or away, matrices
that are not rotations (walked whole), beams of lines of sight past the LDS
copy's room and slices, tiles cut by the grid, and pixels of more rays than a
block has lanes.

Both sides are FP64 and differ in the order of their sums and in crossings
rounded differently (an ulp each): 1e-10 relative, as for the other
deterministic parts; the ray counts are equal."""
import numpy as np
import pytest

from paper_1512_02110_amd import scenes

from ._scene_helpers import look_camera

pytestmark = pytest.mark.gpu


def _cam(pos, R, f, w, h):
    return scenes.Camera(pos=pos, R=tuple(float(x) for x in np.asarray(R).reshape(-1)), fx=f, fy=0.9 * f, cx=w / 2.0,
                         cy=h / 2.0, width=w, height=h)


def _cameras(case, L):
    c = [0.5 * x for x in L]
    if case == "up":
        return scenes.camera_lattice(2, L[0], L[1], 13, 10, 70.0)
    if case == "sideways":
        return [look_camera((-0.2 * L[0], c[1], c[2]), (1, 0.1, 0), (0, 0, 1), 12, 9, 80.0),
                look_camera((c[0], c[1], c[2]), (0.3, 1, 0.2), (0, 0, 1), 11, 12, 110.0),
                look_camera((c[0], 1.3 * L[1], 1.4 * L[2]), (0, -1, -1), (0, 0, 1), 9, 9, 60.0)]
    if case == "away":
        return [look_camera((c[0], c[1], 1.5 * L[2]), (0, 0, 1), (0, 1, 0), 8, 8, 60.0),
                look_camera((c[0], c[1], 0.0), (0, 0, 1), (0, 1, 0), 8, 8, 60.0)]
    if case == "tele":  # a voxel fills the image
        return [look_camera((c[0], c[1], -0.1 * L[2]), (0, 0, 1), (0, 1, 0), 25, 25, 3.0)]
    # matrices that are not rotations: scaled and sheared (an inverse exists), singular (none)
    return [_cam((c[0], c[1], 0.0), [[1.5, 0, 0.2], [0.1, 0.8, 0], [0, 0, 2.0]], 8.0, 10, 9),
            _cam((c[0], c[1], 0.0), [[1, 0, 0], [1, 0, 0], [0, 0, 1]], 8.0, 10, 9)]


@pytest.mark.parametrize("case,n,d,n_side", [
    ("up", (17, 13, 23), (0.05, 0.05, 0.05), 2),
    ("sideways", (19, 16, 14), (0.03, 0.05, 0.04), 3),
    ("away", (9, 9, 9), (0.1, 0.1, 0.1), 1),
    ("tele", (10, 10, 25), (0.1, 0.1, 0.1), 2),
    ("matrix", (14, 15, 16), (0.06, 0.05, 0.07), 2),
    ("sideways", (300, 20, 9), (0.05, 0.04, 0.04), 1),
    ("up", (1, 1, 1), (0.2, 0.2, 0.2), 17),
])
def test_gathers_match_oracle(oracle, case, n, d, n_side):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1512_02110_amd import mcrt as M
    print(f"case voxel gather {case} {n} n_side {n_side}", flush=True)
    rng = np.random.default_rng(11)
    b = rng.uniform(0.0, 3.0, n[0] * n[1] * n[2]) * (rng.random(n[0] * n[1] * n[2]) < 0.6)
    s = scenes.Scene(*n, *d, b, _cameras(case, [x * y for x, y in zip(n, d)]), 0.9, 0.8, 0.4, 0.3, 1000, 0, case)
    # (j also where beta is zero: the local term of the gradient is there)
    j = rng.uniform(0.0, 1.0, size=(s.n_cams, s.n_vox)) * (rng.random((s.n_cams, s.n_vox)) < 0.8)
    dl = rng.normal(size=s.n_pix_total) * (rng.random(s.n_pix_total) < 0.9)
    q = rng.uniform(0.2, 2.0, size=j.shape)
    dev = {k: torch.as_tensor(v, device="cuda") for k, v in dict(b=b, j=j, dl=dl, q=q).items()}
    img = M.mc_voxel_render(s, dev["b"], dev["j"], n_side).cpu().numpy()
    ref = oracle.voxel_render(s, j, n_side)
    assert np.allclose(img, ref, rtol=1e-10, atol=1e-13 * max(np.abs(ref).max(), 1e-300))
    for w, qw in ((None, None), (dev["q"], q)):
        g = M.mc_voxel_grad(s, dev["b"], dev["j"], dev["dl"], n_side, cam_weights=w).cpu().numpy()
        gref = oracle.voxel_grad(s, j, dl, n_side, q=qw)
        assert np.allclose(g, gref, rtol=1e-10, atol=1e-12 * np.abs(gref).max())
    counts, _ = M.mc_voxel_conditioning(s, n_side)
    rc, _ = oracle.voxel_conditioning(s, n_side)
    assert np.array_equal(counts.cpu().numpy(), rc.reshape(-1))
