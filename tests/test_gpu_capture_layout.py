"""The gather capture on the render's own copy of beta: its index steps follow the
axis that the cameras look along where the bitmask's runs are at most an eighth
of the grid along it, and stay x fastest one voxel below that; every captured
index is n_vox or a voxel of a run of that copy that holds extinction; counters
and images are the render's; and the gather ceiling replays these indices."""
import numpy as np
import pytest

from paper_1512_02110_amd import scenes

from ._scene_helpers import look_camera

pytestmark = pytest.mark.gpu


def _scene(axis, n):
    d = 0.02
    L = [a * d for a in n]
    f = [0.03, 0.02, 0.01]
    f[axis] = 1.0
    up = (0, 1, 0) if axis == 2 else (0, 0, 1)
    cams = [look_camera(tuple((0.01 if a == axis else 0.47) * L[a] for a in range(3)), f, up, 32, 32, 75.0)]
    b = np.random.default_rng(3).uniform(1.0, 9.0, n[0] * n[1] * n[2])
    b[np.random.default_rng(4).random(b.size) < 0.85] = 0.0  # most runs of one voxel are empty, few of many
    return scenes.Scene(*n, d, d, d, b, cams, 1.0, 0.8, 0.5, 0.3, 60_000, 3, "capture")


@pytest.mark.parametrize("axis,n,fast", [
    (2, (64, 64, 64), 2),     # runs of 2
    (1, (64, 64, 64), 1),
    (0, (64, 64, 64), 0),
    (2, (128, 128, 32), 2),   # runs of 4, an eighth of 32
    (2, (136, 124, 31), 0),   # of 4, more than an eighth of 31
    (2, (40, 30, 20), 2),     # a bit per voxel
])
def test_capture_walks_the_renders_copy(axis, n, fast):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1512_02110_amd import mcrt as M
    print(f"case capture layout axis {axis} {n}", flush=True)
    s = _scene(axis, n)
    beta = M.beta_tensor(s, "fp32")
    idx, steps, nw, strides, st = M.mc_capture_render_gathers(s, beta, 30, 16, 4096)
    nx, ny, nz = n
    assert strides == {0: (1, nx, nx * ny), 1: (ny, 1, nx * ny), 2: (nz, nx * nz, 1)}[fast]
    _, rst = M.mc_render(s, beta)
    assert st == rst
    msh = 0
    while -(-s.n_vox // (1 << msh)) > 131072:
        msh += 1
    z, y, x = np.meshgrid(*(np.arange(a) for a in (nz, ny, nx)), indexing="ij")
    copy = np.zeros((((s.n_vox - 1) >> msh) + 1) << msh)
    copy[(strides[0] * x + strides[1] * y + strides[2] * z).reshape(-1)] = s.beta
    run = (copy.reshape(-1, 1 << msh) > 0).any(axis=1)
    full = steps[:nw].cpu().numpy() >= 46
    assert full.any()
    got = idx[:nw].cpu().numpy().view(np.uint32)[full].astype(np.int64)
    assert got.max() <= s.n_vox and (got < s.n_vox).any()
    assert np.append(run[np.arange(s.n_vox) >> msh], True)[got].all()


def test_ceiling_reports_the_renders_copy():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1512_02110_amd import micro
    print("case gather ceiling on a flat grid", flush=True)
    s = _scene(2, (136, 124, 31))
    r = micro.gather_ceiling(s, 2_000_000, first_step=30, n_steps=48, reps=2)  # (wavefronts of 80 steps and more)
    assert r["index_strides_xyz"] == [1, 136, 136 * 124]
    assert r["replay_gloads_per_s"] > 0 and r["frac_algorithmic_of_replay"] <= r["frac_issued_of_replay"]
