"""The kernels' copy of beta runs along the axis that the cameras look along:
renders, kept rays, replayed gradients, the voxel pass and the frozen-event
render against the oracle for cameras looking along each axis, on grids whose
sides are not multiples of the copy's tiles and whose bitmask's runs cross its
columns.  FP64 follows the oracle's photons: images and gradients to 1e-9 (the
order of FP64 sums), equal counters of the photons' paths."""
import numpy as np
import pytest

from paper_1512_02110_amd import scenes

from ._scene_helpers import look_camera

pytestmark = pytest.mark.gpu


def _scene(axis, n):
    rng = np.random.default_rng(5 + axis)
    d = (0.05, 0.04, 0.06)
    L = [a * b for a, b in zip(n, d)]
    f = [0.03, 0.02, 0.01]
    f[axis] = 1.0
    up = (0, 1, 0) if axis == 2 else (0, 0, 1)
    cams = [look_camera(tuple(0.13 * L[a] if a == axis else 0.47 * L[a] for a in range(3)), f, up, 9, 8, 75.0),
            look_camera(tuple(-0.21 * L[a] if a == axis else 0.53 * L[a] for a in range(3)), f, up, 11, 7, 60.0)]
    b = rng.uniform(0.5, 6.0, n[0] * n[1] * n[2]) * (rng.random(n[0] * n[1] * n[2]) < 0.5)
    return scenes.Scene(*n, *d, b, cams, 0.95, 0.7, 0.5, 0.3, 3000, 23, "layout")


@pytest.mark.parametrize("axis,n", [(0, (37, 33, 5)), (1, (33, 31, 34)), (2, (35, 17, 65)), (2, (3, 2, 40)),
                                    (1, (64, 90, 48))])
def test_layouts_match_oracle(oracle, axis, n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1512_02110_amd import mcrt as M
    print(f"case layout axis {axis} {n}", flush=True)
    s = _scene(axis, n)
    beta = M.beta_tensor(s, "fp64")
    ref, rst = oracle.render(s)
    assert np.abs(ref).max() > 0
    img, st = M.mc_render(s, beta, transport="fp64")
    for k in ("events", "le_jobs", "vox_free", "esc_top", "esc_bottom", "esc_side", "rr_killed"):
        assert st[k] == rst[k], k
    tol = dict(rtol=1e-9, atol=1e-12 * np.abs(ref).max())
    assert np.allclose(img.cpu().numpy(), ref, **tol)
    assert np.allclose(M.mc_render_noalloc(s, beta, transport="fp64")[0].cpu().numpy(), ref, **tol)
    assert np.allclose(M.mc_render_frozen(s, beta, beta, transport="fp64")[0].cpu().numpy(), ref, **tol)
    mixed = M.mc_render(s, beta, transport="mixed")[0].cpu().numpy()
    assert np.allclose(mixed, ref, rtol=1e-4, atol=1e-4 * np.abs(ref).max())
    dl = np.random.default_rng(1).normal(size=ref.size)
    dlt = torch.as_tensor(dl, device="cuda")
    gref, _ = oracle.grad_beta(s, dl)
    gtol = dict(rtol=1e-9, atol=1e-11 * np.abs(gref).max())
    assert np.allclose(M.mc_grad_beta(s, beta, dlt, transport="fp64")[0].cpu().numpy(), gref, **gtol)
    # (a tape too small for a block of records: device atomics)
    assert np.allclose(M.mc_grad_beta(s, beta, dlt, transport="fp64", tape_limit=100)[0].cpu().numpy(), gref, **gtol)
    _, _, tape = M.mc_render_tape(s, beta, transport="fp64")
    if tape is not None:
        assert np.allclose(M.mc_grad_beta(s, beta, dlt, transport="fp64", tape=tape)[0].cpu().numpy(), gref, **gtol)
        tape.free()
    j = M.mc_voxel_scatter(s, beta, transport="fp64")[0].cpu().numpy()
    jref = np.asarray(oracle.voxel_scatter(s)[0]).reshape(-1)
    assert np.allclose(j, jref, rtol=1e-9, atol=1e-12 * np.abs(jref).max())
