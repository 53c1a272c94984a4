"""The ray bins of the large-grid gradient: one camera, counts around the
powers of two of the camera search, around the cameras whose centres the
kernels keep in LDS (256) and around those whose first pixels they keep
(2048); odd numbers of rays, tiles cut by the grid's faces.  FP64 against the
oracle to 1e-9 (the order of FP64 sums).  FP32 bins against FP32 device
atomics, which deposit the same rays: a bin's walk sums its crossings, so a
segment is off by up to 64 roundings of 2^-24, i.e. 4e-6 of the crossing's
parameter, hence 1e-4 of the largest value."""
import numpy as np
import pytest

from paper_1512_02110_amd import scenes

from ._scene_helpers import look_camera

pytestmark = pytest.mark.gpu


def _scene(n_cams):
    rng = np.random.default_rng(n_cams)
    n, d = (37, 21, 19), (0.05, 0.06, 0.07)
    L = [a * b for a, b in zip(n, d)]
    cams = [look_camera((rng.uniform(0.1, 0.9) * L[0], rng.uniform(0.1, 0.9) * L[1], L[2] * (1.1 + 0.9 * rng.random())),
                        (0.1 * rng.normal(), 0.1 * rng.normal(), -1.0), (0, 1, 0), 1 + i % 3, 1 + i % 2, 100.0)
            for i in range(n_cams)]
    b = rng.uniform(0.5, 6.0, n[0] * n[1] * n[2]) * (rng.random(n[0] * n[1] * n[2]) < 0.5)
    return scenes.Scene(*n, *d, b, cams, 0.95, 0.7, 0.4, 0.3, max(31, 3001 // n_cams), 29, "binning")


@pytest.mark.parametrize("n_cams", [1, 2, 3, 33, 256, 257, 2049])
def test_bins_match_oracle(oracle, n_cams):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1512_02110_amd import mcrt as M
    print(f"case binning {n_cams} cameras", flush=True)
    s = _scene(n_cams)
    dl = np.random.default_rng(1).normal(size=sum(c.n_pix for c in s.cameras))
    dlt = torch.as_tensor(dl, device="cuda")
    ref, _ = oracle.grad_beta(s, dl)
    top = np.abs(ref).max()
    assert top > 0
    beta = M.beta_tensor(s, "fp64")
    assert np.allclose(M.mc_grad_beta(s, beta, dlt, transport="fp64")[0].cpu().numpy(), ref, rtol=1e-9, atol=1e-11 * top)
    _, _, tape = M.mc_render_tape(s, beta, transport="fp64")
    assert tape is not None
    for w in (dlt, -2.0 * dlt):  # a kept tape serves several gradients
        got = M.mc_grad_beta(s, beta, w, transport="fp64", tape=tape)[0].cpu().numpy()
        assert np.allclose(got, ref * (1.0 if w is dlt else -2.0), rtol=1e-9, atol=2e-11 * top)
    tape.free()
    b32 = M.beta_tensor(s, "fp32")
    bins = M.mc_grad_beta(s, b32, dlt, transport="fp32")[0].cpu().numpy()
    atomics = M.mc_grad_beta(s, b32, dlt, transport="fp32", tape_limit=100)[0].cpu().numpy()
    assert np.abs(bins - atomics).max() <= 1e-4 * np.abs(atomics).max()
