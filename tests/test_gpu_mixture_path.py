"""Path scores of the full mixture gradient where the wavefront shares a
collision's cameras: one photon alone, a wavefront's worth, more cameras than
lanes and one camera (every lane walks its own), with collisions past the
sums that a photon's row holds.  FP64 against the oracle, with the tolerance
of the existing dense-aerosol test (its collisions per photon): 1e-9, and
1e-12 of the largest value."""
import numpy as np
import pytest

from paper_1512_02110_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_side,cap", [(1, 2, 0), (64, 9, 0), (130, 1, 0), (700, 3, 0), (700, 3, 400_000)])
def test_path_scores_match_oracle(oracle, n, n_side, cap):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1512_02110_amd import mcrt as M
    print(f"case mixture path {n} photons, {n_side}^2 cameras, tape limit {cap}", flush=True)
    s = scenes.config1(n_photons=n, seed=4)
    s.albedo = 0.99
    s.cameras = scenes.camera_lattice(n_side, 0.79, 0.77, 5, 4, 65.0, z=0.013)
    z = (np.arange(s.nz) + 0.5) * s.dz
    air = np.ascontiguousarray(np.broadcast_to((2.0 * np.exp(-z / 8.0))[:, None, None], (16, 16, 16)).reshape(-1))
    aer = 30.0 * s.beta
    dl = np.random.default_rng(3).normal(size=s.n_pix_total)
    dev = [torch.as_tensor(x, device="cuda") for x in (air, aer, dl)]
    g, st = M.mc_grad_mixture(s, dev[0], dev[1], dev[2], 1.0, full=True, transport="fp64", tape_limit=cap)
    ref, rst = oracle.grad_mix(s, dl, air, aer, sigma=1.0, full=True)
    for k in ("photons", "events", "le_jobs", "vox_free", "rr_killed", "capped"):
        assert st[k] == rst[k], k
    assert np.allclose(g.cpu().numpy(), ref, rtol=1e-9, atol=1e-12 * max(np.abs(ref).max(), 1e-300))
