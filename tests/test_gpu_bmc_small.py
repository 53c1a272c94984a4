"""Backward Monte Carlo at the sizes where its packets run out: fewer packets
than a wavefront has lanes, one more than a launch list holds, cameras whose
rays all miss the domain, and long packets alone in their wavefront, whose
estimates other lanes walk.  FP64 transport follows the oracle's packets:
equal counters, images and second moments to the order of FP64 sums and the
rounding of the walks (1e-9 relative per pixel, as in the larger tests)."""
import numpy as np
import pytest

from paper_1512_02110_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w,h,n_pp,tau,z", [
    (1, 1, 1, 2.0, 0.0), (3, 1, 21, 30.0, 0.0), (13, 5, 1, 8.0, 0.0), (65, 1, 1, 0.5, -0.3), (4, 4, 4, 5.0, 1.5),
])
def test_few_packets_match_oracle(oracle, w, h, n_pp, tau, z):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1512_02110_amd import mcrt as M
    print(f"case bmc {w}x{h} {n_pp} packets a pixel, depth {tau}, camera at {z}", flush=True)
    rng = np.random.default_rng(w + n_pp)
    n, d = (9, 7, 11), 0.1
    b = rng.uniform(0.0, 2.0, 9 * 7 * 11) * (rng.random(9 * 7 * 11) < 0.8) * tau / (11 * d)
    cams = [scenes.upward_camera(0.37, 0.31, z, w, h, 60.0)]  # z = 1.5: above the domain, looking away
    s = scenes.Scene(*n, d, d, d, b, cams, 1.0, 0.8, 0.5, 0.3, 1000, 17, "bmc")
    img, st, m2 = M.mc_bmc_render(s, M.beta_tensor(s, "fp64"), n_pp, transport="fp64", with_m2=True)
    ref, rst, rm2 = oracle.bmc_render(s, n_pp, with_m2=True)
    for k in ("photons", "events", "vox_free", "esc_top", "esc_bottom", "esc_side", "rr_killed", "capped"):
        assert st[k] == rst[k], k
    img, m2 = img.cpu().numpy(), m2.cpu().numpy()
    assert np.allclose(img, ref, rtol=1e-9, atol=1e-300)
    assert np.allclose(m2, rm2, rtol=2e-9, atol=1e-300)
