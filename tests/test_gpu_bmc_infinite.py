"""Backward Monte Carlo under a lid whose depth is past the transport type's
range (finite extinctions times lengths that sum to infinity, and infinite
ones): every path to the sun through it has an estimate of zero and ends there
like any other (exp(-inf) = 0).  The camera looks along a thick layer of almost
forward scattering under the lid, so that no flight reaches the lid, packets
collide many times, and few of them share a wavefront, whose idle lanes walk
the estimates.  Half of the lid is open, so that the images are not all zero.
FP64 follows the oracle's packets: equal counters, images to the order of FP64
sums and the rounding of the walks (1e-9, as in the other tests of few packets).
FP32 packets leave the oracle's where a choice rounds the other way: pixels to
max(1e-3 relative, 3 sigma) as the larger FP32 test has it, with a thousandth
of the events."""
import math

import numpy as np
import pytest

from paper_1512_02110_amd import scenes

from ._scene_helpers import look_camera

pytestmark = pytest.mark.gpu


def _scene(lid, d):
    n = (24, 6, 6)
    b = np.full((n[2], n[1], n[0]), 1.0 / d)
    b[-1] = 0.0
    b[-1, :, :13] = lid
    cam = look_camera((-0.5 * d, 3.1 * d, 2.2 * d), (1.0, 0.0, 0.0), (0, 0, 1), 5, 3, 20.0)
    return scenes.Scene(*n, d, d, d, b.reshape(-1), [cam], 0.98, 0.9995, math.radians(20.0), 0.2, 1, 11, "lid")


@pytest.mark.parametrize("transport,lid,d,n_pp", [
    ("fp64", 1e308, 3.0, 1), ("fp64", 1e308, 3.0, 9), ("fp64", np.inf, 0.1, 4), ("fp32", 3e38, 3.0, 1),
    ("fp32", 3e38, 3.0, 9), ("fp32", np.inf, 0.1, 4),
])
def test_infinite_depth_to_the_sun(oracle, transport, lid, d, n_pp):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1512_02110_amd import mcrt as M
    print(f"case bmc under a lid of {lid}, {transport}, {n_pp} packets a pixel", flush=True)
    s = _scene(lid, d)
    img, st, m2 = M.mc_bmc_render(s, M.beta_tensor(s, transport), n_pp, transport=transport, with_m2=True)
    # (the oracle takes finite extinctions: at 1e6 per voxel the lid is as dark)
    ref, rst, rm2 = oracle.bmc_render(_scene(min(lid, 1e6 / d), d), n_pp, with_m2=True)
    img, m2 = img.cpu().numpy(), m2.cpu().numpy()
    assert np.isfinite(img).all() and (ref > 0).any() and rst["events"] > 3 * rst["photons"]
    if transport == "fp64":
        for k in ("photons", "events", "vox_free", "esc_top", "esc_bottom", "esc_side", "rr_killed", "capped"):
            assert st[k] == rst[k], k
        assert np.allclose(img, ref, rtol=1e-9, atol=1e-300)
        assert np.allclose(m2, rm2, rtol=2e-9, atol=1e-300)
    else:
        sig = np.sqrt(np.maximum(np.maximum(m2, rm2) - ref ** 2, 0.0) / n_pp)
        assert (np.abs(img - ref) <= np.maximum(1e-3 * np.abs(ref), 3 * sig)).all()
        assert abs(st["events"] - rst["events"]) <= max(2, 1e-3 * rst["events"])
