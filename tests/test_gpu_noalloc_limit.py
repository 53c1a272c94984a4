"""The no-allocation render takes inputs up to the last byte of its fixed scratch
(64 MiB): 512 x 512 x 63 voxels, whose bitmask fills its words exactly, and as
many cameras as fit beside them.  One camera table more is refused."""
import numpy as np
import pytest

from paper_1512_02110_amd import scenes

pytestmark = pytest.mark.gpu

LIMIT = 64 << 20


def _round(n):
    return (n + 255) // 256 * 256


def _scratch(s):
    """Bytes of an FP32 render: counters, beta with its zeros and a value a layer,
    a flag, the cameras' tables (184 and 48 bytes each), a bit per run of 128
    voxels, and 256 to spare."""
    nc = len(s.cameras)
    return (256 + _round(4 * (s.n_vox + 64 + s.nz)) + 256 + _round(184 * nc) + _round(48 * nc)
            + _round(4 * (s.n_vox // 128 // 32)) + 256)


def test_the_last_camera_that_fits():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1512_02110_amd import mcrt as M
    print("case noalloc at the end of its scratch, 512x512x63", flush=True)
    n, d = (512, 512, 63), 0.02
    b = np.zeros(n[0] * n[1] * n[2])
    b[::1000] = 5.0
    cams = [scenes.upward_camera(0.05 + 10.1 * (i % 67) / 67, 0.05 + 10.1 * (i // 67) / 67, 0.0, 1, 1, 60.0)
            for i in range(4443)]
    s = scenes.Scene(*n, d, d, d, b, cams, 0.9, 0.8, 0.5, 0.3, 500, 7, "limit")
    assert _scratch(s) == LIMIT and s.n_vox % (128 * 32) == 0
    beta = M.beta_tensor(s, "fp32")
    ref, rst = M.mc_render(s, beta)
    img, st = M.mc_render_noalloc(s, beta)
    assert st == rst and st["le_jobs"] > 0
    assert torch.allclose(img, ref, rtol=1e-12, atol=1e-14 * float(ref.abs().max()))
    more = s.replace(cameras=cams + cams[:6])
    assert _scratch(more) > LIMIT
    with pytest.raises(M.McError) as e:
        M.mc_render_noalloc(more, beta)
    assert e.value.code == M.MC_ERR_SCRATCH_LIMIT
