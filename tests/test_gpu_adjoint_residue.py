"""Events after a path's last light sample score exactly nothing (without an
environment), on recorded paths and on those traced a second time.

Volume: a dense half (x < 0) and an empty one.  Rays run towards +x and the
light shines along +x, so shadow rays leave through the dense half and a path
that has entered the empty half meets no light any more: table entry 0, which
only the empty half reaches, has no gradient."""
import dataclasses

import numpy as np
import pytest
import torch

import lfsynth as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1903_03837_amd as lp
    lp.library()
    return lp


# majorants (max. extinction 10): paths of a few records, of about the 64 that
# are kept, and of several hundred
@pytest.mark.parametrize("majorant", [12.5, 60.0, 250.0, 900.0])
def test_no_score_after_the_last_light(lp, majorant):
    M, N, n = 64, 80, 32
    z, y, x = np.meshgrid(*(np.arange(n),) * 3, indexing="ij")
    data = np.where(x < n // 2, 200, 0).astype(np.uint8).reshape(-1)
    lut = np.zeros((256, 4), np.float32)
    lut[:, :3] = (0.93, 0.87, 0.71)
    lut[2:, 3] = np.minimum(np.arange(2, 256) / 200.0, 1.0)
    sc = S.config(1, M=M, N=N, spp=32, max_bounces=8, g=0.2, majorant=majorant, grid=0)
    sc = dataclasses.replace(sc, volume=S.Volume(data, S.U8, (n, n, n), 0, 0.0, 255.0), medium=S.Medium(lut, 10.0),
                             light=S.Light(S.DIRECTIONAL, (-1.0, 0.0, 0.0), radiance=(3.1, 2.3, 1.7)))
    vol, med, light, prm, _ = lp.device_scene(sc)
    po, pd = lp.points(M)[0], lp.points(N)[0]
    right = pd[None, :, 0] - po[:, None, 0] > 0.1
    g = torch.Generator(device="cuda").manual_seed(1)
    adj = torch.randn((M, N, 3), device="cuda", generator=g) * right[..., None]
    d_lut, d_scale = lp.generate_backward(vol, med, light, prm, adj)
    assert float(d_scale) != 0.0 and float(d_lut[200, 3]) != 0.0 and float(d_lut[200, 0]) != 0.0
    assert d_lut[0].tolist() == [0.0, 0.0, 0.0, 0.0]
