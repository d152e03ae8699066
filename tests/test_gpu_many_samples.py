"""Sample counts at which a product of an item's number and the sample count
passes 32 bits, in the volume tracer, the views and the isosurface variant."""
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


# the last count below the overflow, the first above it, and an odd one there
@pytest.mark.parametrize("spp", [65535, 65536, 70001])
def test_field_is_the_mean_of_its_samples(lp, spp):
    sc = S.config(1, M=2, N=3, spp=spp, vol_n=32, max_bounces=2)
    vol, med, light, prm, _ = lp.device_scene(sc)
    sr = torch.zeros((2, 3, spp, 3), device="cuda")
    lf = lp.generate(vol, med, light, prm, sample_radiance=sr)
    x = sr.cpu().numpy()
    total = np.zeros((2, 3, 3), np.float32)
    for q in range(4):  # four ranges, each summed in sample order in FP32
        total = total + np.cumsum(x[:, :, q * spp // 4:(q + 1) * spp // 4], axis=2, dtype=np.float32)[:, :, -1]
    assert np.any(total > 0)
    assert np.array_equal(lf.cpu().numpy(), total / np.float32(spp))


@pytest.mark.parametrize("surface", [0, 1])
@pytest.mark.parametrize("spp", [65535, 65536, 70001])
def test_white_furnace(lp, surface, spp):
    """Albedo 1 in an environment of 1 and no light: every sample is exactly 1,
    and sums of at most 2^24 ones are exact."""
    sc = S.config(2, vol_n=32, M=2, N=3, spp=spp, views=1, max_bounces=500)
    lut = sc.medium.lut.copy()
    lut[:, :3] = 1.0
    sc = dataclasses.replace(sc, medium=S.Medium(lut, 1.0), light=dataclasses.replace(
        sc.light, radiance=(0.0, 0.0, 0.0), env=(1.0, 1.0, 1.0))).with_params(surface=surface, iso=524.0)
    vol, med, light, prm, cams = lp.device_scene(sc)
    assert bool((lp.generate(vol, med, light, prm) == 1.0).all())
    assert bool((lp.render_views(vol, med, light, prm, cams, 3, 2) == 1.0).all())
