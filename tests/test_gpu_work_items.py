"""The tracer's work items: the last rays of the queue are split into items of
a sample or two whose samples are summed by a second kernel.  The field must be
the mean the header defines, bit for bit, whatever was split: no ray, some rays
or all, ranges of unequal length, ray counts that fill neither tiles nor parts."""
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


def ranges(M, N, spp):
    """Sample ranges of the mean (lf_generate's definition)."""
    r_spp = 4 if spp >= 32 else 2 if spp >= 16 else 1
    r_rays = 4 if M * N < 1572864 else 2 if M * N < 12582912 else 1
    return 1 if M * N * spp > 2 ** 31 else min(r_spp, r_rays)


def mean_of_samples(sr, R):
    spp = sr.shape[2]
    total = None
    for q in range(R):
        acc = torch.zeros_like(sr[:, :, 0])
        for s in range(q * spp // R, (q + 1) * spp // R):
            acc = acc + sr[:, :, s]
        total = acc if total is None else total + acc
    return total / torch.tensor(float(spp), device=sr.device)


# (1, 1): one ray; 7 and 8 samples: the last count that is not split and the
# first that is; 1030 x 1030 at 8: more rays than are split; 9, 17, 33: ranges
# and items of unequal length; 13 x 11, 70 x 9: partial tiles, empty parts
@pytest.mark.parametrize("M,N,spp", [(1, 2, 8), (13, 11, 9), (70, 9, 17), (64, 64, 7), (64, 64, 8), (65, 130, 33),
                                     (600, 601, 33), (1030, 1030, 8)])
def test_field_is_the_mean_of_its_samples(lp, M, N, spp):
    sc = S.config(1, M=M, N=N, spp=spp, vol_n=32)
    vol, med, light, prm, _ = lp.device_scene(sc)
    sr = torch.zeros((M, N, spp, 3), device="cuda")
    lf = lp.generate(vol, med, light, prm, sample_radiance=sr)
    assert torch.equal(lf, mean_of_samples(sr, ranges(M, N, spp)))
    assert torch.equal(lf, lp.generate(vol, med, light, prm))
    if M > 64:  # a slab whose rays are all split, of a field whose rays are not
        p = dataclasses.replace(prm, row_begin=3, row_end=20)
        out = torch.full_like(lf, -1.0)
        lp.generate(vol, med, light, p, out=out)
        assert torch.equal(out[3:20], lf[3:20]) and bool((out[:3] == -1.0).all()) and bool((out[20:] == -1.0).all())


@pytest.mark.parametrize("env", [(0.0, 0.0, 0.0), (0.3, 0.1, 0.2)])
def test_environment_of_missing_rays(lp, env):
    """Rays that miss the box hold the environment exactly, split or not."""
    sc = S.config(1, M=96, N=96, spp=16, vol_n=32)
    sc = dataclasses.replace(sc, light=dataclasses.replace(sc.light, radiance=(0.0, 0.0, 0.0), env=env),
                             medium=S.Medium(sc.medium.lut, 0.0))
    vol, med, light, prm, _ = lp.device_scene(sc)
    lf = lp.generate(vol, med, light, prm)
    # 16 additions of one value and a division by 16, in FP32: 8 + 8 partial sums
    e = np.float32(0.0)
    want = []
    for c in env:
        half = np.float32(0.0)
        for _ in range(8):
            half = np.float32(half + np.float32(c))
        want.append(np.float32((half + half) / np.float32(16.0)))
    off = ~torch.eye(96, dtype=torch.bool, device="cuda")
    assert torch.equal(lf[off], torch.tensor(want, device="cuda").expand(96 * 95, 3))
    assert bool((lf[~off] == float(e)).all())


def test_views_do_not_depend_on_the_batch(lp):
    """A view's pixels are keyed by their index in the batch, so the first view
    is the same alone (every pixel split) and before others (some split)."""
    sc = S.config(2, vol_n=32, spp=33, views=4)
    vol, med, light, prm, cams = lp.device_scene(sc)
    alone = lp.render_views(vol, med, light, prm, cams[:1], 331, 301)
    batch = lp.render_views(vol, med, light, prm, cams, 331, 301)  # 398524 pixels, 262144 of them split
    assert torch.equal(alone[0], batch[0])
