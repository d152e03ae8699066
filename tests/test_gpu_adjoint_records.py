"""The adjoint records a path's events and scores them once its radiance is
known; a path or a shadow ray of more than 64 records is replayed instead.
Majorants from the tight one to 60 times it take paths and shadow rays from a
few records to several hundred, so every route and the change between them is
run, with the radiance kept by the forward and without."""
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


@pytest.mark.parametrize("factor,bounces,lit", [(1.0, 3, True), (1.0, 1, True), (3.0, 3, False), (6.0, 8, True),
                                                (20.0, 3, True), (60.0, 2, True), (60.0, 8, False)])
def test_gradient_over_list_lengths(lp, orc, factor, bounces, lit):
    M, N, spp = 40, 52, 6
    sc = S.config(1, M=M, N=N, spp=spp, max_bounces=bounces, g=0.3)
    lut = (0.05 + 0.9 * sc.medium.lut).astype(np.float32)
    lut[0, 3] = 0.0
    light = dataclasses.replace(sc.light, env=(0.3, 0.2, 0.1))
    if not lit:
        light = dataclasses.replace(light, radiance=(0.0, 0.0, 0.0))
    sc = sc.replace(medium=S.Medium(lut, 25.0), light=light)
    sc = sc.with_params(majorant=factor * orc.majorant(sc.medium, sc.params))
    rng = np.random.default_rng(5)
    ks = np.sort(rng.choice(M * N, 500, replace=False))
    adj = np.zeros((M * N, 3), np.float32)
    adj[ks] = rng.standard_normal((500, 3))
    vol, med, lgt, prm, _ = lp.device_scene(sc)
    d = torch.from_numpy(adj).cuda()
    srad = torch.zeros((M, N, spp, 3), dtype=torch.float32, device="cuda")
    lp.generate(vol, med, lgt, prm, sample_radiance=srad)
    a_lut, a_s = lp.generate_backward(vol, med, lgt, prm, d)
    b_lut, b_s = lp.generate_backward(vol, med, lgt, prm, d, sample_radiance=srad)
    a = np.append(a_lut.double().cpu().numpy(), float(a_s))
    b = np.append(b_lut.double().cpu().numpy(), float(b_s))
    # the same decisions and scores, added up in another order
    assert np.linalg.norm(a - b) <= 1e-5 * np.linalg.norm(a)
    o_lut, o_s = orc.gradient(sc, ks, adj[ks].astype(np.float64))
    o = np.append(o_lut, o_s)
    err = np.linalg.norm(a - o) / np.linalg.norm(o)
    print(f"factor {factor}, {bounces} bounces: adjoint vs oracle {err:.2e}")
    # FP32 decides a collision differently from FP64 about once in 2^22 events
    # (~10^6 here), which replaces one of 3000 samples: 1/sqrt(3000) of the norm
    assert err <= 3e-2
