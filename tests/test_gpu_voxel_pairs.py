"""The tracer's voxel fetch reads each pair of x-neighbours with one load from
the halo-brick copy.  The copy's edges decide whether that can go wrong: the
first and last base voxel of a brick, dimensions of every remainder mod 3,
volumes of one brick, and the last brick of the copy; for each voxel type."""
import dataclasses
import math

import numpy as np
import pytest
import torch

import lfsynth as S

pytestmark = pytest.mark.gpu

DTYPE = {S.U8: np.uint8, S.U16: np.uint16, S.F32: np.float32}


@pytest.fixture(scope="module")
def lp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1903_03837_amd as lp
    lp.library()
    return lp


@pytest.mark.parametrize("dims", [(2, 2, 2), (3, 4, 5), (5, 3, 4), (4, 5, 3), (8, 2, 31), (33, 7, 2), (17, 18, 19)])
@pytest.mark.parametrize("vtype", [S.U8, S.U16, S.F32])
def test_ragged_volumes_match_oracle(lp, orc, vtype, dims):
    rng = np.random.default_rng(17 * vtype + sum(dims))
    top = {S.U8: 255, S.U16: 4000, S.F32: 1.0}[vtype]
    data = (rng.uniform(0.0, top, dims[0] * dims[1] * dims[2])).astype(DTYPE[vtype])
    sc = S.config(1, M=24, N=24, spp=8, grid=3)
    sc = dataclasses.replace(sc, volume=S.Volume(data, vtype, dims, 0, 0.0, float(top)))
    vol, med, light, prm, _ = lp.device_scene(sc)
    got = lp.generate(vol, med, light, prm).reshape(-1, 3).double().cpu().numpy()
    ks = np.arange(24 * 24)
    ks = ks[(ks // 24) != (ks % 24)]
    ref = orc.generate(sc, ks)
    # the bar of the radiance tests: aggregate relative L1, which a wrong
    # voxel (an error of the order of the field itself) exceeds by far
    err = np.abs(got[ks] - ref).sum() / np.abs(ref).sum()
    print(f"type {vtype} dims {dims}: rel L1 {err:.2e}")
    assert err <= 1e-3
