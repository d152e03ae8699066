"""Isosurfaces of long and flat volumes: the march's blocks have a length of
their own along each axis, and forming their kinds costs no more than other
passes over the volume."""
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


def scene(dims, vtype, box, period, iso=1000.3, M=24, N=30, spp=4):
    z, y, x = np.meshgrid(*(np.arange(n) for n in dims[::-1]), indexing="ij")
    v = 1000 + 600 * np.sin(x / period[0]) * np.cos(y / period[1] + 0.5) * np.cos(z / period[2])
    data = (v.astype(np.float32) if vtype == S.F32 else np.rint(v).astype(np.uint16)).reshape(-1)
    sc = S.config(2, vol_n=32, M=M, N=N, spp=spp, max_bounces=3, grid=6, views=1)
    lut = sc.medium.lut.copy()
    lut[:, :3] = np.clip(lut[:, :3], 0.2, 0.9)
    vol = S.Volume(data, vtype, dims, 0, 0.0, 4095.0, tuple(-b for b in box), box)
    return dataclasses.replace(sc, volume=vol, medium=S.Medium(lut, 10.0),
                               light=dataclasses.replace(sc.light, env=(0.05, 0.04, 0.08))).with_params(
        surface=1, iso=iso)


# blocks of 2, 3 and 7 bricks along one axis, 2 along the others; 3 and 2 in
# planes; one block along an axis; a last block of one brick
@pytest.mark.parametrize("dims,box", [((300, 20, 12), (1.0, 0.3, 0.2)), ((9, 500, 31), (0.2, 1.0, 0.3)),
                                      ((13, 12, 900), (0.3, 0.3, 1.0)), ((302, 295, 5), (1.0, 1.0, 0.2)),
                                      ((4, 310, 298), (0.1, 1.0, 1.0))])
@pytest.mark.parametrize("vtype", [S.U16, S.F32])
def test_long_volumes_match_oracle(lp, orc, dims, box, vtype):
    sc = scene(dims, vtype, box, [max(2.0, n / 12.0) for n in dims])
    vol, med, light, prm, cams = lp.device_scene(sc)
    got = lp.generate(vol, med, light, prm).reshape(-1, 3).double().cpu().numpy()
    ref = orc.generate(sc, np.arange(24 * 30))
    err = np.abs(got - ref).sum() / np.abs(ref).sum()
    print(f"{dims} type {vtype}: rel L1 {err:.2e}")
    assert err <= 1e-3  # the bar of the isosurface tests


@pytest.mark.parametrize("dims", [(20000, 64, 64), (64, 64, 20000), (4096, 128, 128), (2048, 128, 128)])
def test_time_of_a_small_field(lp, dims):
    """A small field's time is passes over the volume, in the isosurface variant
    as in the volume tracer.  The former reads it at most once more, with a margin
    of two voxels around blocks of six or more: (8/6)^2 times where two axes are
    short."""
    n = dims[0] * dims[1] * dims[2]
    sc = scene((8, 8, 8), S.U16, (1.0, 1.0, 1.0), (2.0, 2.0, 2.0), M=8, N=9, spp=1)
    vol, med, light, prm, _ = lp.device_scene(sc)
    data = torch.full((n,), 900, dtype=torch.int16, device="cuda")
    data[: n // 2] = 1100
    box = tuple(d / max(dims) for d in dims)
    vol = lp.Volume(data, dims, 0.0, 4095.0, 0, tuple(-b for b in box), box)

    def best(p):
        t = []
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            lp.generate(vol, med, light, p)
            b.record()
            torch.cuda.synchronize()
            t.append(a.elapsed_time(b))
        return min(t)

    volume, surface = best(dataclasses.replace(prm, surface=0)), best(prm)
    print(f"{dims}: volume {volume:.3f} ms, isosurface {surface:.3f} ms")
    assert surface <= 5.0 * volume
