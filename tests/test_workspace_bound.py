"""Workspace of the kept samples: at most 2^25 samples of 12 bytes for any ray
and sample count (size queries, which never touch the device)."""
import ctypes as C
import math
import os

import pytest


@pytest.fixture(scope="module")
def lp():
    import paper_1903_03837_amd as lp
    if not os.path.exists(lp.library_path()):
        pytest.skip("liblumipath.so not built")
    return lp


def scene(lp, M, N, spp):
    vol = lp._Volume()
    vol.data, vol.nx, vol.ny, vol.nz, vol.vmax = 0x10000, 16, 16, 16, 255.0
    vol.box_min[:] = [-1, -1, -1]
    vol.box_max[:] = [1, 1, 1]
    med = lp._Medium(lut=0x20000, lut_size=256, density_scale=10.0)
    light = lp._Light(kind=0)
    light.dir[:] = [0, 0, 1]
    prm = lp._GenParams(M=M, N=N, radius=math.sqrt(3), spp=spp, max_bounces=4)
    prm.surface = 1  # (no range sums beside the kept samples)
    return vol, med, light, prm


def field_bytes(lp, M, N, spp):
    vol, med, light, prm = scene(lp, M, N, spp)
    n = C.c_size_t(0)
    assert lp.library().lf_generate(C.byref(vol), C.byref(med), None, C.byref(light), C.byref(prm), 0,
                                    C.c_void_p(0x30000), None, C.byref(n), None) == 0
    return n.value


def view_bytes(lp, W, H, spp):
    vol, med, light, prm = scene(lp, 8, 8, spp)
    cam = (lp._Camera * 1)()
    cam[0].eye[:], cam[0].target[:], cam[0].up[:], cam[0].vfov = [0, -8, 0], [0, 0, 0], [0, 0, 1], 0.5
    n = C.c_size_t(0)
    assert lp.library().lf_render_views(C.byref(vol), C.byref(med), C.byref(light), C.byref(prm), cam, 1, W, H,
                                        C.c_void_p(0x30000), None, C.byref(n), None) == 0
    return n.value


SPP = [8, 9, 31, 32, 100, 1000, 4097, 65535, 65536, 65537, 100000, 131072, 524288, 524289, 2 ** 31 - 1]


@pytest.mark.parametrize("size,M,N", [(field_bytes, 3, 5), (field_bytes, 300, 301), (field_bytes, 4096, 4095),
                                      (view_bytes, 1, 1), (view_bytes, 1920, 1080), (view_bytes, 16000, 9000)])
def test_kept_samples_stay_within_their_bound(lp, size, M, N):
    plain = size(lp, M, N, 7)  # nothing is kept below 8 samples
    counters = 1024            # of the queue, a cache line each
    for spp in SPP:
        extra = size(lp, M, N, spp) - plain
        assert 0 <= extra <= 12 * 2 ** 25 + counters, (spp, extra)
    assert size(lp, M, N, 8) > plain and size(lp, M, N, 65536) > plain
