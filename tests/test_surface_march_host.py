"""The isosurface march on the host, from the device sources: stepping over
blocks of known sign finds the crossing that fetching every sample finds, on
the same rays, in fields made to be hard (isovalues equal to voxel values,
steps between neighbouring voxels, surfaces on the first and last voxels, long
volumes, voxels that are not finite); and the halo-brick index near its limits."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
U16, F32 = 1, 2


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available to build the probe")
    exe = str(tmp_path_factory.mktemp("march") / "probe")
    # (of the library's host code only its parameter packing is called; the
    # kernels behind it are not linked)
    subprocess.run([hipcc, "-x", "hip", "--cuda-host-only", "-std=c++17", "-O2",
                    "-Wl,--unresolved-symbols=ignore-all", "-o", exe,
                    os.path.join(HERE, "support", "surface_march.cpp")], check=True, capture_output=True)
    return exe


def waves(x, y, z):
    return 600 + 300 * np.sin(0.4 * x) * np.cos(0.3 * y + 0.2 * z)


def steps(x, y, z):
    return np.where((x // 5 + y // 7 + z // 3) % 2 == 0, 100, 900)


def plane(x, y, z):
    return np.where(x < 1, 1000, 10) + np.where(z >= z.max(), 1500, 0)


def far_steps(x, y, z):
    """clear of the isovalue over long stretches"""
    return np.where((x // 24 + y // 24 + z // 24) % 2 == 0, 100, 900)


def slope(x, y, z):
    return 500 + x - 0.25 * y


def spikes(x, y, z):
    """single voxels, the corners and borders of blocks among them"""
    return np.where((x % 13 == 0) & (y % 17 == 0) & (z % 6 == 0) | (x % 29 == 5) & (y % 12 == 11) & (z % 31 == 12), 900, 100)


def hair(x, y, z):
    """regions that keep clear of 500 by about the rounding of the interpolation"""
    r = np.random.default_rng(3)
    off = r.choice([-3.0, -1.01, -0.99, -0.3, 0.0, 0.3, 0.99, 1.01, 3.0], (16, 16, 16))[z // 12 % 16, y // 12 % 16, x // 12 % 16]
    return 500.0 + off * 1e-5 * 1000.0 * (1.0 + 1e-3 * r.standard_normal(x.shape))


def march(probe, dims, field, iso, vtype, box=(1.0, 0.8, 0.9), rays=20000, seed=1, spoil=None):
    z, y, x = np.meshgrid(*(np.arange(n) for n in dims[::-1]), indexing="ij")
    v = field(x, y, z).astype(np.float32)
    if vtype == U16:
        v = np.rint(v)
    if spoil is not None:
        r = np.random.default_rng(5)
        for _ in range(6):
            v[tuple(r.integers(0, n) for n in v.shape)] = spoil
    head = f"{dims[0]} {dims[1]} {dims[2]} {vtype} {iso!r} {box[0]} {box[1]} {box[2]} {rays} {seed}\n".encode()
    out = subprocess.run([probe, "march"], input=head + v.tobytes(), capture_output=True, check=True).stdout.split()
    met, crossings, differ, fast, full = map(int, out)
    print(f"{dims} {field.__name__} iso {iso}: {met} rays, {crossings} crossings, {full / max(fast, 1):.1f} x the steps")
    assert crossings > 300 if v.min() < iso <= v.max() and spoil is None else True  # (a surface to find)
    return met, crossings, differ, fast, full


CASES = [(d, f, i, t) for d, f, i in [
    ((40, 37, 35), waves, 600.5), ((40, 37, 35), waves, 600.0), ((31, 32, 33), steps, 500.0),
    ((31, 32, 33), steps, 100.0), ((31, 32, 33), steps, 900.0), ((7, 8, 160), plane, 500.0),
    ((7, 8, 160), plane, 10.0), ((7, 8, 160), plane, 1510.0), ((2, 2, 2), steps, 400.0), ((3, 4, 5), plane, 300.5),
    ((97, 50, 51), far_steps, 500.0), ((97, 50, 51), far_steps, 100.0), ((97, 50, 51), slope, 540.0),
    ((310, 20, 12), far_steps, 500.0), ((9, 600, 31), waves, 600.0), ((13, 12, 900), slope, 505.25),
    ((302, 295, 5), far_steps, 899.5), ((40, 37, 35), waves, 4000.0),
    ((97, 50, 51), spikes, 500.0), ((97, 50, 51), spikes, 101.0), ((310, 40, 37), spikes, 120.0),
    ((97, 50, 51), hair, 500.0), ((300, 60, 20), hair, 500.0)] for t in (U16, F32) if t == F32 or f is not hair]


@pytest.mark.parametrize("dims,field,iso,vtype", CASES)
def test_skipping_march_finds_the_same_crossings(probe, dims, field, iso, vtype):
    met, crossings, differ, fast, full = march(probe, dims, field, iso, vtype)
    assert met > 5000 and fast <= full
    assert differ == 0


def test_blocks_are_stepped_over(probe):
    """(the comparison above would hold if nothing were skipped)"""
    _, _, differ, fast, full = march(probe, (160, 150, 140), slope, 560.0, U16, rays=4000)
    assert differ == 0 and full >= 2 * fast


@pytest.mark.parametrize("spoil", [float("inf"), float("-inf"), float("nan"), 3.3e38, -3.3e38])
def test_voxels_that_are_not_finite(probe, spoil):
    for field, iso in ((far_steps, 500.0), (slope, 540.0)):
        met, _, differ, _, _ = march(probe, (97, 50, 51), field, iso, F32, spoil=spoil)
        assert met > 5000 and differ == 0


def test_voxels_whose_differences_overflow(probe):
    """2e38 and -2e38 lie on one side of -2.5e38, but interpolating between them
    gives infinities and NaN, which a march that fetches meets."""
    def huge(x, y, z):
        return np.where((x // 3 + y // 4 + z // 5) % 3 == 0, -2e38, 2e38)

    for iso in (-2.5e38, 2.5e38):
        met, _, differ, _, _ = march(probe, (60, 50, 51), huge, iso, F32, spoil=2e38)
        assert met > 5000 and differ == 0


# rows of bricks (nby x nbz) below and above 2^24, the longest axes, and copies
# of nearly 2^32 voxels
@pytest.mark.parametrize("dims", [(2, 2, 2), (65535, 2, 2), (2, 65535, 2), (2, 2, 65535), (2, 30000, 5000),
                                  (2, 65535, 9000), (3, 9000, 65535), (65535, 9000, 2), (65535, 2, 9000),
                                  (1210, 1210, 1210)])
def test_footprint_index(probe, dims):
    out = subprocess.run([probe, "index"], input="%d %d %d\n" % dims, text=True, capture_output=True,
                         check=True).stdout.split()
    assert int(out[1]) < 2 ** 32 and int(out[0]) == 0
