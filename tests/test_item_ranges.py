"""Sample ranges of the tracer's work items: a ray's items must cover its
samples in order for every sample count the entry points take, whatever the
split (host build of the device header's function)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def probe(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available to build the probe")
    exe = str(tmp_path_factory.mktemp("items") / "probe")
    subprocess.run([hipcc, "-x", "hip", "--cuda-host-only", "-std=c++17", "-O1", "-o", exe,
                    os.path.join(HERE, "support", "item_ranges.cpp")], check=True, capture_output=True)
    return exe


# the largest counts before and after 32-bit products of an item and spp
# overflow, the largest that are split finely, and the largest there are
SPP = [1, 2, 3, 7, 8, 9, 17, 33, 100, 46340, 46341, 65535, 65536, 65537, 100000, 131072, 524288, 2 ** 30, 2 ** 31 - 1]


def test_items_cover_the_samples_in_order(probe):
    cases = [(spp, lg) for spp in SPP for lg in range(20) if (1 << lg) <= spp]
    out = subprocess.run([probe], input="".join(f"{s} {l}\n" for s, l in cases), text=True, capture_output=True,
                         check=True).stdout.split()
    assert len(out) == len(cases)
    bad = [(c, int(o)) for c, o in zip(cases, out) if int(o) >= 0]
    assert not bad, bad[:5]
