"""CW-SSIM's DFT passes with the large tile (128 lines x 64 outputs), which is
taken where it leaves enough workgroups: ragged edges in both directions, odd
and prime lengths, lines of the greatest length in either direction; against
the FP64 oracle."""
import os
import re

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

SRC = os.path.join(os.path.dirname(__file__), "..", "paper_1903_03837_amd", "csrc", "metrics.hip")


@pytest.fixture(scope="module")
def lp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1903_03837_amd as lp
    lp.library()
    return lp


def up(a, b):
    return (a + b - 1) // b


def large_tiles(H, W):
    """Workgroups of the large tile: image rows, image columns, and the fewest of
    a subband's inverse columns (rows are those of the image)."""
    few = up(min((W + 1) // 2, W // 4 + 1), 128)  # second scale, one-sided
    return up(W, 64) * up(6 * H, 128), up(H, 64) * up(W, 128) * 6, up(H, 64) * few * 6


# whether rows, columns and the narrowest subband's columns take the large tile
@pytest.mark.parametrize("H,W,takes", [(719, 1279, (True, True, False)), (130, 4096, (False, True, False)),
                                       (4096, 130, (True, True, False)), (2753, 515, (True, True, True))])
def test_large_tiles_match_oracle(lp, H, W, takes):
    least = int(re.search(r"g2\.x \* g2\.y \* g2\.z >= (\d+)\)", open(SRC).read()).group(1))
    assert tuple(n >= least for n in large_tiles(H, W)) == takes
    from oracle import cwssim as cw
    rng = np.random.default_rng(1000 * H + W)
    a = rng.uniform(0, 1, (1, H, W, 3)).astype(np.float32)
    b = np.clip(0.7 * a + rng.normal(0, 0.2, a.shape) + 0.1, 0, 1).astype(np.float32)
    got = lp.cw_ssim(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda()).cpu().numpy()
    ref = cw.cw_ssim(a, b)
    print(f"cw-ssim {H} x {W}: |diff| {np.abs(got - ref).max():.2e}")
    # 1e-6 is the bar at up to 480 points (rounding of a direct sum of n FP32
    # products, at most proportional to n)
    assert np.abs(got - ref).max() <= 1e-6 * max(1.0, max(H, W) / 480.0)
    # each image pair and its swap have one index
    back = lp.cw_ssim(torch.from_numpy(b).cuda(), torch.from_numpy(a).cuda()).cpu().numpy()
    assert np.abs(got - back).max() <= 1e-6 * max(1.0, max(H, W) / 480.0)

