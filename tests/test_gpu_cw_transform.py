"""CW-SSIM's DFT passes on MFMA: sizes on both sides of the tiles' edges (16
steps, 32 and 64 outputs, 64 and 128 lines), odd and prime lengths, the
longest lines, and both tile sizes; against the FP64 oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lp():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1903_03837_amd as lp
    lp.library()
    return lp


@pytest.mark.parametrize("H,W", [(8, 16), (15, 17), (32, 64), (33, 63), (128, 7), (60, 90), (97, 101), (9, 1031),
                                 (7, 4096), (4096, 9), (4093, 7), (540, 721)])
def test_sizes(lp, H, W):
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


def test_batch_equals_single_pairs(lp):
    g = torch.Generator(device="cuda").manual_seed(3)
    a = torch.rand((3, 130, 150, 3), device="cuda", generator=g)
    b = (a + 0.1 * torch.randn(a.shape, device="cuda", generator=g)).contiguous()
    all_ = lp.cw_ssim(a, b)
    assert torch.equal(all_, torch.cat([lp.cw_ssim(a[i:i + 1], b[i:i + 1]) for i in range(3)]))
