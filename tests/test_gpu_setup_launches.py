"""Point sets, queries, point tables and spatial orders are formed in shared
launches whose workgroups are divided among the parts: set sizes and query
counts on both sides of a workgroup (256), and unequal sets."""
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


@pytest.mark.parametrize("n", [1, 2, 255, 256, 257, 65535])
@pytest.mark.parametrize("nq", [0, 1, 255, 256, 257])
def test_points_with_and_without_queries(lp, orc, n, nq):
    g = torch.Generator().manual_seed(n + nq)
    q = torch.nn.functional.normalize(torch.randn((nq, 3), generator=g, dtype=torch.float64), dim=-1).float().cuda()
    K = min(n, 3)
    xyz = lp.points(n)[0]
    both = lp.points(n, q, K)
    assert torch.equal(both[0], xyz)
    if nq == 0:  # (nothing to write at all is refused)
        with pytest.raises(lp.LumiPathError):
            lp.points(n, q, K, want_xyz=False)
    else:
        alone = lp.points(n, q, K, want_xyz=False)
        assert torch.equal(both[1], alone[1]) and torch.equal(both[2], alone[2])
    # a unit vector to FP32 rounding
    assert float((xyz.double().norm(dim=-1) - 1).abs().max()) <= 1e-6
    if nq and n <= 257:
        d = torch.cdist(q.double(), xyz.double())
        near = d.gather(1, both[1][:, :1].long())[:, 0]
        assert float((near - d.min(dim=1).values).abs().max()) <= 1e-6


@pytest.mark.parametrize("M,N", [(1, 1), (1, 300), (257, 1), (255, 256), (256, 511), (40, 513)])
def test_fields_of_unequal_sets(lp, orc, M, N):
    sc = S.config(1, M=M, N=N, spp=4)
    sc = dataclasses.replace(sc, light=dataclasses.replace(sc.light, env=(0.1, 0.2, 0.3)))
    vol, med, light, prm, cams = lp.device_scene(sc)
    got = lp.generate(vol, med, light, prm).reshape(-1, 3).double().cpu().numpy()
    ks = np.arange(M * N) if M != N else np.array([k for k in range(M * N) if k // N != k % N], dtype=np.int64)
    ks = ks[:: max(1, len(ks) // 400)]
    if len(ks) == 0:
        assert not got.any()
        return
    ref = orc.generate(sc, ks)
    assert np.abs(got[ks] - ref).sum() <= 1e-3 * max(np.abs(ref).sum(), 1e-12)
