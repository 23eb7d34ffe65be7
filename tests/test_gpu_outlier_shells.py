"""The outlier filter's second and third search on clouds whose points fill a volume, on
both sides of the lengths of their lists at which they take fewer lanes per query and the
largest cube in shells."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import paper_2511_18441_amd as R
    return R


@pytest.mark.parametrize("k", [4, 8, 16, 32])
@pytest.mark.parametrize("kind,n", [("cube", 700), ("cube", 8_750), ("cube", 20_011), ("cube", 40_003), ("cube", 60_001), ("slab", 9_000), ("fading", 30_000)])
def test_volumes(R, kind, n, k):
    """D against a k-d tree in FP64: 4e-6 relative (a few ulps of the squared distance, half
    of that for its root, one per addition of the mean)."""
    import torch
    from oracle import selection as S
    rng = np.random.default_rng(n + k)
    p = rng.uniform(-1, 1, (3, n))
    if kind == "slab":
        p[1] *= 0.05
    if kind == "fading":   # density falling to a hundredth along x
        p[0] = rng.uniform(0, 1, n) ** 4 * 20
    p = p.astype(np.float32)
    pts = torch.from_numpy(p).cuda()
    nb = R.recogs_outlier_workspace_bytes(n)
    ws = torch.zeros(nb, dtype=torch.uint8, device="cuda")
    dist = torch.empty(n, device="cuda")
    keep = torch.empty(n, dtype=torch.uint8, device="cuda")
    cnt = torch.empty(1, dtype=torch.int32, device="cuda")
    R.recogs_remove_outliers(pts.data_ptr(), n, n, k, 0.3, dist.data_ptr(), keep.data_ptr(), None, n, cnt.data_ptr(),
                             ws.data_ptr(), nb)
    ref = S.knn_mean_distance(p.T.astype(np.float64), k)
    assert np.all(np.abs(dist.cpu().numpy().astype(np.float64) - ref) <= 4e-6 * ref)
    if kind == "cube":   # 1/8 of a point per cell: the 4th neighbour at about 2 cells, the 32nd at 4, twice that in corners
        assert int(ws[52:56].view(torch.int32).item()) > 0   # the workspace header's count of queries left to this search
