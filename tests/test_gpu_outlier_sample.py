"""The outlier filter's cell size comes from a sample of the points: a cloud whose order has
a period must not be judged by one of its phases (the results are the same at any cell size,
the time is not)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import paper_2511_18441_amd as R
    return R


@pytest.mark.parametrize("n,period,phase", [(131_072, 4, 0), (131_072, 4, 3), (100_003, 2, 0), (100_003, 4, 0), (393_216, 12, 0)])
def test_cell_size_of_interleaved_clouds(R, n, period, phase):
    """One point in every `period` lies in a cluster of a hundredth of the others' extent.
    The cell size is the largest 1%-99% extent over ceil(2 n^(1/3)), at most 128; the bins are
    1/1024 of the extent and the sample's quantiles spread by about 1%, so it lies within 5%
    of the whole cloud's; judged by the cluster's phase alone it would be a hundredth."""
    import torch
    rng = np.random.default_rng(n + period)
    p = rng.uniform(-1, 1, (3, n))
    p[:, phase::period] *= 0.01
    p = p.astype(np.float32)
    pts = torch.from_numpy(p).cuda()
    nb = R.recogs_outlier_workspace_bytes(n)
    ws = torch.zeros(nb, dtype=torch.uint8, device="cuda")
    dist = torch.empty(n, device="cuda")
    keep = torch.empty(n, dtype=torch.uint8, device="cuda")
    cnt = torch.empty(1, dtype=torch.int32, device="cuda")
    R.recogs_remove_outliers(pts.data_ptr(), n, n, 4, 0.3, dist.data_ptr(), keep.data_ptr(), None, n, cnt.data_ptr(),
                              ws.data_ptr(), nb)
    h = float(ws[24:28].view(torch.float32).item())   # the workspace begins with the box's six bounds, then the cell size
    q = np.quantile(p.astype(np.float64), [0.01, 0.99], axis=1)
    want = (q[1] - q[0]).max() / min(128, int(np.ceil(2 * n ** (1 / 3))))
    assert abs(h - want) <= 0.05 * want
