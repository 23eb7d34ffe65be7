"""The outlier filter's searches at their edges: fewer points than neighbours, runs of 64
points and one more or less, clouds whose cells wrap around the slot residues, strays that
only the search of the whole cloud settles, coincident points, padded planes; and the
compaction by both of its routes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import paper_2511_18441_amd as R
    return R


def _cloud(kind, n, seed):
    rng = np.random.default_rng(seed)
    if kind == "ball":
        p = rng.standard_normal((3, n))
    elif kind == "sheet":          # a thin slab, long in x: its cells wrap along every axis of few residues
        p = rng.uniform(-1, 1, (3, n)) * np.array([[40.0], [5.0], [0.01]])
    elif kind == "strays":
        p = 0.05 * rng.standard_normal((3, n))
        m = max(1, n // 40)
        p[:, :m] = rng.uniform(-30, 30, (3, m))
    else:                          # few distinct places
        p = rng.integers(0, 3, (3, n)).astype(float)
    return p.astype(np.float32)


@pytest.mark.parametrize("k", [4, 16, 32])
@pytest.mark.parametrize("kind,n", [("ball", 1), ("ball", 2), ("ball", 17), ("ball", 63), ("ball", 64), ("ball", 65),
                                    ("strays", 129), ("sheet", 2049), ("strays", 5000), ("places", 700), ("sheet", 33_000)])
def test_mean_distances_and_keep(R, kind, n, k):
    """D against a k-d tree in FP64. The squared distance carries a few ulps (3 of the
    differences' rounding, 3 of the sum), its root half of that, the mean of k one more per
    addition: 4e-6 relative."""
    import torch
    from oracle import selection as S
    p = _cloud(kind, n, n + k)
    buf = torch.full((3, n + 5), 1e9, device="cuda")
    buf[:, :n] = torch.from_numpy(p).cuda()
    pts = buf[:, :n]
    out, keep, dist = R.remove_outliers(pts, k, 0.3)
    ref = S.knn_mean_distance(p.T.astype(np.float64), k)   # the oracle takes (points, 3)
    got = dist.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(got - ref) <= 4e-6 * ref + 1e-30)
    kp = keep.cpu().numpy() != 0
    if n > 2:
        thr = ref.mean() + 0.3 * ref.std()
        sure = np.abs(ref - thr) > 1e-5 * max(thr, 1e-30)
        assert np.array_equal(kp[sure], (ref <= thr)[sure])
    assert np.array_equal(out.cpu().numpy(), p[:, kp])


@pytest.mark.parametrize("n", [2048 * 1024, 2048 * 1024 + 1])
def test_compaction_on_both_sides_of_its_fold(R, n):
    """2,048 workgroup counts are summed by the compaction itself, more by a scan."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(7)
    pts = torch.randn((3, n), generator=g, device="cuda")
    out, keep, dist = R.remove_outliers(pts, 4, 0.007)
    m = keep.bool()
    assert out.shape[1] == int(m.sum()) and 0 < out.shape[1] < n
    assert torch.equal(out, pts[:, m])
