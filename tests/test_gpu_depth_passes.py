"""The depth order's three passes (the scan's over the low 10 depth bits, then two whose digits
follow the depth range) give the lists of the 64-bit key sort (sort mode 1), bit for bit:
ranges at the edges of 0, 8 + 8, 9 + 8 and wider digits up to depths 2^64 apart, counts at the
edges of the passes' chunks, in eager and graph renders."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import paper_2511_18441_amd as R
    return R


@pytest.mark.parametrize("n", [12290, 16385, 300001])
@pytest.mark.parametrize("spread", [1, 1023, 1025, (1 << 18) - 1, 1 << 18, 1 << 25, (1 << 26) - 1, 1 << 26, 1 << 28, 1 << 29])
def test_same_as_the_key_sort(R, n, spread):
    import torch
    from tests.scenes_by_hand import axis_camera, scene_from
    rng = np.random.default_rng(n + spread)
    lo = int(np.float32(0.5).view(np.uint32))   # a multiple of 1,024
    z = (lo + rng.integers(0, spread + 1, n)).astype(np.uint32)
    z[0], z[1] = lo, lo + spread
    z = z.view(np.float32).astype(np.float64)
    means = np.column_stack([z * rng.uniform(-0.9, 0.9, n), z * rng.uniform(-0.7, 0.7, n), z])
    means[:2, :2] = 0.0
    sc = scene_from(means, np.log(z[:, None] * rng.uniform(0.002, 0.02, (n, 3))), rng.uniform(0.3, 0.95, n),
                    rng.uniform(0.0, 1.0, (n, 3)))
    cam = axis_camera(160, 120, 100.0)
    d = R.DeviceScene(sc)

    def run(cap=None, **kw):
        ws = R.DeviceWorkspace(n, cam.width, cam.height, (16, 16), key_capacity=cap)
        img = R.render(d, cam, ws, (16, 16), 1, **kw)
        k, v = ws.readback()
        return (k, v, int(ws.ws.depth_min_bits), img, ws.vals_sorted()[:k].clone(), ws.ranges().clone(), ws.offsets(n).clone())

    ref = run(sort_mode=1)
    assert ref[1] > n // 2 and ref[2] == lo
    for got in (run(), run(cap=ref[0] + 100, graph_mode=True)):
        assert got[:3] == ref[:3]
        for a, b in zip(got[3:], ref[3:]):
            assert torch.equal(a, b)
