"""Scenes of up to 12,288 Gaussians are ordered by counting over all pairs: the same lists,
offsets, counts and pictures, bit for bit, as the 64-bit key sort's (sort mode 1), at the
edges of its blocks, runs and sizes, with equal depths and with Gaussians outside the view."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import paper_2511_18441_amd as R
    return R


@pytest.mark.parametrize("spread", [0, 2, 1 << 25])
@pytest.mark.parametrize("n", [1, 16, 17, 129, 2047, 2049, 4096, 4097, 8192, 8193, 12288, 12289])
def test_same_as_the_key_sort(R, n, spread):
    import torch
    from tests.scenes_by_hand import axis_camera, scene_from
    rng = np.random.default_rng(n + spread)
    z = np.full(n, np.float32(4.0))
    z = (z.view(np.uint32) + rng.integers(0, spread + 1, n).astype(np.uint32)).view(np.float32)
    # a third of the Gaussians miss the image
    means = np.column_stack([rng.uniform(-4.5, 4.5, n), rng.uniform(-4.0, 4.0, n), z.astype(np.float64)])
    means[0, :2] = 0.0
    sc = scene_from(means, np.log(rng.uniform(0.01, 0.2, (n, 3))), rng.uniform(0.3, 0.95, n), rng.uniform(0.0, 1.0, (n, 3)))
    cam = axis_camera(112, 80, 60.0)
    d = R.DeviceScene(sc)

    def run(cap=None, **kw):
        ws = R.DeviceWorkspace(n, cam.width, cam.height, (16, 16), key_capacity=cap)
        img = R.render(d, cam, ws, (16, 16), 1, **kw)
        k, v = ws.readback()
        return (k, v, int(ws.ws.depth_min_bits), img, ws.vals_sorted()[:k].clone(), ws.ranges().clone(), ws.offsets(n).clone())

    ref = run(sort_mode=1)
    assert ref[0] > 0
    for got in (run(), run(cap=ref[0]), run(cap=ref[0] + 5000, graph_mode=True)):
        assert got[:3] == ref[:3]
        for a, b in zip(got[3:], ref[3:]):
            assert torch.equal(a, b)
    assert run(cap=ref[0] - 1, graph_mode=True)[0] == ref[0]   # overflow: the count, and empty lists
