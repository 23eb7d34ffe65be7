"""The backward takes its tiles longest list first where it can (a value buffer of at least
one word per tile, up to 16,384 tiles) and in their natural order elsewhere: the same
gradients, bit for bit, by every route."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import paper_2511_18441_amd as R
    return R


def _grads(R, sc, cam, tile, cap, graph):
    import torch
    d = R.DeviceScene(sc)
    ws = R.DeviceWorkspace(sc.n, cam.width, cam.height, tile, key_capacity=cap)
    img = R.render(d, cam, ws, tile, 1, keep_backward=True, grow=False, graph_mode=graph)
    g = torch.from_numpy(synth.random_image(3, (cam.height, cam.width, 3))).cuda()
    dop, ddc, dM = (torch.full(s, 9.0, device="cuda") for s in ((sc.n,), (3, sc.n), (9,)))
    o = R.opts_struct(tile, 1, keep_backward=True)
    R.recogs_render_backward(d.c_struct(), R.camera_struct(cam), o, ws.ws, img.data_ptr(), g.data_ptr(), dop.data_ptr(),
                             ddc.data_ptr(), dM.data_ptr())
    keys = ws.readback()[0]
    return keys, dop.cpu().numpy(), ddc.cpu().numpy(), dM.cpu().numpy()


@pytest.mark.parametrize("size,tile,n", [(512, (8, 8), 24), (1100, (8, 8), 24), (100, (32, 32), 4096), (33, (16, 16), 300)])
@pytest.mark.parametrize("graph", [False, True])
def test_order_and_natural_order_agree(R, size, tile, n, graph):
    w = synth.make_tiny()
    sc = w.scene.subset(np.arange(n))
    c = w.view.camera
    s = size / c.width
    cam = synth.Camera(size, size, c.fx * s, c.fy * s, size / 2, size / 2, c.R, c.t, c.znear)
    tiles = (-(-size // tile[0])) * (-(-size // tile[1]))
    keys, *ref = _grads(R, sc, cam, tile, 1 << 17, graph)
    assert np.abs(ref[0]).max() > 0
    for cap in {keys, max(keys, tiles), max(keys, tiles) + 1}:
        k, *got = _grads(R, sc, cam, tile, cap, graph)
        assert k == keys
        for a, b in zip(got, ref):
            assert a.tobytes() == b.tobytes(), (cap, tiles, keys)
