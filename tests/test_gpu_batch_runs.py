"""Batches deal the preprocess blocks of consecutive views of one scene in turn, and take their
depth order in three passes: the images and lists of single renders, bit for bit, for runs of
one to three views, a scene that comes back later, ragged and empty scenes."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import paper_2511_18441_amd as R
    return R


@pytest.mark.parametrize("order", [[0], [0, 0, 0], [0, 1, 1, 2, 0], [3, 0, 0, 3, 1], [2, 2, 1, 1, 1, 0]])
def test_batch_equals_single_views(R, order):
    import torch
    w = synth.make_tiny()
    n = w.scene.n
    sizes = [n, min(n, 2048), min(n, 255), 0]
    scenes = [R.DeviceScene(w.scene.subset(np.arange(k))) for k in sizes]
    c = w.view.camera
    views, cams = [], []
    for k, si in enumerate(order):
        cam = synth.Camera(64 + 24 * k, 48 + 16 * k, c.fx * 0.3, c.fy * 0.3, 32 + 12 * k, 24 + 8 * k, c.R, c.t, c.znear)
        cams.append(cam)
        views.append((si, cam, None, None, None))
    b = R.DeviceBatch(scenes, views, (16, 16), 1)
    b.render()
    imgs = b.images
    torch.cuda.synchronize()
    for k, si in enumerate(order):
        ws = R.DeviceWorkspace(sizes[si], cams[k].width, cams[k].height, (16, 16))
        assert torch.equal(imgs[k], R.render(scenes[si], cams[k], ws, (16, 16), 1)), (k, si)
