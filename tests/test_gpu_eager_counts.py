"""Eager renders get their counts from a note that the scan leaves in pinned memory, with the
depth sort's next pass in flight meanwhile: the same pictures and lists, bit for bit, as a
render without host waits (graph_mode), whatever part of the depth bits differs, from
several threads at once, and after a view that did not fit."""
import threading

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import paper_2511_18441_amd as R
    return R


def _scene(spread, n, seed):
    from tests.scenes_by_hand import axis_camera, scene_from
    rng = np.random.default_rng(seed)
    z = np.full(n, np.float32(4.0))
    z = (z.view(np.uint32) + rng.integers(0, spread + 1, n).astype(np.uint32)).view(np.float32)
    means = np.column_stack([rng.uniform(-2.4, 2.4, n), rng.uniform(-2.0, 2.0, n), z.astype(np.float64)])
    sc = scene_from(means, np.log(rng.uniform(0.01, 0.1, (n, 3))), rng.uniform(0.3, 0.95, n), rng.uniform(0.0, 1.0, (n, 3)))
    return sc, axis_camera(96, 80, 60.0)


def _same(R, d, cam, n, mode, img, ws):
    import torch
    wsg = R.DeviceWorkspace(n, cam.width, cam.height, (16, 16), key_capacity=max(int(ws.ws.num_keys), 1) + 1024)
    ref = R.render(d, cam, wsg, (16, 16), 1, graph_mode=True, sort_mode=mode)
    k, _ = wsg.readback()
    assert k == int(ws.ws.num_keys)
    assert torch.equal(img, ref)
    assert torch.equal(wsg.vals_sorted()[:k], ws.vals_sorted()[:k])


# depth bits that differ: none, within the scan's pass, within the early pass, one, two and
# three passes left; n at the edges of a sort chunk and of the scan's chunks
@pytest.mark.parametrize("mode", [0, 2])
@pytest.mark.parametrize("spread", [0, 255, 65535, 1 << 17, 1 << 23, 1 << 25])
@pytest.mark.parametrize("n", [1, 4097, 20000])
def test_eager_equals_graph(R, mode, spread, n):
    sc, cam = _scene(spread, n, n + spread)
    d = R.DeviceScene(sc)
    ws = R.DeviceWorkspace(n, cam.width, cam.height, (16, 16))
    img = R.render(d, cam, ws, (16, 16), 1, sort_mode=mode)
    _same(R, d, cam, n, mode, img, ws)


def test_threads_on_their_own_streams(R):
    import torch
    jobs = []
    for k in range(4):
        n = 3000 + 5000 * k
        sc, cam = _scene(1 << 24, n, k)
        d = R.DeviceScene(sc)
        jobs.append((d, cam, n, R.DeviceWorkspace(n, cam.width, cam.height, (16, 16)), torch.cuda.Stream()))
    torch.cuda.synchronize()
    out = [None] * len(jobs)

    def run(i):
        d, cam, n, ws, st = jobs[i]
        with torch.cuda.stream(st):
            for _ in range(12):
                img = R.render(d, cam, ws, (16, 16), 1)
        st.synchronize()
        out[i] = img

    th = [threading.Thread(target=run, args=(i,)) for i in range(len(jobs))]
    for t in th:
        t.start()
    for t in th:
        t.join()
    torch.cuda.synchronize()
    for (d, cam, n, ws, _), img in zip(jobs, out):
        _same(R, d, cam, n, 0, img, ws)


@pytest.mark.parametrize("mode", [0, 2])
def test_a_view_that_does_not_fit(R, mode):
    import torch
    n = 9000
    sc, cam = _scene(1 << 24, n, 5)
    d = R.DeviceScene(sc)
    ws = R.DeviceWorkspace(n, cam.width, cam.height, (16, 16), key_capacity=64)
    img = torch.full((cam.height, cam.width, 3), 7.0, device="cuda")
    with pytest.raises(R.RecogsError):
        R.render(d, cam, ws, (16, 16), 1, image=img, grow=False, sort_mode=mode)
    assert bool((img == 7.0).all())
    big = R.DeviceWorkspace(n, cam.width, cam.height, (16, 16), key_capacity=int(ws.ws.num_keys))
    img = R.render(d, cam, big, (16, 16), 1, grow=False, sort_mode=mode)
    _same(R, d, cam, n, mode, img, big)
