"""A thread's first eager render while another thread captures a HIP graph in the global
mode: neither disturbs the other."""
import threading

import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import paper_2511_18441_amd as R
    return R


@pytest.mark.parametrize("n,busy", [(3000, 0), (20_000, 0), (20_000, 24)])
def test_first_eager_render_beside_a_capture(R, n, busy):
    """busy: passes over 1 GiB in front of the render, so that its wait asks for the stream's state."""
    import torch
    w = synth.make_mid(n=n)
    cam = w.view.camera
    d = R.DeviceScene(w.scene)
    ws = [R.DeviceWorkspace(n, cam.width, cam.height, key_capacity=32 * n) for _ in range(2)]
    img = [torch.zeros((cam.height, cam.width, 3), device="cuda") for _ in range(2)]
    ballast = torch.zeros(1 << 28 if busy else 1, device="cuda")
    ref = R.render(d, cam, ws[1], image=img[1]).clone()
    img[1].zero_()
    R.render(d, cam, ws[0], image=img[0], graph_mode=True)   # first launches outside the capture
    ballast.add_(1.0)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    err = []

    def other():
        try:
            with torch.cuda.stream(side):
                for _ in range(busy):
                    ballast.add_(1.0)
                for _ in range(2):
                    R.render(d, cam, ws[1], image=img[1])
        except Exception as e:  # noqa: BLE001
            err.append(e)

    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        R.render(d, cam, ws[0], image=img[0], graph_mode=True)
        t = threading.Thread(target=other)
        t.start()
        t.join(60)
    assert not t.is_alive() and not err, err
    torch.cuda.synchronize()
    assert torch.equal(img[1], ref)
    for _ in range(3):
        img[0].zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(img[0], ref)
