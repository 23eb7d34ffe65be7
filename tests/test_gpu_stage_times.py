"""Stage times of every route of an eager render: each a positive time between events in
stream order, so that together they fill the frame."""
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import paper_2511_18441_amd as R
    return R


# the order by counting pairs; a depth pass in front of the read-back; none (tile-first, 64-bit keys)
@pytest.mark.parametrize("n,mode", [(4096, 0), (60_000, 0), (60_000, 1), (60_000, 2)])
def test_stages_fill_the_frame(R, n, mode):
    """The stages' sum against the time between two events around the call: it lacks what
    the call does outside its first and last event (the events themselves), and is no
    more than it by the events' resolution (1 us, ten of them)."""
    import torch
    w = synth.make_mid(n=n)
    cam = w.view.camera
    d = R.DeviceScene(w.scene)
    ws = R.DeviceWorkspace(n, cam.width, cam.height)
    img = R.render(d, cam, ws, sort_mode=mode).clone()
    again = torch.empty_like(img)
    runs = []
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        R.render(d, cam, ws, image=again, sort_mode=mode, profile=1)
        b.record()
        b.synchronize()
        ms = list(ws.ws.stage_ms)
        assert torch.equal(again, img)
        assert all(x > 0 for k, x in enumerate(ms) if k != 7 or mode == 2), ms
        assert sum(ms) <= a.elapsed_time(b) + 0.01, ms
        runs.append(ms)
    if mode == 0 and n > 12_288:   # two passes over 60,000 pairs against a read-back that ran beside the first
        assert min(m[3] for m in runs) > min(m[2] for m in runs), runs
