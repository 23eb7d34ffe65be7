"""The general chain of an eager render (more than 12,288 Gaussians, sort mode 0): its first
depth pass is in flight while the counts travel. A view that does not fit then, depths that
leave its passes nothing to do, and sizes at the edges of the chunks of the scan and of the
passes."""
import numpy as np
import pytest

import synth
from tests.gpu_common import assert_pixels, gpu_run, pull
from tests.test_gpu_eager_counts import _same, _scene
from tests.test_gpu_parity import TOL_F32, _check_integer_steps, _oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import paper_2511_18441_amd as R
    return R


@pytest.mark.parametrize("mode", [0, 1, 2])
def test_a_view_that_does_not_fit(R, mode):
    """The error comes with nothing of the call left in flight: its workspace is overwritten at
    once on another stream, and carved again for a render that fits."""
    import torch
    n = 20_000
    sc, cam = _scene(1 << 24, n, 7)
    d = R.DeviceScene(sc)
    ws = R.DeviceWorkspace(n, cam.width, cam.height, (16, 16), key_capacity=64)
    img = torch.full((cam.height, cam.width, 3), 7.0, device="cuda")
    side = torch.cuda.Stream()
    for _ in range(3):
        with pytest.raises(R.RecogsError):
            R.render(d, cam, ws, (16, 16), 1, image=img, grow=False, sort_mode=mode)
        need = int(ws.ws.num_keys)
        with torch.cuda.stream(side):
            ws.mem.fill_(0xA5)
        side.synchronize()
        torch.cuda.synchronize()
        assert bool((ws.mem == 0xA5).all()) and bool((img == 7.0).all())
    big = R.DeviceWorkspace(n, cam.width, cam.height, (16, 16), key_capacity=need)
    img = R.render(d, cam, big, (16, 16), 1, grow=False, sort_mode=mode)
    assert int(big.ws.num_keys) == need
    _same(R, d, cam, n, 0 if mode == 1 else mode, img, big)   # (64-bit keys have no graph form)


# float32 steps that the depths span, and the passes that the bits above the scan's ten need
@pytest.mark.parametrize("spread,passes", [(0, 0), (100, 0), (3000, 1), (200_000, 1), (1 << 20, 2), (1 << 25, 2)])
def test_depth_bits_left_for_the_passes(R, orc, spread, passes):
    rng = np.random.default_rng(spread + 3)
    n = 14_000
    z = np.full(n, np.float32(4.0))
    if spread:
        z = (z.view(np.uint32) + rng.integers(0, spread, n).astype(np.uint32)).view(np.float32)
    from tests.scenes_by_hand import axis_camera, scene_from
    means = np.column_stack([rng.uniform(-0.6, 0.6, n) * z, rng.uniform(-0.5, 0.5, n) * z, z.astype(np.float64)])
    sc = scene_from(means, np.log(rng.uniform(0.005, 0.02, (n, 3)) * z[:, None]), rng.uniform(0.05, 0.5, n),
                    rng.uniform(0.0, 1.0, (n, 3)))
    cam = axis_camera(96, 80, 60.0)
    base = synth.make_tiny()
    w = synth.Workload(f"early{spread}", [sc], [synth.View(0, cam, base.view.select, base.view.recolor)])
    out = gpu_run(w, keep_backward=True)
    p = pull(out, n)
    pr = _oracle(w, orc)
    _check_integer_steps(w, orc, p, pr, n)
    ref = orc.render_image(pr, brute=True)
    assert_pixels(p["img"], ref.rgb, ref.slack, TOL_F32, f"depth spread {spread}")
    assert int(out["ws"].ws.depth_passes) == passes
    _same(R, out["dscene"], cam, n, 0, out["img"], out["ws"])


@pytest.mark.parametrize("n", [12_288, 12_289, 13_312, 13_313, 16_384, 16_385, 20_479, 20_481])
def test_edges_of_the_chunks(R, n):
    sc, cam = _scene(1 << 23, n, n)
    d = R.DeviceScene(sc)
    ws = R.DeviceWorkspace(n, cam.width, cam.height, (16, 16))
    img = R.render(d, cam, ws, (16, 16), 1)
    _same(R, d, cam, n, 0, img, ws)
    wide = R.DeviceWorkspace(n, cam.width, cam.height, (16, 16), key_capacity=int(ws.ws.num_keys))
    assert (R.render(d, cam, wide, (16, 16), 1, sort_mode=1) == img).all()   # 64-bit keys: another sort altogether
    assert (wide.vals_sorted() == ws.vals_sorted()).all()


# the order by counting pairs, the general chain, and more than 2,048 emission chunks
@pytest.mark.parametrize("n", [4096, 20_000, 2_300_000])
def test_a_workspace_of_any_content(R, n):
    """Nothing is taken from the workspace but what the render wrote there."""
    import torch
    sc, cam = _scene(1 << 23, n, 3)
    d = R.DeviceScene(sc)
    ws = R.DeviceWorkspace(n, cam.width, cam.height, (16, 16), key_capacity=64)
    with pytest.raises(R.RecogsError):
        R.render(d, cam, ws, (16, 16), 1, grow=False)
    ws = R.DeviceWorkspace(n, cam.width, cam.height, (16, 16), key_capacity=int(ws.ws.num_keys))
    got = []
    for fill in (0, 0xFF, 0xA5):
        for graph in (False, True):
            ws.mem.fill_(fill)
            img = R.render(d, cam, ws, (16, 16), 1, grow=False, graph_mode=graph)
            k, _ = ws.readback()
            got.append((img, ws.vals_sorted()[:k].clone()))
    for img, vals in got[1:]:
        assert torch.equal(img, got[0][0]) and torch.equal(vals, got[0][1])
