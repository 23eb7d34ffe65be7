"""The region form composites four records at a time out of a ring of 96: the same image,
transmittance and list positions, bit for bit, as the tile form (8x8 tiles at 2 pixels per
thread), for lists that end at every place in a group, a chunk of 64 and the ring, with
splats that miss a region, and for pixels that stop at any record of a group or never."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import paper_2511_18441_amd as R
    return R


@pytest.mark.parametrize("opacity", [0.05, 0.6, 0.97])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 63, 64, 65, 66, 97, 128, 191, 400])
def test_region_form_equals_tile_form(R, n, opacity):
    import torch
    from tests.scenes_by_hand import axis_camera, scene_from
    rng = np.random.default_rng(n)
    means = np.column_stack([rng.uniform(-0.8, 0.8, n), rng.uniform(-0.8, 0.8, n), rng.uniform(3.0, 6.0, n)])
    sc = scene_from(means, np.log(rng.uniform(0.02, 0.5, (n, 3))), np.clip(rng.normal(opacity, 0.02, n), 0.01, 0.99),
                    rng.uniform(0.0, 1.0, (n, 3)))
    cam = axis_camera(37, 29, 40.0)
    d = R.DeviceScene(sc)
    out = []
    for tile, ppt in (((8, 8), 2), ((16, 16), 1), ((32, 32), 1), ((16, 16), 2), ((32, 32), 4)):
        ws = R.DeviceWorkspace(n, cam.width, cam.height, tile)
        kw = dict(depth=torch.empty((cam.height, cam.width), device="cuda")) if ppt != 2 or tile != (8, 8) else {}
        img = R.render(d, cam, ws, tile, ppt, (0.2, 0.4, 0.6), keep_backward=True, **kw)
        plain = R.render(d, cam, ws, tile, ppt, (0.2, 0.4, 0.6), chw=True)
        R.render(d, cam, ws, tile, ppt, (0.2, 0.4, 0.6), keep_backward=True, image=img)
        # nproc counts list entries, which depend on the tile: compared through the blended value
        last = ws.nproc().long() - 1
        r = ws.ranges().long()
        ty = torch.arange(cam.height, device="cuda")[:, None] // tile[1]
        tx = torch.arange(cam.width, device="cuda")[None, :] // tile[0]
        first = r[(ty * (-(-cam.width // tile[0])) + tx).flatten(), 0].view(cam.height, cam.width)
        v = ws.vals_sorted().long()
        owner = torch.where(last >= 0, v[(first + last).clamp(0, max(len(v) - 1, 0))], last)
        out.append((img, plain.permute(1, 2, 0).contiguous(), ws.final_T().clone(), owner, kw.get("depth")))
    for o in out:
        assert torch.equal(o[0], out[0][0]) and torch.equal(o[1], out[0][0])
        assert torch.equal(o[2], out[0][2]) and torch.equal(o[3], out[0][3])
        if o[4] is not None:
            assert torch.equal(o[4], out[1][4])
