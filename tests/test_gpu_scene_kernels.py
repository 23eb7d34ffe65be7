"""Selection and baked recolour at the edges of their vector and workgroup sizes: counts
around 4 and 8 elements per thread and around the one-workgroup selection, plane strides
and mask addresses that are and are not aligned for the vector accesses."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import paper_2511_18441_amd as R
    return R


@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("n,pad,shift", [(1, 0, 0), (3, 1, 0), (5, 3, 1), (4096, 0, 0), (4095, 1, 0), (16384, 0, 0),
                                         (16385, 3, 0), (16387, 0, 3), (300_001, 7, 0)])
def test_select_sizes_and_alignment(R, orc, n, pad, shift, storage):
    """mask and count against the oracle's predicate (decisions it flags excepted)."""
    import torch
    w = synth.make_mid(n=max(n, 64))
    sc = w.scene.subset(np.arange(n))
    sc = sc if storage == "f32" else sc.with_storage(storage)
    sel = synth.SelectParams(400.0, 400.0, 300.0, np.float32([0.5, 0.5, 0.5]), 0.6)
    d = R.DeviceScene(sc, stride=n + pad)
    buf = torch.full((n + 8,), 7, dtype=torch.uint8, device="cuda")
    mask = buf[shift:shift + n]
    count = torch.full((1,), 99, dtype=torch.int32, device="cuda")
    R.recogs_select(d.c_struct(), R.camera_struct(w.view.camera), R.select_struct(sel), mask.data_ptr(), count.data_ptr())
    got = mask.cpu().numpy()
    ref, flag = orc.select(sc, w.view.camera, sel)
    assert not ((got != ref) & (flag == 0)).any()
    assert int(count.item()) == int(got.sum())
    rest = buf.cpu().numpy()
    assert (rest[:shift] == 7).all() and (rest[shift + n:] == 7).all()


@pytest.mark.parametrize("storage", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("n,deg,pad", [(1, 0, 0), (7, 1, 0), (8, 3, 0), (9, 2, 7), (2047, 3, 1), (2048, 1, 0), (4099, 3, 5)])
def test_recolor_into_a_whole_copy(R, n, deg, pad, storage):
    """The copy holds the bits of a cloned scene recoloured in place; columns past n stay."""
    import torch
    rng = np.random.default_rng(n + deg)
    sc = synth.scenes.make_scene_mid_like(rng, max(n, 64), deg).subset(np.arange(n))
    sc = sc if storage == "f32" else sc.with_storage(storage)
    d = R.DeviceScene(sc, stride=n + pad)
    mask = torch.from_numpy((rng.random(n) < 0.4).astype(np.uint8)).cuda()
    M = torch.from_numpy((np.eye(3) + 0.2 * rng.standard_normal((3, 3))).astype(np.float32).reshape(9)).cuda()
    b = torch.from_numpy(rng.uniform(-0.1, 0.1, 3).astype(np.float32)).cuda()
    want = d.sh.clone()
    R.recogs_recolor(d.c_struct(), want.data_ptr(), mask.data_ptr(), M.data_ptr(), b.data_ptr(), 0)
    got = torch.full_like(d.sh, 3.0)
    R.recogs_recolor(d.c_struct(), got.data_ptr(), mask.data_ptr(), M.data_ptr(), b.data_ptr(), 1)
    assert torch.equal(got[:, :n], want[:, :n])
    assert bool((got[:, n:] == 3.0).all())
