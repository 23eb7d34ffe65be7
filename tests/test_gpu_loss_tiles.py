"""The SSIM passes at the edges of their 64 x 8 tiles and their halos, on the smallest
images and on images narrower or shorter than the window."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import paper_2511_18441_amd as R
    return R


@pytest.mark.parametrize("H,W", [(1, 1), (1, 200), (130, 1), (8, 64), (7, 63), (9, 65), (17, 129), (16, 16), (5, 191),
                                 (24, 69), (67, 320)])
def test_dssim_at_tile_edges(R, orc, H, W):
    """Loss and gradient against the oracle; nothing written past the workspace. The
    gradient's bound is that of a float32 evaluation of two 121-tap windows: 1e-4 of the
    largest entry."""
    import torch
    y = synth.random_image(11, (H, W, 3), 0.3)
    t = (0.7 * y + synth.random_image(12, (H, W, 3), 0.1)).astype(np.float32)
    ty, tt = torch.from_numpy(y).cuda(), torch.from_numpy(t).cuda()
    nb = R.recogs_dssim_workspace_bytes(W, H)
    ws = torch.full((nb // 4 + 64,), 12345.0, device="cuda")
    lam, n = 0.2, y.size
    loss = torch.empty(1, device="cuda")
    dl = torch.full_like(ty, 5.0)
    R.recogs_loss_l1_dssim(ty.data_ptr(), tt.data_ptr(), W, H, (1 - lam) / n, lam, dl.data_ptr(), 0, loss.data_ptr(),
                           ws.data_ptr(), nb)
    val, g = orc.ssim(y, t)
    ref = (1 - lam) * orc.loss_l1_grad(y, t) - lam * g
    assert abs(loss.item() - ((1 - lam) * orc.loss_l1(y, t) + lam * (1.0 - val))) <= 1e-5
    assert np.abs(dl.cpu().numpy() - ref).max() <= 1e-4 * np.abs(ref).max()
    assert bool((ws[nb // 4:] == 12345.0).all())
