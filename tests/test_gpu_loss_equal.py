"""The SSIM term of equal images: 1 - S cancels, so what is left of the loss is rounding."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import paper_2511_18441_amd as R
    return R


@pytest.mark.parametrize("kind", [0.1, 0.3, 0.7, 0.9, "random", "smooth"])
def test_dssim_of_equal_images(R, kind):
    """Equal images make the two factors of S's denominator those of its numerator, bit for
    bit, so S is 1 to the rounding of three products and a reciprocal (2^-22), and its sum
    over 23,040 values in 20 workgroups (25 additions deep) and the two of the loss keep 27
    2^-24 of it: 2e-6 in all."""
    import torch
    H, W = 80, 96
    if kind == "random":
        y = synth.random_image(5, (H, W, 3), 0.3)
    elif kind == "smooth":
        y = np.broadcast_to((0.5 + 0.3 * np.sin(np.arange(W) / 20.0))[None, :, None], (H, W, 3))
    else:
        y = np.full((H, W, 3), kind)
    ty = torch.from_numpy(np.ascontiguousarray(y, np.float32)).cuda()
    tt = ty.clone()
    nb = R.recogs_dssim_workspace_bytes(W, H)
    ws = torch.empty(nb // 4, device="cuda")
    loss, dl = torch.empty(1, device="cuda"), torch.empty_like(ty)
    R.recogs_loss_l1_dssim(ty.data_ptr(), tt.data_ptr(), W, H, 0.0, 1.0, dl.data_ptr(), 0, loss.data_ptr(), ws.data_ptr(), nb)
    assert abs(loss.item()) <= 2e-6
