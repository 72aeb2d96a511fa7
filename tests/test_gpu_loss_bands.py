"""The loss and its gradient where the streaming window sums change shape: columns of a workgroup
(256 floats of a row: 85 pixels and one channel), bands of 8, 16 and 32 rows and their remainders,
images smaller than the window. Tolerances as in test_gpu_loss.py: fp32 sums of up to 15 taps twice
(2e-6 of a moment), carried through D >= 9e-4."""

import numpy as np
import pytest
import torch

from oracle import loss as OL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,w,radius", [(8, 85, 5), (9, 86, 5), (17, 171, 7), (2, 3, 7), (7, 256, 1), (500, 1366, 5),
                                        (529, 2731, 2)])
def test_loss_at_band_and_strip_edges(h, w, radius):
    from paper_2501_19196_amd import renderer as R
    print("case", h, w, radius, flush=True)
    rng = np.random.default_rng(h * 1000 + w)
    a = rng.random((h, w, 3)).astype(np.float32)
    b = np.clip(a + 0.2 * rng.standard_normal((h, w, 3)), 0, 1).astype(np.float32)
    loss, g = R.image_loss(torch.from_numpy(a).cuda(), torch.from_numpy(b).cuda(), w, h,
                           0.4, radius, 1.5)
    torch.cuda.synchronize()
    assert float(loss.cpu()[0]) == pytest.approx(OL.loss(a, b, 0.4, radius, 1.5), rel=2e-5)
    gr = OL.loss_grad(a, b, 0.4, radius, 1.5)
    gg = g.cpu().numpy().reshape(gr.shape)
    assert np.abs(gg - gr).max() <= 2e-4 * np.abs(gr).max()
    assert np.linalg.norm(gg - gr) <= 1e-4 * np.linalg.norm(gr)
