"""The grid correction of the convolutional path over its parameters: one visibility on the origin's
cell makes a constant plane, so the image of blink_image_batch_conv is the correction's product
1 / (c(X/N) c(Y/N)) times the same constant; its profile along the axes is compared with the
oracle's correction at the smallest and largest width, flat to narrow kernels and both shift forms.
Bound: the correction and the row pass round to FP32 a few times, and a placement's tap weights
(relative error below 1e-6 each, of one sign pattern) act as one smooth factor: 2e-5 of the peak.
"""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch as _t
    if not _t.cuda.is_available():
        pytest.skip("no GPU")
    return _t


@pytest.mark.parametrize("shift", [True, False])
@pytest.mark.parametrize("N,width,beta", [(64, 4, 9.2), (1024, 8, 18.4), (256, 16, 36.8), (256, 7, 16.1), (512, 2, 4.6),
                                          (128, 16, 100.0), (4096, 6, 13.8)])
def test_profile(torch, N, width, beta, shift):
    import paper_2505_15204_amd as blink
    print(f"[gpu-case] conv correction N={N} width={width} beta={beta} shift={shift}", flush=True)
    d = "cuda:0"
    vis = torch.ones((1, 1, 1, 1), dtype=torch.complex64, device=d)
    uvw = torch.zeros((1, 1, 3), dtype=torch.float64, device=d)
    freq = torch.full((1,), 150.0e6, dtype=torch.float64, device=d)
    with blink.Context(0) as ctx:
        res = ctx.blink_image_batch_conv(vis, None, uvw, freq, N, 1.0e-3, width, beta, shift=shift)
        torch.cuda.synchronize()
        img = res["images"].cpu().numpy().reshape(N, N).astype(np.float64)
    want = oracle.image_batch_conv(vis.cpu().numpy(), None, uvw.cpu().numpy(), freq.cpu().numpy(), N, 1.0e-3, width,
                                   beta, shift=shift)["images"].reshape(N, N)
    # the corner pixels are divided by the smallest values of c: compare relative to each pixel's
    # correction, over which FP32 errors are spread
    c = oracle.conv_correction(N, width, beta, shift)
    scale = np.max(np.abs(c)) ** 2 / (c[:, None] * c[None, :])
    assert np.max(np.abs(img - want) / scale) <= 2e-5 * np.max(np.abs(want))
