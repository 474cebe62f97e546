"""Magnitudes of the PSNR terms are correctly rounded FP64 roots: an image of one pixel against a
truth of zero has the square of its magnitude as its mean squared error, which no neighbouring
value of the magnitude gives.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [1e-15, 1.0, 3e7])
def test_magnitudes_are_correctly_rounded(gpu_lib, scale):
    import torch
    from paper_2311_13177_amd import binding as B

    rng = np.random.default_rng(11)
    n = 2_000_000
    im = (scale * (rng.standard_normal(n) + 1j * rng.standard_normal(n))).astype(np.complex64).reshape(n, 1, 1)
    d = torch.from_numpy(im).to("cuda")
    _, mse, _ = B.vp_psnr(d, torch.zeros_like(d))
    x, y = im.real.astype(np.float64), im.imag.astype(np.float64)
    mag = np.sqrt(x * x + y * y).reshape(-1)  # both squares are exact, one rounding in the sum
    wrong = int(np.count_nonzero(mse.cpu().numpy() != mag * mag))
    assert wrong == 0, wrong
