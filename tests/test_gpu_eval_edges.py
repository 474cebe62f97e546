"""Edges of the evaluation kernels on the GPU against the FP64 oracle: image sizes around a trip
of the block, magnitudes whose FP32 squares overflow or vanish, windows across the loads in flight.
"""

import numpy as np
import pytest

import oracle as O
from parity import both_bounds
from synth import configs

pytestmark = pytest.mark.gpu


# images below, at and above the elements a block takes in one trip; an FP32 square of these
# magnitudes overflows or underflows. FP64 sums of exact differences: 1e-12.
@pytest.mark.parametrize("npx", [1, 255, 4096, 4097, 70001])
@pytest.mark.parametrize("scale", [1.0, 1e-30, 1e30])
def test_psnr_sizes_and_ranges(gpu_lib, npx, scale):
    import torch
    from paper_2311_13177_amd import binding as B

    rng = np.random.default_rng(npx)
    t = scale * (rng.standard_normal((2, npx, 1)) + 1j * rng.standard_normal((2, npx, 1)))
    t[:, 0] = 0 if npx > 1 else t[:, 0]
    im = t + 0.1 * scale * rng.standard_normal(t.shape)
    t, im = t.astype(np.complex64), im.astype(np.complex64)
    p, mse, peak = (x.cpu().numpy() for x in B.vp_psnr(torch.from_numpy(im).to("cuda"), torch.from_numpy(t).to("cuda")))
    for k in range(2):
        t64, i64 = t[k].astype(np.complex128), im[k].astype(np.complex128)
        np.testing.assert_allclose(p[k], O.psnr(i64, t64), rtol=1e-12)
        np.testing.assert_allclose(mse[k], np.mean((np.abs(i64) - np.abs(t64)) ** 2), rtol=1e-12)
        np.testing.assert_allclose(peak[k], np.abs(t64).max(), rtol=1e-15)


# pairs of pixels (even n) and single pixels; windows below, at and above the masks in flight
@pytest.mark.parametrize("n", [16, 45, 64])
def test_baseline_pairs_and_windows(gpu_lib, n):
    import torch
    from paper_2311_13177_amd import binding as B

    case = configs.small_case(n=n, n_spec=2, n_time=3, n_blades=12, lines=6, f=1.0)
    plan = B.Plan.from_geometry(case.geometry())
    y = O.simulate_measurements(case)
    masks = O.blade_masks(O.Geometry.from_dict(case.geometry()))
    for window in (1, 4, 5, 6, 11):
        want = O.window_baseline(y.astype(np.complex128), masks, window)
        got = B.vp_baseline(plan, torch.from_numpy(y).to("cuda"), window=window, first_frame=0, n_frames=12)
        assert both_bounds(got.cpu().numpy(), want) <= 1e-4, window
