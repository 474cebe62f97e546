"""A projection tile whose exact region fits the staging limit while the region from even columns
does not (43 x 95 and 43 x 96 of 4096 elements): asked for or met by the tuner, it fits as the
default shape does, bit for bit.
"""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,shift", [(128, np.linspace(-15, 15, 31)), (192, np.linspace(-14.5, 15.5, 31))])
def test_region_at_the_limit(gpu_lib, n, shift):
    from paper_2311_13177_amd import binding as B

    nb = 8
    plan = B.Plan.from_geometry(dict(n=n, n_spec=31, n_time=1, angle_rad=np.deg2rad(180.0 * np.arange(nb) / nb),
                                     lines=np.full(nb, 16, np.int32), blade_time=None, spec_shift_px=shift))
    rng = np.random.default_rng(n)
    y = ((rng.standard_normal(plan.blade_shape) + 1j * rng.standard_normal(plan.blade_shape))
         * plan.masks()).astype(np.complex64)
    want = B.vp_reconstruct(plan, y, B.vp_options_default(n_steps=2))
    asked = B.vp_options_default(n_steps=2, tiles=(12, 1, 2, 1, 0, 4, 8))
    for opts in (asked, B.vp_options_default(n_steps=2, autotune=1)):
        got = B.vp_reconstruct(plan, y, opts)
        assert np.array_equal(got["vol"], want["vol"]) and got["final_loss"] == want["final_loss"]
