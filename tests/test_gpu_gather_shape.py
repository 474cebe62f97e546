"""The default gather shapes on the GPU: a fit is the same bit for bit whatever tile shape it takes.
"""

import numpy as np
import pytest

import oracle as O
from synth import configs

pytestmark = pytest.mark.gpu


# 512k voxels a step of the rule: one side of each line, and the line itself
@pytest.mark.parametrize("n,S", [(64, 16), (125, 32), (128, 32), (180, 32), (256, 16)])
def test_gather_shapes_give_the_same_fit(gpu_lib, n, S):
    from paper_2311_13177_amd import binding as B

    case = configs.small_case(n=n, n_spec=S, n_blades=3, lines=8, f=2.0)
    plan = B.Plan.from_geometry(case.geometry())
    y = O.simulate_measurements(case)
    got = B.vp_reconstruct(plan, y, B.vp_options_default(n_steps=2))
    pr, gw = plan.tiles()[:2]
    for rows, sc in ((4, 4), (2, 1)):
        want = B.vp_reconstruct(plan, y, B.vp_options_default(n_steps=2, tiles=(pr, gw, rows, sc)))
        assert np.array_equal(got["vol"], want["vol"]) and got["final_loss"] == want["final_loss"]
