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


# knots whose parts do not fit LDS at once, with voxels for sixteen sums a lane: the fused gather
# takes fewer bins than the storing one, and each finds the tables the other has uploaded
@pytest.mark.parametrize("first", ["operator", "session"])
def test_phased_shapes_of_fits_and_operators(gpu_lib, first):
    import torch
    from parity import assert_close
    from paper_2311_13177_amd import binding as B

    case = configs.small_case(n=256, n_spec=64, n_blades=8, lines=8, f=6.0)
    plan = B.Plan.from_geometry(case.geometry())
    geom = O.Geometry.from_dict(case.geometry())
    y = O.simulate_measurements(case)
    pr, gw, rows, sc, _, _, _, res = plan.tiles()
    assert res == 0 and rows * sc <= 8
    d_y = torch.from_numpy(y).to("cuda")
    vol = torch.randn(plan.volume_shape, dtype=torch.complex64, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    out = torch.empty(plan.blade_shape, dtype=torch.complex64, device="cuda")
    if first == "operator":
        k = B.vp_forward(plan, vol)
        B.vp_forward_noalloc(plan, vol, out)
    else:
        B.vp_reconstruct(plan, y, B.vp_options_default(n_steps=1))
        B.vp_forward_noalloc(plan, vol, out)
        k = B.vp_forward(plan, vol)
    assert torch.equal(k, out)
    assert_close(B.vp_adjoint(plan, d_y).cpu().numpy(), O.adjoint(y.astype(np.complex128), geom), 1e-4)
    got = B.vp_reconstruct(plan, y, B.vp_options_default(n_steps=2))
    want = B.vp_reconstruct(plan, y, B.vp_options_default(n_steps=2, tiles=(pr, gw, 4, 4)))
    assert np.array_equal(got["vol"], want["vol"]) and got["final_loss"] == want["final_loss"]
