"""The DFT passes on the GPU by kind of length: compiled, radices at run time, and several
lengths in one launch.

A transform's radices follow its length alone, so a slice's batch result equals its own fit bit
for bit whatever lengths run beside it. Operators take the 1e-4 relative tolerance of the FP32
passes against the FP64 oracle.
"""

import numpy as np
import pytest

import oracle as O
from parity import assert_close
from synth import configs

pytestmark = pytest.mark.gpu


# powers and products of every radix, one row (and column) per item to sixteen
@pytest.mark.parametrize("n", [15, 16, 27, 60, 75, 81, 96, 100, 125, 144, 225, 243, 250, 270, 375, 400, 486, 500])
def test_run_time_lengths_match_the_oracle(gpu_lib, n):
    import torch
    from paper_2311_13177_amd import binding as B

    case = configs.small_case(n=n, n_spec=2, n_blades=2, lines=6, f=1.0)
    plan = B.Plan.from_geometry(case.geometry())
    geom = O.Geometry.from_dict(case.geometry())
    rng = np.random.default_rng(n)
    shape = (case.n_time, case.n_spec, n, n)
    vol = (rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64)
    k = B.vp_forward(plan, torch.from_numpy(vol).to("cuda"))
    assert_close(k.cpu().numpy(), O.forward(vol.astype(np.complex128), geom), 1e-4)
    g = B.vp_adjoint(plan, k)
    assert_close(g.cpu().numpy(), O.adjoint(k.cpu().numpy().astype(np.complex128), geom), 1e-4)


# the kinds alone and together: one compiled length, several, 512, and lengths without a plan
@pytest.mark.parametrize("lengths", [(64, 64), (64, 128, 192), (512, 512), (48, 512, 64), (512, 100, 256, 60, 320, 384)])
def test_batches_of_mixed_lengths_equal_solo_fits(gpu_lib, lengths):
    from paper_2311_13177_amd import binding as B

    plans, ys = [], []
    for i, n in enumerate(lengths):
        case = configs.small_case(n=n, n_spec=2, n_blades=2 + i % 2, lines=8, f=1.0, seed=i)
        plans.append(B.Plan.from_geometry(case.geometry()))
        ys.append(O.simulate_measurements(case))
    opts = B.vp_options_default(n_steps=3)
    got = B.vp_batch_reconstruct(plans, ys, [opts] * len(plans))
    for p, y, g in zip(plans, ys, got):
        want = B.vp_reconstruct(p, y, opts)
        assert np.array_equal(g["vol"], want["vol"]) and g["final_loss"] == want["final_loss"]


# one block per blade against the separate passes, which a batch takes: one to four groups of 16
# rows and columns, whole and partial, one and two knots a blade, steps that skip blades
@pytest.mark.parametrize("n", [5, 16, 18, 32, 36, 45, 48, 50, 64])
@pytest.mark.parametrize("n_time,schedule", [(1, "all"), (3, "all"), (3, "cyclic"), (2, "random")])
def test_whole_blades_equal_the_passes(gpu_lib, n, n_time, schedule):
    import torch
    from paper_2311_13177_amd import binding as B

    case = configs.small_case(n=n, n_spec=2, n_time=n_time, n_blades=4, lines=min(5, n), f=0.5)
    plan = B.Plan.from_geometry(case.geometry())
    y = O.simulate_measurements(case)
    sched = {"all": B.VP_SCHED_ALL_BLADES, "cyclic": B.VP_SCHED_CYCLIC, "random": B.VP_SCHED_RANDOM}[schedule]
    opts = B.vp_options_default(n_steps=5, schedule=sched, seed=3)
    (want,) = B.vp_batch_reconstruct([plan], [y], [opts])
    got = B.vp_reconstruct(plan, y, opts)
    assert np.array_equal(got["vol"], want["vol"]) and got["final_loss"] == want["final_loss"]
    geom = O.Geometry.from_dict(case.geometry())
    rng = np.random.default_rng(n)
    vol = (rng.standard_normal(plan.volume_shape) + 1j * rng.standard_normal(plan.volume_shape)).astype(np.complex64)
    d_y = torch.from_numpy(y).to("cuda")
    k = B.vp_forward(plan, torch.from_numpy(vol).to("cuda"), d_y)
    assert_close(k.cpu().numpy(), O.residual(vol.astype(np.complex128), geom, y.astype(np.complex128)), 1e-4)
    g = B.vp_adjoint(plan, d_y).cpu().numpy()
    assert_close(g, O.adjoint(y.astype(np.complex128), geom), 1e-4)
