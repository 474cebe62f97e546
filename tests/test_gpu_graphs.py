"""Fits stepped by graphs of one and of eight steps against eager steps, bit for bit: counts below,
at and above eight and sixteen, in calls of changing length with reads between them.
"""

import numpy as np
import pytest

import oracle as O
from synth import configs
from synth.kplanes_init import init_params

pytestmark = pytest.mark.gpu

CALLS = [(1, 2, 1), (7, 8), (8, 8, 3), (15, 1, 9), (16, 5), (17, 24, 1), (40,)]


def _make(B, kind):
    case = configs.small_case(n=48, n_spec=4, n_time=2, n_blades=5, lines=8, f=1.0)
    plan = B.Plan.from_geometry(case.geometry())
    y = O.simulate_measurements(case)
    opts = B.vp_options_default(n_steps=64, lr=1e-2)
    if kind == "cartesian":
        s = B.Session(plan, y, opts)
        return s, lambda: s.read()["vol"]
    if kind == "nu":
        rng = np.random.default_rng(3)
        smp = (rng.standard_normal(B.nu_shape(plan)) + 1j * rng.standard_normal(B.nu_shape(plan))).astype(np.complex64)
        s = B.NuSession(plan, smp, opts)
        return s, lambda: s.read()["vol"]
    if kind == "kplanes":
        s = B.KPlanesSession(plan, B.vp_kplanes.make(2, 2, (48,), 0.01, 0.02, 0.005, 1e-2), y,
                             init_params(4, 2, 2, (48,), seed=5), opts)
        return s, lambda: s.read()["params"]
    # slices that stop at 5, 20 and 64 steps, inside and between graphs
    b = B.Batch([plan] * 3, [y, 2 * y, 3 * y], [B.vp_options_default(n_steps=k, lr=1e-2) for k in (5, 20, 64)])
    return b, lambda: np.stack([b.read(i)["vol"] for i in range(3)])


@pytest.mark.parametrize("kind", ["cartesian", "nu", "kplanes", "batch"])
@pytest.mark.parametrize("calls", CALLS)
def test_graph_steps_equal_eager_steps(gpu_lib, kind, calls):
    from paper_2311_13177_amd import binding as B

    g, read_g = _make(B, kind)
    e, read_e = _make(B, kind)
    for n in calls:
        g.step(n)
        e.step(n, use_graph=False)
        assert np.array_equal(read_g(), read_e()), (n, calls)
