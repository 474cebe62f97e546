"""The projection's staging on the GPU: units of 16 and of 4 bytes, rings of planes, regions of
every size class, against the FP64 oracle.

A gradient-descent fit is linear in the projection, so its volume agrees with the oracle's to
the operators' tolerance (1e-4 relative); two steps run the projection of a nonzero volume.
"""

import numpy as np
import pytest

import oracle as O
from parity import assert_close
from synth import configs

pytestmark = pytest.mark.gpu

CASES = {
    # one, two and three bins: rings longer than the bins, a last phase half full
    "bins_1": (dict(n=48, n_spec=1, n_blades=3, lines=9, f=0.5), [(8, 1, 2, 1), (2, 1, 2, 1, 0, 4, 8)]),
    "bins_3": (dict(n=64, n_spec=3, n_blades=5, lines=9, f=2.0), [(4, 1, 2, 1), (1, 2, 2, 1, 0, 4, 8)]),
    # odd n: the last column has no neighbour to share a 16-byte unit with
    "odd_45": (dict(n=45, n_spec=5, n_blades=4, lines=9, f=2.0), [(1, 1, 2, 1), (8, 1, 2, 1, 0, 4, 8), (12, 1, 2, 1)]),
    "odd_135": (dict(n=135, n_spec=4, n_time=3, n_blades=6, lines=12, f=6.0), [(4, 2, 2, 1), (12, 1, 2, 1, 0, 4, 8)]),
    # wide shears: regions above 1024 elements, and above 2048 (both parities of n)
    "wide_96": (dict(n=96, n_spec=6, n_blades=4, lines=12, f=7.0), [(8, 1, 2, 1), (2, 4, 2, 1, 0, 4, 8)]),
    "wider_72": (dict(n=72, n_spec=4, n_blades=5, lines=12, f=13.0), [(8, 1, 2, 1), (8, 2, 2, 1, 0, 4, 8)]),
    "wider_75": (dict(n=75, n_spec=4, n_blades=5, lines=12, f=13.0), [(8, 1, 2, 1), (4, 1, 2, 1, 0, 4, 8)]),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_staged_projection_matches_the_oracle(gpu_lib, name):
    from paper_2311_13177_amd import binding as B

    kw, shapes = CASES[name]
    case = configs.small_case(**kw)
    plan = B.Plan.from_geometry(case.geometry())
    y = O.simulate_measurements(case)
    want = O.reconstruct(O.Geometry.from_dict(case.geometry()), y, 2, optimizer="gd")
    ref = B.vp_reconstruct(plan, y, B.vp_options_default(n_steps=2, optimizer=B.VP_OPT_GD))
    assert_close(ref["vol"], want["vol"], 1e-4)
    for sh in shapes:
        got = B.vp_reconstruct(plan, y, B.vp_options_default(n_steps=2, optimizer=B.VP_OPT_GD, tiles=sh))
        assert np.array_equal(got["vol"], ref["vol"]), sh
