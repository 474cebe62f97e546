"""The tile shapes that plans choose by themselves, on the host, at sizes where both sides of the
rule have been measured (`best`: the fastest compiled shapes there, within three per cent).
"""

import numpy as np
import pytest

from paper_2311_13177_amd import binding as B


def _plan(n, S, T, nb, f):
    tau = None if T == 1 else np.arange(nb) / nb
    ang = 180.0 * np.arange(nb) / nb if T == 1 else np.mod(np.arange(nb) * 111.246, 180.0)
    return B.Plan.from_geometry(dict(n=n, n_spec=S, n_time=T, angle_rad=np.deg2rad(ang), lines=np.full(nb, 16, np.int32),
                                     blade_time=tau, spec_shift_px=(np.arange(S) - S / 4.0) * 2.0 * f / S))


# (rows, parts per wave, waves) of the projection
@pytest.mark.parametrize("case,best", [
    ((150, 64, 4, 9, 2.0), {(4, 1, 8), (4, 2, 8)}),    # few parts a knot: 35 us, 54 with two rows
    ((128, 32, 4, 9, 2.5), {(2, 1, 8), (2, 1, 4)}),    # 18 us, 28 with one row
    ((300, 64, 1, 4, 7.2), {(2, 1, 4), (2, 1, 8), (4, 1, 8)}),  # 34 us, 57 with one row
    ((225, 64, 4, 9, 6.0), {(8, 1, 8)}),               # 53 us, 78 with four rows
    ((225, 64, 1, 12, 2.0), {(4, 1, 8), (4, 1, 4)}),   # 42 us, 68 with two rows
    ((256, 32, 1, 12, 2.0), {(4, 1, 4)}),              # 22 us, 25 with eight rows
    ((64, 32, 16, 32, 2.0), {(2, 1, 4), (2, 1, 8), (4, 1, 8), (4, 1, 4)}),  # 18 us, 27 with one row
    ((192, 32, 16, 32, 3.0), {(8, 1, 8)}),
    ((64, 16, 1, 5, 2.0), {(1, 1, 8), (2, 1, 8), (1, 1, 4)}),
    ((384, 64, 1, 24, 6.5), {(8, 1, 8)}),              # 101 us, 134 in groups of sixteen
    ((150, 64, 1, 8, 4.8), {(1, 1, 8)}),               # 28 us, 34 with two rows
])
def test_projection_shapes(case, best):
    pr, gw, _, _, _, _, pw, _ = _plan(*case).tiles()
    assert (pr, gw, pw) in best


# (rows, bins per wave, resident) of the gather with the update
@pytest.mark.parametrize("case,best", [
    ((300, 4, 1, 8, 7.2), {(4, 1, 0)}),                # 18 us, 24 with two rows
    ((300, 4, 1, 24, 2.0), {(4, 1, 0)}),               # 29 us, 38
    ((225, 16, 1, 8, 6.0), {(4, 1, 0), (4, 2, 0)}),    # 22 and 23 us, 30 with two rows
    ((300, 16, 1, 24, 7.2), {(4, 2, 0)}),              # 46 us, 58 with one bin
    ((128, 4, 8, 16, 2.5), {(4, 1, 0), (4, 1, 1)}),    # 14 and 15 us, 18 with two rows
    ((256, 32, 1, 12, 4.0), {(4, 2, 0)}),
    ((192, 32, 16, 32, 3.0), {(4, 4, 1)}),
    ((64, 16, 1, 5, 2.0), {(2, 1, 0), (2, 1, 1)}),
])
def test_gather_shapes(case, best):
    _, _, gr, gb, _, _, _, res = _plan(*case).tiles()
    assert (gr, gb, res) in best
