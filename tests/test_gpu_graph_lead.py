"""Calls around the capture of a fit's larger graph against eager steps, bit for bit: at its shortest
call, in the middle of a call, and after many short ones; slices stop before, in and behind it.
"""

import numpy as np
import pytest

from test_gpu_graphs import _make

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["cartesian", "nu", "kplanes", "batch"])
@pytest.mark.parametrize("calls", [(31, 1, 32), (33, 8, 3), (47, 16, 7), (8,) * 19])
def test_steps_around_the_larger_graph(gpu_lib, kind, calls):
    from paper_2311_13177_amd import binding as B

    g, read_g = _make(B, kind)
    e, read_e = _make(B, kind)
    for n in calls:
        g.step(n)
    e.step(sum(calls), use_graph=False)
    assert np.array_equal(read_g(), read_e())
