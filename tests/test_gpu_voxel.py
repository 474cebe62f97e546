"""Edges of the voxel-wise TV/L1 gradient on the GPU against the FP64 oracle: planes of less than
a block and of remainders, missing neighbours of every kind, both weights, accumulation.
"""

import numpy as np
import pytest

import oracle as O
from parity import assert_close
from synth import configs

pytestmark = pytest.mark.gpu


# n 16: less than a block; 32: exactly two blocks; 45, 75: odd remainders; one bin or knot
@pytest.mark.parametrize("n,S,T", [(16, 1, 1), (16, 3, 2), (32, 1, 3), (45, 2, 1), (75, 4, 3)])
def test_tv_gradient_edges(gpu_lib, n, S, T):
    import torch
    from paper_2311_13177_amd import binding as B

    case = configs.small_case(n=n, n_spec=S, n_time=T, n_blades=3, lines=6, f=1.0)
    plan = B.Plan.from_geometry(case.geometry())
    rng = np.random.default_rng(n * S + T)
    vol = (rng.standard_normal((T, S, n, n)) + 1j * rng.standard_normal((T, S, n, n))).astype(np.complex64)
    v64 = vol.astype(np.complex128)
    d = torch.from_numpy(vol).to("cuda")
    for tv, l1 in ((0.5, 0.0), (0.0, 0.3), (0.5, 0.3)):
        want = tv * O.tv_grad(v64, 1e-2) + l1 * O.l1_grad(v64, 1e-2)
        assert_close(B.vp_tv_grad(plan, d, tv, l1, 1e-2).cpu().numpy(), want, 1e-4)
        acc = d.clone()
        B.vp_tv_grad(plan, d, tv, l1, 1e-2, grad=acc, accumulate=True)
        assert_close(acc.cpu().numpy(), want + v64, 1e-4)
