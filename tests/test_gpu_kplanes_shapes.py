"""The K-Planes kernels over their compiled features, one and two scales, grids of less than a
wave's 64 samples, of remainders and of odd size, and odd numbers of bins and blades, against the
FP64 oracle: decode to 1e-5 and the gradient to 1e-4 relative, as for the other shapes.
"""

import numpy as np
import pytest

import oracle as O
from parity import both_bounds
from oracle import kplanes as K
from synth import configs

pytestmark = pytest.mark.gpu

#        n, bins, times, blades, features, scales
SHAPES = [(15, 1, 1, 1, 1, (15,)), (27, 3, 2, 3, 2, (27, 9)), (45, 5, 3, 5, 16, (45,)), (64, 2, 2, 3, 4, (64, 20)),
          (75, 3, 3, 5, 8, (75, 30)), (96, 9, 2, 3, 1, (40, 96)), (135, 2, 2, 2, 8, (135, 60)), (72, 5, 2, 4, 16, (72, 36)),
          # two (b, s) a wave: an even and an odd number of them
          (80, 40, 2, 14, 2, (33,)), (75, 27, 2, 19, 8, (25, 75))]


@pytest.mark.parametrize("n,S,T,nb,F,res", SHAPES)
def test_decode_and_gradient(gpu_lib, n, S, T, nb, F, res):
    import torch
    from paper_2311_13177_amd import binding as B

    case = configs.small_case(n=n, n_spec=S, n_time=T, n_blades=nb, lines=5, f=1.0)
    plan = B.Plan.from_geometry(case.geometry())
    geom = O.Geometry.from_dict(case.geometry())
    cfg = K.KPConfig(features=F, time_res=2, spatial_res=res)
    regs = (0.02, 0.05, 0.01)
    model = B.vp_kplanes.make(F, 2, res, *regs, 1e-2)
    y = O.simulate_measurements(case)
    _, _, total = K.layout(S, cfg)
    rng = np.random.default_rng(n + F)
    p = (0.5 * (rng.standard_normal(total) + 1j * rng.standard_normal(total))).astype(np.complex64)
    p64, d_p = p.astype(np.complex128), torch.from_numpy(p).cuda()
    times = [0.0, 0.4, 1.0]
    got = B.vp_kplanes_decode(plan, model, d_p, times).cpu().numpy()
    for i, t in enumerate(times):
        assert both_bounds(got[i], K.decode(p64, n, S, cfg, t)) <= 1e-5, t
    g, _, _ = B.vp_kplanes_gradient(plan, model, d_p, torch.from_numpy(y).cuda())
    kp = O.Geometry(n=n, n_spec=S, n_time=1, angle_rad=geom.angle_rad, lines=geom.lines,
                    blade_time=geom.blade_time if geom.blade_time is not None else np.zeros(nb),
                    spec_shift_px=geom.spec_shift_px)
    _, want, _ = K.objective_and_gradient(p64, kp, y, cfg, *regs, 1e-2)
    assert both_bounds(g.cpu().numpy(), want) <= 1e-4
