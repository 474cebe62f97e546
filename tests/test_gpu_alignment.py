"""Operator calls on arrays that start 8 bytes past a 16-byte boundary, the alignment that the C
interface asks for: the same bits as on aligned arrays.
"""

import pytest

from synth import configs

pytestmark = pytest.mark.gpu


def _shifted(t):
    import torch

    buf = torch.empty(t.numel() + 3, dtype=t.dtype, device=t.device)
    at = 1 if buf.data_ptr() % 16 == 0 else 0
    out = buf[at:at + t.numel()].view(t.shape)
    out.copy_(t)
    assert out.data_ptr() % 16 == 8
    return out


# regions of each size class of the staging, one and several knots, an odd size beside the even ones
@pytest.mark.parametrize("kw", [dict(n=48, n_spec=3, n_blades=3, lines=9, f=0.5), dict(n=64, n_spec=5, n_blades=9, lines=9, f=2.0),
                                dict(n=96, n_spec=6, n_time=3, n_blades=6, lines=12, f=7.0),
                                dict(n=72, n_spec=4, n_blades=5, lines=12, f=13.0),
                                dict(n=45, n_spec=4, n_blades=4, lines=9, f=2.0)])
def test_eight_byte_aligned_arrays(gpu_lib, kw):
    import torch
    from paper_2311_13177_amd import binding as B

    plan = B.Plan.from_geometry(configs.small_case(**kw).geometry())
    g = torch.Generator(device="cuda").manual_seed(3)
    vol = torch.randn(plan.volume_shape, dtype=torch.complex64, device="cuda", generator=g)
    y = torch.randn(plan.blade_shape, dtype=torch.complex64, device="cuda", generator=g)
    off, y_off = _shifted(vol), _shifted(y)
    want = B.vp_forward(plan, vol, y)
    assert torch.equal(B.vp_forward(plan, off, y_off, out=_shifted(y)), want)
    out = _shifted(y)
    B.vp_forward_noalloc(plan, off, out, y=y_off)
    assert torch.equal(out, want)
    assert torch.equal(B.vp_adjoint(plan, _shifted(want), grad=_shifted(vol)), B.vp_adjoint(plan, want))
    s = B.vp_nu_forward(plan, vol)
    assert torch.equal(B.vp_nu_forward(plan, off), s)
    assert torch.equal(B.vp_nu_adjoint(plan, _shifted(s)), B.vp_nu_adjoint(plan, s))
    assert torch.equal(B.vp_tv_grad(plan, off, 0.5, 0.3, 1e-2), B.vp_tv_grad(plan, vol, 0.5, 0.3, 1e-2))
    opts = B.vp_options_default(tv_weight=1e-3)
    m, v = [0.1 * vol, vol.abs().to(torch.complex64)], [0.1 * vol, vol.abs().to(torch.complex64)]
    new = B.vp_step(plan, opts, vol, vol, m[0], m[1], 3)
    mo, vo = _shifted(v[0]), _shifted(v[1])
    assert torch.equal(B.vp_step(plan, opts, off, off.clone(), mo, vo, 3), new)
    assert torch.equal(mo, m[0]) and torch.equal(vo, m[1])
    for a, b in zip(B.vp_render(plan, off, 2), B.vp_render(plan, vol, 2)):
        assert torch.equal(a, b)


def test_eight_byte_aligned_evaluation(gpu_lib):
    import torch
    from paper_2311_13177_amd import binding as B

    plan = B.Plan.from_geometry(configs.small_case(n=48, n_spec=2, n_time=3, n_blades=7, lines=9).geometry())
    g = torch.Generator(device="cuda").manual_seed(4)
    y = torch.randn(plan.blade_shape, dtype=torch.complex64, device="cuda", generator=g)
    a, b = y[:3].contiguous(), y[3:6].contiguous()
    kw = dict(window=3, first_frame=0, n_frames=7)
    assert torch.equal(B.vp_baseline(plan, _shifted(y), **kw), B.vp_baseline(plan, y, **kw))
    for p, q in zip(B.vp_psnr(_shifted(a), _shifted(b)), B.vp_psnr(a, b)):
        assert torch.equal(p, q)
