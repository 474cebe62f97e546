"""Workspaces kept by a plan for its operator calls: calls on more streams than there are slots,
of several sizes on one stream, from several threads on one stream, and a captured update replayed
between eager calls all return what a call on its own returns, bit for bit."""

import threading

import numpy as np
import pytest

from synth import configs

pytestmark = pytest.mark.gpu


def _setup():
    import torch
    from paper_2311_13177_amd import binding as B

    case = configs.small_case(n=96, n_spec=6, n_time=3, n_blades=7, lines=12, f=2.0)
    plan = B.Plan.from_geometry(case.geometry())
    g = torch.Generator(device="cuda").manual_seed(5)
    vols = [torch.randn(plan.volume_shape, dtype=torch.complex64, device="cuda", generator=g) for _ in range(6)]
    want = []
    for v in vols:
        k = B.vp_forward(plan, v)
        want.append((k, B.vp_adjoint(plan, k)))
        torch.cuda.synchronize()
    return torch, B, plan, vols, want


@pytest.mark.parametrize("streams", [1, 3, 6])
def test_calls_on_many_streams(gpu_lib, streams):
    torch, B, plan, vols, want = _setup()
    ss = [torch.cuda.Stream() for _ in range(streams)]
    got = []
    for rep in range(4):
        for i, v in enumerate(vols):
            with torch.cuda.stream(ss[i % streams]):
                k = B.vp_forward(plan, v)
                got.append((i, k, B.vp_adjoint(plan, k)))
    torch.cuda.synchronize()
    for i, k, a in got:
        assert torch.equal(k, want[i][0]) and torch.equal(a, want[i][1])


def test_threads_on_one_stream(gpu_lib):
    torch, B, plan, vols, want = _setup()
    got = [[] for _ in vols]

    def work(i):
        for _ in range(10):
            k = B.vp_forward(plan, vols[i])
            got[i].append((k, B.vp_adjoint(plan, k)))

    ts = [threading.Thread(target=work, args=(i,)) for i in range(len(vols))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    torch.cuda.synchronize()
    for i, r in enumerate(got):
        assert len(r) == 10 and all(torch.equal(k, want[i][0]) and torch.equal(a, want[i][1]) for k, a in r)


def test_blade_aligned_and_cartesian_calls_share_a_stream(gpu_lib):
    torch, B, plan, vols, want = _setup()
    alone = B.vp_nu_forward(plan, vols[0])
    torch.cuda.synchronize()
    for _ in range(3):
        k = B.vp_forward(plan, vols[1])
        s = B.vp_nu_forward(plan, vols[0])
        a = B.vp_adjoint(plan, k)
        assert torch.equal(s, alone) and torch.equal(k, want[1][0]) and torch.equal(a, want[1][1])


@pytest.mark.parametrize("t", [1, 2, 7])
def test_captured_update_replays(gpu_lib, t):
    torch, B, plan, vols, want = _setup()
    opts = B.vp_options_default(tv_weight=1e-3)
    m0, v0 = vols[2] * 0.1, vols[3].abs().to(torch.complex64)
    m, v, out = m0.clone(), v0.clone(), torch.empty_like(vols[0])
    ref_m, ref_v = m0.clone(), v0.clone()
    ref = B.vp_step(plan, opts, vols[0], vols[1], ref_m, ref_v, t)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.vp_step(plan, opts, vols[0], vols[1], m, v, t, out)
    for _ in range(3):
        m.copy_(m0)
        v.copy_(v0)
        out.zero_()
        graph.replay()
        k = B.vp_forward(plan, vols[1])
        torch.cuda.synchronize()
        assert torch.equal(out, ref) and torch.equal(m, ref_m) and torch.equal(v, ref_v)
        assert torch.equal(k, want[1][0])
