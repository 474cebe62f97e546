"""Operator calls whose workspace is not simply the stream's own kept one: streams that come and go,
captured calls replayed beside eager ones, and workspaces above the size that is kept.
"""

import numpy as np
import pytest

import oracle as O
from parity import assert_close
from synth import configs
from test_gpu_workspace import _setup

pytestmark = pytest.mark.gpu


def test_streams_that_come_and_go(gpu_lib):
    torch, B, plan, vols, want = _setup()
    big = B.vp_nu_forward(plan, vols[0])
    for rep in range(3):
        for i, v in enumerate(vols):
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                k = B.vp_forward(plan, v)
                a = B.vp_adjoint(plan, k)
                n = B.vp_nu_forward(plan, vols[0])
            if (rep + i) % 2:  # its slots finished, or still at work when the next stream asks
                s.synchronize()
            torch.cuda.current_stream().wait_stream(s)
            assert torch.equal(k, want[i][0]) and torch.equal(a, want[i][1]) and torch.equal(n, big)


# a graph may not share a kept workspace with the calls that run while it is replayed
def test_captured_calls_replay_beside_eager_ones(gpu_lib):
    torch, B, plan, vols, want = _setup()
    cs, es = torch.cuda.Stream(), torch.cuda.Stream()
    vol = vols[0].clone()
    k, a = torch.empty_like(want[0][0]), torch.empty_like(want[0][1])

    def both():
        B.vp_forward(plan, vol, out=k)
        B.vp_adjoint(plan, k, grad=a)

    with torch.cuda.stream(cs):
        both()  # the stream has its slot
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=cs):
        both()
    for rep in range(4):
        i, j = rep % 3, 3 + rep % 3
        vol.copy_(vols[i])
        k.zero_()
        a.zero_()
        torch.cuda.synchronize()
        got = []
        with torch.cuda.stream(cs):
            graph.replay()
            e = B.vp_forward(plan, vols[j])  # on the capture stream itself
            got.append((e, B.vp_adjoint(plan, e)))
        with torch.cuda.stream(es):
            for _ in range(3):
                e = B.vp_forward(plan, vols[j])
                got.append((e, B.vp_adjoint(plan, e)))
        torch.cuda.synchronize()
        assert torch.equal(k, want[i][0]) and torch.equal(a, want[i][1]), rep
        assert all(torch.equal(x, want[j][0]) and torch.equal(y, want[j][1]) for x, y in got), rep


def test_workspace_above_the_kept_size(gpu_lib):
    import torch
    from paper_2311_13177_amd import binding as B

    case = configs.small_case(n=512, n_spec=1, n_time=2, n_blades=17, lines=12, f=1.0)
    plan = B.Plan.from_geometry(case.geometry())
    assert 2 * 17 * 512 * 512 * 8 > 64 << 20
    rng = np.random.default_rng(2)
    vol = (rng.standard_normal(plan.volume_shape) + 1j * rng.standard_normal(plan.volume_shape)).astype(np.complex64)
    d = torch.from_numpy(vol).to("cuda")
    first, second = B.vp_forward(plan, d), B.vp_forward(plan, d)
    assert torch.equal(first, second)
    assert_close(first.cpu().numpy(), O.forward(vol.astype(np.complex128), O.Geometry.from_dict(case.geometry())), 1e-4)
