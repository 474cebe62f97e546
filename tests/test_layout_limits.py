"""Projection regions at the staging limit, on the host: whatever shape a plan accepts, the launch
accepts too, and a plane of the ring holds the region that the kernel stages.
"""

import numpy as np

from host_build import run_host
from paper_2311_13177_amd import binding


def _geometry(n, S, T, nb, shift):
    ang = np.deg2rad(180.0 * np.arange(nb) / nb) if T == 1 else np.deg2rad(np.mod(np.arange(nb) * 111.246, 180.0))
    return " ".join(map(str, [n, S, T, nb, *shift, *ang, *(np.arange(nb) / nb)]))


def test_accepted_shapes_can_be_launched(tmp_path):
    binding.lib()
    rng = np.random.default_rng(4)
    text = [_geometry(128, 31, 1, 8, np.linspace(-15, 15, 31)),  # 43 x 95 exact, 43 x 96 from even columns
            _geometry(192, 31, 1, 12, np.linspace(-14.5, 15.5, 31)),
            _geometry(192, 31, 16, 32, np.linspace(-14.5, 15.5, 31)),
            _geometry(125, 31, 1, 8, np.linspace(-15, 15, 31))]
    for _ in range(120):
        hi = rng.uniform(0.5, 16.0)
        lo = -rng.uniform(0.0, 16.0)
        S = int(rng.integers(2, 40))
        T = int(rng.choice([1, 4]))
        text.append(_geometry(int(rng.choice([48, 75, 128, 135, 192])), S, T, int(rng.integers(2, 16)),
                              np.linspace(lo, hi, S)))
    rc, out = run_host(tmp_path, "layouts", "\n".join(text) + "\n")
    last = out.strip().splitlines()[-1].split()
    assert rc == 0 and last[:1] == ["accepted"], out
    assert int(last[1]) > 1000 and int(last[3]) > 0 and int(last[5]) == 0, out
