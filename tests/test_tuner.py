"""What the tuner times, on the host: projections and gathers as a step runs them, not behind their like."""

from host_build import run_host
from paper_2311_13177_amd import binding


def test_kernels_are_timed_as_in_a_step(tmp_path):
    binding.lib()
    rc, out = run_host(tmp_path, "tuner")
    assert rc == 0, out
