"""The tile shape of a batch on the host: a shape asked for stays, a plan's own follows the group."""

from host_build import run_host
from paper_2311_13177_amd import binding


def test_asked_shapes_stay(tmp_path):
    binding.lib()
    rc, out = run_host(tmp_path, "group_shape")
    assert rc == 0, out
