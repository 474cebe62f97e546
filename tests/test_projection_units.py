"""The unit of the projection's staging on the host: 16 bytes only where the volume is on 16."""

from host_build import run_host
from paper_2311_13177_amd import binding


def test_volumes_on_eight_bytes_take_the_narrow_units(tmp_path):
    binding.lib()
    rc, out = run_host(tmp_path, "project_units")
    assert rc == 0 and out.count("ok") == 16, out
