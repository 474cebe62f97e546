"""Workspaces that a plan keeps for its operator calls, on the host: which calls allocate and how
much stays, with stand-in memory, stream and event functions.
"""

import pytest

from host_build import run_host
from paper_2311_13177_amd import binding


@pytest.mark.parametrize("what", ["sizes", "own", "streams"])
def test_kept_workspaces(tmp_path, what):
    binding.lib()
    rc, out = run_host(tmp_path, "workspaces", what)
    assert rc == 0 and out.strip() == "0 bad", out
