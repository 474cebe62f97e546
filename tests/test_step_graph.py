"""When a fit captures its larger graph, on the host: never ahead of the first steps, and only
where the call or the fit so far is long enough to repay it.
"""

from host_build import run_host


def test_captures_follow_the_rule(tmp_path):
    rc, out = run_host(tmp_path, "step_graph")
    assert rc == 0 and out.strip().endswith(" 0 bad"), out
