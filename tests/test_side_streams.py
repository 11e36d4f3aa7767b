"""Streams of the solvers' least-squares steps: none is destroyed while an
event recorded on it is still to be waited for or destroyed (the runtime
aborts over such events).  Read from the source: only the pool of leases
destroys streams, events first, and in every solver the flags whose event is
recorded on a leased stream are declared after the lease, so that they are
destroyed before it."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2111_11058_amd", "csrc")


def _src(name):
    return open(os.path.join(CSRC, name)).read()


def test_only_the_pool_destroys_streams():
    solve = _src("solve.hip")
    body = re.search(r"void SideLease::give_back\(.*?\n}\n", solve, re.S).group(0)
    assert body.index("hipEventDestroy") < body.index("hipStreamDestroy")
    assert "hipStreamDestroy" not in _src("bgmres.hip")
    rest = solve.replace(body, "")
    # (run_cycle's own stream of a graph capture, which nothing else uses)
    assert [m for m in re.findall(r"hipStreamDestroy\((\w+)\)", rest) if m != "cs"] == []


def test_flags_end_before_their_streams():
    solve = _src("solve.hip")
    run = re.search(r"\nGmresResult gmres_run\(.*?\n}\n", solve, re.S).group(0)
    assert run.index("PinnedFlags flags") > run.index("ColumnSide side(")
    assert run.index("PinnedFlags flags") > run.index("unique_ptr<SStep> sst")
    block = _src("bgmres.hip")
    assert "SideLease lease_;" in block and re.search(r"void solve\(.*PinnedFlags flags\(1\)", block, re.S)
