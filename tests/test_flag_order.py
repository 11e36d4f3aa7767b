"""The least-squares stream of a Krylov cycle copies the convergence flags to
pinned host words, and the next cycle's start, on the caller's stream, changes
the flags and copies them to the same words.  Only the event that the caller's
stream waits for at the end of a cycle orders the two, so in the source of
both cycle forms the copy must be queued before that event is recorded."""
import os
import re

import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2111_11058_amd", "csrc", "solve.hip")


@pytest.mark.parametrize("name, post, record", [
    ("run_cycle", r"check\(side->ls\)", r"hipEventRecord\(side->ev_done\[par\], side->ls\)"),
    ("run_sstep_cycle", r"flags\.post\(gs\.active, q\)", r"hipEventRecord\(ss\.ev_read\[par\], q\)"),
])
def test_flags_are_copied_before_the_event(name, post, record):
    src = open(SRC).read()
    body = re.search(r"\nstatic \w+ %s\(.*?\n}\n" % name, src, re.S).group(0)
    last = body.rindex("hipStreamWaitEvent(s, ")  # the end of the cycle
    posts, records = ([m.start() for m in re.finditer(x, body[:last])] for x in (post, record))
    assert len(posts) == 1 and len(records) == 1
    assert posts[0] < records[0], "the copy of the flags is not covered by the event"
