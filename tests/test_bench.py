"""What bench.py says about a launch is what the library launches."""

import pytest

import bench
from paper_2506_20252_amd import pat


@pytest.mark.parametrize("coll,n,count,dtype,env,walk", [
    ("rs", 64, 262144, "float32", None, 1), ("rs", 64, 15, "float32", None, 0), ("rs", 4097, 64, "float32", None, 0),
    ("rs", 64, 262144, "float32", "PAT_TREE_TILE", 0), ("ag", 64, 4096, "bfloat16", "PAT_STREAMING", 0),
    ("ag", 64, 4096, "bfloat16", None, 1),
])
def test_launches_are_the_librarys(coll, n, count, dtype, env, walk, monkeypatch):
    """Both sides of the walk's limits and of a step-kernel setting.  A walk is
    one launch; the schedule's are pat_plan_info's."""
    if env:
        monkeypatch.setenv(env, "1")
    info = bench.launch_info(coll, n, count, dtype)
    st, plan = pat.pat_plan_info(pat.PAT_REDUCESCATTER if coll == "rs" else pat.PAT_ALLGATHER, n, count, dtype)
    assert (info["walk"], info["launches"]) == (walk, 1 if walk else plan["launches_per_op"])


def test_nontemporal_is_the_launchs_own():
    """N = 1000, 256 B chunks: 256 MB of send buffers, read by a nontemporal
    walk, while the step schedule moves under 1e9 bytes and is cached."""
    st, plan = pat.pat_plan_info(pat.PAT_REDUCESCATTER, 1000, 64, "float32")
    assert bench.launch_info("rs", 1000, 64, "float32")["nontemporal"] == 1 and plan["streaming"] == 0
