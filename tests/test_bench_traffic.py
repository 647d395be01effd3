"""bench.py's lookup of measured HBM traffic: only a counter summary of the schedule that ran."""
import os

import pytest

import bench

HEAD = "# columns: kernel, launches, fetch MiB/launch, write MiB/launch, total bytes/launch\n"


def summary(tmp_path, rows):
    p = os.path.join(str(tmp_path), "t.txt")
    with open(p, "w") as f:
        f.write(HEAD + "".join("%s\t%d\t1.0\t1.0\t%d\n" % r for r in rows))
    return p


def test_summary_of_the_same_schedule(tmp_path):
    p = summary(tmp_path, [("a<1, 2>", 12, 1000), ("b", 4, 500)])
    assert bench.measured_traffic(p, {"a<1, 2>": 3, "b": 1}) == {"a<1, 2>": 1000.0, "b": 500.0}


@pytest.mark.parametrize("launches", [
    {"a<1, 2>": 1, "b": 1},             # one launch for what were three: same name, other traffic
    {"a<1, 2>": 3, "b": 1, "c": 1},     # a kernel that the summary does not know
    {"a<1, 2>": 3},                     # one that no longer runs
])
def test_summary_of_another_schedule(tmp_path, launches):
    p = summary(tmp_path, [("a<1, 2>", 12, 1000), ("b", 4, 500)])
    assert bench.measured_traffic(p, launches) == {}


def test_no_summary(tmp_path):
    assert bench.measured_traffic(os.path.join(str(tmp_path), "none.txt"), {"a": 1}) == {}
