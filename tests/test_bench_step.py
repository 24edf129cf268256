"""bench.py's timed step makes the calls a program makes, whole (their y and z
passes are not those of the phase calls), and nothing besides."""
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
pytest.importorskip("torch")
import bench  # noqa: E402


class Recorder:
    def __init__(self):
        self.calls = []

    def __getattr__(self, name):
        return lambda *a, **k: self.calls.append(name)


class Buffers:
    desc = bmin = bmax = pdms = dist = None


def test_step_makes_whole_calls():
    pdm, marks = Recorder(), []

    def event():
        marks.append(len(pdm.calls))
        return len(marks) - 1

    e, tf = bench.tube_tree_step(pdm, Buffers(), None, None, 64, ["a", "b"], None, None, None, event)
    per_tf = ["tf_update", "full_recompute", "full_recompute_cached"]
    assert pdm.calls == ["build_bricks", "build_partitions"] + per_tf * 2
    # every call stands alone between two events
    assert [marks[i] for i in e] == [0, 1, 2]
    assert [[marks[i] for i in f] for f in tf] == [[2, 3, 4, 5], [5, 6, 7, 8]]
