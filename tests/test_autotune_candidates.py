"""The autotuner's candidates are different launches: lines_mult, which only the
single cooperative launch uses, varies only there."""
from paper_2407_21552_amd import autotune


def test_grouped_candidates_differ_in_what_they_launch():
    seen = set()
    for c in autotune.CANDIDATES:
        key = (c["single_launch"], c["rows_per_item"], c["largest_first"],
               c["lines_mult"] if c["single_launch"] else None)
        assert key not in seen
        seen.add(key)
    assert {c["single_launch"] for c in autotune.CANDIDATES} == {0, 1}
    assert {c["lines_mult"] for c in autotune.CANDIDATES if c["single_launch"]} == {1, 2, 4}
