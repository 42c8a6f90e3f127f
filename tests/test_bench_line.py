"""CPU test of bench.py's result line."""
import json

import pytest

import bench


@pytest.mark.parametrize("legs", [0, 3, 40])
def test_the_line_stays_short(legs):
    """A full run's line once was longer than the end of the output that is kept of a run, and could not be read back."""
    out = {"metric": "m", "value": 1.5, "unit": "u", "ms_per_step": 2.0, "vs_baseline": None,
           "config": {"model": "x" * 500}, "restore": {"us_per_layer": 43.8}}
    out.update({f"leg{i}": {"rows": list(range(100 * (i + 1)))} for i in range(legs)})
    line, rest = bench.split_line(out)
    assert len(json.dumps(line)) <= bench.LINE_LIMIT < 16000
    assert {**line, **rest} == (out if not rest else {**out, "legs_on_stderr": list(rest)})
    assert bool(rest) == (legs == 40) and "restore" in line and "config" in line
