"""bench.py's result line."""
import json

import bench


def test_the_result_line_is_short_and_whole():
    """Whoever reads a log has the last few thousand bytes of it: the other runs' reports, of any length, go elsewhere."""
    out = {"metric": "m", "value": 1.5, "config": {"model": "x"}, "memory_bytes": {"workspace": 1, "measured": {"rows": ["r" * 100] * 100}},
           "cpu_baseline": {"value": 2.0}}
    out.update({k: [{"row": "v" * 100}] * 100 for k in bench.DETAILS})
    line, details = bench.report_lines(out)
    assert len(line) < 500 and json.loads(line) == {"metric": "m", "value": 1.5, "config": {"model": "x"}, "memory_bytes": {"workspace": 1},
                                                    "cpu_baseline": {"value": 2.0}}
    kept = json.loads(details)
    assert all(kept[k] == out[k] for k in bench.DETAILS) and kept["memory_measured"] == out["memory_bytes"]["measured"]
    assert bench.report_lines({"metric": "m"}) == ('{"metric": "m"}', None)
