"""bench.py prints one JSON line that a reader of the last 8 kB of its output gets whole."""
import json

import bench


def test_one_short_line(tmp_path, capsys):
    out = {"metric": bench.METRIC, "value": 1.0, "unit": "DOF/s", "mixed": {"fgmres_iterations": list(range(20))}}
    detail = {"newton_iterations": [{"index": i, "solve_ms": 1.0 / 3.0} for i in range(5000)]}
    path = tmp_path / "record.json"
    bench.emit(out, detail, str(path))
    text = capsys.readouterr().out
    assert text.count("\n") == 1 and len(text) < 8000
    assert json.loads(text) == out
    assert json.loads(path.read_text()) == {**out, "detail": detail}
    bench.emit(out, detail, "")
    assert json.loads(capsys.readouterr().out) == out
