"""bench.py's output: stdout carries one JSON line short enough to be kept whole by whatever records it, however much the sections
hold; the sections are on stderr and, if asked for, in a file."""
import json

import bench


def test_one_short_line_on_stdout(capsys, tmp_path):
    line = dict(metric="m", value=1.0, unit="u", n_gpus=1, steps=20, warmup=5, ms_per_step=0.7, config=dict(workload="w"))
    sections = {f"section{i}": dict(rows=[dict(layer=j, us=1.0) for j in range(400)]) for i in range(10)}
    bench.report(line, sections, str(tmp_path / "details.json"))
    out, err = capsys.readouterr()
    assert out.count("\n") == 1 and len(out) < 4096
    assert json.loads(out) == line
    assert {r["section"]: r["data"] for r in map(json.loads, err.splitlines())} == sections
    assert json.load(open(tmp_path / "details.json")) == sections
