"""The benchmark's result line stays short whatever the other workloads record."""
import json

import bench


def test_result_line_is_short_and_details_go_to_stderr(capsys):
    extra = {f"workload{i}": {"per_layer": [dict(layer=j, us=1.0) for j in range(60)]} for i in range(20)}
    line = {"metric": "m", "value": 1.5, "config": {"workload": "w"}, "extra": extra, "oracle_samples": {"a": 1}}
    bench.emit(line)
    out, err = capsys.readouterr()
    assert json.loads(out) == {"metric": "m", "value": 1.5, "config": {"workload": "w"}} and out.count("\n") == 1
    detail = [l for l in err.splitlines() if l.startswith("[bench] detail ")]
    assert len(detail) == 1 and json.loads(detail[0].split(" ", 2)[2]) == {"extra": extra, "oracle_samples": {"a": 1}}
