"""CPU test of the benchmark's record of counter measurements: their entries per launch go with them."""
import json

import bench


def test_stored_traffic_is_scaled_to_the_launches_it_stands_beside(tmp_path, monkeypatch):
    monkeypatch.setattr(bench, "traffic_path", lambda workload: str(tmp_path / f"{workload}.json"))
    rec = {"source_sha256": bench.kernel_source_hash(), "entries_per_launch": 8, "kernels": {"a": {"bytes_per_launch": 800.0}}}
    (tmp_path / "w.json").write_text(json.dumps(rec))
    none = {"traffic": None, "traffic_entries": None}
    assert bench.stored_traffic("a", "w", 4) == {"traffic": 400.0, "traffic_entries": 8}
    assert bench.stored_traffic("a", "w") == {"traffic": 800.0, "traffic_entries": 8}
    assert bench.stored_traffic("b", "w", 4) == none and bench.stored_traffic("a", "other", 4) == none
    (tmp_path / "w.json").write_text(json.dumps(dict(rec, source_sha256="0")))
    assert bench.stored_traffic("a", "w", 4) == none
    assert bench.entries_per_launch(16) == (2, 8) and bench.entries_per_launch(15) == (1, 15)
