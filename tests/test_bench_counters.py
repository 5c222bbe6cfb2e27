"""The bench's counter summaries take the variant that the steps run: the tuner
launches the other variants of the same form, a few times each."""
import json
import os
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402


def _write(d, rows):
    os.makedirs(d, exist_ok=True)
    with open(os.path.join(d, "run_counter_collection.csv"), "w") as f:
        f.write("Kernel_Name,Counter_Name,Counter_Value\n")
        for k, c, v in rows:
            f.write(f'"{k}",{c},{v}\n')


@pytest.mark.parametrize("other", ["void mdk::k_force_brick<false, 2, 4, false, 2, false>(int)",
                                   "void mdk::k_force_brick<false, 2, 2, true, 2, false>(int)"])
def test_tuner_launches_are_left_out(tmp_path, monkeypatch, other):
    kept = "void mdk::k_force_brick<false, 2, 2, false, 2, false>(int)"
    t = str(tmp_path)
    _write(t + "/f", [(other, "FETCH_SIZE", 900.0)] * 2 + [(kept, "FETCH_SIZE", 100.0)] * 5)
    _write(t + "/w", [(kept, "WRITE_SIZE", 10.0)] * 5 + [(other, "WRITE_SIZE", 900.0)] * 2)
    _write(t + "/cf", [("copyBuffer", "FETCH_SIZE", 524288.0)])
    _write(t + "/cw", [("copyBuffer", "WRITE_SIZE", 1048576.0)])
    out = tmp_path / "c.json"
    monkeypatch.setattr(bench, "COUNTERS_JSON", str(out))
    bench.counters_summary(type("A", (), dict(
        fetch_dir=t + "/f", write_dir=t + "/w", copy_fetch_dir=t + "/cf", copy_write_dir=t + "/cw",
        large_fetch_dir=None, large_write_dir=None, commands=""))())
    assert json.loads(out.read_text())["forms"] == {
        "fp64": {"fetch_kib": 100.0, "write_kib": 10.0, "dispatches": 5}}
