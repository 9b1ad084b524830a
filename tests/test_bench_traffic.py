"""The byte record of bench.py (no GPU): runs are counted by the passes' own kernels, launches of other ops are left
out, and collections whose runs cannot be counted are refused."""
import json
import types

import pytest

from test_bench_host import _bench

HDR = "Kernel_Name,Counter_Name,Counter_Value\n"
ROOT_PASS, SUB_PASS = "void ot::k_block<float, {m}, 6, true>(x)", "void ot::k_block<float, {m}, 6, false>(x)"
RANGES, OTHER = "void ot::k_node_ranges<float, 6, {m}, true>(x)", "void ot::k_block<float, 0, 4, true>(x)"


def _csv(path, counter, kernels, copy):
    path.write_text(HDR + "".join(f'"{k}",{counter},{v}\n' for k, v in kernels) + f"copyBuffer,{counter},{copy}\n")


@pytest.mark.parametrize("mode,m", [("fixed", 1), ("atomic", 0)])
def test_runs_of_several_dispatches(tmp_path, monkeypatch, mode, m):
    b = _bench()
    out = tmp_path / "traffic.json"
    monkeypatch.setattr(b, "PROFILE_TRAFFIC", str(out))
    run = [(ROOT_PASS.format(m=m), 1000), (SUB_PASS.format(m=m), 10), (RANGES.format(m=m), 100)]
    _csv(tmp_path / "f.csv", "FETCH_SIZE", run * 3 + [(OTHER, 5000)], 524288)
    _csv(tmp_path / "w.csv", "WRITE_SIZE", run * 2 + [(OTHER, 5000)], 1048576)
    args = types.SimpleNamespace(config=2, dtype="f32", mode=mode)
    b.write_traffic(args, str(tmp_path / "f.csv"), str(tmp_path / "w.csv"))
    rec = json.loads(out.read_text())
    assert rec["kernel"] == "k_block + k_node_ranges"
    assert rec["bytes_per_launch"] == 1110 * 1024 * 2 + 1110 * 1024
    out.unlink()
    _csv(tmp_path / "f.csv", "FETCH_SIZE", run * 3 + run[:1], 524288)   # another plan's runs among them
    with pytest.raises(SystemExit):
        b.write_traffic(args, str(tmp_path / "f.csv"), str(tmp_path / "w.csv"))
    assert not out.exists()
