"""The counter summary of the finest-level kernels when two levels' launches
share a grid: only the finest level's dispatches count."""
import csv
import json

import bench


def _rows(path, counter, copy, values):
    with open(path, "w", newline="") as fh:
        w = csv.DictWriter(fh, ["Dispatch_Id", "Kernel_Name", "Grid_Size", "Counter_Name", "Counter_Value"])
        w.writeheader()
        for i, (name, v) in enumerate([("__amd_rocclr_copyBuffer", copy)] * 3 +
                                      [("void ebmg::k_rb<float, 3>(args)", v) for v in values]):
            w.writerow({"Dispatch_Id": i, "Kernel_Name": name, "Grid_Size": 1024, "Counter_Name": counter,
                        "Counter_Value": v})


def test_levels_that_share_a_grid(tmp_path, monkeypatch):
    kib = (1 << 29) / 1024.0
    _rows(tmp_path / "f.csv", "FETCH_SIZE", kib / 2, [1000.0, 1010.0, 125.0, 130.0, 990.0])
    _rows(tmp_path / "w.csv", "WRITE_SIZE", kib, [500.0, 500.0, 62.5, 62.5, 500.0])
    monkeypatch.setattr(bench, "TRAFFIC_FILE", str(tmp_path / "out.json"))
    assert bench.pmc_summary(str(tmp_path / "f.csv"), str(tmp_path / "w.csv"), "none") == 0
    k = json.load(open(tmp_path / "out.json"))["kernels"]["k_rb<float,3>"]
    assert k["dispatches"] == 3
    assert abs(k["hbm_bytes_per_launch"] - (1000.0 * 2 + 500.0) * 1024) < 1e-6 * 2500 * 1024
