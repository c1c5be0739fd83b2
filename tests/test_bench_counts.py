"""The bench's account of a profiled run: bytes and launches per step from the
counters of the whole run."""
from __future__ import annotations

import csv
import json

import pytest

import bench


@pytest.mark.parametrize("pipelines", [1, 2, 3])
def test_traffic_summary_divides_by_the_steps_of_the_run(tmp_path, monkeypatch, pipelines):
    steps, warmup = 5, 2
    # the run, counted as main() issues it
    regions = [warmup, 1, steps, steps]
    ran, built = sum(regions), sum(regions) + pipelines
    if pipelines > 1:
        ran, built = ran + 5 + steps, built + 5 + steps + 1
    launches = {"k_conv_lds<x>": 7 * ran, "k_insert_points": built, "k_clear_tables": built}
    for d, counter in (("fetch", "FETCH_SIZE"), ("write", "WRITE_SIZE")):
        for name, rows in ((d, launches), ("copy" + d, {"copy": 3})):
            (tmp_path / name).mkdir()
            with open(tmp_path / name / "x_counter_collection.csv", "w", newline="") as fh:
                w = csv.writer(fh)
                w.writerow(["Kernel_Name", "Counter_Name", "Counter_Value"])
                for kernel, count in rows.items():
                    w.writerows([[kernel, counter, 1024.0 if kernel == "copy" else 10.0]] * count)
    (tmp_path / "fetch" / "source_hash.txt").write_text("hash")
    monkeypatch.setattr(bench, "TRAFFIC_FILE", str(tmp_path / "traffic.json"))
    bench.summarize_pmc(*(str(tmp_path / d) for d in ("fetch", "write", "copyfetch", "copywrite")), 1, steps, warmup, "key",
                        pipelines)
    fams = json.load(open(tmp_path / "traffic.json"))["key"]["families"]
    for fam, n in (("conv", 7), ("insert", 1), ("fill", 1)):
        assert fams[fam]["dispatches_per_step"] == pytest.approx(n)
        assert fams[fam]["fetch_bytes_per_step"] == pytest.approx(10.0 * 1024 * n)   # a unit is 1 MiB / 1024
        assert fams[fam]["write_bytes_per_step"] == pytest.approx(10.0 * 1024 * n)
