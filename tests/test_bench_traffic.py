"""The benchmark's committed traffic counters count only for the sources and the workload they were taken on."""
import hashlib
import os

import bench


def test_counters_of_other_sources_are_left_out(tmp_path, monkeypatch):
    srcs = []
    for name in ("dst_runs.hip", "dst_stage.hip", "dst_forms.hip"):
        srcs.append(str(tmp_path / name))
        (tmp_path / name).write_text(name)
    profile = tmp_path / "traffic.md"
    kernel = "k_unbin_staged<double, true, true>"

    def write():
        shas = ", ".join(f"{os.path.basename(f)} sha256 {hashlib.sha256(open(f, 'rb').read()).hexdigest()}" for f in srcs)
        profile.write_text(f"Kernel sources: {shas}\n\n| `{kernel}` | 298 | 408743 | 2663.97 | 8.4e+08 |\n")

    monkeypatch.setattr(bench, "TRAFFIC_PROFILE", str(profile))
    monkeypatch.setattr(bench, "ITERATION_SRC", srcs)
    assert bench.measured_traffic(kernel, 1) is None  # no summary
    write()
    assert bench.measured_traffic(kernel, 1) == 8.4e8 and bench.measured_traffic(kernel, 2) == 8.4e8
    assert bench.measured_traffic(kernel, 0) is None and bench.measured_traffic("k_other", 1) is None
    for f in srcs:
        write()
        open(f, "a").write("changed")
        assert bench.measured_traffic(kernel, 1) is None, f


def test_the_sources_are_there():
    assert all(os.path.exists(f) for f in bench.ITERATION_SRC)
    assert {os.path.basename(f) for f in bench.ITERATION_SRC} >= {"dst_runs.hip", "dst_stage.hip"}
