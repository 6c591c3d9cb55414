"""Host logic of the traffic summary for the whole count (CPU): all count-mode
kernels per call, scaled by the calibration copy; other modes' kernels and
runs that mix graphs are kept out."""
import json

import pytest

import importlib.util
import os

_spec = importlib.util.spec_from_file_location(
    "rocprof_summary", os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1907_09575_amd",
                                    "rocprof_summary.py"))
rs = importlib.util.module_from_spec(_spec)
_spec.loader.exec_module(rs)

NAMES = ["void tc::(anonymous namespace)::k_count_bits<0, 8>(tc::CountArgs)", "void tc::(anonymous namespace)::k_count_packs<0, 0>(x)",
         "void tc::(anonymous namespace)::k_count_packs16<0, 7, 4>(x)"]


def write(path, counter, copy_kib, rows):
    with open(path, "w") as f:
        f.write("Kernel_Name,Grid_Size,Counter_Name,Counter_Value\n")
        f.write('"copyBuffer",1024,%s,%f\n' % (counter, copy_kib))
        for name, grid, val in rows:
            f.write('"%s",%d,%s,%f\n' % (name, grid, counter, val))


def run(tmp_path, rows):
    # the copy reads half of what it moves in FETCH_SIZE, all of it in WRITE_SIZE
    write(tmp_path / "f.csv", "FETCH_SIZE", (1 << 20) / 2, rows)
    write(tmp_path / "w.csv", "WRITE_SIZE", 1 << 20, [(k, g, 1.0) for k, g, _ in rows])
    bench = {"config": {"workload": "x", "seed": 1}, "roofline": {"kernel": "count", "algorithmic_bytes_per_launch": 5}}
    (tmp_path / "b.json").write_text(json.dumps(bench))
    return rs.traffic(str(tmp_path / "f.csv"), str(tmp_path / "w.csv"), str(tmp_path / "b.json"), "count",
                      str(tmp_path / "o.json"))


def test_sum_over_the_kernels_of_a_call(tmp_path):
    rows = [(n, 64 * (i + 1), 100.0 * (i + 1)) for i, n in enumerate(NAMES)] * 3
    rows += [("void tc::(anonymous namespace)::k_count_bits<1, 5>(x)", 64, 1e9)]  # support: not the count's
    res = run(tmp_path, rows)
    assert res["fetch_kib_per_launch"] == 600.0 and res["write_kib_per_launch"] == 3.0
    assert res["fabric_bytes_per_launch"] == 1024 * (600 * 2 + 3)
    assert res["algorithmic_bytes_per_launch"] == 5


def test_two_graphs_are_refused(tmp_path):
    with pytest.raises(AssertionError):
        run(tmp_path, [(NAMES[0], 64, 1.0)] * 2 + [(NAMES[0], 128, 1.0)])
