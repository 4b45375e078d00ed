"""bench.py names the kernels that a 3D step launches, and its summaries keep them."""
import csv
import os
import re

import pytest

import bench
from test_march_rule import rule  # noqa: F401  (the library's rule, built on the CPU)

CSRC = os.path.join(bench.ROOT, "paper_2003_09145_amd", "csrc")


@pytest.mark.parametrize("n", [(256, 256, 256), (252, 252, 252), (512, 256, 128), (300, 200, 100),
                               (260, 140, 300)])
def test_sweep_kernels_follow_the_dispatch(rule, n):  # noqa: F811
    y, z = rule(*n)[:2]
    names = [[k for k, _ in bench.sweep_kernels(n, d)] for d in range(3)]
    assert all(sum(c for _, c in bench.sweep_kernels(n, d)) == 3 for d in range(3))
    assert names[0] == ["k_sweep<3,0,4,false>"]
    assert names[1] == (["k_march<3,1,false,0>"] if y else ["k_sweep<3,1,4,false>"])
    assert names[2] == (["k_march<3,2,false,1>", "k_march<3,2,false,2>"] if z else ["k_sweep<3,2,8,false>"])


def test_sources_hold_every_header_of_the_sweeps():
    seen, todo = set(), ["teno_kernels.hip", "teno_march.hip"]
    while todo:
        f = todo.pop()
        seen.add(f)
        for inc in re.findall(r'#include "(teno_\w+\.hpp)"', open(os.path.join(CSRC, f)).read()):
            todo += [inc] if inc not in seen else []
    have = {os.path.basename(p) for p in bench.SWEEP_SOURCES}
    assert seen <= have, seen - have


def _write(path, rows):
    os.makedirs(os.path.dirname(path), exist_ok=True)
    with open(path, "w", newline="") as f:
        w = csv.writer(f)
        w.writerow(["Dispatch_Id", "Kernel_Name", "Counter_Name", "Counter_Value",
                    "Start_Timestamp", "End_Timestamp"])
        w.writerows(rows)


def test_march_summaries(tmp_path, monkeypatch):
    for name in ("TRAFFIC_FILE", "CLOCK_FILE", "MARCH_TRAFFIC_FILE", "MARCH_CLOCK_FILE"):
        monkeypatch.setattr(bench, name, str(tmp_path / (name + ".txt")))
    k = "void teno::k_march<3, 2, false, %d>(teno::MarchArgs)"
    copy = "void at::native::vectorized_elementwise_kernel<4, copy>(int)"
    ncell = 256 ** 3
    alg = {1: 8 * 5 * ncell * 3, 2: 8 * 5 * ncell * 4}
    kib = 1024.0
    for cal, c in (("calf", "FETCH_SIZE"), ("calw", "WRITE_SIZE")):
        _write(str(tmp_path / cal / "c_counter_collection.csv"),
               [[0, copy, c, bench.COPY_BYTES / kib, 0, 1]])
    # stage 1 moves 1.1 of its algorithmic bytes, the later ones 1.2
    _write(str(tmp_path / "fetch" / "f_counter_collection.csv"),
           [[m, k % m, "FETCH_SIZE", 0.7 * alg[m] / kib, 0, 1] for m in (1, 2)])
    _write(str(tmp_path / "write" / "w_counter_collection.csv"),
           [[m, k % m, "WRITE_SIZE", (0.4 if m == 1 else 0.5) * alg[m] / kib, 0, 1] for m in (1, 2)])
    _write(str(tmp_path / "valu" / "v_counter_collection.csv"),
           [[m, k % m, "SQ_INSTS_VALU_FMA_F64", 100.0 * m, 0, 1] for m in (1, 2)])
    bench.summarize_counters(str(tmp_path))
    _write(str(tmp_path / "grbm" / "g_counter_collection.csv"),
           [[m, k % m, "GRBM_GUI_ACTIVE", 8 * 1e6 * (2.0 + 0.1 * m), 0, 1_000_000] for m in (1, 2)])
    bench.summarize_clock(str(tmp_path))
    assert not os.path.exists(bench.TRAFFIC_FILE) and not os.path.exists(bench.CLOCK_FILE)
    text = open(bench.MARCH_TRAFFIC_FILE).read()
    assert "ratio=1.100" in text and "ratio=1.200" in text
    z = bench.sweep_kernels([256] * 3, 2)
    assert bench.mean_over(bench.load_traffic, z) == pytest.approx((1.1 * alg[1] + 2 * 1.2 * alg[2]) / 3, rel=1e-6)
    assert bench.mean_over(bench.load_executed_flop, z) == pytest.approx(128 * (100 + 2 * 200) / 3)
    assert bench.mean_over(bench.load_clock_ghz, z) == pytest.approx((2.1 + 2 * 2.2) / 3, abs=1e-3)
    # of other sources, or without one of the kernels: none
    assert bench.mean_over(bench.load_traffic, z + [("k_march<3,1,false,0>", 3)]) is None
    open(bench.MARCH_TRAFFIC_FILE, "w").write(text.replace(bench.sources_sha(), "0" * 16))
    assert bench.mean_over(bench.load_traffic, z) is None


def test_sweep_names_resolve_in_the_committed_summaries():
    for path, prefix in ((bench.MARCH_TRAFFIC_FILE, "kernel "), (bench.MARCH_CLOCK_FILE, "clock ")):
        names = [line[len(prefix):].split(":", 1)[0].strip()
                 for line in open(path) if line.startswith(prefix)]
        for d in range(3):
            for k, _ in bench.sweep_kernels([256] * 3, d):
                assert len(bench.match_kernel(names, k)) == 1, (path, k, names)
