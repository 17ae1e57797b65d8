"""Counter summary of the profiling helpers: times and counters are taken over a kernel's
dispatches of the largest grid, not over every launch that shares its name."""
import argparse
import csv
import sqlite3

from paper_2604_09993_amd import profiling

NAME = "void cis::k_tangent<double, cis::Topo<4, 3, 6, 1, false>, true>(int)"
SHORT = "k_tangent<double, Topo<4, 3, 6, 1, false>, true>"


def test_largest_grid_alone(tmp_path):
    (tmp_path / "kt").mkdir()
    db = sqlite3.connect(tmp_path / "kt" / "kt_results.db")
    db.execute("create table kernels (name, grid_x, grid_y, grid_z, duration)")
    db.executemany("insert into kernels values (?, ?, 1, 1, ?)",
                   [(NAME, 1000, 1000000), (NAME, 1000, 1200000), (NAME, 16, 50000)])
    db.commit()
    db.close()
    with open(tmp_path / "c.csv", "w", newline="") as fh:
        w = csv.writer(fh)
        w.writerow(["Dispatch_Id", "Kernel_Name", "Grid_Size", "Counter_Name", "Counter_Value"])
        for d, grid, v in ((1, 1000, 64e6), (2, 16, 1e6), (3, 1000, 66e6)):
            w.writerow([d, NAME, grid, "SQ_INSTS_VALU_FMA_F64", v])
    md = tmp_path / "out.md"
    profiling.valu_summary(argparse.Namespace(csv=[str(tmp_path / "c.csv")], note="",
                                              trace=str(tmp_path / "kt"), commands=[],
                                              cmd_trace="", md=str(md), title="t"))
    row = next(l for l in md.read_text().splitlines() if l.startswith(f"| `{SHORT}`"))
    cell = [x.strip() for x in row.split("|")]
    assert cell[2] == "1100.0" and float(cell[3]) == 64 * 2 * 65e6
    # the headline's algorithmic FLOPs over the headline's time
    algo = profiling.bench_algorithmic_flops()
    assert abs(float(cell[7]) - algo["k_tangent<double, Topo<4, 3"] / 1.1e-3 / 1e12) <= 0.005


def test_only_batches_that_run():
    """FP32 is timed on the quad13 batch alone: no work of the mixed batch by its name."""
    for table in (profiling.bench_algorithmic_flops(), profiling.bench_algorithmic_bytes()):
        assert [k for k in table if k.startswith("k_tangent<float")] == \
            ["k_tangent<float, Topo<4, 3"]
