"""Host-side tests of the profile summaries on synthetic profiler output: passes that run small steps several
to a launch, blocks among the step launches, and the program runs that bench.py ends with."""
import csv
import json
from argparse import Namespace

from paper_2103_11595_amd import profsum

PER = [{"kernel": "fma", "kS": 2, "kN": 2, "L": 4, "steps": 1, "bytes": 100.0, "flops": 10.0, "us": 4.0},
       {"kernel": "fma", "kS": 2, "kN": 2, "L": 4, "steps": 1, "bytes": 100.0, "flops": 10.0, "us": 4.0},
       {"kernel": "block", "kS": 5, "kN": 6, "L": 13, "steps": 2, "bytes": 100.0, "flops": 4000.0, "us": 20.0},
       {"kernel": "chain", "kS": 5, "kN": 5, "L": 12, "steps": 2, "bytes": 100.0, "flops": 4000.0, "us": 30.0}]
STEPS = ["void jf::k_absorb<float>(jf::StepDesc const*)", "void jf::k_absorb<float>(jf::StepDesc const*)",
         "void jf::k_block<float, 16>(jf::BlockDesc const*)", "void jf::k_chain<256>(jf::ChainDesc const*)"]


def _log(tmp_path, kernel="k_block<float>"):
    line = {"value": 1.0, "unit": "u", "ms_per_step": 1.0, "dtype": "c64", "config": {"workload": "w"},
            "roofline": {"kernel": kernel, "avg_launch_us": 20.0, "pass": {
                "launches": 4, "algorithmic_bytes_per_pass": 400.0, "avg_launch_us": 14.5, "kernel_ms_per_pass": 0.058}},
            "per_launch": PER}
    (tmp_path / "b.log").write_text(json.dumps(line) + "\n")
    return str(tmp_path / "b.log")


def test_a_trace_summary_counts_the_launches_of_a_pass(tmp_path):
    # passes: one launch for the two small steps, the block, the chain, the sum; then the program runs with a
    # launch for every step, which are no passes
    one_pass = [("jf::k_grid(jf::GridArgs)", 5), (STEPS[2], 20), (STEPS[3], 30), ("jf::k_sumsq_one(double2)", 2)]
    one_run = list(zip(STEPS, (4, 4, 20, 30))) + [("jf::k_sumsq_one(double2)", 2), ("jf::k_assemble(jf::AssembleArgs)", 1)]
    with open(tmp_path / "bench_kernel_trace.csv", "w", newline="") as f:
        w = csv.writer(f)
        w.writerow(["Kernel_Name", "Start_Timestamp", "End_Timestamp"])
        t = 0
        for name, us in [("void jf::k_absorb_mfma<tune>(jf::StepDesc const*)", 9)] * 3 + one_pass * 5 + one_run * 3:
            w.writerow([name, t, t + 1000 * us])
            t += 1000 * us + 500
    out = tmp_path / "t.md"
    profsum.trace(Namespace(dir=str(tmp_path), log=_log(tmp_path), passes=4, out=str(out), title="t", command="c",
                            live_log=None, live_command="x"))
    text = out.read_text()
    assert "Last 4 passes of the trace, 4 launches each" in text
    for row in ("| `k_grid` | 4 | 5.0 |", "| `k_block<float, 16>` | 4 | 20.0 |", "| `k_chain<256>` | 4 | 30.0 |"):
        assert row in text
    assert "k_absorb" not in text and "0.057 ms" in text
    assert "(`roofline.kernel` = `k_block<float>`): 1 launches per run, average **20.0 us**" in text


def test_counters_of_blocks_join_their_launches(tmp_path):
    with open(tmp_path / "bench_counter_collection.csv", "w", newline="") as f:
        w = csv.writer(f)
        w.writerow(["Dispatch_Id", "Kernel_Name", "Counter_Name", "Counter_Value"])
        names = ["void jf::k_absorb_mfma<tune>(...)", "jf::k_grid(jf::GridArgs)"] + STEPS
        for i, (k, util, mops) in enumerate(zip(names, (50, 9, 0, 0, 40, 60), (7, 7, 0, 0, 5, 6))):
            w.writerow([i + 1, k, "MfmaUtil", float(util)])
            w.writerow([i + 1, k, "SQ_INSTS_VALU_MFMA_MOPS_F32", float(mops)])
    profsum.mfma(Namespace(dir=str(tmp_path), log=_log(tmp_path), live_log=None, out=str(tmp_path / "m.md"),
                           json=str(tmp_path / "m.json"), title="t", command="c"))
    rec = json.loads((tmp_path / "m.json").read_text())
    assert rec["by_kernel"]["block"]["mfma_busy_pct_time_weighted"] == 40.0
    assert rec["by_kernel"]["chain"]["mfma_busy_pct_time_weighted"] == 60.0
    assert rec["by_kernel"]["fma"]["mfma_busy_pct_time_weighted"] == 0.0
