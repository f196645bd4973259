"""Collect the rocprofv3 evidence behind one ``bench.py`` line and write the short text summary
that is kept under ``profiles/``.

    python -m paper_2202_05868_amd.rocprof_summary --workload c4 --out /tmp/prof_c4
    python -m paper_2202_05868_amd.rocprof_summary --case csr_graph --out /tmp/prof_csr

(the second form profiles a multiply of ``perf/cases.py``, run by this file itself with ``--run-case``.)

Runs, one after the other, each as its own process and under its own time limit:

  1. ``rocprofv3 --kernel-trace --stats``  on  ``python3 bench.py --workload W --timed-only``
  2. ``rocprofv3 --pmc FETCH_SIZE``        on the same command with ``--no-ramp --steps 5 --warmup 2 --calib-copy``
  3. ``rocprofv3 --pmc WRITE_SIZE``        likewise
  4. ``rocprofv3 --pmc SQ_BUSY_CU_CYCLES SQ_VALU_MFMA_BUSY_CYCLES SQ_WAVE_CYCLES SQ_LDS_BANK_CONFLICT``  likewise
  5. ``rocprofv3 --pmc TA_BUSY_avr SQ_BUSY_CU_CYCLES SQ_INSTS_VMEM_RD SQ_WAIT_ANY SQ_WAVE_CYCLES``  likewise

and writes ``<out>/summary.txt``.  The kernel trace holds every dispatch of the run: the launches
that let the clocks settle, the warm-up and the timed steps.  The summary therefore gives the
average over the dispatches of the TIMED steps (the last ``steps`` calls) beside the average over
all dispatches, and the ``ms_per_step`` the benchmark printed in that same run.  HBM bytes are the
counters scaled by what they read for a plain 256 MiB streaming kernel in the same process.
The process that collects never touches the GPU itself; the profiled program is the one named after ``--``.
"""
from __future__ import annotations

import argparse
import json
import os
import sqlite3
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
COPY_BYTES = 256 * 1024 * 1024
MULTIPLY = "(name like '%vbr_spmm%' or name like '%entry_rows%')"      # the kernels a multiply launches


def is_multiply(kernel: str) -> bool:
    return "vbr_spmm" in kernel or "entry_rows" in kernel


def short(kernel: str, n: int) -> str:
    return kernel[kernel.find("vbr_spmm" if "vbr_spmm" in kernel else "entry_rows"):][:n]


def run_case(args) -> int:
    """The profiled program of ``--case``: the multiply again and again, one JSON line with what the summary needs."""
    sys.path.insert(0, ROOT)
    os.chdir(ROOT)
    import torch
    from perf import cases
    case = next(c for c in cases.listed() if c["name"] == args.run_case)
    state = cases.prepare(case, 1)
    work = cases.work(case)
    ramp = 0 if args.no_ramp else 300
    for _ in range(ramp + args.warmup):
        cases.run(state)
    start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    start.record()
    for _ in range(args.steps):
        cases.run(state)
    end.record()
    torch.cuda.synchronize()
    ms = start.elapsed_time(end) / args.steps
    if args.calib_copy:
        x = torch.zeros(COPY_BYTES // 4, dtype=torch.float32, device="cuda:0")
        y = torch.empty_like(x)
        torch.neg(x, out=y)                # a kernel that making the inputs has not used
        torch.cuda.synchronize()
    kernels = state["M"].launches(case["n"]) if case["path"] == "multiply" else [dict(kernel="entry_rows_kernel")]
    print(json.dumps(dict(ms_per_step=ms, value=work["flops"] / ms * 1e-9, unit="TFLOP/s of entries", clock_ramp_launches=ramp,
                          roofline=dict(kernel=kernels, algorithmic_hbm_bytes=work["bytes"]))), flush=True)
    return 0


def run(cmd, log, limit):
    print("[rocprof_summary] " + " ".join(cmd), flush=True)
    env = dict(os.environ, TMPDIR="/tmp")
    with open(log, "w") as f:
        rc = subprocess.run(["timeout", "-s", "KILL", str(limit)] + cmd, cwd="/tmp", env=env, stdout=subprocess.PIPE,
                            stderr=f, text=True)
    if rc.returncode != 0:
        raise SystemExit("pass failed (%d): see %s" % (rc.returncode, log))
    lines = [ln for ln in rc.stdout.splitlines() if ln.startswith("{")]
    return json.loads(lines[-1]) if lines else None


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("--workload", default="c4")
    ap.add_argument("--clean", action="store_true")
    ap.add_argument("--dense", action="store_true", help="the dense product on the zero-filled matrix (bench.py --dense)")
    ap.add_argument("--case", help="a multiply of perf/cases.py instead of a workload of the benchmark")
    ap.add_argument("--run-case", help="run that multiply here (the profiled program)")
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--no-ramp", action="store_true")
    ap.add_argument("--calib-copy", action="store_true")
    ap.add_argument("--out")
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--no-counters", action="store_true", help="kernel trace only")
    args = ap.parse_args()
    if args.run_case:
        return run_case(args)
    if not args.out:
        ap.error("--out is needed")
    out_dir = os.path.abspath(args.out)
    os.makedirs(out_dir, exist_ok=True)
    bench = ["python3", os.path.join(ROOT, "bench.py"), "--workload", args.workload, "--timed-only"]
    flags = (" --clean" if args.clean else "") + (" --dense" if args.dense else "")
    bench += flags.split()
    shown = "python3 bench.py --workload %s --timed-only%s" % (args.workload, flags)
    what, how = "workload " + args.workload, "--workload %s%s" % (args.workload, flags)
    if args.case:
        bench = ["python3", os.path.abspath(__file__), "--run-case", args.case]
        shown = "python3 paper_2202_05868_amd/rocprof_summary.py --run-case " + args.case
        what, how = "case %s of perf/cases.py" % args.case, "--case " + args.case
    pmc_tail = ["--no-ramp", "--steps", "5", "--warmup", "2", "--calib-copy"]
    text = ["# rocprofv3 summary: vbr_spmm on %s%s (MI355X, gfx950)" % (
                what, (" (noise-free)" if args.clean else "") + (" stored zero-filled: the dense product" if args.dense else "")),
            "",
            "made by             : python -m paper_2202_05868_amd.rocprof_summary %s --out <out>" % how,
            "kernel trace command: cd /tmp && export TMPDIR=/tmp && rocprofv3 --kernel-trace --stats -d <out>/trace -o t -- %s --steps %d" % (shown, args.steps)]

    bj = run(["rocprofv3", "--kernel-trace", "--stats", "-d", os.path.join(out_dir, "trace"), "-o", "t", "--"] + bench +
             ["--steps", str(args.steps)], os.path.join(out_dir, "trace.err"), 400)
    con = sqlite3.connect(os.path.join(out_dir, "trace", "t_results.db"))
    rows = con.execute("select name, start, end from kernels where %s order by start" % MULTIPLY).fetchall()
    per_step = len(bj["roofline"]["kernel"])
    timed = rows[-args.steps * per_step:] if per_step else []
    text += ["", "## kernel trace: per kernel, dispatches / average us, over ALL dispatches of the run and over the",
             "## dispatches of the %d timed steps (the last %d dispatches)" % (args.steps, len(timed))]
    names = []
    for r in rows:
        if r[0] not in names:
            names.append(r[0])
    step_us = 0.0
    for nm in names:
        all_d = [(e - s) / 1e3 for k, s, e in rows if k == nm]
        tim_d = [(e - s) / 1e3 for k, s, e in timed if k == nm]
        text.append("  %-70s all %5d / %9.3f us    timed %4d / %9.3f us" % (
            short(nm, 70), len(all_d), sum(all_d) / len(all_d), len(tim_d), sum(tim_d) / max(1, len(tim_d))))
        step_us += sum(tim_d) / max(1, args.steps)
    text.append("  kernel time per timed step (sum over its launches): %.3f us" % step_us)
    if per_step > 1:
        spans = [max(e for _, _, e in timed[i:i + per_step]) - min(b for _, b, _ in timed[i:i + per_step])
                 for i in range(0, len(timed), per_step)]
        text.append("  the launches of one call follow each other: first start to last end of a timed step, average %.3f us" % (
            sum(spans) / len(spans) / 1e3))
    text.append(("the case" if args.case else "bench.py") + " in the same run: ms_per_step %.4f (HIP events around the %d timed steps), value %.1f %s, clock-ramp launches %d" % (
        bj["ms_per_step"], args.steps, bj["value"], bj["unit"], bj["clock_ramp_launches"]))
    text.append("(under the profiler every dispatch is followed by a completion signal, so the GPU idles between launches and")
    text.append(" its clocks settle lower than in an unprofiled run; compare with the ms_per_step of this run, not of another)")

    if not args.no_counters:
        res, spmm_sum = {}, {}
        for tag, sub in (("FETCH_SIZE", "fetch"), ("WRITE_SIZE", "write")):
            run(["rocprofv3", "--pmc", tag, "-d", os.path.join(out_dir, sub), "-o", "p", "--"] + bench + pmc_tail,
                os.path.join(out_dir, sub + ".err"), 180)
            con = sqlite3.connect(os.path.join(out_dir, sub, "p_results.db"))
            q = con.execute("select kernel_name, avg(value), count(*) from counters_collection where counter_name=? "
                            "group by kernel_name", (tag,)).fetchall()
            text += ["", "## %s (KiB per dispatch, average over dispatches): rocprofv3 --pmc %s -d <out>/%s -o p -- %s %s" % (
                tag, tag, sub, shown, " ".join(pmc_tail))]
            spmm_sum[tag] = 0.0
            for k, val, cnt in q:
                if is_multiply(k):
                    text.append("  %-70s %14.1f KiB (n=%d)" % (short(k, 70), val, cnt))
                    spmm_sum[tag] += val
                elif "neg_kernel" in k if args.case else "elementwise" in k and "Fill" not in k:
                    text.append("  %-70s %14.1f KiB (n=%d)" % ("256 MiB streaming kernel (torch.%s out=)" % ("neg" if args.case else "mul"), val, cnt))
                    res[tag] = val
        if "FETCH_SIZE" in res and "WRITE_SIZE" in res:
            sf = COPY_BYTES / (res["FETCH_SIZE"] * 1024)
            sw = COPY_BYTES / (res["WRITE_SIZE"] * 1024)
            fb = spmm_sum["FETCH_SIZE"] * 1024 * sf
            wb = spmm_sum["WRITE_SIZE"] * 1024 * sw
            text += ["", "calibration: the streaming kernel reads 256 MiB and writes 256 MiB -> scale factors %.4f (fetch), %.4f (write)" % (sf, sw),
                     "vbr_spmm FETCH_SIZE per call (all its launches): %.1f MB scaled" % (fb / 1e6),
                     "vbr_spmm WRITE_SIZE per call (all its launches): %.1f MB scaled" % (wb / 1e6),
                     "HBM traffic per launch: %.1f MB (algorithmic: %.1f MB)" % ((fb + wb) / 1e6, bj["roofline"]["algorithmic_hbm_bytes"] / 1e6)]
        ctrs = ["SQ_BUSY_CU_CYCLES", "SQ_VALU_MFMA_BUSY_CYCLES", "SQ_WAVE_CYCLES", "SQ_LDS_BANK_CONFLICT"]
        run(["rocprofv3", "--pmc"] + ctrs + ["-d", os.path.join(out_dir, "mfma"), "-o", "p", "--"] + bench + pmc_tail[:-1],
            os.path.join(out_dir, "mfma.err"), 180)
        con = sqlite3.connect(os.path.join(out_dir, "mfma", "p_results.db"))
        q = con.execute("select kernel_name, counter_name, avg(value), count(*) from counters_collection "
                        "where %s group by kernel_name, counter_name" % MULTIPLY.replace("name", "kernel_name")).fetchall()
        text += ["", "## matrix-unit and LDS counters (per dispatch, average): rocprofv3 --pmc %s -d <out>/mfma -o p -- %s %s" % (
            " ".join(ctrs), shown, " ".join(pmc_tail[:-1]))]
        per = {}
        for k, c, val, cnt in q:
            text.append("  %-60s %-28s %16.1f (n=%d)" % (short(k, 60), c, val, cnt))
            per.setdefault(k, {})[c] = val
        for k, cs in per.items():
            if cs.get("SQ_BUSY_CU_CYCLES"):
                text.append("  -> MFMA busy = SQ_VALU_MFMA_BUSY_CYCLES / (4 SIMDs x SQ_BUSY_CU_CYCLES) = %.1f %%  (%s)" % (
                    100.0 * cs.get("SQ_VALU_MFMA_BUSY_CYCLES", 0.0) / (4.0 * cs["SQ_BUSY_CU_CYCLES"]), short(k, 50)))
        # the load path: how busy the texture-address unit is (every direct-to-LDS load goes through it)
        ctrs = ["TA_BUSY_avr", "SQ_BUSY_CU_CYCLES", "SQ_INSTS_VMEM_RD", "SQ_WAIT_ANY", "SQ_WAVE_CYCLES"]
        run(["rocprofv3", "--pmc"] + ctrs + ["-d", os.path.join(out_dir, "ta"), "-o", "p", "--"] + bench + pmc_tail[:-1],
            os.path.join(out_dir, "ta.err"), 180)
        con = sqlite3.connect(os.path.join(out_dir, "ta", "p_results.db"))
        q = con.execute("select kernel_name, counter_name, avg(value), count(*) from counters_collection "
                        "where %s group by kernel_name, counter_name" % MULTIPLY.replace("name", "kernel_name")).fetchall()
        text += ["", "## load path (per dispatch, average): rocprofv3 --pmc %s -d <out>/ta -o p -- %s %s" % (
            " ".join(ctrs), shown, " ".join(pmc_tail[:-1]))]
        per = {}
        for k, c, val, cnt in q:
            text.append("  %-60s %-28s %16.1f (n=%d)" % (short(k, 60), c, val, cnt))
            per.setdefault(k, {})[c] = val
        for k, cs in per.items():
            if cs.get("SQ_BUSY_CU_CYCLES") and cs.get("SQ_INSTS_VMEM_RD"):
                per_cu = cs["SQ_BUSY_CU_CYCLES"] / 256.0
                text.append("  -> TA busy %.0f %% of the kernel's cycles (TA_BUSY_avr / (SQ_BUSY_CU_CYCLES / 256 CUs)); %.1f busy cycles and "
                            "%.1f kernel cycles per vector-memory load instruction and CU; waves waiting %.0f %% of their time  (%s)" % (
                                100.0 * cs.get("TA_BUSY_avr", 0.0) / per_cu, cs.get("TA_BUSY_avr", 0.0) * 256.0 / cs["SQ_INSTS_VMEM_RD"],
                                cs["SQ_BUSY_CU_CYCLES"] / cs["SQ_INSTS_VMEM_RD"],
                                100.0 * cs.get("SQ_WAIT_ANY", 0.0) / max(1.0, cs.get("SQ_WAVE_CYCLES", 1.0)), short(k, 50)))
    with open(os.path.join(out_dir, "summary.txt"), "w") as f:
        f.write("\n".join(text) + "\n")
    print("\n".join(text))
    return 0


if __name__ == "__main__":
    sys.exit(main())
