"""rocprofv3 summaries of the library's kernels, and reading them back.

The roofline figures of ``bench.py`` compare a kernel's algorithmic bytes per
launch with its launch time; the HBM bytes it really moves come from two
rocprofv3 counter runs (FETCH_SIZE, then WRITE_SIZE, KiB per dispatch), each
scaled by what the same counter reads for a 1 GiB device-to-device copy of
known size.  This module turns the CSV output of those runs (and of a
``--kernel-trace --stats`` run, and optionally of an SQ instruction-counter
run) into a short markdown summary under ``profiles/``, with machine-readable
lines that ``bench.py`` reads:

    kernel_source_sha256: <hash of the kernel and launch-plan sources>
    traffic_bytes_per_launch: <calibrated HBM bytes per dispatch>
    steps_per_launch: <time steps one dispatch advances>
    avg_launch_ns: <mean dispatch duration in the counter runs>

A summary is used only while its hash matches the current sources (comments
and blank lines do not count), so a kernel edit invalidates it.

    python -m paper_1810_07642_amd.profiling step --storage fp64 \\
        --fetch DIR --write DIR [--sq DIR] --out profiles/step_fp64_dewetting4096_traffic.md
    python -m paper_1810_07642_amd.profiling adjoint --fetch DIR --write DIR [--sq DIR] --out ...
    python -m paper_1810_07642_amd.profiling trace --trace DIR --out ... --command "..."
"""
import argparse
import csv
import glob
import hashlib
import os
import re
import statistics

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")

# Sources a kernel's traffic depends on: the kernel and the launch plan that
# sets its tiles (hence its halo re-reads).
STEP_SOURCES = [os.path.join(CSRC, f) for f in ("step.h", "step_form.hip", "march.h", "march_form.hip",
                                                  "march.hip", "fwd.hip", "device.h", "api.hip")]
ADJ_SOURCES = [os.path.join(CSRC, f) for f in ("adj.h", "adj.hip", "device.h", "api.hip")]

N4096 = 4096 * 4096
# Algorithmic bytes per site of one pass: the three moments (FP64, FP32: a pass
# between two others) or the record (FP16S) read and written once, plus the kappa
# field read once.
STEP_BYTES = {"fp64": (32, 24), "fp32": (16, 12), "fp16s": (24, 20)}  # (read, write) per site
# The kernel the benchmark workload (tau = 1, 4096^2, g = 0) runs per form and the
# steps one launch of it advances: three steps from moments to moments in FP64
# and FP32, two in FP16S.
STEP_KERNEL = {"fp64": ("march_kernel<0, 1, false, 3, true, true, true, 3, 3>", 3),
               "fp32": ("march_kernel<1, 1, false, 3, true, true, true, 3, 6>", 3),
               "fp16s": ("step_kernel<2, 1, false, 2, true, true>", 2)}
PROFILE_STEPS = 26  # a first pass of two steps and eight of three; thirteen of two (FP16S)
# The two-step reverse pass of the benchmark workload (tau = 1: the adjoint
# between steps as three fields per site), FP32: fields 12 + two captures 24 +
# kappa 4 + g_kappa 8 read; fields 12 + g_kappa 8 written.  (The general pass
# moves nine adjoint populations: 72 read, 44 written.)
ADJ_BYTES = (48, 20)
ADJ_KERNEL = "adj_step2_kernel<float, true, true, true>"
CALIB_BYTES = 1 << 30  # the 1 GiB calibration copy
CLOCK_GHZ = 2.4
SIMDS = 256 * 4


def source_hash(paths):
    """Hash of the given sources with comments and blank lines removed."""
    h = hashlib.sha256()
    for p in paths:
        text = open(p).read()
        text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
        for line in text.splitlines():
            code = line.split("//", 1)[0].rstrip()
            if code:
                h.update(code.encode() + b"\n")
    return h.hexdigest()[:16]


def read_summary(path, sources):
    """(traffic bytes per launch, steps per launch, avg launch ns) from a
    committed summary taken on the current sources, else None."""
    if not os.path.exists(path):
        return None
    text = open(path).read()
    m_hash = re.search(r"kernel_source_sha256:\s*([0-9a-f]+)", text)
    m_val = re.search(r"traffic_bytes_per_launch:\s*([0-9.eE+]+)", text)
    m_steps = re.search(r"steps_per_launch:\s*([0-9]+)", text)
    m_ns = re.search(r"avg_launch_ns:\s*([0-9.eE+]+)", text)
    if not m_hash or not m_val or m_hash.group(1) != source_hash(sources):
        return None
    return (float(m_val.group(1)), int(m_steps.group(1)) if m_steps else 1,
            float(m_ns.group(1)) if m_ns else None)


# ---- rocprofv3 CSV ---------------------------------------------------------------

def _find(dirpath, suffix):
    hits = sorted(glob.glob(os.path.join(dirpath, "**", f"*{suffix}"), recursive=True))
    if not hits:
        raise FileNotFoundError(f"no *{suffix} under {dirpath}")
    return hits


def _rows(path):
    with open(path, newline="") as fh:
        return list(csv.DictReader(fh))


def counters(dirpath):
    """{(kernel name, grid size): {counter: [value per dispatch]}} from a
    --pmc run (values of one dispatch summed over the counter's instances)."""
    out = {}
    for path in _find(dirpath, "counter_collection.csv"):
        per = {}
        for r in _rows(path):
            key = (r["Kernel_Name"], int(r.get("Grid_Size", 0) or 0), r["Dispatch_Id"])
            per.setdefault(key, {}).setdefault(r["Counter_Name"], 0.0)
            per[key][r["Counter_Name"]] += float(r["Counter_Value"])
        for (name, grid, _), vals in per.items():
            d = out.setdefault((name, grid), {})
            for c, v in vals.items():
                d.setdefault(c, []).append(v)
    return out


def trace(dirpath):
    """{(kernel name, grid size): [duration ns per dispatch]} from a
    --kernel-trace run."""
    out = {}
    for path in _find(dirpath, "kernel_trace.csv"):
        for r in _rows(path):
            grid = int(r.get("Grid_Size_X", r.get("Grid_Size", 0)) or 0)
            dur = float(r["End_Timestamp"]) - float(r["Start_Timestamp"])
            out.setdefault((r["Kernel_Name"], grid), []).append(dur)
    return out


def headline_mean(durations):
    """(mean, number left out) of the dispatch durations of the headline
    lattice.  The bench also steps smaller lattices (its sweep over the
    paper's sizes), and the launch plan fills the GPU with the same grid at
    every size, so their launches can share the kernel name and grid; the
    headline lattice's launches are the large majority, and the others are
    many times shorter: keep those within a factor of two of the median."""
    med = statistics.median(durations)
    keep = [d for d in durations if 0.5 * med <= d <= 2.0 * med]
    return statistics.mean(keep), len(durations) - len(keep)


def _pick(table, pattern, grid=None):
    """The (name, grid) entry whose name matches `pattern` (and whose grid is
    `grid`, if given): the one with the most dispatches."""
    cands = [(k, v) for k, v in table.items() if re.search(pattern, k[0]) and (grid is None or k[1] == grid)]
    if not cands:
        raise KeyError(f"no kernel matching {pattern!r}" + ("" if grid is None else f" with grid {grid}"))

    def count(item):
        v = item[1]
        return len(next(iter(v.values()))) if isinstance(v, dict) else len(v)
    return max(cands, key=count)


def _calibration(fetch, write):
    """Bytes moved per counter byte of the 1 GiB runtime copy: (fetch, write)."""
    _, fv = _pick(fetch, r"[Cc]opy[Bb]uffer")
    _, wv = _pick(write, r"[Cc]opy[Bb]uffer")
    f_kib = statistics.mean(fv["FETCH_SIZE"])
    w_kib = statistics.mean(wv["WRITE_SIZE"])
    return CALIB_BYTES / (f_kib * 1024.0), CALIB_BYTES / (w_kib * 1024.0), f_kib, w_kib


def _sq_lines(sq, pattern, grid, dur_ns):
    _, vals = _pick(sq, pattern, grid)
    mean = {c: statistics.mean(v) for c, v in vals.items()}
    lines = ["", "SQ instruction counters of the same kernel (means over its dispatches in the counter run):", "",
             "| counter | per launch |", "|---|---|"]
    for c in sorted(mean):
        lines.append(f"| {c} | {mean[c]:.4g} |")
    if dur_ns:
        cyc = dur_ns * CLOCK_GHZ
        lines.append("")
        if "SQ_INSTS_VALU" in mean:
            # a wave64 VALU instruction holds a 16-lane SIMD for 4 cycles, FP64
            # FMA included (78.6 TFLOP/s = 1024 SIMDs x 16 lanes x 2 x 2.4 GHz);
            # transcendental and packed forms take longer, so this is a lower
            # bound of the busy share
            issue = mean["SQ_INSTS_VALU"] * 4.0 / (SIMDS * cyc)
            lines.append(f"VALU issue share: SQ_INSTS_VALU x 4 cycles / ({SIMDS} SIMDs x {cyc:.4g} cycles of a "
                         f"{dur_ns / 1e3:.1f} us launch at {CLOCK_GHZ} GHz) = {issue:.3f}")
            lines.append(f"valu_issue_share: {issue:.4f}")
        if "SQ_ACTIVE_INST_VALU" in mean:
            act = mean["SQ_ACTIVE_INST_VALU"] * 4.0 / (SIMDS * cyc)
            lines.append(f"VALU active share: SQ_ACTIVE_INST_VALU x 4 / ({SIMDS} SIMDs x launch cycles) = {act:.3f}")
        if "SQ_INSTS_LDS" in mean and "SQ_WAVES" in mean:
            lines.append(f"LDS instructions per wavefront: {mean['SQ_INSTS_LDS'] / mean['SQ_WAVES']:.0f}")
    return lines


def traffic_summary(title, kernel_desc, pattern, fetch_dir, write_dir, alg_read, alg_write, steps_per_launch,
                    sources, commands, notes=(), sq_dir=None, trace_dir=None, alg_desc=""):
    fetch, write = counters(fetch_dir), counters(write_dir)
    cf, cw, cf_kib, cw_kib = _calibration(fetch, write)
    (kname, grid), fv = _pick(fetch, pattern)
    _, wv = _pick(write, pattern, grid)
    f_kib = statistics.mean(fv["FETCH_SIZE"])
    w_kib = statistics.mean(wv["WRITE_SIZE"])
    rd = f_kib * 1024.0 * cf
    wr = w_kib * 1024.0 * cw
    dur, excluded = None, 0
    if trace_dir:
        t = trace(trace_dir)
        # trace grids count workgroups x 64 lanes like the counter runs' Grid_Size
        hits = [d for (name, g), d in t.items() if name == kname and g == grid]
        if hits:
            dur, excluded = headline_mean(hits[0])
    lines = [f"# {title}", "", f"Kernel: `{kname}` ({kernel_desc}), grid {grid} lanes.", "",
             "Commands (each a run of its own, on one MI355X; <repo> is the repository root):", "",
             "    cd /tmp && export TMPDIR=/tmp"]
    lines += [f"    {c}" for c in commands]
    lines += ["", "| kernel | dispatches | FETCH_SIZE (KiB/dispatch) | WRITE_SIZE (KiB/dispatch) |", "|---|---|---|---|",
              f"| {kname.split('(')[0]} | {len(fv['FETCH_SIZE'])} | {f_kib:.1f} | {w_kib:.1f} |",
              f"| 1 GiB runtime copy | 1 | {cf_kib:.1f} | {cw_kib:.1f} |", "",
              f"Calibration (bytes moved / counter bytes of the 1 GiB copy): fetch x {cf:.4f}, write x {cw:.4f}.", "",
              f"| per launch ({steps_per_launch} step{'s' if steps_per_launch > 1 else ''}) | read | write | total |",
              "|---|---|---|---|",
              f"| measured HBM bytes (calibrated) | {rd / 1e6:.1f} MB | {wr / 1e6:.1f} MB | {(rd + wr) / 1e6:.1f} MB |",
              f"| algorithmic{': ' + alg_desc if alg_desc else ''} | {alg_read / 1e6:.1f} MB | {alg_write / 1e6:.1f} MB | "
              f"{(alg_read + alg_write) / 1e6:.1f} MB |",
              f"| measured / algorithmic | {rd / alg_read:.3f} | {wr / alg_write:.3f} | "
              f"{(rd + wr) / (alg_read + alg_write):.3f} |"]
    if dur:
        lines += ["", f"Mean launch duration in the traced bench run ({excluded} shorter dispatches of smaller "
                      f"lattices with the same kernel and grid left out): {dur / 1e3:.1f} us: "
                      f"{(alg_read + alg_write) / dur:.1f} GB/s algorithmic "
                      f"({(alg_read + alg_write) / dur / 8000.0:.3f} of 8 TB/s), "
                      f"{(rd + wr) / dur:.1f} GB/s measured HBM traffic."]
    lines += [""] + list(notes)
    if sq_dir:
        lines += _sq_lines(counters(sq_dir), re.escape(kname), grid, dur)
    lines += ["", f"kernel_source_sha256: {source_hash(sources)}",
              f"traffic_bytes_per_launch: {rd + wr:.6e}",
              f"algorithmic_bytes_per_launch: {alg_read + alg_write:.6e}",
              f"steps_per_launch: {steps_per_launch}"]
    if dur:
        lines.append(f"avg_launch_ns: {dur:.1f}")
    return "\n".join(lines) + "\n"


def trace_summary(trace_dir, command, title):
    t = trace(trace_dir)
    lines = [f"# {title}", "", "Command (one MI355X; <repo> is the repository root):", "",
             "    cd /tmp && export TMPDIR=/tmp", f"    {command}", "",
             "Per kernel and grid (lanes = workgroups x 64), durations in ns from the kernel trace.  "
             "Smaller lattices can share a kernel and grid with the 4096^2 launches (the launch plan fills "
             "the GPU with the same grid at every size); `avg (majority)` averages the launches within a "
             "factor of two of the median, as the traffic summaries do:", "",
             "| kernel | grid | launches | avg | avg (majority) | left out | median | min | max |",
             "|---|---|---|---|---|---|---|---|---|"]
    for (name, grid), d in sorted(t.items(), key=lambda kv: -sum(kv[1])):
        short = name.split("(")[0]
        hm, left = headline_mean(d)
        lines.append(f"| `{short}` | {grid} | {len(d)} | {statistics.mean(d):.0f} | {hm:.0f} | {left} | "
                     f"{statistics.median(d):.0f} | {min(d):.0f} | {max(d):.0f} |")
    return "\n".join(lines) + "\n"


def _step_cmds(storage):
    base = f"python3 <repo>/bench.py --profile-steps {PROFILE_STEPS} --profile-storage {storage}"
    return [f"rocprofv3 --pmc {c} --output-format csv -d <repo>/gpurun_out/step_{storage}_{c} -o run -- {base}"
            for c in ("FETCH_SIZE", "WRITE_SIZE")]


def main(argv=None):
    ap = argparse.ArgumentParser(description=__doc__, formatter_class=argparse.RawDescriptionHelpFormatter)
    sub = ap.add_subparsers(dest="what", required=True)
    s = sub.add_parser("step")
    s.add_argument("--storage", choices=("fp64", "fp32", "fp16s"), required=True)
    a = sub.add_parser("adjoint")
    for p in (s, a):
        p.add_argument("--fetch", required=True)
        p.add_argument("--write", required=True)
        p.add_argument("--sq")
        p.add_argument("--sq-command", default="")
        p.add_argument("--trace", help="kernel-trace run of the bench (launch durations)")
        p.add_argument("--out", required=True)
    t = sub.add_parser("trace")
    t.add_argument("--trace", required=True)
    t.add_argument("--command", required=True)
    t.add_argument("--title", default="Kernel trace")
    t.add_argument("--out", required=True)
    args = ap.parse_args(argv)
    if args.what == "trace":
        text = trace_summary(args.trace, args.command, args.title)
    elif args.what == "step":
        r, w = STEP_BYTES[args.storage]
        cmds = _step_cmds(args.storage)
        if args.sq_command:
            cmds.append(args.sq_command)
        kname, spp = STEP_KERNEL[args.storage]
        text = traffic_summary(
            f"HBM traffic of the {args.storage.upper()} step kernel, patterned dewetting 4096 x 4096",
            f"{args.storage.upper()} storage, kappa field, {spp} time steps per launch, omega = 1 stages",
            re.escape(kname), args.fetch, args.write,
            r * N4096, w * N4096, spp, STEP_SOURCES, cmds, sq_dir=args.sq, trace_dir=args.trace,
            alg_desc=f"{'records' if args.storage == 'fp16s' else 'moments'} read and written once and the kappa field "
                     f"read once ({r}/{w} B/site)",
            notes=[f"`bench.py --profile-steps {PROFILE_STEPS}` runs {PROFILE_STEPS} steps "
                   "of the benchmark workload, a record copy of one population "
                   "buffer (tflbm_state_save) and a 1 GiB runtime copy that calibrates the counters."])
    else:
        cmds = [f"rocprofv3 --pmc {c} --output-format csv -d <repo>/gpurun_out/adj_{c} -o run -- "
                f"python3 <repo>/bench.py --profile-adjoint 16" for c in ("FETCH_SIZE", "WRITE_SIZE")]
        if args.sq_command:
            cmds.append(args.sq_command)
        text = traffic_summary(
            "Reverse pass, two steps per launch: FP32 adjoint, patterned dewetting 4096 x 4096",
            "FP32 adjoint carried as three fields per site (tau = 1), kappa field, two reverse time steps per "
            "launch", re.escape(ADJ_KERNEL),
            args.fetch, args.write, ADJ_BYTES[0] * N4096, ADJ_BYTES[1] * N4096, 2, ADJ_SOURCES, cmds, sq_dir=args.sq,
            trace_dir=args.trace,
            alg_desc="adjoint fields 12 + two captures 24 + kappa 4 + g_kappa 8 read; fields 12 + g_kappa 8 written "
                     "(B/site)",
            notes=["`bench.py --profile-adjoint 16` captures 16 FP32 steps of the benchmark workload, runs the "
                   "reverse pass over them (8 launches of the two-step kernel), then a 1 GiB runtime copy that "
                   "calibrates the counters."])
    with open(args.out, "w") as fh:
        fh.write(text)
    print(text)


if __name__ == "__main__":
    main()
