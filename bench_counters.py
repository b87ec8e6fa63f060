"""Sums the hardware counters of rocprofv3 --pmc runs of `bench.py --pmc-pass` over the dispatches of
one kernel and writes the short table kept under profiles/ (counter values per attention call), with
the figures derived from them: matrix-core busy share, LDS bytes per cycle, where the wavefronts'
time goes.

    python bench_counters.py --kernel attn_prefill_mfma_queued_kernel --calls 8 --title "..." \
        --command "<the rocprofv3 commands>" --out profiles/<name>.md <run a>/p_counter_collection.csv <run b>/...
"""
from __future__ import annotations

import argparse
import csv
from collections import defaultdict


def main() -> int:
    ap = argparse.ArgumentParser()
    ap.add_argument("csv", nargs="+")
    ap.add_argument("--kernel", required=True)
    ap.add_argument("--calls", type=int, required=True, help="calls of the entry point in the pass")
    ap.add_argument("--waves-per-simd", type=int, default=2, help="wavefronts of the kernel that a SIMD holds")
    ap.add_argument("--title", required=True)
    ap.add_argument("--command", default="")
    ap.add_argument("--note", default="")
    ap.add_argument("--out", required=True)
    args = ap.parse_args()

    tot = defaultdict(float)
    disp = defaultdict(set)
    for path in args.csv:
        with open(path, newline="") as f:
            for row in csv.DictReader(f):
                if args.kernel in row["Kernel_Name"]:
                    tot[row["Counter_Name"]] += float(row["Counter_Value"])
                    disp[row["Counter_Name"]].add(row["Dispatch_Id"])
    n = args.calls
    lines = [f"# {args.title}", ""]
    if args.command:
        lines += ["Commands (from /tmp, TMPDIR=/tmp; one counter group per run):", "", "```",
                  args.command, "```", ""]
    lines += [f"Sums over the dispatches of {args.kernel} in one pass, divided by the {n} calls of the pass "
              f"({len(next(iter(disp.values()), ()))} dispatches).", "",
              "| counter | per call |", "|---|---:|"]
    lines += [f"| {k} | {tot[k] / n:,.0f} |" for k in sorted(tot)]
    lines.append("")
    g = lambda k: tot.get(k, 0.0) / n
    if g("SQ_INSTS_MFMA") and g("SQ_VALU_MFMA_BUSY_CYCLES"):
        lines.append(f"* Matrix-core instructions per call: {g('SQ_INSTS_MFMA'):,.0f} (wavefront level; 32x32x16 bf16: "
                     f"{g('SQ_INSTS_MFMA') * 32 * 32 * 16 * 2 / 1e9:.1f} GFLOP issued); busy cycles per instruction "
                     f"{g('SQ_VALU_MFMA_BUSY_CYCLES') / g('SQ_INSTS_MFMA'):.1f}.")
    # Cycles are those in which the kernel's wavefronts are resident: SQ_WAVE_CYCLES counts them per wavefront in units of
    # four.  (GRBM_GUI_ACTIVE and SQ_BUSY_CYCLES also count what goes on between a dispatch and the next: 11 to 18 and 43 to
    # 68 million a call for the same kernel, 574 to 582 here.)
    if g("SQ_WAVE_CYCLES") and g("SQ_VALU_MFMA_BUSY_CYCLES"):
        simd_cycles = 4 * g("SQ_WAVE_CYCLES") / args.waves_per_simd
        lines.append(f"* Matrix-core busy cycles / cycles of the SIMDs that hold its wavefronts ({args.waves_per_simd} each; 4 x "
                     f"SQ_WAVE_CYCLES / {args.waves_per_simd}) = {100 * g('SQ_VALU_MFMA_BUSY_CYCLES') / simd_cycles:.1f} %.")
        if g("SQ_INSTS_LDS"):
            lines.append(f"* LDS instructions per call: {g('SQ_INSTS_LDS'):,.0f} (1 KB operand reads almost all of "
                         f"them): {g('SQ_INSTS_LDS') * 1024 / (simd_cycles / 4):.0f} bytes per cycle and "
                         f"compute unit in use; bank conflict cycles {g('SQ_LDS_BANK_CONFLICT'):,.0f}.")
    if g("SQ_WAVE_CYCLES"):
        w = g("SQ_WAVE_CYCLES")
        lines.append(f"* Wavefront time (SQ_WAVE_CYCLES): waiting (SQ_WAIT_ANY) {100 * g('SQ_WAIT_ANY') / w:.0f} %, "
                     f"issuing (SQ_ACTIVE_INST_ANY) {100 * g('SQ_ACTIVE_INST_ANY') / w:.0f} %, of which vector ALU "
                     f"including matrix-core issue (SQ_ACTIVE_INST_VALU) {100 * g('SQ_ACTIVE_INST_VALU') / w:.0f} %.")
    if args.note:
        lines += ["", args.note]
    with open(args.out, "w") as f:
        f.write("\n".join(lines) + "\n")
    print("\n".join(lines))
    return 0


if __name__ == "__main__":
    raise SystemExit(main())
