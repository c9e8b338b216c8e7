"""Turn rocprofv3 CSV output into a short text summary (per kernel: calls, mean duration,
counter means) and, on request, into the HBM bytes per launch that bench.py reports.

    python -m paper_2502_08145_amd.profile_summary <dir> [<dir> ...]
    python -m paper_2502_08145_amd.profile_summary --traffic <workload> <copy MiB> <FETCH dir> <WRITE dir>

Each <dir> is the -d directory of one rocprofv3 run (--kernel-trace, with --stats and/or --pmc).
--traffic prints a JSON object {workload: {kernel: bytes per launch}}: FETCH_SIZE and WRITE_SIZE
(KiB per dispatch) of every GEMM kernel, each scaled by what the same counter read for a kernel of
exactly known traffic that ran in the same process: the tiled transpose of a <copy MiB> MiB matrix
(bench.py --calibrate-copy; every element read once and written once).  The object also carries
the hash of the kernel sources it was measured with ("_source", build.source_id()).
"""
from __future__ import annotations

import collections
import csv
import glob
import os
import re
import sys


_LAYOUT = {("true", "false"): "NN", ("true", "true"): "NT", ("false", "false"): "TN"}   # (A, B) K-contiguous
_BOOL = "(true|false)"


def short(name: str) -> str:
    """The name of a kernel symbol: the library's (axonn_linear_part_kernel) without what is a run-time argument (the
    number of K ranges, the waves per wave-K tile), and the mode; kernel_key() gives the same from the library's side."""
    m = re.search(rf"gemm_tile_kernel16<(\d+), (\d+), (\d+), (\d+), {_BOOL}, {_BOOL}, {_BOOL}>", name)
    if m:
        bm, bn, wm, wn, akc, bkc, split = m.groups()
        waves = "_w8" if int(wm) * int(wn) == 8 else ""
        return f"mfma16_{bm}x{bn}{waves}{'_sk' if split == 'true' else ''}/{_LAYOUT.get((akc, bkc), '??')}"
    m = re.search(rf"gemm_tile_kernel_k64<(\d+), (\d+), (\d+), {_BOOL}, {_BOOL}, {_BOOL}, \d+, {_BOOL}>", name)
    if m:
        bm, bn, wn, akc, bkc, split, tail = m.groups()
        waves = "_w8" if wn == "4" else ""
        return f"mfma16k64_{bm}x{bn}{waves}{'_sk' if split == 'true' else ''}{'_ktail' if tail == 'true' else ''}/{_LAYOUT.get((akc, bkc), '??')}"
    m = re.search(rf"gemm_tile_kernel_k64g<(\d+), (\d+), (\d+), {_BOOL}, {_BOOL}, {_BOOL}>", name)
    if m:
        bm, bn, groups, akc, bkc, tail = m.groups()
        return f"mfma16k64g_{bm}x{bn}{'_g2' if groups == '2' else ''}{'_ktail' if tail == 'true' else ''}/{_LAYOUT.get((akc, bkc), '??')}"
    m = re.search(rf"gemm_tile_kernel_k64gs<(\d+), (\d+), {_BOOL}, {_BOOL}>", name)
    if m:
        bm, bn, akc, bkc = m.groups()
        return f"mfma16k64g_{bm}x{bn}_sk/{_LAYOUT.get((akc, bkc), '??')}"
    m = re.search(rf"gemm_tile_kernel_k64p<{_BOOL}, {_BOOL}>", name)
    if m:
        return f"mfma16k64p_256x256_w8/{_LAYOUT.get(m.groups(), '??')}"
    m = re.search(rf"gemm_wavek_kernel<{_BOOL}, {_BOOL}, (\d+), (\d+)>", name)
    if m:
        akc, bkc, mi, ni = m.groups()
        return f"wavek_{16 * int(mi)}x{16 * int(ni)}/{_LAYOUT.get((akc, bkc), '??')}"
    m = re.search(rf"gemm_shortk_kernel<(\d), {_BOOL}>", name)
    if m:
        return f"wavek_64x64_k{32 * int(m.group(1))}{'_xcd' if m.group(2) == 'true' else ''}/TN"
    m = re.search(rf"gemm_edge_kernel<{_BOOL}, {_BOOL}>", name)
    if m:
        return f"edge_128x128/{_LAYOUT.get(m.groups(), '??')}"
    m = re.search(r"gemm_naive_kernel<(\d)>", name)
    if m:
        return f"naive/{('NN', 'NT', 'TN')[int(m.group(1))]}"
    if "transpose_tile_kernel" in name:   # in rows or in bands of tiles: the same traffic
        return "transpose_tile"
    if "transpose_window_kernel" in name:   # reads rows twice: no copy to calibrate counters with
        return "transpose_window"
    if "transpose_naive_kernel" in name:
        return "transpose_naive"
    return re.sub(r"\(.*", "", name)[:60]


GEMMS = ("mfma", "wavek", "edge", "naive")   # what the names of the product kernels start with


def summarize(d: str, out=sys.stdout):
    traces = glob.glob(os.path.join(d, "**", "*kernel_trace.csv"), recursive=True)
    counters = glob.glob(os.path.join(d, "**", "*counter_collection.csv"), recursive=True)
    dur = collections.defaultdict(list)
    for f in traces:
        for r in csv.DictReader(open(f)):
            dur[short(r["Kernel_Name"])].append(int(r["End_Timestamp"]) - int(r["Start_Timestamp"]))
    ctr = collections.defaultdict(lambda: collections.defaultdict(list))
    for f in counters:
        for r in csv.DictReader(open(f)):
            ctr[short(r["Kernel_Name"])][r["Counter_Name"]].append(float(r["Counter_Value"]))
    print(f"== {d}", file=out)
    keys = [k for k in dur if k.startswith(GEMMS + ("transpose",))]
    for k in sorted(keys, key=lambda k: -sum(dur[k])):
        v = dur[k]
        print(f"{k:<22s} calls {len(v):5d}  mean {sum(v) / len(v) / 1e3:9.2f} us  min {min(v) / 1e3:9.2f}  "
              f"max {max(v) / 1e3:9.2f}  total {sum(v) / 1e6:9.3f} ms", file=out)
        means = {c: sum(vals) / len(vals) for c, vals in ctr.get(k, {}).items()}
        for c in sorted(means):
            print(f"    {c:<28s} mean per dispatch {means[c]:.6g}  (n={len(ctr[k][c])})", file=out)
        # derived: GRBM_GUI_ACTIVE is summed over the 8 XCDs, SQ_VALU_MFMA_BUSY_CYCLES over 256 CUs x 4 SIMDs
        if "SQ_VALU_MFMA_BUSY_CYCLES" in means and means.get("GRBM_GUI_ACTIVE"):
            print(f"    -> MFMA busy {means['SQ_VALU_MFMA_BUSY_CYCLES'] / 1024.0 / (means['GRBM_GUI_ACTIVE'] / 8.0) * 100:.1f} % of "
                  f"the kernel's cycles", file=out)
        if "SQ_LDS_BANK_CONFLICT" in means and means.get("SQ_LDS_IDX_ACTIVE"):
            print(f"    -> LDS bank-conflict cycles / LDS-active cycles {means['SQ_LDS_BANK_CONFLICT'] / means['SQ_LDS_IDX_ACTIVE'] * 100:.1f} %",
                  file=out)
    return dur, ctr


def kernel_key(kernel: str, layout: str) -> str:
    """The name short() gives the symbol behind a kernel name of the library (binding.kernel_name): split-K over any
    number of K ranges, and wave-K tiles over any number of waves, are one kernel."""
    kernel = re.sub(r"^(wavek_\d+x\d+)_w\d+$", r"\1", kernel)
    return re.sub(r"_sk\d+$", "_sk", kernel) + "/" + layout


def traffic(workload: str, copy_mib: float, fetch_dir: str, write_dir: str) -> dict:
    import io
    _, fetch = summarize(fetch_dir, io.StringIO())
    _, write = summarize(write_dir, io.StringIO())
    mean = lambda v: sum(v) / len(v)
    kib = copy_mib * 1024.0
    f_scale = kib / mean(fetch["transpose_tile"]["FETCH_SIZE"])
    w_scale = kib / mean(write["transpose_tile"]["WRITE_SIZE"])
    out = {}
    for k in fetch:
        if k.startswith(GEMMS) and k in write:
            out[k] = int(round(1024.0 * (mean(fetch[k]["FETCH_SIZE"]) * f_scale + mean(write[k]["WRITE_SIZE"]) * w_scale)))
    from .build import source_id
    return {workload: out, "_scale": {"FETCH_SIZE": round(f_scale, 4), "WRITE_SIZE": round(w_scale, 4)},
            "_source": source_id(),
            "_note": "bytes per launch = FETCH_SIZE x scale + WRITE_SIZE x scale (KiB -> bytes), scales from a tiled "
                     "transpose of known size in the same process; _source = hash of the kernel sources measured"}


def main(argv):
    if len(argv) < 2:
        sys.exit(__doc__)
    if argv[1] == "--traffic":
        import json
        if len(argv) != 6:
            sys.exit(__doc__)
        print(json.dumps(traffic(argv[2], float(argv[3]), argv[4], argv[5]), indent=1))
        return
    for d in argv[1:]:
        summarize(d)


if __name__ == "__main__":
    main(sys.argv)
