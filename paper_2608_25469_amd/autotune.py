"""Offline block-size tuner for the blocked path (paper Sec. 4.3.2).

Pre-build phase of the paper's adaptive blocking: for every (data type, m, n)
scale point, time the blocked solve with each candidate I_B (the rows of a
panel) and keep the fastest.  The results go to a JSON file (written after every
measurement, so an interrupted sweep resumes) and are turned into the
compiled-in table ``csrc/tuning_gfx950.h``; at run time the library picks the
entry of the nearest tested scale (``hsma_lookup_block_size``).  A solve that
is given no block size reports that entry, and ``hsma_trsm_noalloc`` takes the
sizes whose workspace of inverted blocks of that edge would fit its array; the
solve itself has panels as tall as the kernel takes.

  python -m paper_2608_25469_amd.autotune sweep  --out results.json   (GPU)
  python -m paper_2608_25469_amd.autotune header --json results.json  (CPU)
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HEADER = os.path.join(HERE, "csrc", "tuning_gfx950.h")
CANDIDATES = (16, 32, 64, 128, 256)
SCALES_REAL = [(m, m) for m in (128, 256, 512, 1024, 2048, 4096, 8192, 16384)] + \
              [(m, 256) for m in (1024, 4096, 16384)]
SCALES_COMPLEX = [(m, m) for m in (128, 256, 512, 1024, 2048, 4096, 8192)] + \
                 [(m, 256) for m in (1024, 4096)]


def sweep(out_path: str, reps: int = 3, scales=None) -> dict:
    import numpy as np
    import torch
    sys.path.insert(0, ROOT)
    import paper_2608_25469_amd as hs
    import workloads as W

    torch.cuda.set_device(0)
    res = {"device": torch.cuda.get_device_name(0), "candidates": list(CANDIDATES), "points": []}
    if os.path.exists(out_path):
        with open(out_path) as f:
            res = json.load(f)
    done = {(p["complex"], p["m"], p["n"]) for p in res["points"]}
    todo = scales or ([(False, m, n) for m, n in SCALES_REAL] + [(True, m, n) for m, n in SCALES_COMPLEX])
    for cx, m, n in todo:
        if (cx, m, n) in done:
            continue
        L, B = W.problem(7, m, n, cx)
        Ld, Bd, B0 = hs.to_colmajor(L), hs.to_colmajor(B), hs.to_colmajor(B)
        del L, B
        times = {}
        for ib in CANDIDATES:
            hs.trsm(Ld, Bd, 1.0, block_size=ib, path=2)
            torch.cuda.synchronize()
            ts = []
            for _ in range(reps):
                Bd.copy_(B0)
                torch.cuda.synchronize()
                t = time.perf_counter()
                hs.trsm(Ld, Bd, 1.0, block_size=ib, path=2)
                torch.cuda.synchronize()
                ts.append((time.perf_counter() - t) * 1e3)
            times[str(ib)] = float(np.median(ts))
        best = min(times, key=lambda k: times[k])
        fl = W.flops(m, n, cx)
        point = {"complex": cx, "m": m, "n": n, "ms": times, "best": int(best),
                 "best_gflops": fl / (times[best] * 1e-3) / 1e9}
        res["points"].append(point)
        print(json.dumps(point), flush=True)
        with open(out_path + ".tmp", "w") as f:
            json.dump(res, f, indent=1)
        os.replace(out_path + ".tmp", out_path)
        del Ld, Bd, B0
        torch.cuda.empty_cache()
    return res


def write_header(res: dict, path: str = HEADER, source: str = "") -> None:
    pts = sorted(res["points"], key=lambda p: (p["complex"], p["m"], p["n"]))
    lines = [
        "// Diagonal-block edge I_B for the blocked path on gfx950, by problem scale",
        "// and data type (paper Sec. 4.3.2: offline profiling builds a \"scale x data",
        "// type -> block\" table; the runtime picks the entry of the nearest tested",
        "// scale).  Generated by paper_2608_25469_amd/autotune.py from measurements;",
        "// regenerate with that script after kernel changes.",
        "//",
        f"// Source: {source or 'sweep results'} ({res.get('device', 'gfx950')}),",
        "// candidates " + ", ".join(str(c) for c in res.get("candidates", CANDIDATES)) +
        "; median of timed solves per candidate.",
        "#pragma once",
        "",
        "namespace hsma {",
        "namespace tuning {",
        "",
        "struct Entry {",
        "    int dtype;   // 0 real, 1 complex",
        "    int m, n;    // tested scale",
        "    int ib;      // best diagonal-block edge",
        "};",
        "",
        "static const Entry kTable[] = {",
    ]
    for p in pts:
        lines.append(f"    {{{1 if p['complex'] else 0}, {p['m']}, {p['n']}, {p['best']}}},"
                     f"  // {p['best_gflops']:.0f} GFLOP/s")
    lines += ["};", "", f"static const char kSource[] = \"{os.path.basename(source) or 'sweep'}\";", "",
              "}  // namespace tuning", "}  // namespace hsma", ""]
    with open(path, "w") as f:
        f.write("\n".join(lines))


def main():
    ap = argparse.ArgumentParser()
    sub = ap.add_subparsers(dest="cmd", required=True)
    s1 = sub.add_parser("sweep")
    s1.add_argument("--out", required=True)
    s1.add_argument("--reps", type=int, default=3)
    s2 = sub.add_parser("header")
    s2.add_argument("--json", required=True)
    s2.add_argument("--out", default=HEADER)
    a = ap.parse_args()
    if a.cmd == "sweep":
        sweep(a.out, a.reps)
    else:
        with open(a.json) as f:
            write_header(json.load(f), a.out, source=a.json)


if __name__ == "__main__":
    main()
