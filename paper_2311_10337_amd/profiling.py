"""Roofline bookkeeping for bench.py: algorithmic bytes per kernel and HBM
traffic from rocprofv3 counter runs.

Algorithmic bytes are the bytes a kernel must move at minimum width, with each
input and output touched once (random gathers count their element size, not
the cache line they pull). ``traffic`` comes from two rocprofv3 ``--pmc`` runs
(FETCH_SIZE, then WRITE_SIZE, KiB per dispatch), each scaled by what the same
counter reads for a plain copy kernel of known size.
"""
from __future__ import annotations

import csv
import glob
import hashlib
import json
import os

HERE = os.path.dirname(os.path.abspath(__file__))
HBM_PEAK_GBS = 8000.0  # MI355X HBM3E


def _bits(x: int) -> int:
    """Bits of a sort key that holds the values 0..x, as the library counts them (at least one)."""
    return max(1, int(x).bit_length())


def sorts(n: int, m: int, num_vertices: int, span: int, causal: bool = False) -> list:
    """The radix sorts of one call on one graph, as the library makes them: (elements, key bytes, value bytes,
    passes, whether the values are implicit in the first pass). span = max t - min t; a causal key's tie field
    is taken as one bit."""
    tb, idb = _bits(span), _bits(n - 1)
    packed = tb <= 32 and not causal
    passes = lambda bits: -(-bits // 8)
    return [(n, 8, 8 if packed else 16, passes(tb), False),
            (2 * n, 4, 4, passes(_bits(num_vertices - 1)), not causal),
            (m, 8, 4, passes(tb + idb + 1), True),
            (m, 4, 8, passes(_bits(n - 1)), False)]


def algorithmic_bytes_per_step(kernel: str, n: int, m: int, num_vertices: int, span: int,
                               causal: bool = False) -> tuple:
    """(unit description, bytes per step): what the launches of a kernel must move in one call."""
    if kernel == "k_rs_scatter":
        # per element and pass: key and value read and written (the first pass of an implicit value reads the key)
        total = sum(k * (2 * (kb + vb) * p - (vb if iota else 0))
                    for k, kb, vb, p, iota in sorts(n, m, num_vertices, span, causal))
        return ("element x pass: key and value read and written (records by time, incidences by vertex, rows by "
                "key, rows by chain)", total)
    raise KeyError(kernel)


def source_hash(files=None) -> str:
    """Hash of every kernel source under csrc/ (sorted by name)."""
    if files is None:
        files = sorted(os.path.relpath(f, HERE) for f in glob.glob(os.path.join(HERE, "csrc", "*"))
                       if f.endswith((".hip", ".h")))
    h = hashlib.sha256()
    for f in files:
        with open(os.path.join(HERE, f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def _counter_rows(d):
    paths = glob.glob(os.path.join(d, "**", "*counter_collection.csv"), recursive=True)
    rows = []
    for p in paths:
        with open(p) as fh:
            rows.extend(csv.DictReader(fh))
    rows.sort(key=lambda r: int(r["Dispatch_Id"]))
    return rows


def _is_library(name: str) -> bool:
    return name.startswith("ce::") or name.startswith("void ce::")


def _calibration_kib(rows):
    """Counter value of the calibration copy: the largest runtime copy issued before the first library
    kernel (the pipeline's own device copies come later and can be larger)."""
    first = next((i for i, r in enumerate(rows) if _is_library(r["Kernel_Name"])), len(rows))
    copies = [float(r["Counter_Value"]) for r in rows[:first] if "copyBuffer" in r["Kernel_Name"]]
    return max(copies) if copies else None


def summarize_pmc(fetch_dir: str, write_dir: str, kernel: str, copy_bytes: int) -> dict:
    """Per-dispatch HBM traffic of `kernel`, calibrated against the largest copy dispatch."""
    out = {"kernel": kernel, "copy_bytes": copy_bytes}
    for name, d in (("FETCH_SIZE", fetch_dir), ("WRITE_SIZE", write_dir)):
        rows = [r for r in _counter_rows(d) if r["Counter_Name"] == name]
        ref_kib = _calibration_kib(rows)
        factor = (copy_bytes / 1024.0) / ref_kib if ref_kib else None
        mine = [float(r["Counter_Value"]) for r in rows if kernel in r["Kernel_Name"]]
        out[name] = {"dispatches": len(mine), "avg_kib": (sum(mine) / len(mine)) if mine else None,
                     "copy_kib": ref_kib, "scale": factor}
    f, w = out["FETCH_SIZE"], out["WRITE_SIZE"]
    if f["avg_kib"] is not None and w["avg_kib"] is not None and f["scale"] and w["scale"]:
        out["traffic_bytes_per_launch"] = 1024.0 * (f["avg_kib"] * f["scale"] + w["avg_kib"] * w["scale"])
    else:
        out["traffic_bytes_per_launch"] = None
    out["source_hash"] = source_hash()
    return out


def _is_host_side(name: str) -> bool:
    # torch's own kernels (input fills and copies made by the benchmark harness)
    return "at::native" in name


def summarize_pipeline_pmc(fetch_dir: str, write_dir: str, copy_bytes: int, steps: int = 1) -> dict:
    """HBM traffic of the whole pipeline per step: every dispatch from the first to the last library
    kernel (library kernels and the runtime copies they issue), calibrated like summarize_pmc."""
    out = {"scope": "pipeline", "copy_bytes": copy_bytes, "steps": steps}
    for name, d in (("FETCH_SIZE", fetch_dir), ("WRITE_SIZE", write_dir)):
        rows = [r for r in _counter_rows(d) if r["Counter_Name"] == name]
        ref_kib = _calibration_kib(rows)
        factor = (copy_bytes / 1024.0) / ref_kib if ref_kib else None
        lib = [i for i, r in enumerate(rows) if _is_library(r["Kernel_Name"])]
        span = rows[lib[0]:lib[-1] + 1] if lib else []
        mine = [float(r["Counter_Value"]) for r in span if not _is_host_side(r["Kernel_Name"])]
        out[name] = {"dispatches": len(mine), "total_kib": sum(mine), "copy_kib": ref_kib, "scale": factor}
    f, w = out["FETCH_SIZE"], out["WRITE_SIZE"]
    if f["scale"] and w["scale"]:
        out["traffic_bytes_per_step"] = 1024.0 * (f["total_kib"] * f["scale"] + w["total_kib"] * w["scale"]) / steps
    else:
        out["traffic_bytes_per_step"] = None
    out["source_hash"] = source_hash()
    return out


def load_pipeline_traffic(path: str) -> float | None:
    """Pipeline traffic per step from a committed summary, or None if the kernels changed since."""
    if not os.path.exists(path):
        return None
    with open(path) as fh:
        text = fh.read()
    start = text.find("```json")
    if start < 0:
        return None
    blob = json.loads(text[start + 7:text.find("```", start + 7)])
    if blob.get("scope") != "pipeline" or blob.get("source_hash") != source_hash():
        return None
    return blob.get("traffic_bytes_per_step")


# algorithmic bytes per temporal edge of the whole path, by stage: each intermediate written once and read
# once at minimal width (input 16, incidence 48, skeleton 64, MSF rows 32, dendrogram rows 20, per-record
# outputs 12, labels 4)
STAGE_BYTES = {"input": 16, "incidence": 48, "skeleton": 64, "msf": 32, "dendrogram": 20, "condensed": 12,
               "labels": 4}
PATH_BYTES_PER_EDGE = sum(STAGE_BYTES.values())


def load_traffic(kernel: str, path: str) -> float | None:
    """Traffic per launch from a committed PMC summary, or None if the kernels changed since."""
    if not os.path.exists(path):
        return None
    with open(path) as fh:
        text = fh.read()
    start = text.find("```json")
    if start < 0:
        return None
    blob = json.loads(text[start + 7:text.find("```", start + 7)])
    if blob.get("kernel") != kernel or blob.get("source_hash") != source_hash():
        return None
    return blob.get("traffic_bytes_per_launch")


if __name__ == "__main__":
    import sys
    fetch_dir, write_dir, kernel, copy_bytes = sys.argv[1], sys.argv[2], sys.argv[3], int(sys.argv[4])
    if kernel == "pipeline":
        steps = int(sys.argv[5]) if len(sys.argv) > 5 else 1
        print(json.dumps(summarize_pipeline_pmc(fetch_dir, write_dir, copy_bytes, steps), indent=1))
    else:
        print(json.dumps(summarize_pmc(fetch_dir, write_dir, kernel, copy_bytes), indent=1))
