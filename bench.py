#!/usr/bin/env python3
"""Benchmark of the stencil hot path on one MI355X.

One "step" = one pass of the stencil over the workload's matrix (all of its iterations) at
the workgroup size the sweep found best.  Before the timed region the script runs the sweep
of Section 5 over the workload's whole size list (every size: 3 warm-ups + `--reps` samples),
reduces it (best size, speedup over the fixed sizes 4x4 and 32x4 / 4x32, best/worst) and asks
the predictor for a size.  Inputs are generated from a seed and are resident in HBM before
anything is timed.

The default workload is C5 (8192^2, 256 MiB each way): the one configuration that no cache
holds.  Passes of a single-application workload are timed on a rotation of matrix pairs, so that
no pass finds part of its input in the 256 MB last-level cache, where the pass before left it: its
bandwidth figure is then an HBM figure (the figure on one pair is reported beside it).  The other
workloads, and four heat steps on 8192^2 and 16384^2 matrices, follow as sub-records with the
same fields.

Prints ONE JSON line, short enough for a reader that keeps a few thousand characters: of the other
workloads and the sweeps it holds the outcome only (--record FILE writes the complete record).  `value` = Gcells/s (cell updates per second) of the timed steps;
`roofline` prices the stencil kernel's algorithmic bytes (one read + one write per cell
update) over its HIP-event-measured launch time against the 8 TB/s HBM peak, with the
arithmetic views beside it; `cpu_baseline` is the CPU oracle timed on a bounded sample of the
same workload on the host cores.
"""
from __future__ import annotations

import argparse
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
FP32_VECTOR_PEAK_TFLOPS = 157.3      # published: packed fp32 fma on 256 CUs x 4 SIMDs x 16 lanes at 2.4 GHz
# vector instructions the chip can issue per second, one lane each: 256 CUs x 4 SIMDs x 16 lanes x 2.4 GHz
VALU_LANE_ISSUE_PEAK = 256 * 4 * 16 * 2.4e9
ROTATION_BYTES = 512 << 20           # what lies between two uses of a matrix pair in the timed passes (twice the last-level cache)
ROTATION_MAX_PAIRS = 24
PRECONDITION_SECONDS = 0.06          # continuous untimed work ahead of every timed region (clock ramp)

WORKLOADS = ["C1", "C2", "C3", "C4", "C5", "H8192", "H16384", "W8192", "G5", "G7", "D5", "I5"]


def flops_per_cell_update(w):
    """fp32 operations the customising function states per cell and application (None: integer)."""
    n, s_, e, w_ = w.halo
    taps = (n + s_ + 1) * (e + w_ + 1)
    if w.kernel == "heat":
        return 7                     # three adds, 4u, the subtraction, alpha * t, the final add
    if w.kernel == "weighted_sum":
        return 2 * taps - 1 if w.dtype == "f32" else None
    if w.kernel == "sincos":
        return 3 * taps + 1          # per cell of the region: w * sin + cos and the running sum; sin and cos once
    return None

# mappings swept besides the paper's one element per work-item with a local-memory tile:
# (staging, cells_rows, cells_cols)
# ... or ("temporal", cells_rows, 4, applications per launch) for the iterated heat workload
MAPPINGS = {
    "weighted_sum": [("local", 1, 1), ("local", 2, 4), ("local", 4, 4), ("direct", 1, 4), ("direct", 2, 4),
                     ("direct", 4, 4), ("stream", 5, 4), ("stream", 10, 4), ("stream", 20, 4)],
    "heat": [("local", 1, 1), ("local", 2, 4), ("local", 4, 4), ("direct", 1, 4), ("direct", 2, 4),
             ("temporal", 2, 4, 2), ("temporal", 4, 4, 2), ("temporal", 4, 4, 3), ("temporal", 2, 4, 4),
             ("temporal", 4, 4, 4), ("temporal", 8, 4, 4),
             ("stream", 16, 4, 4), ("stream", 36, 4, 4), ("stream", 40, 4, 6), ("stream", 38, 4, 8),
             ("stream", 74, 4, 8)],
    "sincos": [("local", 1, 1), ("local", 2, 4), ("local", 4, 4), ("local", 8, 4),
               ("stream", 64, 4), ("stream", 67, 4), ("stream", 89, 4), ("stream", 134, 4)],
    "life": [("local", 1, 1), ("local", 1, 16), ("local", 2, 16), ("direct", 1, 16), ("direct", 2, 16),
             ("direct", 4, 16), ("direct", 8, 16), ("temporal", 2, 16, 2), ("temporal", 4, 16, 2), ("temporal", 2, 16, 4), ("temporal", 4, 16, 4),
             ("temporal", 8, 16, 4), ("stream", 16, 4, 4), ("stream", 40, 4, 6), ("stream", 20, 8, 8)],
}


def parse_args():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=0, help="timed steps (0 = per-workload default)")
    ap.add_argument("--warmup", type=int, default=-1)
    ap.add_argument("--workload", default="C5", choices=WORKLOADS,
                    help="C1..C5; four heat steps on a 8192^2 / 16384^2 matrix (H8192, H16384); a 28-tap weighted sum "
                         "with C5's border region, given at run time, on C5's matrix (W8192); a 5x5 / 7x7 Gaussian blur "
                         "of a 8192^2 matrix (G5, G7); the 5x5 blur of a 4096^2 matrix of doubles / of 32-bit "
                         "integers with binomial weights (D5, I5)")
    ap.add_argument("--iters", type=int, default=0,
                    help="applications per step instead of the workload's own number (profiling runs of iterated workloads)")
    ap.add_argument("--reps", type=int, default=30, help="timed samples per workgroup size in the sweep")
    ap.add_argument("--cpu-seconds", type=float, default=12.0, help="target CPU time of the oracle sample")
    ap.add_argument("--same-matrices", action="store_true",
                    help="time the passes of single-application workloads on one matrix pair (part of the input then comes "
                         "from the last-level cache) instead of a rotation of pairs")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-predictor", action="store_true", help="skip the leave-one-out predictor study")
    ap.add_argument("--no-others", action="store_true", help="skip the sub-records of the other workloads")
    ap.add_argument("--quick", action="store_true", help="sweep a thinned size list (development only)")
    ap.add_argument("--wg", default="", help="R,C: skip the sweep and time this workgroup size (profiling runs)")
    ap.add_argument("--mapping", default="", help="staging,cells_rows,cells_cols[,depth] to go with --wg, e.g. direct,2,4")
    ap.add_argument("--nt-store", default=None, choices=["0", "1"],
                    help="force plain (0) or non-temporal (1) output stores instead of timing both")
    ap.add_argument("--xcd-remap", default=None, choices=["0", "1"], help="workgroup numbering to go with --wg")
    ap.add_argument("--record", default="", metavar="FILE", help="write the complete record (the printed line is its summary)")
    ap.add_argument("--copy-only", action="store_true",
                    help="launch only the plain copy kernel on the workload's matrix (counter calibration)")
    return ap.parse_args()


def named_workload(wl, name):
    if name.startswith("C"):
        return wl.config(int(name[1]) - 1)
    if name in ("D5", "I5"):
        # the synthetic template's other element types (Section 3.3) on the paper's largest matrix
        import numpy as np
        if name == "D5":
            return wl.Workload("D5 gaussian5x5 4096x4096 f64 clamp", 4096, 4096, "f64", (2, 2, 2, 2), "clamp", 0.0,
                               wl.WEIGHTED_SUM, 1, wl.BASE_SEED + 20, "pow2", weights=wl.gaussian_weights(2, 1.0))
        b = np.array([1.0, 4.0, 6.0, 4.0, 1.0])
        return wl.Workload("I5 binomial5x5 4096x4096 i32 clamp", 4096, 4096, "i32", (2, 2, 2, 2), "clamp", 0.0,
                           wl.WEIGHTED_SUM, 1, wl.BASE_SEED + 21, "pow2", weights=np.outer(b, b).astype(np.float32))
    if name.startswith("G"):
        # Table 2's gaussian goes beyond C2's 5x5: the same blur, and the next size up, on a matrix no cache holds
        radius = {"G5": 2, "G7": 3}[name]
        w = wl.config(1, rows=8192, cols=8192)
        w.halo = (radius,) * 4
        w.weights = wl.gaussian_weights(radius, radius / 2.0)
        w.name = "%s gaussian%dx%d 8192x8192 f32 clamp" % (name, 2 * radius + 1, 2 * radius + 1)
        return w
    n = int(name[1:])
    if name.startswith("W"):
        # the lightweight synthetic stencil (Section 3.3) with C5's region: a border region the
        # library has no compiled variant for, so the run-time-region kernels serve it
        c5 = wl.config(4)
        weights = c5.weights / c5.weights.sum()
        return wl.Workload("%s weighted_sum N1S5E3W0 %dx%d f32 const0" % (name, n, n), n, n, "f32", c5.halo, "constant",
                           0.0, wl.WEIGHTED_SUM, 1, c5.seed, "pow2", weights=weights.astype("float32"))
    # four steps, so that every launch but the first reads what the launch before it wrote: nothing
    # of its input can have stayed in the 256 MB last-level cache from an earlier pass
    w = wl.config(3, rows=n, cols=n, iters=4)
    w.name = "%s heat %dx%d f32 wrap x4" % (name, n, n)
    return w


def device_matrices(torch, w):
    """(in, out) tensors of the workload, resident on the device.  The two matrices larger than C5
    are drawn on the device (the same distribution as C4's uniform fill)."""
    if w.rows * w.cols > 8192 * 8192:
        gen = torch.Generator(device="cuda")
        gen.manual_seed(w.seed)
        a = torch.rand(w.rows * w.cols, generator=gen, device="cuda", dtype=torch.float32) * 100.0
    else:
        a = torch.from_numpy(w.grid()).cuda()
    types = {"f32": torch.float32, "u8": torch.uint8, "i32": torch.int32, "f64": torch.float64}
    return a, torch.empty(a.shape, dtype=types[w.out_dtype], device="cuda")


def sweep_summary(res, cells_per_sample):
    import math as m
    legal = res.legal()
    out = {
        "sizes": len(res.sizes),
        "refused": sum(1 for s in res.status if s != 0),
        "best_wg": list(res.best) if res.best else None,
        "best_ms": res.best_ms,
        "best_gcells_s": cells_per_sample / res.best_ms / 1e6 if res.best else None,
        "worst_ms": res.worst_ms,
        "best_over_worst": res.worst_ms / res.best_ms if res.best else None,
    }
    for name, wg in (("4x4", (4, 4)), ("32x4", (32, 4)), ("4x32", (4, 32))):
        t = res.ms_of(wg)
        out["speedup_over_" + name] = (t / res.best_ms) if (res.best and not m.isnan(t)) else None
        out["gcells_s_" + name] = (cells_per_sample / t / 1e6) if not m.isnan(t) else None
    return out, legal


def apply_mapping(st, mapping):
    st.set_mapping(*mapping[:3])
    if len(mapping) > 3 and mapping[3]:
        st.set_option(1, mapping[3])      # STENCIL_OPT_TEMPORAL_DEPTH


def mapping_name(mapping):
    return "%s %dx%d" % tuple(mapping[:3]) + (" depth %d" % mapping[3] if len(mapping) > 3 and mapping[3] else "")


def sweep_burst(w):
    """Applications per timed sample.  An event pair costs a few microseconds, so a sample is
    a burst of back-to-back applications long enough (>= ~100 us at a nominal 4 TB/s) to make
    that negligible; at least 10 for the iterated workloads."""
    est_us = w.rows * w.cols * w.bytes_per_cell_update / 4e12 * 1e6
    burst = int(min(20, max(1, math.ceil(100.0 / max(est_us, 1e-3)))))
    return max(burst, 24) if w.iters > 1 else burst      # 24: a multiple of every temporal depth swept


# the vectorised mapping each kernel is usually fastest with (predictor study)
FAST_MAPPING = {"weighted_sum": ("local", 2, 4), "heat": ("direct", 2, 4), "sincos": ("local", 2, 4),
                "life": ("direct", 2, 16)}


# strong configurations of each kernel, swept together (stencil_sweep_configs) for the sub-records:
# (staging, cells_rows, cells_cols, applications per launch or 0, workgroup size[, numbering, non-temporal stores])
STRONG_CONFIGS = {
    "weighted_sum": [("local", 2, 4, 0, (16, 8)), ("local", 2, 4, 0, (8, 8)), ("direct", 2, 4, 0, (8, 16)),
                     ("direct", 4, 4, 0, (4, 128)), ("local", 4, 4, 0, (16, 8)), ("stream", 10, 4, 0, (1, 64)),
                     # the same with non-temporal output stores (numbering as is)
                     ("local", 2, 4, 0, (16, 8), -1, 1), ("direct", 2, 4, 0, (8, 16), -1, 1),
                     ("stream", 10, 4, 0, (1, 64), -1, 1), ("stream", 5, 4, 0, (1, 64), -1, 1)],
    "life": [("direct", 2, 16, 0, (2, 128)), ("direct", 4, 16, 0, (1, 256)), ("direct", 4, 16, 0, (1, 256), -1, 1),
             ("direct", 8, 16, 0, (2, 128), -1, 1), ("direct", 8, 16, 0, (1, 256), -1, 1),
             # (under "stream" only the generations per launch and the workgroup make a difference)
             ("temporal", 2, 16, 4, (64, 8)), ("stream", 20, 8, 8, (1, 64)), ("stream", 20, 8, 8, (2, 64)),
             ("stream", 20, 8, 8, (4, 64)), ("stream", 40, 4, 6, (4, 64))],
    "heat": [("direct", 2, 4, 0, (4, 16)), ("temporal", 2, 4, 4, (32, 32)), ("stream", 38, 4, 8, (1, 64)),
             ("stream", 38, 4, 8, (2, 64)), ("stream", 38, 4, 8, (1, 128)), ("stream", 40, 4, 6, (1, 64))],
    "sincos": [("local", 4, 4, 0, (8, 32)), ("local", 2, 4, 0, (18, 14)), ("stream", 89, 4, 0, (4, 64)),
               ("stream", 134, 4, 0, (32, 8)), ("stream", 134, 4, 0, (1, 64)),
               ("stream", 134, 4, 0, (32, 8), -1, 1), ("stream", 89, 4, 0, (4, 64), -1, 1),
               ("stream", 67, 4, 0, (32, 8), -1, 1)],
}
# one application of the heat step on matrices that no cache holds (256 MiB and 1 GiB each way): the
# workgroup sizes that win there are not those of the 4096^2 matrix, and the workgroup numbering and
# non-temporal output stores matter the other way round - the reason to sweep per dataset
LARGE_HEAT_CONFIGS = [(m, cr, 4, 0, wg, remap, nt)
                      for m, cr in (("direct", 2), ("direct", 4), ("local", 2), ("local", 4))
                      for wg in ((4, 16), (4, 64), (2, 256), (8, 64), (1, 512))
                      for remap in (1, 0) for nt in (0, 1)]


def marching_heights(w, slots=(2, 3, 4, 5, 6)):
    """Segment heights at which the marching kernel's wavefronts (strips x segments) just fill so many slots per SIMD."""
    from paper_1511_02490_amd import libstencil as ls
    st = ls.Stencil.from_workload(w)
    st.set_mapping("stream", 64, 4)
    heights = sorted({st.stream_segment_rows(k) for k in slots}, reverse=True)
    st.close()
    return heights


def strong_configs(w):
    if w.name.startswith("W"):
        return ([("local", cr, 4, 0, wg, -1, nt) for cr in (2, 4) for wg in ((8, 32), (4, 64), (8, 16)) for nt in (0, 1)] +
                [("stream", h, 4, 0, wg, -1, 1) for h in marching_heights(w) for wg in ((1, 64), (4, 64))])
    if w.name.startswith(("D5", "I5")):
        cc = 2 if w.dtype == "f64" else 4
        return ([("local", cr, cc, 0, wg, -1, nt) for cr in (2, 4) for wg in ((8, 32), (4, 64), (16, 16)) for nt in (0, 1)] +
                [("direct", cr, cc, 0, wg, -1, nt) for cr in (2, 4) for wg in ((4, 64), (4, 16)) for nt in (0, 1)] +
                [("local", 1, 1, 0, (16, 32), -1, 0)])
    if w.name.startswith("G"):
        return ([("local", cr, 4, 0, wg, remap, 1) for cr in (2, 4) for wg in ((8, 32), (4, 64), (8, 64)) for remap in (1, 0)] +
                [("direct", cr, 4, 0, wg, remap, 1) for cr in (2, 4) for wg in ((4, 64), (1, 512)) for remap in (1, 0)] +
                [("stream", h, 4, 0, wg, -1, 1) for h in marching_heights(w, (2, 3, 4, 5, 6, 8)) for wg in ((1, 64), (4, 64))])
    return LARGE_HEAT_CONFIGS if w.name.startswith("H") else STRONG_CONFIGS[w.kernel]


def kernel_label(w, mapping, info, nt, remap=1):
    """Name under which a kernel's rocprofv3 counters are kept in profiles/traffic.json: the kernel that runs
    (Stencil.describe_run), which need not be the mapping's own, its cells per work-item and its workgroup."""
    kernel = info["kernel"].split()[0]
    cells = (2, 4) if mapping[0] == "stream" and kernel == "tile_kernel" else mapping[1:3]
    return "%s: %s<%s>%s, wg %dx%d" % (
        w.name.split()[0], kernel, w.kernel,
        "" if kernel in ("register_tile_kernel", "life_stream_kernel") else " %dx%d cells/work-item" % tuple(cells), *info["wg"]) + (
        ", %d applications/launch" % info["applications"] if info["applications"] > 1 else "") + (
        ", non-temporal stores" if nt else "") + ("" if remap else ", plain workgroup numbering")


def recorded_counters(label):
    """What the committed rocprofv3 summaries hold for this kernel (HBM bytes per launch, vector
    instructions), or None when there is nothing for it or the kernel's sources have changed since
    the counters were taken."""
    from paper_1511_02490_amd import rocprof_summary as rs
    import re
    try:
        with open(rs.TRAFFIC_JSON) as fh:
            table = json.load(fh)
    except (OSError, ValueError):
        return None
    rec = table.get(label)
    if rec is None and any(k in label for k in (" stream_kernel<", " stream_through_kernel<", " march_kernel<", " march_masked_kernel<")):
        # in the streaming kernels a wavefront's accesses do not depend on how wavefronts are grouped
        # into workgroups: a record taken with another workgroup size of the same mapping serves
        strip = lambda k: re.sub(r", wg \d+x\d+", "", k)
        rec = next((v for k, v in sorted(table.items()) if strip(k) == strip(label)), None)
    if not rec or rec.get("source_hash") != rs.kernel_source_hash(rs.family_of(label)):
        return None
    return rec


def cpu_baseline(w, target_seconds):
    """The oracle, as it stands, on (the first rows of) the workload's matrix: whole passes of a
    bounded number of iterations, repeated until about `target_seconds` of CPU time have gone by
    (never less than one second), the sample sized from a short calibration run."""
    from oracle import stencil as oracle
    import copy
    threads = oracle.max_threads()
    ws = copy.copy(w)
    ws.rows = min(w.rows, 8192)            # the matrices beyond C5: their first 8192 rows
    g = ws.grid()
    run = lambda it, grid=g, th=0: oracle.apply(grid, w.kernel, w.halo, w.border, w.pad, w.weights, w.scalars, it, th)
    run(1, g[:64])                         # load the library, spawn the threads
    iters, dt = 1, 0.0
    while True:                            # calibration: the iterations one pass makes
        t0 = time.perf_counter()
        run(iters)
        dt = time.perf_counter() - t0
        if dt >= target_seconds / 3 or iters >= w.iters:
            break
        iters = int(min(w.iters, max(2 * iters, iters * 0.8 * target_seconds / max(dt, 1e-3))))
    passes = int(max(1, min(100000, math.ceil(max(1.0, 0.7 * target_seconds) / max(dt, 1e-6)))))
    t0 = time.perf_counter()
    for _ in range(passes):
        run(iters)
    dt = time.perf_counter() - t0
    # the same oracle on one thread, on a sample a tenth the size (context for the threaded figure)
    it1 = max(1, iters // 10)
    rows1 = ws.rows if iters >= 10 else max(64, ws.rows // 10)
    t1 = time.perf_counter()
    n1 = 0
    while True:
        run(it1, g[:rows1], 1)
        n1 += 1
        if time.perf_counter() - t1 >= min(1.0, target_seconds / 8):
            break
    dt1 = time.perf_counter() - t1
    run(1, g[:8], threads)                 # thread count back
    return {
        "value": ws.rows * w.cols * iters * passes / dt / 1e9,
        "unit": "Gcells/s",
        "cores": threads,
        "kind": "oracle",
        "sample": "%s %d x %d matrix, %d of %d iterations, %d passes, %.1f s" % (
            "whole" if ws.rows == w.rows else "first %d rows of the" % ws.rows, w.rows, w.cols, iters, w.iters, passes, dt),
        "single_thread": {"value": rows1 * w.cols * it1 * n1 / dt1 / 1e9, "unit": "Gcells/s", "cores": 1,
                          "sample": "first %d rows, %d iterations, %d passes, %.1f s" % (rows1, it1, n1, dt1)},
    }


class Bench:
    """One workload on the device: its handle, matrices and the measurements made on them."""

    def __init__(self, ls, torch, w, args):
        self.ls, self.torch, self.w, self.args = ls, torch, w, args
        self.st = ls.Stencil.from_workload(w)
        self.tin, self.tout = device_matrices(torch, w)
        self.cells = w.rows * w.cols
        self.burst = w.iters if w.name.startswith("H") else sweep_burst(w)
        self.alg_bytes = self.cells * w.bytes_per_cell_update
        self.pairs = [(self.tin, self.tout)]

    def close(self):
        self.st.close()
        del self.tin, self.tout, self.pairs

    def rotation(self):
        """The matrix pairs the timed passes of a single-application workload go round: copies of the
        input and outputs of their own, so many that a pair has left the last-level cache (256 MB, on
        the memory side: it holds what was read and what was written) when its turn comes again.
        Passes over one pair find part of the input there - 8192^2 floats: 96 instead of 118 us for
        the sin/cos stencil - which no stream of fresh matrices would.  Iterated workloads keep their
        one pair: what their applications leave in the caches for each other is theirs."""
        if len(self.pairs) == 1 and self.w.iters == 1 and not self.args.same_matrices:
            pair_bytes = self.tin.numel() * self.tin.element_size() + self.tout.numel() * self.tout.element_size()
            n = int(min(ROTATION_MAX_PAIRS, max(3, 1 + math.ceil(ROTATION_BYTES / pair_bytes))))
            self.pairs += [(self.tin.clone(), self.torch.empty_like(self.tout)) for _ in range(n - 1)]
            self.st.set_sweep_rotation(self.pairs)       # the library's sweeps go round the same pairs
        return self.pairs

    def run_pass(self, k, size):
        """The k-th pass of the workload, on the pair whose turn it is."""
        tin, tout = self.pairs[k % len(self.pairs)]
        self.st.run(tin, tout, self.w.iters, size)

    def timed_kernel(self, size, reps, one_pair=False):
        """Mean milliseconds per pass of the handle's current kernel: `reps` x `burst` passes back to back round
        the rotation (or on its first pair only) between two events on the launch stream.  Back to back: from idle
        the device needs some 30 ms of continuous work before a kernel's time settles."""
        torch = self.torch
        n_pairs = 1 if one_pair else len(self.rotation())
        n = reps * self.burst
        for k in range(min(n, 3 * n_pairs)):
            self.run_pass(k % n_pairs, size)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for k in range(n):
            self.run_pass(k % n_pairs, size)
        e1.record()
        e1.synchronize()
        return e0.elapsed_time(e1) / n

    def copy_reference(self, n=20):
        """GB/s of the plain copy kernel on this matrix (read + write), timed like a sweep sample."""
        mean_ms, _ = self.ls.time_copy(self.tin, self.tin.new_empty(self.tin.shape), burst=max(self.burst, 2), reps=n)
        return 2.0 * self.tin.numel() * self.tin.element_size() / (mean_ms * 1e-3) / 1e9

    def choose_stores(self, mapping, size):
        """Plain or non-temporal output stores for this configuration, whichever the sweep's clock
        prefers (forced by --nt-store); leaves the handle on that choice."""
        a, st, ls = self.args, self.st, self.ls
        if a.nt_store is not None:
            nt = int(a.nt_store)
        elif a.wg or mapping[2] == 1:      # one cell per work-item: no 16-byte stores to switch
            nt = 0
        else:
            depth = mapping[3] if len(mapping) > 3 else 0
            pair = [(mapping[0], mapping[1], mapping[2], depth, size, -1, flag) for flag in (0, 1)]
            mean, status, _ = st.sweep_configs(self.tin, self.tout, pair, iters=self.burst, reps=a.reps)
            # plain stores unless the others win by more than the run-to-run noise
            nt = 1 if (status[0] == ls.OK and status[1] == ls.OK and mean[1] < 0.98 * mean[0]) else 0
        apply_mapping(st, mapping)
        st.set_option(ls.OPT_NT_STORE, nt)
        return nt

    def choose_stores_for_steps(self, mapping, size):
        """The same choice for the timed steps, made on whole steps (all iterations of the workload):
        a short burst does not show what the stores do to a long chain of dependent launches."""
        a, st, ls, w, torch = self.args, self.st, self.ls, self.w, self.torch
        if a.nt_store is not None or a.wg or mapping[2] == 1 or w.iters == 1:
            return self.choose_stores(mapping, size)
        apply_mapping(st, mapping)
        took = []
        per_trial = 1
        for flag in (0, 1):
            st.set_option(ls.OPT_NT_STORE, flag)
            t_a = time.perf_counter()
            st.run(self.tin, self.tout, w.iters, size)
            torch.cuda.synchronize()
            if flag == 0:     # a trial lasts a few milliseconds, so that the host's part does not decide
                per_trial = max(1, min(500, int(0.004 / max(time.perf_counter() - t_a, 1e-6))))
            trials = []
            for _ in range(3):
                t_a = time.perf_counter()
                for _ in range(per_trial):
                    st.run(self.tin, self.tout, w.iters, size)
                torch.cuda.synchronize()
                trials.append(time.perf_counter() - t_a)
            took.append(min(trials))
        nt = 1 if took[1] < 0.98 * took[0] else 0
        st.set_option(ls.OPT_NT_STORE, nt)
        return nt

    def precondition(self, size, seconds=PRECONDITION_SECONDS):
        """Untimed passes of the workload, back to back, for `seconds`: from idle the chip needs some
        30 ms of continuous work before its clocks settle (a kernel of 95 us steady state takes 120 us
        during the first milliseconds), and it falls back within a second of idling."""
        w, torch = self.w, self.torch
        t0 = time.perf_counter()
        batch = max(1, min(8, 256 // max(1, w.iters)))       # a few hundred launches between synchronisations
        k = 0
        while time.perf_counter() - t0 < seconds:
            for _ in range(batch):
                self.run_pass(k, size)
                k += 1
            torch.cuda.synchronize()

    def timed_steps(self, size, steps, warmup):
        """(ms per step, Gcells/s) of `steps` whole passes, the handle as configured."""
        w, torch = self.w, self.torch
        self.rotation()
        self.precondition(size)
        for k in range(warmup):
            self.run_pass(k, size)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for k in range(steps):
            self.run_pass(warmup + k, size)
        torch.cuda.synchronize()
        dt = time.perf_counter() - t0
        return dt / steps * 1e3, self.cells * w.iters * steps / dt / 1e9

    def kernel_roofline(self, mapping, size, nt=None, remap=1):
        """Launch duration of one kernel by HIP events on the launch stream (the sweep's own clock)
        against what a launch must move: the matrix once each way, whatever the number of
        applications it fuses."""
        w, st, a = self.w, self.st, self.args
        if nt is None:
            nt = self.choose_stores(mapping, size)
        else:
            apply_mapping(st, mapping)
            st.set_option(self.ls.OPT_NT_STORE, nt)
        # what a sample's launches are (with a rotation of pairs: single applications)
        chain = self.burst if len(self.rotation()) == 1 else 1
        info = st.describe_run(chain, size)
        depth = info["applications"]
        per_launch = chain / info["launches"]            # on average: the last launch makes what is left
        self.precondition(size)
        k_res = st.sweep(self.tin, self.tout, [size], iters=self.burst, fixed=(0, 0), reps=max(a.reps, 30))
        launches = info["launches"] * (self.burst // chain)
        kernel_ms = same_ms = k_res.mean_ms[0] / launches
        if len(self.pairs) > 1:
            kernel_ms = self.timed_kernel(size, max(a.reps, 30))
            same_ms = self.timed_kernel(size, max(a.reps, 30), one_pair=True)
        achieved = self.alg_bytes / (kernel_ms * 1e-3) / 1e9
        label = kernel_label(w, mapping, info, nt, remap)
        rec = recorded_counters(label)
        out = {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
               "frac": achieved / HBM_PEAK_GBS, "traffic": rec["traffic_bytes_per_launch"] if rec else None,
               "kernel": label, "kernel_ms": kernel_ms, "algorithmic_bytes_per_launch": self.alg_bytes,
               "applications_per_launch": depth, "nt_store": nt,
               "gcells_s": self.cells * per_launch / (kernel_ms * 1e-3) / 1e9,
               "matrix_pairs_in_rotation": len(self.pairs)}
        if len(self.pairs) > 1:
            # the same launches on one matrix pair, part of whose input the last-level cache still holds
            same = self.alg_bytes / (same_ms * 1e-3) / 1e9
            out["on_one_matrix_pair"] = {"kernel_ms": same_ms, "achieved": same, "frac": same / HBM_PEAK_GBS,
                                         "note": "cache-assisted: not an HBM figure"}
        # the arithmetic views: algorithmic fp32 operations against the published vector peak ...
        flops = flops_per_cell_update(w)
        if flops:
            tflops = flops * self.cells * per_launch / (kernel_ms * 1e-3) / 1e12
            out["alu"] = {"bound": "alu", "achieved": tflops, "peak": FP32_VECTOR_PEAK_TFLOPS, "unit": "TFLOP/s",
                          "frac": tflops / FP32_VECTOR_PEAK_TFLOPS, "flops_per_cell_update": flops}
        # ... and vector instructions issued (rocprofv3 SQ_INSTS_VALU, 64 lanes each; an instruction of
        # the transcendental unit holds its issue slot four times as long) against the chip's issue rate
        if rec and rec.get("valu_insts_per_launch"):
            slots = (rec["valu_insts_per_launch"] + 3.0 * rec.get("valu_trans_insts_per_launch", 0.0)) * 64.0
            rate = slots / (kernel_ms * 1e-3)
            out["valu_issue"] = {"bound": "alu", "achieved": rate / 1e12, "peak": VALU_LANE_ISSUE_PEAK / 1e12,
                                 "unit": "T lane-instructions/s", "frac": rate / VALU_LANE_ISSUE_PEAK,
                                 "valu_insts_per_cell_update": rec["valu_insts_per_launch"] * 64.0 / (self.cells * per_launch),
                                 "issue_slots_per_cell_update": slots / (self.cells * per_launch),
                                 "valu_busy_frac_in_profile": rec.get("valu_busy_frac")}
        return out


def sub_record(ls, torch, wl, name, args):
    """A workload other than the benchmarked one, with the same fields: the fastest of its strong
    configurations (stencil_sweep_configs), timed steps with it, the roofline of its best kernel
    that makes one application per launch (and of the fused one the steps used), the oracle."""
    w = named_workload(wl, name)
    b = Bench(ls, torch, w, args)
    reps = max(5, args.reps // 3)
    configs = strong_configs(w)
    b.rotation()
    mean, status, best = b.st.sweep_configs(b.tin, b.tout, configs, iters=b.burst, reps=reps)
    ok = [k for k in range(len(configs)) if status[k] == ls.OK]
    if not ok:
        b.close()
        return None
    as_mapping = lambda c: (c[0], c[1], c[2]) + ((c[3],) if c[3] else ())
    flags = lambda c: (c[5] if len(c) > 5 else -1, c[6] if len(c) > 6 and c[6] >= 0 else 0)
    def configure(cfg):
        apply_mapping(b.st, as_mapping(cfg))
        remap, nt = flags(cfg)
        if remap >= 0:
            b.st.set_option(ls.OPT_XCD_REMAP, remap)
        b.st.set_option(ls.OPT_NT_STORE, nt)
        return nt

    if len(b.rotation()) > 1:
        # the sweep's samples are short; the ranking that counts is over longer runs of back-to-back passes
        for k in ok:
            configure(configs[k])
            b.precondition(configs[k][4], 0.01)
            mean[k] = b.timed_kernel(configs[k][4], max(reps, 20)) * b.burst
        best = min(ok, key=lambda k: mean[k])
    c = configs[best]
    single = [k for k in ok if not configs[k][3]]
    c1 = configs[min(single, key=lambda k: mean[k])] if single else None

    nt = configure(c)
    info = b.st.describe_run(w.iters, c[4])
    steps = {"C1": 200, "C2": 200, "C3": 10, "C4": 3, "C5": 30, "H8192": 50, "H16384": 20, "W8192": 30, "G5": 30, "G7": 30, "D5": 50, "I5": 50}[name]
    ms_per_step, value = b.timed_steps(c[4], steps, max(1, steps // 10))
    out = {"workload": w.name, "metric": "Gcells/s", "value": value, "unit": "Gcells/s", "ms_per_step": ms_per_step,
           "steps": steps, "dtype": w.dtype,
           "config": {"rows": w.rows, "cols": w.cols, "iters": w.iters, "mapping": mapping_name(as_mapping(c)),
                      "wg": list(c[4]), "xcd_remap": flags(c)[0], "nt_store": nt,
                      "applications_per_launch": info["applications"], "kernel": info["kernel"], "configurations_swept": len(configs),
                      "matrix_pairs_in_rotation": len(b.pairs)}}
    if c1 is not None:
        nt1 = configure(c1)
        out["roofline"] = b.kernel_roofline(as_mapping(c1), c1[4], nt=nt1, remap=0 if flags(c1)[0] == 0 else 1)
        out["roofline"]["xcd_remap"] = flags(c1)[0]
    if c[3]:
        nt = configure(c)
        out["roofline_timed_kernel"] = b.kernel_roofline(as_mapping(c), c[4], nt=nt)
    if "roofline" in out:
        out["roofline"]["copy_kernel_gbs"] = b.copy_reference()
        if name.startswith("H"):
            at = configs.index(("direct", 2, 4, 0, (4, 16), 1, 0))          # the 4096^2 matrix's best
            if status[at] == ls.OK:
                gbs = b.alg_bytes / (mean[at] / b.burst) / 1e6
                out["with_the_4096_best"] = {"algorithmic_gbs": gbs, "frac_of_hbm_peak": gbs / HBM_PEAK_GBS}
    b.close()
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(w, min(3.0, args.cpu_seconds))
    return out


def leave_one_out_prediction(ls, wl, torch, index, mapping_of, reps):
    """Section 7's leave-one-out evaluation in miniature: sweep the other four workloads, train
    the classifier on their (f(s), Omega(s)) pairs, predict for workload `index` with the
    NearestNeighbour fallback of Algorithm 1.  Returns (predictor, training table)."""
    pred = ls.Predictor()
    table = []
    for i in range(5):
        if i == index:
            continue
        o = wl.config(i)
        st = ls.Stencil.from_workload(o)
        st.set_mapping(*mapping_of(o))
        st.set_option(ls.OPT_SWEEP_CUTOFF, 300)      # training sweeps: adaptive sampling
        a = torch.from_numpy(o.grid()).cuda()
        b = torch.empty_like(a)
        burst = sweep_burst(o)
        res = st.sweep(a, b, o.wg_sizes(), iters=burst, fixed=(0, 0), reps=reps)
        if res.best:
            pred.add(st.features(), res.best)
            table.append({"workload": o.name.split()[0], "oracle_wg": list(res.best),
                          "mapping": mapping_name(mapping_of(o)), "ms_per_application": res.best_ms / burst})
        st.close()
        del a, b
    return pred, table


def rounded(x):
    """The record with its floats to six significant digits."""
    if isinstance(x, float):
        return float("%.6g" % x) if math.isfinite(x) else None
    if isinstance(x, dict):
        return {k: rounded(v) for k, v in x.items()}
    if isinstance(x, (list, tuple)):
        return [rounded(v) for v in x]
    return x


def summary(out):
    """What goes to stdout of the complete record: the same fields, the sweeps and the other workloads by their outcome."""
    pick = lambda d, *keys: {k: d[k] for k in keys if d and d.get(k) is not None}
    short = dict(out)
    short["sweep"] = {"seconds": out["sweep"]["seconds"],
                      "best_by_mapping": {name: [s["best_wg"], s["best_gcells_s"]] for name, s in out["sweep"]["by_blocking"].items()}}
    short["predictor"] = {tag: pick(p, "mapping", "predicted_wg", "oracle_wg", "performance") for tag, p in out["predictor"].items()}
    short["other_workloads"] = {
        name: dict(pick(r, "value", "ms_per_step"), **pick(r["config"], "mapping", "wg", "nt_store"),
                   **{"one_per_launch": pick(r.get("roofline"), "kernel_ms", "achieved", "frac")})
        for name, r in out["other_workloads"].items() if r}
    return rounded({k: v for k, v in short.items() if v not in (None, {}) or k in ("vs_baseline", "roofline", "config")})


def main():
    args = parse_args()
    if args.gpus != 1:
        print("bench.py: this build measures one GPU only (--gpus 1); no multi-GPU path exists.", file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_1511_02490_amd import libstencil as ls
    from paper_1511_02490_amd import workloads as wl

    if not torch.cuda.is_available():
        print("bench.py: no GPU visible", file=sys.stderr)
        sys.exit(1)
    torch.cuda.set_device(0)

    w = named_workload(wl, args.workload)
    if args.iters > 0:
        w.iters = args.iters
    index = int(args.workload[1]) - 1 if args.workload.startswith("C") else -1
    sizes = w.wg_sizes()
    if args.quick:
        sizes = sizes[::5]
    b = Bench(ls, torch, w, args)
    b.rotation()            # single-application workloads: every sweep below goes round fresh matrix pairs
    st, tin, tout, burst, cells = b.st, b.tin, b.tout, b.burst, b.cells
    cells_per_sample = cells * burst

    steps = args.steps if args.steps > 0 else {"C1": 200, "C2": 200, "C3": 20, "C4": 5, "C5": 100, "H8192": 100,
                                               "H16384": 30, "W8192": 100, "G5": 100, "G7": 100, "D5": 100, "I5": 100}[args.workload]
    warmup = args.warmup if args.warmup >= 0 else max(1, steps // 10)

    if args.copy_only:
        gbs = b.copy_reference(max(steps, 20))
        print(json.dumps({"metric": "plain copy kernel GB/s (read+write)", "value": gbs, "unit": "GB/s",
                          "config": {"workload": w.name, "bytes_each_way": tin.numel() * tin.element_size()}}))
        return

    sweeps, sweep_seconds, predictor, best_vs_fixed, confirmation = {}, 0.0, {}, None, None
    confirmed_nt = best1_nt = None       # the kind of output stores the confirmation pass settled on
    ls.time_copy(tin, tin.new_empty(tin.shape), burst=20, reps=max(10, int(4e9 / max(tin.numel() * tin.element_size(), 1)) // 20))   # clocks up before the first sweep
    if args.wg:
        wg = tuple(int(x) for x in args.wg.split(","))
        m = args.mapping.split(",") if args.mapping else ["local", "1", "1"]
        blocking = (m[0],) + tuple(int(x) for x in m[1:])
        apply_mapping(st, blocking)
        if args.xcd_remap is not None:
            st.set_option(ls.OPT_XCD_REMAP, int(args.xcd_remap))
        best1 = (float("nan"), blocking, wg) if len(blocking) == 3 else None
    else:
        t_sweep0 = time.perf_counter()
        best = None    # (ms per sample, mapping, wg) over every mapping
        best1 = None   # the same over the mappings that make one application per launch
        best_wg_tuned = None   # ... and over those in which the workgroup size is the tunable (local, direct)
        candidates = []        # every (ms per sample, mapping, wg) that was timed
        mappings = list(MAPPINGS[w.kernel])
        if w.kernel == "weighted_sum" and w.dtype == "f32" and w.rows >= 4096:
            try:        # the marching kernel at the heights that fill whole wavefront slots on a matrix of this size
                mappings += [("stream", h, 4) for h in marching_heights(w, (2, 3, 4, 6)) if ("stream", h, 4) not in mappings]
            except ls.StencilError:
                pass    # a region the marching kernels do not have
        for mapping in mappings:
            try:
                apply_mapping(st, mapping)
            except ls.StencilError:
                continue                 # a mapping this scenario does not have (border mode, region)
            res = st.sweep(tin, tout, sizes, iters=burst, fixed=(4, 4), reps=args.reps)
            summ, _ = sweep_summary(res, cells_per_sample)
            summ["w_max"] = st.max_wg_size()
            sweeps[mapping_name(mapping)] = summ
            candidates.extend((t, mapping, sz) for sz, t in res.legal())
            if res.best and (best is None or res.best_ms < best[0]):
                best = (res.best_ms, mapping, res.best)
            if res.best and len(mapping) == 3 and (best1 is None or res.best_ms < best1[0]):
                best1 = (res.best_ms, mapping, res.best)
            if res.best and mapping[0] in ("local", "direct") and (best_wg_tuned is None or res.best_ms < best_wg_tuned[0]):
                best_wg_tuned = (res.best_ms, mapping, res.best)
        sweep_seconds = time.perf_counter() - t_sweep0
        assert best is not None, "no legal workgroup size"
        # Confirmation pass.  A size's samples last a few milliseconds, the sweeps use plain output
        # stores only, and near the top the landscape is flat: the best size of every mapping that
        # came within 15 % of the best, and the three best sizes overall, are timed again with both
        # kinds of store, each over a longer run of back-to-back passes after PRECONDITION_SECONDS
        # of its own launches, and the fastest is taken.
        per_mapping = {}
        for c in sorted(candidates, key=lambda c: c[0]):
            per_mapping.setdefault(mapping_name(c[1]), c)
        close = [c for c in per_mapping.values() if c[0] <= 1.15 * best[0]]
        close += [c for c in sorted(candidates, key=lambda c: c[0])[:3] if c not in close]
        # The sweeps ran with plain output stores; here both kinds of store are timed (where the
        # mapping has 16-byte stores to switch), since which is better depends on the kernel.
        confirmed = []
        b.rotation()
        for ms, mapping, size in close:
            for nt in ((0, 1) if (mapping[2] > 1 and args.nt_store is None) else (int(args.nt_store or 0),)):
                apply_mapping(st, mapping)
                st.set_option(ls.OPT_NT_STORE, nt)
                b.precondition(size)
                if len(b.rotation()) > 1:
                    confirmed.append((b.timed_kernel(size, args.reps) * burst, mapping, size, ms, nt))
                else:
                    res = st.sweep(tin, tout, [size], iters=burst, fixed=(0, 0), reps=args.reps)
                    confirmed.append((res.mean_ms[0], mapping, size, ms, nt))
        st.set_option(ls.OPT_NT_STORE, 0)
        # plain stores (the library's default) unless the others win by more than the run-to-run noise
        plain = {(c[1], c[2]): c[0] for c in confirmed if c[4] == 0}
        confirmed = [c for c in confirmed if c[4] == 0 or (c[1], c[2]) not in plain or c[0] < 0.98 * plain[(c[1], c[2])]]
        confirmed.sort(key=lambda c: c[0])
        best = confirmed[0][:3]
        confirmed_nt = confirmed[0][4]
        singles = [c for c in confirmed if len(c[1]) == 3]
        if singles:
            best1 = singles[0][:3]
            best1_nt = singles[0][4]
        confirmation = [{"mapping": mapping_name(m), "wg": list(sz), "nt_store": nt, "ms_in_sweep": ms0, "ms_confirmed": ms}
                        for ms, m, sz, ms0, nt in confirmed]
        _, blocking, wg = best
        apply_mapping(st, blocking)
        # The paper's question - what the best workgroup size is worth over a fixed one - put to the
        # mappings in which the workgroup size decides the decomposition (in the register-streaming
        # mappings it only groups wavefronts and most sizes are refused): the paper's own mapping
        # first, then the fastest of them.
        if best_wg_tuned is not None:
            pick = lambda name: {k: sweeps[name][k] for k in (
                "sizes", "refused", "best_wg", "best_gcells_s", "best_over_worst", "speedup_over_4x4", "gcells_s_4x4",
                "speedup_over_32x4", "speedup_over_4x32")}
            best_vs_fixed = {"paper_mapping": dict(mapping="local 1x1", **pick("local 1x1")) if "local 1x1" in sweeps else None,
                             "fastest_tile_or_direct_mapping": dict(mapping=mapping_name(best_wg_tuned[1]),
                                                                    **pick(mapping_name(best_wg_tuned[1])))}

        # Algorithm 1 on this scenario, for the best mapping's family and for the paper's
        # mapping: train on the other four workloads' sweeps, predict, repair an illegal
        # prediction (NearestNeighbour), and score it on this workload's own sweep table.
        if not args.no_predictor and index >= 0:
            for tag, mapping_of in (("fast", lambda o: FAST_MAPPING[o.kernel]), ("paper", lambda o: ("local", 1, 1))):
                pred, table = leave_one_out_prediction(ls, wl, torch, index, mapping_of, max(5, args.reps // 3))
                mine = mapping_of(w)
                apply_mapping(st, mine)
                res = st.sweep(tin, tout, sizes, iters=burst, fixed=(4, 4), reps=max(5, args.reps // 3))
                p = st.predict(pred, sizes)
                t_p = res.ms_of(p)
                if math.isnan(t_p) and st.is_legal(*p):
                    t_p = st.sweep(tin, tout, [p], iters=burst, fixed=(0, 0), reps=args.reps).mean_ms[0]
                t4 = res.ms_of((4, 4))
                pretrained = None
                if mine == ("local", 1, 1):
                    # the classifier shipped with the library (trained offline on the 128-scenario study)
                    shipped = ls.pretrained_predictor("local,1,1")
                    q = st.predict(shipped, sizes)
                    shipped.close()
                    t_q = res.ms_of(q)
                    pretrained = {"predicted_wg": list(q),
                                  "performance": (res.best_ms / t_q) if not math.isnan(t_q) else None}
                predictor[tag] = {"mapping": mapping_name(mine), "pretrained": pretrained,
                                  "trained_on": table, "predicted_wg": list(p),
                                  "oracle_wg": list(res.best), "performance": res.best_ms / t_p,
                                  "speedup_over_4x4": (t4 / t_p) if not math.isnan(t4) else None}
            apply_mapping(st, blocking)

    if confirmed_nt is not None and w.iters == 1:
        nt_store = confirmed_nt
        apply_mapping(st, blocking)
        st.set_option(ls.OPT_NT_STORE, nt_store)
    else:
        nt_store = b.choose_stores_for_steps(blocking, wg)
    timed_run = st.describe_run(w.iters, wg)
    ms_per_step, value = b.timed_steps(wg, steps, warmup)

    # `roofline` prices the best kernel that makes ONE application per launch: that is the
    # kernel whose bytes are all compulsory.  A temporally blocked kernel moves the matrix once
    # per `depth` applications, so its per-launch figure says little about HBM; it is reported
    # beside it as `roofline_timed_kernel` when it is the one the timed steps used.
    roofline_timed = None
    if len(blocking) > 3 and best1 is not None:
        roofline = b.kernel_roofline(best1[1], best1[2], nt=best1_nt)
        roofline_timed = b.kernel_roofline(blocking, wg)
        roofline["note"] = ("single-application kernel; the timed steps used the temporally blocked kernel "
                            "in roofline_timed_kernel")
    else:
        roofline = b.kernel_roofline(blocking, wg, nt=nt_store, remap=0 if args.xcd_remap == "0" else 1)
    roofline["copy_kernel_gbs"] = b.copy_reference()
    n_pairs = len(b.pairs)
    b.close()

    others = {}
    if not (args.wg or args.quick or args.no_others):
        for name in ("C4", "H8192", "H16384", "C3", "C2", "C1", "C5", "W8192", "G5", "G7", "D5", "I5"):
            if name != args.workload:
                others[name] = sub_record(ls, torch, wl, name, args)

    out = {
        "metric": "Gcells/s at best swept workgroup size (achieved HBM GB/s in roofline)",
        "value": value, "unit": "Gcells/s", "n_gpus": 1, "steps": steps, "warmup": warmup,
        "ms_per_step": ms_per_step, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": w.dtype, "data": "synthetic",
        "config": {"workload": w.name, "rows": w.rows, "cols": w.cols, "iters": w.iters,
                   "halo_nsew": list(w.halo), "border": w.border, "best_wg": list(wg),
                   "staging": blocking[0], "cells_per_work_item": list(blocking[1:3]),
                   "applications_per_launch": timed_run["applications"],
                   "nt_store": nt_store, "sweep_burst": burst, "sweep_reps": args.reps,
                   "preconditioning_seconds": PRECONDITION_SECONDS, "matrix_pairs_in_rotation": n_pairs},
        "roofline": roofline,
        "roofline_timed_kernel": roofline_timed,
        "best_vs_fixed": best_vs_fixed,
        "sweep": {"seconds": sweep_seconds, "confirmation_pass": confirmation, "by_blocking": sweeps},
        "predictor": predictor,
        "other_workloads": others,
    }
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(w, args.cpu_seconds)
    if args.record:
        with open(args.record, "w") as fh:
            json.dump(rounded(out), fh, indent=1)
    print(json.dumps(summary(out)))


if __name__ == "__main__":
    main()
