"""Benchmark of the wavefront sweep on one MI355X.

    python bench.py [--gpus 1] [--steps K] [--warmup W] [--n 16384] [--no-cpu] [--no-batch]
                    [--calib-copy]

Workload: one 16384 x 16384 float32 instance, values normal(0,1) clipped to [-4, 4]
(seed 2), resident in HBM before timing.  A step is the whole differentiable sweep:
  1. wf_forward: the table D, the score and the checkpoint grid (band rows every 64 rows,
     block columns every K = 64 columns), one persistent kernel;
  2. wf_backward with g_score = 1 and no g_D (the score's gradient): the selections
     recomputed from C and the checkpoint grid together with the exits of every band's
     last row and the zeroed gradient, the exits composed over groups of bands, and the
     walk of the argmin path per band.
Prints ONE JSON line: cells/s of the step (value), per-sweep cells/s and effective HBM
rates (3 m n sizeof(elem) per sweep), method-byte HBM rates of the forward kernel and of
the adjoint call measured with HIP events on the launch stream (the selection bit-planes
and the exits, intermediates of the adjoint, are reported apart), the roofline entry of
the one that takes the longest, the adjoint with an upstream gradient of the table (the
reverse pipeline) timed beside it, the CPU oracle timed on a bounded sample on this host
(the whole matrix when it fits the budget), and the error of this run's table, score and
gradient against that oracle.  Also measured,
as extra keys: the ragged batch (512 instances, one graph replay), the batched
differentiable sweep (64 instances of 2048 x 2048, forward with checkpoints + adjoint), the
smooth (soft-min) sweep of the same 16384 x 16384 matrix, and the tridiagonal partition
solver on a system of 10^8 unknowns in float64.
"""
from __future__ import annotations

import argparse
import hashlib
import json
import os
import re
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_HBM_GBPS = 8000.0  # MI355X published HBM3E bandwidth
CKPT_K = 64
PROFILES = os.path.join(ROOT, "profiles")
# kernel -> (summary file of its measured HBM traffic, sources its code comes from)
KERNELS = {
    "fwd_kernel": ("fwd_kernel_f32_16384_traffic.txt", ["wf_fwd.hip", "wf_common.h", "wf_internal.h"]),
    "sel_kernel": ("sel_kernel_f32_16384_traffic.txt", ["wf_bwd.hip", "wf_common.h", "wf_internal.h"]),
    "adj_kernel": ("adj_kernel_f32_16384_traffic.txt", ["wf_bwd.hip", "wf_common.h", "wf_internal.h"]),
    "path_adjoint": ("path_adjoint_f32_16384_traffic.txt",
                     ["wf_bwd.hip", "wf_common.h", "wf_internal.h", "wf_path.h", "wf_api.hip"]),
    "stage1_level0": ("tri_stage1_f64_1e8_traffic.txt", ["tri.hip"]),
    "stage3_level0": ("tri_stage3_f64_1e8_traffic.txt", ["tri.hip"]),
}


def parse():
    p = argparse.ArgumentParser()
    p.add_argument("--gpus", type=int, default=1)
    p.add_argument("--steps", type=int, default=20)
    p.add_argument("--warmup", type=int, default=3)
    p.add_argument("--n", type=int, default=16384)
    p.add_argument("--no-cpu", action="store_true", help="skip the CPU oracle baseline")
    p.add_argument("--no-batch", action="store_true", help="skip the ragged-batch and batched-adjoint measurements")
    p.add_argument("--no-tri", action="store_true", help="skip the tridiagonal partition solver measurement")
    p.add_argument("--no-soft", action="store_true", help="skip the soft-min sweep measurement")
    p.add_argument("--calib-copy", action="store_true",
                   help="first run one plain device copy of m*n elements (HBM counter calibration)")
    return p.parse_args()


def source_hash(files) -> str:
    h = hashlib.sha256()
    for f in files:
        with open(os.path.join(ROOT, "paper_2510_27351_amd", "csrc", f), "rb") as fh:
            h.update(fh.read())
    return h.hexdigest()[:16]


def measured_traffic(kernel: str):
    """HBM bytes per launch of 'kernel' from the committed counter summary, or None when the
    summary is missing or was taken on other kernel sources."""
    fname, files = KERNELS[kernel]
    try:
        text = open(os.path.join(PROFILES, fname)).read()
    except OSError:
        return None
    src = re.search(r"^source_hash:\s*(\S+)", text, re.M)
    val = re.search(r"^hbm_bytes_per_launch:\s*([0-9.eE+]+)", text, re.M)
    if not src or not val or src.group(1) != source_hash(files):
        return None
    return float(val.group(1))


def host_cpu() -> dict:
    """The host's CPU model and core counts (the oracle runs on one of them)."""
    model = None
    try:
        with open("/proc/cpuinfo") as fh:
            for line in fh:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    return {"cpu_model": model, "logical_cpus": os.cpu_count(), "cpus_available": len(os.sched_getaffinity(0))}


def cpu_baseline(C_cpu, budget_s: float = 15.0):
    """Times the CPU oracle (single-threaded C, float64, row by row) on a bounded leading
    block of the same matrix: forward with the selection map, then the adjoint of the score.
    The block edge is grown from a probe so that the timed call takes about budget_s (capped
    at the whole matrix).  Returns the baseline entry and, when the block is the whole matrix,
    the oracle's float64 table, selections and adjoint for the error report."""
    import numpy as np

    import oracle
    oracle.build(force=False)
    n = C_cpu.shape[0]

    def run(r):
        block = C_cpu[:r, :r].numpy().astype(np.float64)
        t0 = time.perf_counter()
        D64, sel = oracle.forward(block, "f64", want_sel=True)
        g64 = oracle.backward(sel, None, 1.0, "f64")
        return time.perf_counter() - t0, (D64, sel, g64)

    r = min(n, 1024)
    dt, _ = run(r)
    r2 = int(min(n, r * max(1.0, (budget_s / max(dt, 1e-3)) ** 0.5)))
    dt, outs = run(r2)
    entry = {"value": r2 * r2 / dt, "unit": "cells/s", "cores": 1, "kind": "oracle",
             "sample": f"top-left {r2}x{r2} block of the same matrix; f64 row-by-row C oracle, "
                       f"forward with selection map then adjoint of the score, one thread, {dt:.2f} s",
             "host": host_cpu()}
    return entry, (outs if r2 == n else None)


def result_errors(C_cpu, D, score, gC, oracle64):
    """Error of this run's results against the oracle: the table and score against the float64
    forward (normwise, and elementwise with the worst cell: the inputs are signed, so D crosses
    zero), the score's gradient against the float32 oracle (bitwise) and the float64 one
    (cells that differ are float32/float64 selection flips at near-ties)."""
    import numpy as np

    import oracle
    D64, sel64, g64 = oracle64
    Dn = D.cpu().numpy()
    diff = np.abs(Dn.astype(np.float64) - D64)
    normwise = float(diff.max() / np.abs(D64).max())
    rel = diff / np.maximum(np.abs(D64), np.finfo(np.float64).tiny)
    w = np.unravel_index(int(np.argmax(rel)), rel.shape)
    s64 = float(D64[-1, -1])
    fwd = {"vs": "float64 oracle", "normwise_max_err": normwise, "elementwise_max_rel_err": float(rel[w]),
           "worst_cell": [int(w[0]), int(w[1])], "score_rel_err": abs(float(score) - s64) / abs(s64)}
    del diff, rel
    D32, sel32 = oracle.forward(C_cpu.numpy(), "f32", want_sel=True)
    fwd["bitwise_equal_f32_oracle"] = bool(np.array_equal(Dn, D32))
    del Dn, D32
    g = gC.cpu().numpy()
    g32 = oracle.backward(sel32, None, 1.0, "f32")
    g64s = oracle.backward(sel32, None, 1.0, "f64")
    adj = {"bitwise_equal_f32_oracle": bool(np.array_equal(g, g32)),
           "max_rel_err_vs_f64_adjoint_on_same_selections": float(np.abs(g - g64s).max()),
           "cells_differing_from_f64_oracle": int(np.count_nonzero(g != g64)),
           "selection_flips_f32_f64": int(np.count_nonzero(sel32 != sel64))}
    return {"fwd": fwd, "adjoint": adj}


def batch_rate(steps: int, warmup: int):
    """The ragged batch (512 instances, m and n uniform in [64, 2048], seed 3, float32
    uniform [0,1)): one autotuned plan, tables written, graph replays timed with events."""
    import torch

    import paper_2510_27351_amd as wf
    from paper_2510_27351_amd import inputs

    ms, ns, mats = inputs.ragged_batch_f32()
    plan = wf.Plan(ms, ns)
    C = plan.pack([x.cuda() for x in mats])
    del mats
    D = torch.empty(plan.elems, device=C.device)
    scores = torch.empty(plan.batch, device=C.device)
    for _ in range(max(warmup, 1)):
        plan.forward(C, D=D, scores=scores)
    wf.last_async_error()
    stream = torch.cuda.current_stream()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    e0.record(stream)
    for _ in range(steps):
        plan.forward(C, D=D, scores=scores)
    e1.record(stream)
    torch.cuda.synchronize()
    wf.last_async_error()
    ms_per = e0.elapsed_time(e1) / steps
    cells = sum(m * n for m, n in zip(ms, ns))
    out = {"workload": "512 instances, m and n uniform in [64, 2048] (seed 3), float32 uniform [0,1), "
                       "tables written; one persistent launch per replay of the captured graph",
           "cells": cells, "ms": ms_per, "cells_per_s": cells / (ms_per * 1e-3),
           "effective_GBps": 3 * cells * 4 / (ms_per * 1e-3) / 1e9, "tile": plan.tile, "rows": plan.table_rows}
    plan.close()
    return out


def c5_rate(steps: int, warmup: int):
    """The batched differentiable sweep: 64 instances of 2048 x 2048 float32 uniform [0,1)
    (seed 4), one plan; a step is the batched forward (scores and every instance's checkpoint
    grid, K = 64) and the batched adjoint of the sum of the scores from those grids, each
    timed with HIP events on the launch stream."""
    import torch

    import paper_2510_27351_amd as wf
    from paper_2510_27351_amd import inputs

    C3, _ = inputs.batch_2048_f32()
    B, m, n = C3.shape
    plan = wf.Plan([m] * B, [n] * B, offsets=[b * m * n for b in range(B)])
    C = C3.reshape(-1).cuda()
    del C3
    scores = torch.empty(B, device=C.device)
    ones = torch.ones(B, device=C.device)
    ck = torch.empty(plan.ckpt_elems(CKPT_K), device=C.device)
    gC = torch.empty_like(C)
    for _ in range(max(warmup, 1)):
        plan.forward_ckpt(C, CKPT_K, scores=scores, ckpt=ck)
        plan.backward(C, g_scores=ones, ckpt=ck, ckpt_k=CKPT_K, g_C=gC)
    wf.last_async_error()
    stream = torch.cuda.current_stream()
    ev = [[torch.cuda.Event(enable_timing=True) for _ in range(3)] for _ in range(steps)]
    torch.cuda.synchronize()
    for k in range(steps):
        ev[k][0].record(stream)
        plan.forward_ckpt(C, CKPT_K, scores=scores, ckpt=ck)
        ev[k][1].record(stream)
        plan.backward(C, g_scores=ones, ckpt=ck, ckpt_k=CKPT_K, g_C=gC)
        ev[k][2].record(stream)
    torch.cuda.synchronize()
    wf.last_async_error()
    f_ms = sum(e[0].elapsed_time(e[1]) for e in ev) / steps
    b_ms = sum(e[1].elapsed_time(e[2]) for e in ev) / steps
    cells = B * m * n
    eff = lambda t: 3 * cells * 4 / (t * 1e-3) / 1e9  # noqa: E731
    out = {"workload": f"{B} instances of {m}x{n} float32 uniform [0,1) (seed 4); forward writes scores and "
                       f"checkpoint grids (K={CKPT_K}), adjoint of sum(scores) from the grids; one plan",
           "cells": cells, "tile": plan.tile, "rows": plan.rows,
           "fwd": {"ms": f_ms, "cells_per_s": cells / (f_ms * 1e-3), "effective_GBps": eff(f_ms)},
           "adjoint": {"ms": b_ms, "cells_per_s": cells / (b_ms * 1e-3), "effective_GBps": eff(b_ms)},
           "fwd_adjoint": {"ms": f_ms + b_ms, "cells_per_s": cells / ((f_ms + b_ms) * 1e-3),
                           "effective_GBps": 2 * eff(f_ms + b_ms)}}
    plan.close()
    return out


def _events_ms(stream, fn, steps: int) -> float:
    """Average milliseconds of fn() over 'steps' calls, HIP events on 'stream'."""
    import torch
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    e0.record(stream)
    for _ in range(steps):
        fn()
    e1.record(stream)
    torch.cuda.synchronize()
    return e0.elapsed_time(e1) / steps


def soft_rate(C, steps: int, warmup: int, gamma: float = 1.0, block: int = 2048):
    """The smooth (soft-min) sweep of the benchmark matrix: forward (table and score) and the
    adjoint of the score from the table, each timed with HIP events.  Error: the table's
    top-left block x block against the float64 oracle (D[i][j] depends on C[:i+1, :j+1]
    only, so the block is exact); the adjoint's first and last cells against their exact
    value 1."""
    import numpy as np
    import torch

    import paper_2510_27351_amd as wf
    m, n = C.shape
    D = torch.empty_like(C)
    gC = torch.empty_like(C)
    one = torch.ones((), dtype=C.dtype, device=C.device)
    for _ in range(max(warmup, 1)):
        wf.soft_forward(C, gamma, D=D)
        wf.soft_backward(C, D, gamma, g_score=one, g_C=gC)
    wf.last_async_error()
    stream = torch.cuda.current_stream()
    f_ms = _events_ms(stream, lambda: wf.soft_forward(C, gamma, D=D), steps)
    b_ms = _events_ms(stream, lambda: wf.soft_backward(C, D, gamma, g_score=one, g_C=gC), steps)
    wf.last_async_error()
    cells = m * n
    es = C.element_size()
    out = {"workload": f"soft-min recurrence, gamma={gamma}, the same {m}x{n} float32 matrix; forward writes the "
                       "table, adjoint of the score reads C and the table",
           "fwd": {"ms": f_ms, "cells_per_s": cells / (f_ms * 1e-3),
                   "achieved_GBps": 2 * cells * es / (f_ms * 1e-3) / 1e9},
           "adjoint": {"ms": b_ms, "cells_per_s": cells / (b_ms * 1e-3),
                       "achieved_GBps": 3 * cells * es / (b_ms * 1e-3) / 1e9}}
    try:
        import oracle
        oracle.build(force=False)
        blk = C[:block, :block].cpu().numpy().astype(np.float64)
        ref = oracle.soft_forward(blk, gamma)
        got = D[:block, :block].cpu().numpy().astype(np.float64)
        diff = np.abs(got - ref)
        out["errors"] = {"vs": f"float64 oracle on the top-left {block}x{block} block of the table",
                         "normwise_max_err": float(diff.max() / np.abs(ref).max()),
                         "elementwise_max_rel_err": float((diff / np.maximum(np.abs(ref), 1e-300)).max())}
    except Exception as e:  # noqa: BLE001 -- the timing stands without the check
        out["errors"] = {"skipped": str(e)}
    # the adjoint of the score is the probability that a path passes through each cell:
    # exactly 1 at the first and the last cell, which every path visits
    out["adjoint_check"] = {"first_cell": float(gC[0, 0]), "last_cell": float(gC[-1, -1]), "exact": 1.0,
                            "min": float(gC.min())}
    return out


def tri_rate(steps: int, warmup: int, N: int = 100_000_000):
    """The tridiagonal partition solver (the paper's own method) on one diagonally dominant
    float64 system of N unknowns (seed 8), resident in HBM, with the predicted sub-system
    size and recursion depth.  The whole solve (2R+3 launches) is timed with HIP events, and
    so are the level-0 Stage 1 and Stage 3 kernels alone (they move nearly all the bytes).
    Algorithmic bytes: Stage 1 reads a, b, c, d (4 elements per unknown) and writes the
    interface system (8 per sub-system); Stage 3 reads a, b, c, d and the interface values
    and writes x (5 per unknown); each deeper level moves the same on its interface system."""
    import numpy as np
    import torch

    from paper_2510_27351_amd import inputs, tri
    a, b, c, d = (v.cuda() for v in inputs.tridiagonal_dd(N, seed=8))
    plan = tri.Plan(1, N, torch.float64)
    x = torch.empty_like(a)
    for _ in range(max(warmup, 1)):
        plan.solve(a, b, c, d, x)
    stream = torch.cuda.current_stream()
    ms = _events_ms(stream, lambda: plan.solve(a, b, c, d, x), steps)
    es = 8
    P0 = tri.subsystems(N, plan.m)
    A, B, Cc, Dd = tri.stage1(a, b, c, d, plan.m)
    z = torch.zeros(2 * P0, dtype=torch.float64, device=a.device)
    x3 = torch.empty_like(a)
    s1_ms = _events_ms(stream, lambda: tri.stage1(a, b, c, d, plan.m), steps)
    s3_ms = _events_ms(stream, lambda: tri.stage3(a, b, c, d, z, plan.m, x=x3), steps)
    del A, B, Cc, Dd, x3
    sizes = plan.sizes
    ms_l = [plan.m] + plan.ms
    algo = 0
    for lvl in range(plan.R + 1):
        nl, Pl = sizes[lvl], tri.subsystems(sizes[lvl], ms_l[lvl])
        algo += (4 * nl + 8 * Pl) * es + (5 * nl + 2 * Pl) * es
    algo += 7 * sizes[plan.R + 1] * es  # the Thomas solve of the deepest system
    s1_bytes = (4 * N + 8 * P0) * es
    s3_bytes = (5 * N + 2 * P0) * es
    gb = lambda nbytes, t: nbytes / (t * 1e-3) / 1e9  # noqa: E731
    kern = {"stage1_level0": {"ms": s1_ms, "bytes_per_launch": s1_bytes, "achieved_GBps": gb(s1_bytes, s1_ms),
                              "frac": gb(s1_bytes, s1_ms) / PEAK_HBM_GBPS,
                              "measured_traffic_bytes": measured_traffic("stage1_level0")},
            "stage3_level0": {"ms": s3_ms, "bytes_per_launch": s3_bytes, "achieved_GBps": gb(s3_bytes, s3_ms),
                              "frac": gb(s3_bytes, s3_ms) / PEAK_HBM_GBPS,
                              "measured_traffic_bytes": measured_traffic("stage3_level0")}}
    dom = max(kern, key=lambda k: kern[k]["ms"])
    out = {"workload": f"one tridiagonal system of {N} unknowns, float64, diagonally dominant (seed 8), resident "
                       f"in HBM; predicted m={plan.m}, R={plan.R}, m_1..m_R={plan.ms}, level sizes {sizes}",
           "ms": ms, "unknowns_per_s": N / (ms * 1e-3), "algorithmic_bytes": algo,
           "achieved_GBps": gb(algo, ms), "frac_of_peak": gb(algo, ms) / PEAK_HBM_GBPS, "kernels": kern,
           "roofline": {"bound": "hbm", "kernel": dom, "achieved": kern[dom]["achieved_GBps"], "peak": PEAK_HBM_GBPS,
                        "unit": "GB/s", "frac": kern[dom]["frac"], "traffic": kern[dom]["measured_traffic_bytes"]},
           "paper_context": "N=1e8 FP64 partition method, wall-clock incl. transfers: 643.11 ms (RTX 2080 Ti, "
                            "non-recursive, m=64, 32 streams); 241.161 ms (RTX A5000, 3 recursive steps)"}
    try:
        from oracle import tridiag
        ha, hb, hc, hd = (v.cpu().numpy() for v in (a, b, c, d))
        got = x.cpu().numpy()
        t0 = time.perf_counter()
        want = tridiag.c_partition_solve(ha, hb, hc, hd, [plan.m] + plan.ms)
        t_or = time.perf_counter() - t0
        ref = tridiag.c_thomas(ha, hb, hc, hd)
        out["errors"] = {"bitwise_equal_oracle_partition": bool(np.array_equal(got, want)),
                         "max_abs_err_vs_thomas": float(np.max(np.abs(got - ref))),
                         "max_abs_x": float(np.max(np.abs(ref)))}
        out["cpu_oracle"] = {"ms": t_or * 1e3, "cores": 1,
                             "kind": "oracle (plain C partition method, same m and R, one thread)"}
    except Exception as e:  # noqa: BLE001
        out["errors"] = {"skipped": str(e)}
    del plan
    return out


def main():
    args = parse()
    if args.gpus != 1:
        print(json.dumps({"error": "this build measures one GPU only (one process, one device); "
                                   "run with --gpus 1"}))
        sys.exit(2)
    import torch

    import paper_2510_27351_amd as wf
    from paper_2510_27351_amd import inputs

    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    n = m = args.n
    C_cpu = inputs.single_16384_f32(n)
    C = C_cpu.to(dev)
    D = torch.empty_like(C)
    gC = torch.empty_like(C)
    one = torch.ones((), dtype=C.dtype, device=dev)
    ckpt = torch.empty(wf.ckpt_elems(m, n, CKPT_K), dtype=C.dtype, device=dev)
    stream = torch.cuda.current_stream(dev)
    lib = wf._lib.load()
    code = wf._lib.WF_F32
    sp = stream.cuda_stream

    def fwd():
        wf._lib.check(lib.wf_forward(code, m, n, C.data_ptr(), n, D.data_ptr(), n, wf_score.data_ptr(),
                                     ckpt.data_ptr(), CKPT_K, sp), "wf_forward")

    def bwd():
        wf._lib.check(lib.wf_backward(code, m, n, C.data_ptr(), n, ckpt.data_ptr(), CKPT_K, None, n, one.data_ptr(),
                                      None, n, gC.data_ptr(), n, sp), "wf_backward")

    wf_score = torch.empty((), dtype=C.dtype, device=dev)
    if args.calib_copy:
        D.copy_(C)
        torch.cuda.synchronize()
    for _ in range(args.warmup):
        fwd()
        bwd()
    wf.last_async_error()
    torch.cuda.synchronize()
    K = args.steps
    ev = [[torch.cuda.Event(enable_timing=True) for _ in range(3)] for _ in range(K)]
    t_start = torch.cuda.Event(enable_timing=True)
    t_end = torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    t_start.record(stream)
    for k in range(K):
        ev[k][0].record(stream)
        fwd()
        ev[k][1].record(stream)
        bwd()
        ev[k][2].record(stream)
    t_end.record(stream)
    torch.cuda.synchronize()
    wf.last_async_error()
    total_ms = t_start.elapsed_time(t_end)
    fwd_ms, bwd_ms = [sum(e[i].elapsed_time(e[i + 1]) for e in ev) / K for i in range(2)]
    ms = total_ms / K
    cells = m * n
    es = C.element_size()
    ck_bytes = ckpt.numel() * es
    nb = (m + 63) // 64
    Ks = (n + 63 + 63) // 64
    plane_bytes = nb * Ks * 64 * 32  # selection bit-planes: 32 bytes per band row and 64 slots
    top_bytes = (nb - 1) * n * es     # band top rows read back from the checkpoint grid
    exit_bytes = nb * n * 4           # exits of every band's last row
    # The general adjoint (an upstream gradient of the table given: the reverse pipeline),
    # timed beside the step on the same matrix with a zero g_D.
    gD = torch.zeros_like(C)

    def bwd_general():
        wf._lib.check(lib.wf_backward(code, m, n, C.data_ptr(), n, ckpt.data_ptr(), CKPT_K, None, n, one.data_ptr(),
                                      gD.data_ptr(), n, gC.data_ptr(), n, sp), "wf_backward")

    bwd_general()
    gen_ms = _events_ms(stream, bwd_general, max(2, min(K, 5)))
    wf.last_async_error()
    del gD
    bwd()  # the step's own gradient for the error report
    torch.cuda.synchronize()
    # Method bytes per launch: the inputs and outputs of the differentiable sweep each launch
    # must move at least.  The adjoint call's intermediates (selection bit-planes and exits,
    # written by its sweep and read by its walk) are reported apart.
    kern = {
        "fwd_kernel": (fwd_ms, 2 * cells * es + ck_bytes, 0, "read C, write D and the checkpoint grid"),
        "path_adjoint": (bwd_ms, 2 * cells * es + top_bytes, plane_bytes + exit_bytes,
                         "wf_backward, score alone (sel_path_kernel + compose_kernel + walk_kernel): read C and "
                         "the checkpoint grid's band rows, write g_C (intermediate: the selection bit-planes "
                         "and the exits written)"),
    }
    eff = lambda nbytes, t_ms: nbytes / (t_ms * 1e-3) / 1e9  # noqa: E731
    kernels = {k: {"ms": t, "bytes_per_launch": b, "intermediate_bytes_per_launch": ib,
                   "achieved_GBps": eff(b, t), "frac": eff(b, t) / PEAK_HBM_GBPS,
                   "measured_traffic_bytes": measured_traffic(k), "bytes": what}
               for k, (t, b, ib, what) in kern.items()}
    dom = max(kernels, key=lambda k: kernels[k]["ms"])
    tile_fwd, rows_fwd = wf.forward_config(m, n)
    out = {
        "metric": "cells/sec and effective HBM GB/s (% peak), fwd and fwd+adjoint, n=16384",
        "value": cells / (ms * 1e-3),
        "unit": "cells/s",
        "n_gpus": 1,
        "steps": K,
        "warmup": args.warmup,
        "ms_per_step": ms,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f32",
        "data": "synthetic",
        "config": {"workload": f"single {m}x{n} float32, normal(0,1) clipped to [-4,4], seed 2; step = "
                               f"forward (table, score, checkpoint grid K={CKPT_K}) + adjoint of the score "
                               "from the checkpoint grid (wf_backward: selection recompute with the bands' "
                               "exits, then the walk of the argmin path)",
                   "m": m, "n": n, "ckpt_k": CKPT_K,
                   "tile_forward": tile_fwd, "rows_per_lane_forward": rows_fwd,
                   "tile_reverse": wf.predict_tile(m, n, reverse=True)},
        "fwd": {"ms": fwd_ms, "cells_per_s": cells / (fwd_ms * 1e-3),
                "effective_GBps": eff(3 * cells * es, fwd_ms),
                "effective_pct_peak": 100 * eff(3 * cells * es, fwd_ms) / PEAK_HBM_GBPS},
        "adjoint": {"ms": bwd_ms, "cells_per_s": cells / (bwd_ms * 1e-3),
                    "effective_GBps": eff(3 * cells * es, bwd_ms),
                    "effective_pct_peak": 100 * eff(3 * cells * es, bwd_ms) / PEAK_HBM_GBPS},
        "adjoint_with_gD": {"ms": gen_ms, "cells_per_s": cells / (gen_ms * 1e-3),
                            "note": "wf_backward with an upstream gradient of the table (zero here): selection "
                                    "recompute then the reverse pipeline; not part of the step"},
        "fwd_adjoint": {"ms": ms, "effective_GBps": eff(6 * cells * es, ms),
                        "effective_pct_peak": 100 * eff(6 * cells * es, ms) / PEAK_HBM_GBPS},
        "kernels": kernels,
        "roofline": {"bound": "hbm", "achieved": kernels[dom]["achieved_GBps"], "peak": PEAK_HBM_GBPS,
                     "unit": "GB/s", "frac": kernels[dom]["frac"], "traffic": measured_traffic(dom),
                     "kernel": dom, "kernel_ms": kernels[dom]["ms"],
                     "bytes_per_launch": kernels[dom]["bytes_per_launch"]},
    }
    if not args.no_batch:
        b = batch_rate(K, args.warmup)
        b["ratio_single_over_batch"] = (cells / (fwd_ms * 1e-3)) / b["cells_per_s"]
        out["batch"] = b
        out["c5"] = c5_rate(K, args.warmup)
    if not args.no_soft:
        out["soft"] = soft_rate(C, K, args.warmup)
    if not args.no_tri:
        out["tri"] = tri_rate(K, args.warmup)
    if not args.no_cpu:
        base, oracle64 = cpu_baseline(C_cpu)
        out["cpu_baseline"] = base
        if oracle64 is not None:
            out["errors"] = result_errors(C_cpu, D, wf_score.item(), gC, oracle64)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
