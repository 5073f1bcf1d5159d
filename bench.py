"""Benchmark: UniQuan_F optimisation steps on one MI355X.

A step is one pass of the whole hot path over one batch, for every
(matrix, k) of the workload:
    fq_fwd (transform, level table, nearest-level mapping, detransform; it
            stores the residual What - W)
    -> reconstruction forward GEMM + loss (Et = (What - W) X^T, sum Et^2; the
       same error as What X^T - X W^T without the stored fp32 target)
    -> weight-gradient GEMM (dL/dWhat = 2 Et X)
    -> fq_bwd fused with the SGD update (straight-through gradients of s,
       alpha, z_B applied in place in the same pass)
with the mapping schedule of the paper's local and periodic mapping (p = 2:
local remap on even steps, frozen codes otherwise; the initial full mapping
is part of set-up).  Inputs are synthetic and resident in HBM before timing.
Set-up initialises every layer with the unified initialisation (grid search
over clipping ranges with the general alternating update, G = 30, T = 15 by
default); its kernel time is reported under ``init`` with an ALU roofline and
its own CPU-oracle baseline, outside the timed steps.

Output: one JSON line.  The headline workload is the 70B MLP slice
(``mlp70b``: gate/up 28672x8192 and down 8192x28672, 4096 tokens, k = 2 and
3), the largest single-GPU configuration.  ``value`` is the fake-quant
fwd+bwd throughput in Gweights/s (weights quantized forward and backward per
second of quantizer kernel time inside the timed steps); the reconstruction
GEMM throughput is ``gemm_tflops``.  Per-kernel averages come from HIP events
recorded on the stream the kernels run on.  ``roofline`` describes the kernel
with the largest share of step time; ``ceilings`` holds the streaming and
MFMA rates this GPU reaches (measured in the same run) and each headline
fraction against them; ``workloads`` holds the other configurations (the
4096x4096 projection, the 7B MLP, the 7B block's seven matrices over 100
timed steps) as sub-records; ``cpu_baseline`` times the CPU oracle on a
bounded sample on all host cores.

Usage: python bench.py [--gpus 1] [--steps K] [--warmup W] [--workload NAME]
       python bench.py --summarize-profiles WORKLOAD   (CPU: profiles/ from rocprofv3 CSVs)
"""
from __future__ import annotations

import argparse
import ctypes
import hashlib
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0          # MI355X HBM3E, GB/s
MFMA_BF16_PEAK_TFLOPS = 2500.0  # MI355X dense bf16 MFMA
# Plain (unpacked) 32-bit VALU operations per second: 256 CUs x 4 SIMDs x 16
# lanes x 2.4 GHz.  The 157.3 TFLOP/s fp32 vector peak counts a packed FMA as
# 4 flops; a timed chain of independent v_add_f32 / v_fma_f32 reaches 37 T of
# these lane-operations per second, so 39.3 T is the issue limit.
VALU_PEAK_TOPS = 256 * 4 * 16 * 2.4e9 / 1e12
PROFILES = os.path.join(ROOT, "profiles")
CSRC = os.path.join(ROOT, "paper_2506_03781_amd", "csrc")


_HIP = None
HIP_EVENT_DISABLE_SYSTEM_FENCE = 0x20000000


class TimingEvent:
    """A HIP timing event created with hipEventDisableSystemFence, recorded on
    torch's current stream.  A default event writes back and invalidates the
    caches when it completes: a few microseconds of idle GPU per event and
    the next kernel starts on cold caches, both counted in the phase it
    brackets.  These events skip that fence; they are read only after a
    device-wide synchronisation, so their timestamps are complete.  The HIP
    runtime is the one torch already loaded (one runtime per process)."""

    def __init__(self):
        global _HIP
        import torch
        if _HIP is None:
            torch.zeros(1, device="cuda")
            path = next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l)
            h = ctypes.CDLL(path)
            h.hipEventCreateWithFlags.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.c_uint]
            h.hipEventRecord.argtypes = [ctypes.c_void_p, ctypes.c_void_p]
            h.hipEventElapsedTime.argtypes = [ctypes.POINTER(ctypes.c_float), ctypes.c_void_p, ctypes.c_void_p]
            h.hipEventDestroy.argtypes = [ctypes.c_void_p]
            _HIP = h
        self._torch = torch
        self.ev = ctypes.c_void_p()
        rc = _HIP.hipEventCreateWithFlags(ctypes.byref(self.ev), HIP_EVENT_DISABLE_SYSTEM_FENCE)
        if rc != 0:
            raise RuntimeError(f"hipEventCreateWithFlags failed ({rc})")

    def record(self):
        rc = _HIP.hipEventRecord(self.ev, ctypes.c_void_p(self._torch.cuda.current_stream().cuda_stream))
        if rc != 0:
            raise RuntimeError(f"hipEventRecord failed ({rc})")

    def elapsed_time(self, end) -> float:
        """Milliseconds from this event to ``end`` (call after a device synchronisation)."""
        ms = ctypes.c_float()
        rc = _HIP.hipEventElapsedTime(ctypes.byref(ms), self.ev, end.ev)
        if rc != 0:
            raise RuntimeError(f"hipEventElapsedTime failed ({rc})")
        return ms.value

    def __del__(self):
        if _HIP is not None and self.ev:
            _HIP.hipEventDestroy(self.ev)


def parse():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=50)
    ap.add_argument("--warmup", type=int, default=50)
    ap.add_argument("--workload", default="mlp70b")
    ap.add_argument("--sub-workloads", default="attn4096,mlp7b,block7b,mlp7b_rows",
                    help="comma-separated workloads reported as sub-records ('' for none)")
    ap.add_argument("--sub-steps", type=int, default=20, help="timed steps of each sub-record")
    ap.add_argument("--block7b-steps", type=int, default=100,
                    help="timed steps of the 7B block's seven matrices (the configuration times 100)")
    ap.add_argument("--no-ceilings", action="store_true", help="skip the streaming and MFMA ceiling probes")
    ap.add_argument("--unfused", action="store_true",
                    help="time the step as four passes (fq_fwd, loss GEMM, gradient GEMM, fq_bwd with SGD) instead "
                         "of two GEMMs and the fused backward + SGD + next forward pass")
    ap.add_argument("--summarize-block-profile", action="store_true",
                    help="write profiles/decoder_block7b.md from gpurun_out/prof_block7b (no GPU needed)")
    ap.add_argument("--summarize-profiles", default=None, metavar="WORKLOAD",
                    help="(no GPU) write profiles/ summaries from the rocprofv3 CSVs under gpurun_out/")
    ap.add_argument("--mode", default="paper", choices=["paper", "full", "local", "frozen"])
    ap.add_argument("--seed", type=int, default=0)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--init", default="unified", choices=["unified", "greedy"],
                    help="parameter initialisation (set-up, timed separately from the steps)")
    ap.add_argument("--init-grid", type=int, default=30, help="grid points G of the unified init")
    ap.add_argument("--init-rounds", type=int, default=15, help="alternating rounds T of the unified init")
    ap.add_argument("--init-clip", type=int, default=0, help="0 fixed min, 1 fixed max, 2 balanced")
    ap.add_argument("--target", action="store_true",
                    help="loss against a stored fp32 target Y = X W^T instead of the residual form")
    ap.add_argument("--no-block", action="store_true",
                    help="skip the block-level step on a 7B decoder block (8192 tokens, 32 heads, I = 11008)")
    ap.add_argument("--block-kv", type=int, default=None,
                    help="key/value heads of the decoder block (default 32, multi-head; 8 for grouped-query)")
    ap.add_argument("--calib-copy", action="store_true",
                    help="also run a plain 256 MiB device copy (counter calibration)")
    return ap.parse_args()


# Sources of the step's kernels: counters taken on other sources do not
# describe the kernels that run.
STEP_SOURCES = ("fq_fwd.hip", "fq_bwd.hip", "gemm.hip", "uq_device.h", "uq_launch.h")


def src_hash() -> str:
    """Hash of the step kernels' sources with comments and blank space taken
    out, so that an edit of a comment keeps the counters that were taken."""
    import re
    h = hashlib.sha256()
    for f in STEP_SOURCES:
        text = open(os.path.join(CSRC, f)).read()
        text = re.sub(r"/\*.*?\*/", " ", text, flags=re.S)
        text = re.sub(r"//[^\n]*", " ", text)
        h.update(" ".join(text.split()).encode())
    return h.hexdigest()[:16]


def fq_bytes_per_weight(k, g, mode, w_bytes=2, what_bytes=2, grad_bytes=2):
    """Algorithmic HBM bytes per weight of the quantizer forward and of the
    fused backward + SGD update (gradients not stored)."""
    fwd = w_bytes + 4 + what_bytes + 1 + (1 if mode != "full" else 0) + (4 * k + 12) / g
    # dL/dWhat, W, s, code in; s out; per group Delta, z_U in, alpha, z_B in and out
    bwd = grad_bytes + w_bytes + 4 + 1 + 4 + (8 + 2 * (4 * k + 4)) / g
    return fwd, bwd


def fq_step_bytes_per_weight(k, g, w_bytes=2, what_bytes=2, grad_bytes=2):
    """Algorithmic bytes per weight of uniquan_fq_step (backward + SGD of one
    step, forward of the next), as (read, written).  One pass for g <= 512:
    dL/dWhat, W, s, code in; s, What, code out; per group Delta, z_U, s_r,
    alpha, z_B in and alpha, z_B out.  Groups of 513 to 16384 bf16 weights
    (bf16 dL/dWhat) take one pass too, one workgroup per group; other large
    groups run the two passes."""
    if g > 512 and (g > 16384 or w_bytes != 2 or grad_bytes != 2):
        return fq_read_write_bytes(k, g, "local", w_bytes, what_bytes, grad_bytes)
    rd = grad_bytes + w_bytes + 4 + 1 + (4 * k + 12) / g
    wr = 4 + what_bytes + 1 + (4 * k + 4) / g
    return rd, wr


def fq_read_write_bytes(k, g, mode, w_bytes=2, what_bytes=2, grad_bytes=2):
    """The read and written parts of fq_bytes_per_weight (forward + backward)."""
    rd = (w_bytes + 4 + (1 if mode != "full" else 0) + (4 * k + 12) / g
          + grad_bytes + w_bytes + 4 + 1 + (8 + 4 * k + 4) / g)
    wr = what_bytes + 1 + 4 + (4 * k + 4) / g
    return rd, wr


def init_ops_per_weight(k, G, T):
    """Algorithmic VALU operations per weight of the unified initialisation:
    per grid point the transform (2) and shifted copy (1), the greedy start
    (4 per bit: |r|, sum, sign test, residual update), per alternating round
    the signed sums (2k), the C^T C counts (k(k-1)/2), the nearest-level search
    (k compares, 2 distances, 2 |.|, 1 compare) and with a one-point grid the
    shift update (k + 3), and the candidate error (search k + 5, detransform 2,
    difference, square, sum)."""
    rnd = 2 * k + k * (k - 1) // 2 + (k + 5) + ((k + 3) if G == 1 else 0)
    per_point = 3 + 4 * k + T * rnd + (k + 5) + 5
    return G * per_point


def cpu_baseline_init(W, k, g, G, T, clip, budget_s=3.0):
    """The oracle's unified initialisation on the first groups of a matrix,
    numpy restricted to one thread."""
    import numpy as np
    from threadpoolctl import threadpool_limits
    import oracle.unified_init as UI
    Wg = np.asarray(W, np.float32).reshape(-1, g)
    n = 2
    with threadpool_limits(1):
        while True:
            t0 = time.perf_counter()
            UI.unified_init(Wg[:n], k, g, G=G, T=T, clip=clip)
            dt = time.perf_counter() - t0
            if dt >= budget_s / 3 or n * 2 > Wg.shape[0]:
                break
            n *= 2
    return {"value": n * g / dt / 1e9, "unit": "Gweights/s", "cores": 1, "kind": "oracle",
            "sample": f"oracle unified_init (G={G}, T={T}, k={k}) on the first {n} groups of "
                      f"{g} weights, numpy on one thread: {dt:.2f} s"}


def schedule(mode, step):
    from paper_2506_03781_amd import uniquan as uq
    if mode == "full":
        return uq.MAP_FULL
    if mode == "local":
        return uq.MAP_LOCAL
    if mode == "frozen":
        return uq.MAP_FROZEN
    return uq.MAP_LOCAL if step % 2 == 0 else uq.MAP_FROZEN


def load_counters(workload):
    """HBM traffic per launch from committed rocprofv3 counter runs, if they were
    taken on the current kernel sources."""
    path = os.path.join(PROFILES, f"pmc_{workload}.json")
    if not os.path.exists(path):
        return None
    d = json.load(open(path))
    if d.get("src_hash") != src_hash():
        return None
    return d


def host_cores() -> int:
    return len(os.sched_getaffinity(0))


def cpu_baseline(layers_np, X, mode, budget_s=20.0):
    """The oracle on a bounded row sample of the headline workload's first
    (matrix, k) layers, on the host cores of this machine: fq_fwd + fq_bwd
    (the metric's unit; vectorised numpy, effectively one thread), the
    reconstruction loss and weight gradient (fp64 matmuls, BLAS on every
    core) and the fold.  Rows double until each part has used its share of
    the budget."""
    from threadpoolctl import threadpool_limits
    cores = host_cores()
    with threadpool_limits(cores):
        return _cpu_baseline(layers_np, X, mode, budget_s, cores)


def _timed_rows(fn, R, per, rows=8):
    """Run fn(rows) with rows doubling until it takes >= per / 3 (or all rows)."""
    while True:
        t0 = time.perf_counter()
        fn(rows)
        dt = time.perf_counter() - t0
        if dt >= per / 3 or rows >= R:
            return rows, dt
        rows = min(R, rows * 2)


def _cpu_baseline(layers_np, X, mode, budget_s, cores):
    import numpy as np
    import oracle.uniquan as O
    omode = {"full": O.MAP_FULL, "local": O.MAP_LOCAL, "frozen": O.MAP_FROZEN}.get(mode, O.MAP_LOCAL)
    per = budget_s / (3 * max(1, len(layers_np)))
    fq_w = fq_t = rc_f = rc_t = fo_w = fo_t = 0.0
    parts = []
    Xb = np.asarray(X, np.float32)
    T = Xb.shape[0]
    for (W, s, k, g) in layers_np:
        R, C = W.shape
        cache = {}

        def params(rows):
            if rows not in cache:
                Wr, sr = W[:rows], s[:rows]
                p = O.init_param_set_a(Wr, sr, k, g)
                prev = O.fq_fwd(Wr, sr, p["alpha"], p["z_b"], k, g)["codes"]
                cache.clear()
                cache[rows] = (Wr, sr, p["alpha"], p["z_b"], prev)
            return cache[rows]

        def fq(rows):
            Wr, sr, a, z, prev = params(rows)
            Gr = np.random.default_rng(0).standard_normal(Wr.shape).astype(np.float32)
            t0 = time.perf_counter()
            f = O.fq_fwd(Wr, sr, a, z, k, g, mode=omode, codes_prev=prev)
            O.fq_bwd(Wr, sr, a, z, f["codes"], Gr, k, g)
            return time.perf_counter() - t0

        # fq: time only the oracle calls (parameter set-up excluded)
        rows = 8
        while True:
            dt = fq(rows)
            if dt >= per / 3 or rows >= R:
                break
            rows = min(R, rows * 2)
        fq_w += rows * C
        fq_t += dt
        Wr, sr, a, z, _ = params(rows)
        Rw = O.residual_f32(O.fq_fwd(Wr, sr, a, z, k, g)["what32"], Wr)
        rr, dt2 = _timed_rows(lambda n: O.recon_residual(Xb, Rw[:n]), rows, per)
        rc_f += 4.0 * T * rr * C
        rc_t += dt2
        fr, dt3 = _timed_rows(lambda n: O.fold(Wr[:n], sr[:n], a[: n * C // g], z[: n * C // g], k, g), rows, per)
        fo_w += fr * C
        fo_t += dt3
        parts.append(f"{rows} rows x {C} cols at k={k} (recon on {rr} rows x {T} tokens, fold on {fr} rows)")
    return {"value": fq_w / fq_t / 1e9, "unit": "Gweights/s", "cores": cores, "kind": "oracle",
            "sample": "oracle fq_fwd (" + ("local" if mode == "paper" else mode) + " mapping) + fq_bwd, "
                      "recon (fp64 matmuls) and fold on the first rows of the headline layers: "
                      + "; ".join(parts) + f"; fq {int(fq_w)} weights in {fq_t:.2f} s",
            "threads": {"fq": "vectorised numpy (one thread)", "recon": f"BLAS on {cores} threads",
                        "fold": "vectorised numpy (one thread)"},
            "recon_tflops": rc_f / rc_t / 1e12 if rc_t else None,
            "fold_gweights_per_s": fo_w / fo_t / 1e9 if fo_t else None,
            "seconds": {"fq": fq_t, "recon": rc_t, "fold": fo_t}}


def ceilings(n_bytes=1 << 30, reps=3, grids=(2048, 8192, 32768)):
    """What this GPU reaches: 16-byte nontemporal streaming read, write and
    copy over n_bytes buffers (best over grid sizes and reps launches, each
    launch timed by HIP events) and independent MFMA chains on registers."""
    import torch

    from paper_2506_03781_amd import uniquan as uq
    sink = torch.zeros(16, dtype=torch.float32, device="cuda")
    src = torch.ones(n_bytes // 4, dtype=torch.int32, device="cuda")
    dst = torch.empty_like(src)
    out = {}
    for name, op, moved in (("read", 0, n_bytes), ("write", 1, n_bytes), ("copy", 2, 2 * n_bytes)):
        best, best_grid = None, None
        for blocks in grids:
            for _ in range(reps + 1):
                a, b = TimingEvent(), TimingEvent()
                a.record()
                uq.uniquan_probe_stream(op, n_bytes, src, dst, sink, blocks)
                b.record()
                torch.cuda.synchronize()
                ms = a.elapsed_time(b)
                if best is None or ms < best:
                    best, best_grid = ms, blocks
        out[f"{name}_gbs"] = moved / (best * 1e-3) / 1e9
        out[f"{name}_grid"] = best_grid
    iters = 20000
    best = None
    for _ in range(reps + 1):
        a, b = TimingEvent(), TimingEvent()
        a.record()
        uq.uniquan_probe_mfma(iters, sink)
        b.record()
        torch.cuda.synchronize()
        ms = a.elapsed_time(b)
        best = ms if best is None else min(best, ms)
    out["mfma_bf16_tflops"] = uq.uniquan_probe_mfma_flops(iters) / (best * 1e-3) / 1e12
    out["note"] = (f"streaming probes over {n_bytes >> 20} MiB buffers (best of {reps + 1} launches at each of "
                   f"{list(grids)} workgroups); MFMA probe: 8 independent v_mfma_f32_32x32x16_bf16 chains per "
                   "wavefront, one wavefront per SIMD")
    del src, dst, sink
    return out


def bcq_inference(layers, batches=(1, 8), target_bytes=512 << 20):
    """The deployed layer after the timed steps: fold (Theorem 1) -> stored
    form -> Y = X What^T for a batch of T activation rows.  Copies of the
    stored form are rotated so that the bytes touched between two reads of one
    copy exceed the 256 MB last-level cache (cold-cache decode, as one token's
    pass over a model reads each layer once)."""
    import torch

    from paper_2506_03781_amd import uniquan as uq
    res = []
    for lay in layers:
        R, C, k, g = lay.R, lay.C, lay.k, lay.g
        if C % 128 or g % 128 or k > 4:
            continue
        a, z, c = lay.fold()
        Gn = R * C // g
        per_copy = R * C * k // 8 + 2 * (k + 1) * Gn
        n_copy = int(min(64, max(2, -(-target_bytes // per_copy))))
        copies = []
        for _ in range(n_copy):
            st = (torch.empty(R * C * k // 32, dtype=torch.int32, device="cuda"),
                  torch.empty(Gn * k, dtype=torch.float16, device="cuda"),
                  torch.empty(Gn, dtype=torch.float16, device="cuda"))
            uq.uniquan_bcq_pack(R, C, k, g, c, a, z, *st)
            copies.append(st)
        for T in batches:
            X = lay.X[:T].contiguous()
            Y = torch.empty(T, R, device="cuda")
            ws = torch.empty(max(1, uq.uniquan_bcq_matmul_ws(T, R, C)), device="cuda")
            for i in range(3):
                uq.uniquan_bcq_matmul(T, R, C, k, g, X, *copies[i % n_copy], Y, ws)
            n_it = max(20, 2 * n_copy)
            e0, e1 = TimingEvent(), TimingEvent()
            e0.record()
            for i in range(n_it):
                uq.uniquan_bcq_matmul(T, R, C, k, g, X, *copies[i % n_copy], Y, ws)
            e1.record()
            torch.cuda.synchronize()
            us = e0.elapsed_time(e1) / n_it * 1e3
            byt = per_copy + 2 * T * C + 4 * T * R
            gbs = byt / (us * 1e-6) / 1e9
            res.append({"R": R, "C": C, "k": k, "g": g, "T": T, "us_per_call": us, "algorithmic_bytes": byt,
                        "achieved_gbs": gbs, "frac_hbm": gbs / HBM_PEAK_GBS, "copies_rotated": n_copy})
        del copies
    return res


def block_decoder(seed, k=3, steps=5, warmup=2, n_kv=None):
    """Block-level reconstruction of a 7B decoder block (Algorithm 1 with f =
    one rotary causal attention module and one SiLU-gated MLP module): per
    step the seven fake-quant forwards, the block's forward on What, the
    loss, backpropagation to all seven matrices and the straight-through
    backward with the SGD update.  8192 tokens as 4 sequences of 2048,
    C = 4096 in 32 heads of 128, I = 11008; n_kv key/value heads (32 by
    default; 8 gives the grouped-query form with k, v of [1024, 4096])."""
    import numpy as np
    import torch

    from paper_2506_03781_amd import synth
    from paper_2506_03781_amd import uniquan as uq
    from paper_2506_03781_amd.block import DecoderBlock, QuantMatrix
    wl = synth.WORKLOADS["block7b"]
    g = wl.group_size
    n_seq, H = 4, 32
    n_kv = H if n_kv is None else n_kv
    mats, X = {}, None
    for name, spec in zip(DecoderBlock.NAMES, wl.matrices):
        # only the first matrix's activations are used; the weights do not depend on T
        sc = synth.scaled(spec, T=8) if X is not None else spec
        if name in ("k", "v"):
            sc = synth.scaled(sc, R=spec.R * n_kv // H)
        m = synth.make_matrix(sc, seed)
        if X is None:
            X = m.X
        q = QuantMatrix(m.W, m.s, k, g)
        q.init_unified()
        mats[name] = q
        del m
    rs = np.random.default_rng(seed + 1000)
    C = mats["q"].C
    g1 = (1.0 + 0.1 * rs.standard_normal(C)).astype(np.float32)
    g2 = (1.0 + 0.1 * rs.standard_normal(C)).astype(np.float32)
    blk = DecoderBlock(mats, g1, g2, X.shape[0], n_seq, H, n_kv=n_kv)
    blk.prepare(X)
    blk.set_input(X)
    # SGD on L / L0 (one step with zero learning rates measures L0)
    blk.step(uq.MAP_FULL, 0.0, 0.0)
    l0 = float(blk.loss.item())
    lr_f, lr_b = 0.005 / l0, 0.0005 / l0
    rel = []
    for i in range(warmup):
        blk.step(uq.MAP_FULL if i == 0 else uq.MAP_LOCAL, lr_f, lr_b)
        rel.append(float(blk.loss.item()) / l0)
    step_local = uq.record(blk.step, uq.MAP_LOCAL, lr_f, lr_b)
    torch.cuda.synchronize()
    e0, e1 = TimingEvent(), TimingEvent()
    e0.record()
    for _ in range(steps):
        step_local()
    e1.record()
    torch.cuda.synchronize()
    ms_unfused = e0.elapsed_time(e1) / steps
    # the fused step form: the straight-through backward + SGD of each matrix
    # fused with its next fake-quant forward (What left by the last quantize)
    blk.quantize(uq.MAP_LOCAL)
    step_fused = uq.record(blk.step_fused, uq.MAP_LOCAL, lr_f, lr_b)
    torch.cuda.synchronize()
    e0.record()
    for _ in range(steps):
        step_fused()
    e1.record()
    torch.cuda.synchronize()
    ms = e0.elapsed_time(e1) / steps
    # one instrumented step for the split between phases
    ev = [TimingEvent() for _ in range(6)]
    ev[0].record()
    blk.quantize(uq.MAP_LOCAL)
    ev[1].record()
    blk.forward()
    ev[2].record()
    blk.compute_loss()
    ev[3].record()
    blk.backward()
    ev[4].record()
    blk.update(lr_f, lr_b)
    ev[5].record()
    torch.cuda.synchronize()
    phases = dict(zip(("fq_fwd", "forward", "loss", "backward", "ste_sgd"),
                      (ev[i].elapsed_time(ev[i + 1]) for i in range(5))))
    flops = blk.flops_per_step()
    tf = flops / (ms * 1e-3) / 1e12
    n_w = sum(q.R * q.C for q in mats.values())
    last = float(blk.loss.item()) / l0
    return {"T": blk.T, "C": blk.C, "I": blk.I, "heads": H, "kv_heads": n_kv, "seq_len": blk.L, "n_seq": n_seq, "k": k, "g": g,
            "steps": steps, "ms_per_step": ms, "ms_per_step_unfused": ms_unfused,
            "gweights_per_s": n_w / (ms * 1e-3) / 1e9,
            "gemm_flops_per_step": flops, "tflops_effective": tf, "frac_mfma": tf / MFMA_BF16_PEAK_TFLOPS,
            "phase_ms": phases, "loss_init": l0, "rel_loss_warmup": rel, "rel_loss_last": last,
            "state_finite": bool(math.isfinite(last)),
            "optimiser": "SGD on L / L_init (learning rates 0.005 / 0.0005 divided by the initial loss)",
            "note": "whole step over the seven matrices in the fused form (block forward on What with the "
                    "quantized input, loss, backpropagation, then per matrix the straight-through backward + "
                    "SGD fused with the next fake-quant forward); ms_per_step_unfused: the same step with the "
                    "fake-quant forward and the backward + SGD as separate passes; phase_ms splits an unfused "
                    "step; flops count the GEMMs only"}


# Kernel-name patterns of the step's four phases in rocprofv3 output.
PHASE_PATTERNS = {
    "fq_fwd": r"fq_fwd_kernel<1, 1, [23], ",
    "gemm_fwd": r"gemm_(?:pp_kernel<256, \d+, |w4_kernel<)[14], ",
    "gemm_bwd": r"gemm_(?:pp_kernel<256, \d+, |w4_kernel<)2, ",
    "fq_bwd": r"fq_bwd_kernel<1, 1, ",
    "fq_step": r"fq_step_kernel<1, 1, 1, [023], ",
}


def summarize_profiles(workload, steps, warmup, fused=True, out_dir=PROFILES, run_dir=os.path.join(ROOT, "gpurun_out")):
    """Write profiles/uniquan_kernels_<workload>.md and pmc_<workload>.json from
    the CSVs of three rocprofv3 runs of this script (commands in the summary):
    a kernel trace with statistics, then FETCH_SIZE and WRITE_SIZE counter
    runs.  Counters are scaled by what they read for a plain 256 MiB device
    copy (run by --calib-copy in the counter runs)."""
    import csv
    import collections
    import re
    from paper_2506_03781_amd import synth
    wl = synth.WORKLOADS[workload]
    n_layers = len(wl.matrices) * len(wl.ks)
    pdir = os.path.join(run_dir, f"prof_{workload}")
    stats = list(csv.DictReader(open(os.path.join(pdir, "trace_kernel_stats.csv"))))
    trace = list(csv.DictReader(open(os.path.join(pdir, "trace_kernel_trace.csv"))))

    def counters(path):
        d = collections.defaultdict(list)
        for r in csv.DictReader(open(path)):
            d[r["Kernel_Name"]].append(float(r["Counter_Value"]))
        return d

    fetch = counters(os.path.join(run_dir, f"pmc_fetch_{workload}", "fetch_counter_collection.csv"))
    write = counters(os.path.join(run_dir, f"pmc_write_{workload}", "write_counter_collection.csv"))
    kib_copy = 256 * 1024
    cf = [v for k, vs in fetch.items() if "copyBuffer" in k for v in vs if v > kib_copy / 4]
    cw = [v for k, vs in write.items() if "copyBuffer" in k for v in vs if v > kib_copy / 4]
    fscale = kib_copy / (sum(cf) / len(cf))
    wscale = kib_copy / (sum(cw) / len(cw))

    def mean_kib(d, pat):
        vals = [v for k, vs in d.items() if re.search(pat, k) for v in vs]
        return sum(vals) / len(vals), len(vals)

    phases = FUSED_PHASES if fused else PHASES
    patterns = {ph: PHASE_PATTERNS[ph] for ph in phases}
    kern = {}
    for ph, pat in patterns.items():
        f, nf = mean_kib(fetch, pat)
        w, nw = mean_kib(write, pat)
        kern[ph] = {"pattern": pat, "fetch_kib_raw": f, "write_kib_raw": w, "dispatches": [nf, nw],
                    "hbm_bytes_per_launch": (f * fscale + w * wscale) * 1024}
    win = {}
    for ph, pat in list(patterns.items()) + [("loss_reduce", r"reduce_loss_kernel")]:
        d = sorted((int(r["Start_Timestamp"]), int(r["End_Timestamp"])) for r in trace
                   if re.search(pat, r["Kernel_Name"]))
        sel = d[warmup * n_layers:(warmup + steps) * n_layers]
        win[ph] = (len(sel), sum(e - b for b, e in sel) / max(1, len(sel)) / 1e3)
    js = {"workload": workload, "src_hash": src_hash(), "fetch_scale": fscale, "write_scale": wscale,
          "calibration": "plain 256 MiB device copy (torch copy_ -> __amd_rocclr_copyBuffer): FETCH_SIZE and "
                         "WRITE_SIZE scaled so that it reads and writes 262144 KiB",
          "kernels": kern, "trace_timed_avg_us": {ph: v[1] for ph, v in win.items()}}
    json.dump(js, open(os.path.join(out_dir, f"pmc_{workload}.json"), "w"), indent=1)
    cmd_common = (f"--workload {workload} --no-cpu-baseline --no-block --no-ceilings --sub-workloads ''"
                  + ("" if fused else " --unfused"))
    lines = [f"# rocprofv3 summary: UniQuan_F step kernels, workload `{workload}`", "",
             f"Workload: {wl.description}; bench.py step (unified initialisation G = 30, T = 15 at set-up, "
             "residual loss form, LOCAL/FROZEN mapping alternating, " + (
                 "two GEMMs and the fused backward + SGD + next forward pass" if fused else
                 "four passes") + "); MI355X.", "",
             "Commands (run from the repository root on the GPU box; the summary is then written on the CPU "
             f"with `python bench.py --summarize-profiles {workload} --steps {steps} --warmup {warmup}`):", "",
             "```",
             f"rocprofv3 --kernel-trace --stats -f csv -d gpurun_out/prof_{workload} -o trace -- "
             f"python3 bench.py --steps {steps} --warmup {warmup} {cmd_common}",
             f"rocprofv3 --pmc FETCH_SIZE -f csv -d gpurun_out/pmc_fetch_{workload} -o fetch -- "
             f"python3 bench.py --steps 2 --warmup 1 {cmd_common} --calib-copy",
             f"rocprofv3 --pmc WRITE_SIZE -f csv -d gpurun_out/pmc_write_{workload} -o write -- "
             f"python3 bench.py --steps 2 --warmup 1 {cmd_common} --calib-copy",
             "```", "", f"Kernel sources hash (bench.src_hash): `{src_hash()}`", "",
             f"## Timed steps only ({steps} steps after {warmup} warm-up steps, {n_layers} layers)", "",
             "Per-dispatch durations from the trace (`trace_kernel_trace.csv`), each phase kernel's dispatches in "
             "time order after the warm-up steps.  The bench's per-phase HIP events bracket a phase: gemm_fwd "
             "is the loss GEMM plus its loss reduction.", "",
             "| Phase | Kernel pattern | Dispatches | Average (us) |", "|---|---|---|---|"]
    for ph, (n, avg) in win.items():
        lines.append(f"| {ph} | `{patterns.get(ph, 'reduce_loss_kernel')}` | {n} | {avg:.1f} |")
    lines += ["", "## HBM traffic per launch (`--pmc FETCH_SIZE`, `--pmc WRITE_SIZE`)", "",
              f"Calibration on a plain 256 MiB device copy: FETCH_SIZE x {fscale:.3f}, WRITE_SIZE x {wscale:.3f}.",
              "", "| Phase | Kernel pattern | FETCH_SIZE raw (KiB) | WRITE_SIZE (KiB) | HBM bytes / launch (scaled) |",
              "|---|---|---|---|---|"]
    for ph, k in kern.items():
        lines.append(f"| {ph} | `{k['pattern']}` | {k['fetch_kib_raw']:.0f} | {k['write_kib_raw']:.0f} | "
                     f"{k['hbm_bytes_per_launch'] / 1e6:.1f} MB |")
    lines += ["", "## Kernel trace statistics (`--kernel-trace --stats`, whole run)", "",
              "| Kernel | Calls | Average (us) | Min (us) | Max (us) | Share of GPU time |", "|---|---|---|---|---|---|"]
    for r in stats:
        n = r["Name"]
        if "uq::" not in n:
            continue
        n = re.sub(r"\(uq::\w+\)", "", n).replace("void ", "")
        lines.append(f"| `{n[:90]}` | {r['Calls']} | {float(r['AverageNs']) / 1e3:.1f} | "
                     f"{float(r['MinNs']) / 1e3:.1f} | {float(r['MaxNs']) / 1e3:.1f} | {float(r['Percentage']):.1f}% |")
    open(os.path.join(out_dir, f"uniquan_kernels_{workload}.md"), "w").write("\n".join(lines) + "\n")
    print("\n".join(lines))


def summarize_block_profile(out_dir=PROFILES, run_dir=os.path.join(ROOT, "gpurun_out")):
    """Write profiles/decoder_block7b.md from a kernel trace of the bench's two
    decoder-block legs (command in the summary): per step (the kernels from
    one attention forward to the next), the median fused-form step of the
    multi-head leg and of the grouped-query leg (they run in that order), by
    kernel, with the attention kernels' rates."""
    import collections
    import csv
    import re
    pdir = os.path.join(run_dir, "prof_block7b")
    rows = sorted(csv.DictReader(open(os.path.join(pdir, "trace_kernel_trace.csv"))),
                  key=lambda r: int(r["Start_Timestamp"]))
    marks = [i for i, r in enumerate(rows) if "attn_fwd_kernel" in r["Kernel_Name"]]
    cycles = []
    for i0, i1 in zip(marks, marks[1:]):
        ks = rows[i0:i1]
        if not any("fq_step_kernel" in r["Kernel_Name"] for r in ks):
            continue
        agg, cnt = collections.defaultdict(float), collections.Counter()
        for r in ks:
            n = re.sub(r"\(.*", "", r["Kernel_Name"]).replace("void ", "")
            agg[n] += (int(r["End_Timestamp"]) - int(r["Start_Timestamp"])) / 1e3
            cnt[n] += 1
        wall = (int(rows[i1]["Start_Timestamp"]) - int(rows[i0]["Start_Timestamp"])) / 1e3
        cycles.append((wall, agg, cnt))
    half = len(cycles) // 2
    legs = {"multi-head (32 key/value heads)": cycles[:half], "grouped-query (8 key/value heads)": cycles[half:]}
    B, L, d = 128, 2048, 128
    per_product = 2.0 * B * (L * (L + 32) / 2) * d        # causal, diagonal tiles whole
    flops = {"attn_fwd_kernel": 3 * per_product, "attn_bwd_dq_kernel": 3 * per_product,
             "attn_bwd_dkv_kernel": 4 * per_product}
    cmd = ("rocprofv3 --kernel-trace --stats -f csv -d gpurun_out/prof_block7b -o trace -- python3 bench.py "
           "--steps 3 --warmup 1 --workload mlp7b --no-cpu-baseline --no-ceilings --sub-workloads ''")
    lines = ["# rocprofv3 summary: the 7B decoder block step, kernel by kernel", "",
             "Workload: one 7B decoder block (C = 4096 in 32 heads of 128, I = 11008), 8192 tokens as 4 "
             "sequences of 2048, k = 3, g = 128, all seven matrices quantized, the fused step form (block "
             "forward, loss, backpropagation, one fused backward + SGD + next forward per matrix); the bench's "
             "block legs (`block_decoder`, `block_decoder_gqa`).  MI355X.", "",
             "Command (run from the repository root on the GPU box; the summary is then written on the CPU "
             "with `python bench.py --summarize-block-profile`):", "", "```", cmd, "```", ""]
    for leg, cyc in legs.items():
        if not cyc:
            continue
        cyc = sorted(cyc, key=lambda c: c[0])
        wall, agg, cnt = cyc[len(cyc) // 2]
        tot = sum(agg.values())
        lines += [f"## {leg}: median of {len(cyc)} fused steps", "",
                  f"Step {wall / 1e3:.2f} ms from one attention forward to the next, {tot / 1e3:.2f} ms of kernel "
                  "time.", "", "| Kernel | Calls | Time (us) | Share | Rate |", "|---|---|---|---|---|"]
        for n, v in sorted(agg.items(), key=lambda x: -x[1]):
            base = re.sub(r"<.*", "", n).replace("uq::", "")
            rate = f"{flops[base] / (v / cnt[n] * 1e-6) / 1e12:.0f} TFLOP/s" if base in flops else ""
            lines.append(f"| `{n[:80]}` | {cnt[n]} | {v:.1f} | {100 * v / tot:.1f}% | {rate} |")
        lines.append("")
    open(os.path.join(out_dir, "decoder_block7b.md"), "w").write("\n".join(lines))
    print("\n".join(lines))


def progress(msg):
    """One progress line on stderr (stdout carries only the JSON line)."""
    print(f"[bench {time.strftime('%H:%M:%S')}] {msg}", file=sys.stderr, flush=True)


def build_layers(wl, args, want_cpu):
    """Device state of every (matrix, k) of a workload: synthetic data,
    unified initialisation (timed), the initial FULL mapping and L0."""
    import torch

    from paper_2506_03781_amd import synth
    from paper_2506_03781_amd import uniquan as uq
    from paper_2506_03781_amd.layer import QuantLayer
    layers, host_np, init_ms = [], [], []
    init_np, X_np = None, None
    for spec in wl.matrices:
        g = wl.group_size or spec.C
        m = synth.make_matrix(spec, args.seed)
        progress(f"{wl.name}: {spec.name} {spec.R}x{spec.C} generated")
        wdt = torch.bfloat16 if spec.dtype == "bf16" else torch.float32
        for k in wl.ks:
            lay = QuantLayer(m.W, m.X, m.s, k, g, w_dtype=wdt, residual=not args.target)
            if args.init == "unified":
                if not layers:
                    lay.init_unified(args.init_grid, args.init_rounds, args.init_clip)  # first-launch warm-up
                e0, e1 = TimingEvent(), TimingEvent()
                e0.record()
                lay.init_unified(args.init_grid, args.init_rounds, args.init_clip)
                e1.record()
                torch.cuda.synchronize()
                init_ms.append(e0.elapsed_time(e1))
                if init_np is None and want_cpu:
                    init_np = (m.W[:64].copy(), k, g)
            else:
                lay.init_greedy()
            lay.prepare()
            lay.fq_fwd(uq.MAP_FULL)        # initial mapping computes every distance
            # SGD on L / L0 (L0 the loss at the initialisation): the paper's
            # learning rates on the plain sum diverge within a step at these
            # sizes, and timing a non-finite state would not time the method
            lay.recon(backward=False)
            lay.l0 = float(lay.loss.item())
            lay.lr = (0.005 / lay.l0, 0.0005 / lay.l0)
            layers.append(lay)
            if want_cpu and len(host_np) < 2:
                nr = min(m.R, 4096)
                host_np.append((m.W[:nr].copy(), m.s[:nr].copy(), k, g))
                if X_np is None:
                    X_np = m.X.copy()
        del m
    torch.cuda.synchronize()
    return layers, init_ms, host_np, init_np, X_np


PHASES = ["fq_fwd", "gemm_fwd", "gemm_bwd", "fq_bwd"]
FUSED_PHASES = ["gemm_fwd", "gemm_bwd", "fq_step"]


class StepRunner:
    """The timed steps of a list of layers.  Each phase's launches are
    recorded through the checked wrappers the first time it runs (a warm-up
    step) and replayed afterwards, so the host enqueues a phase in a few
    microseconds and the stream stays ahead of the GPU; the timing events are
    created before the timed steps.

    fused = False: fq_fwd -> loss GEMM -> weight-gradient GEMM -> fq_bwd with
    SGD.  fused = True: loss GEMM -> weight-gradient GEMM -> fq_step (the
    backward with SGD and the next step's forward in one pass); the first
    step's forward is the initial mapping done at set-up, so every step still
    runs the whole hot path once."""

    def __init__(self, layers, mode, fused=False):
        self.layers, self.mode, self.fused = layers, mode, fused
        self.phases = FUSED_PHASES if fused else PHASES
        self.launches = {}

    def phase(self, li, name, mode, fn, *a):
        from paper_2506_03781_amd import uniquan as uq
        key = (li, name, mode)
        if key in self.launches:
            self.launches[key]()
        else:
            self.launches[key] = uq.record(fn, *a)

    def step(self, step, evs=None):
        from paper_2506_03781_amd import uniquan as uq
        mode = schedule(self.mode, step)
        nxt = schedule(self.mode, step + 1)
        for li, lay in enumerate(self.layers):
            es = evs[li] if evs is not None else None
            calls = ([] if self.fused else [("fq_fwd", mode, lay.fq_fwd, (mode,))]) + [
                ("gemm_fwd", 0, lay.recon, (False,)),
                ("gemm_bwd", 0, uq.uniquan_layer_grad, (lay.T, lay.R, lay.C, lay.Et, lay.Xt, lay.G))]
            if self.fused:
                calls.append(("fq_step", nxt, lay.fq_step, (*lay.lr, nxt)))
            else:
                calls.append(("fq_bwd", 0, lay.fq_bwd_sgd, lay.lr))
            for i, (name, md, fn, a) in enumerate(calls):
                if es:
                    es[i].record()
                self.phase(li, name, md, fn, *a)
            if es:
                es[len(calls)].record()

    def run(self, steps, warmup, first_step=0):
        """warmup untimed steps, then `steps` timed ones; per-phase HIP events."""
        import torch
        nph = len(self.phases)
        pool = [[[TimingEvent() for _ in range(nph + 1)] for _ in self.layers] for _ in range(steps)]
        for s_ in range(warmup):
            self.step(first_step + s_)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for s_ in range(steps):
            self.step(first_step + warmup + s_, pool[s_])
        torch.cuda.synchronize()
        t1 = time.perf_counter()
        tot = {p: 0.0 for p in self.phases}
        per_layer = []
        for li in range(len(self.layers)):
            d = {p: 0.0 for p in self.phases}
            for es_step in pool:
                es = es_step[li]
                for i, p in enumerate(self.phases):
                    d[p] += es[i].elapsed_time(es[i + 1])
            for p in self.phases:
                d[p] /= steps
                tot[p] += d[p]
            per_layer.append(d)
        self.next_step = first_step + warmup + steps
        return {"ms_per_step": (t1 - t0) * 1e3 / steps, "wall_s": t1 - t0, "tot": tot, "per_layer": per_layer}


def layer_kernel_stats(layers, tot, mode0):
    """Per-phase achieved rates, averaged over the layers' launches."""
    import torch
    n = len(layers)
    out = {}
    for ph in tot:
        dur_ms = tot[ph] / n
        if ph in ("gemm_fwd", "gemm_bwd"):
            work = sum(2.0 * l.T * l.R * l.C for l in layers) / n
            ach = work / (dur_ms * 1e-3) / 1e12
            out[ph] = dict(bound="mfma", achieved=ach, peak=MFMA_BF16_PEAK_TFLOPS, unit="TFLOP/s",
                           frac=ach / MFMA_BF16_PEAK_TFLOPS, avg_ms=dur_ms, algorithmic_flops=work)
            continue
        byt = 0.0
        for l in layers:
            wb = 2 if l.W.dtype == torch.bfloat16 else 4
            if ph == "fq_step":
                byt += sum(fq_step_bytes_per_weight(l.k, l.g, wb)) * l.R * l.C
            else:
                f, b = fq_bytes_per_weight(l.k, l.g, mode0, wb)
                byt += (f if ph == "fq_fwd" else b) * l.R * l.C
        byt /= n
        ach = byt / (dur_ms * 1e-3) / 1e9
        out[ph] = dict(bound="hbm", achieved=ach, peak=HBM_PEAK_GBS, unit="GB/s", frac=ach / HBM_PEAK_GBS,
                       avg_ms=dur_ms, algorithmic_bytes=byt)
    return out


def step_summary(layers, res, mode0):
    import torch
    tot = res["tot"]
    weights = sum(l.R * l.C for l in layers)
    flops = sum(4.0 * l.T * l.R * l.C for l in layers)
    fused = "fq_step" in tot
    fq_ms = tot["fq_step"] if fused else tot["fq_fwd"] + tot["fq_bwd"]
    gemm_ms = tot["gemm_fwd"] + tot["gemm_bwd"]
    fq_bytes = 0.0
    for l in layers:
        wb = 2 if l.W.dtype == torch.bfloat16 else 4
        if fused:
            fq_bytes += sum(fq_step_bytes_per_weight(l.k, l.g, wb)) * l.R * l.C
        else:
            f, b = fq_bytes_per_weight(l.k, l.g, mode0, wb)
            fq_bytes += (f + b) * l.R * l.C
    fq_gbs = fq_bytes / (fq_ms * 1e-3) / 1e9
    gemm_tflops = flops / (gemm_ms * 1e-3) / 1e12
    rel = [float(l.loss.item()) / l.l0 for l in layers]
    finite = all(math.isfinite(r) for r in rel) and all(bool(torch.isfinite(l.s).all()) for l in layers)
    return {"value": weights / (fq_ms * 1e-3) / 1e9, "fq_hbm_gbs": fq_gbs, "fq_frac_hbm": fq_gbs / HBM_PEAK_GBS,
            "gemm_tflops": gemm_tflops, "gemm_frac_mfma": gemm_tflops / MFMA_BF16_PEAK_TFLOPS,
            "rel_loss": rel, "finite": finite}


def sub_record(name, args, steps, warmup):
    """A compact record of another configuration: the same step, kernels and
    method as the headline; only the sizes differ."""
    import torch

    from paper_2506_03781_amd import synth
    wl = synth.WORKLOADS[name]
    layers, init_ms, _, _, _ = build_layers(wl, args, False)
    mode0 = "local" if args.mode == "paper" else args.mode
    res = StepRunner(layers, args.mode, fused=not args.unfused).run(steps, warmup)
    sm = step_summary(layers, res, mode0)
    ks = layer_kernel_stats(layers, res["tot"], mode0)
    rec = {"description": wl.description, "matrices": [[l.R, l.C] for l in layers], "T": layers[0].T,
           "k": [l.k for l in layers], "g": [l.g for l in layers], "steps": steps, "warmup": warmup,
           "ms_per_step": res["ms_per_step"], "timed_s": res["wall_s"],
           "value": sm["value"], "unit": "Gweights/s", "fq_frac_hbm": sm["fq_frac_hbm"],
           "gemm_tflops": sm["gemm_tflops"], "gemm_frac_mfma": sm["gemm_frac_mfma"],
           "phase_ms_per_step": res["tot"],
           "kernels": {p: {"avg_ms": v["avg_ms"], "achieved": v["achieved"], "unit": v["unit"], "frac": v["frac"]}
                       for p, v in ks.items()},
           "init_ms_total": sum(init_ms), "rel_loss_after_timed_steps": sm["rel_loss"],
           "state_finite": sm["finite"]}
    del layers
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    return rec


def main():
    args = parse()
    if args.summarize_profiles:
        summarize_profiles(args.summarize_profiles, args.steps, args.warmup, fused=not args.unfused)
        return
    if args.summarize_block_profile:
        summarize_block_profile()
        return
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (got --gpus {args.gpus}); this build has no multi-GPU path.",
              file=sys.stderr)
        sys.exit(2)
    import torch

    from paper_2506_03781_amd import synth
    from paper_2506_03781_amd import uniquan as uq

    assert torch.cuda.is_available(), "bench.py needs a GPU"
    torch.cuda.set_device(0)
    uq.lib()
    wl = synth.WORKLOADS[args.workload]
    g = wl.group_size
    want_cpu = not args.no_cpu_baseline
    layers, init_ms, host_np, init_np, X_np = build_layers(wl, args, want_cpu)
    mode0 = "local" if args.mode == "paper" else args.mode

    runner = StepRunner(layers, args.mode, fused=not args.unfused)
    if args.calib_copy:
        src = torch.empty(64 << 20, dtype=torch.float32, device="cuda")
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        del src, dst
    res = runner.run(args.steps, args.warmup)
    progress(f"{args.workload}: {args.steps} timed steps, {res['ms_per_step']:.3f} ms per step")
    tot, per_layer = res["tot"], res["per_layer"]
    sm = step_summary(layers, res, mode0)
    ks = layer_kernel_stats(layers, tot, mode0)
    dom = max(ks, key=lambda p: ks[p]["avg_ms"])
    counters = load_counters(args.workload)
    for p, st in ks.items():
        tr = None
        if counters and p in counters.get("kernels", {}):
            tr = counters["kernels"][p].get("hbm_bytes_per_launch")
        st["traffic"] = tr
    roof = {k2: ks[dom][k2] for k2 in ("bound", "achieved", "peak", "unit", "frac", "traffic")}
    roof["kernel"] = dom

    # per-mode forward times (after the timed region)
    by_mode = {}
    for name, md in (("full", uq.MAP_FULL), ("local", uq.MAP_LOCAL), ("frozen", uq.MAP_FROZEN)):
        lay = layers[0]
        a, b = TimingEvent(), TimingEvent()
        fwd = uq.record(lay.fq_fwd, md)
        a.record()
        for _ in range(10):
            fwd()
        b.record()
        torch.cuda.synchronize()
        by_mode[name] = a.elapsed_time(b) / 10 * 1e3

    # the same steps with the backward quantizer fused into the weight-gradient
    # GEMM's epilogue (after the timed region; not part of `value`)
    fused = None
    if all(l.k <= 4 and l.g <= 128 and l.T % 32 == 0 for l in layers):
        nfs = min(args.steps, 10)
        fev = []
        fpool = [[TimingEvent() for _ in range(2)] for _ in range(nfs)]
        for s_ in range(nfs + 2):
            mode = schedule(args.mode, runner.next_step + s_)
            e = fpool.pop() if s_ >= 2 else None
            if e:
                e[0].record()
            for li, lay in enumerate(layers):
                runner.phase(li, "fq_fwd", mode, lay.fq_fwd, mode)
                runner.phase(li, "gemm_fwd", 0, lay.recon, False)
                runner.phase(li, "ste_sgd", 0, lay.grad_ste_sgd, *lay.lr)
            if e:
                e[1].record()
                fev.append(e)
        torch.cuda.synchronize()
        fused_ms = sum(a.elapsed_time(b) for a, b in fev) / len(fev)
        fused = {"ms_per_step": fused_ms, "headline_ms_per_step_events": sum(tot.values()), "steps": nfs,
                 "note": "fq_fwd -> loss GEMM -> weight-gradient GEMM with the straight-through backward "
                         "and SGD update in its epilogue (dL/dWhat never written)"}

    # the other form of the step (four passes, or the fused one), for comparison
    alt_runner = StepRunner(layers, args.mode, fused=args.unfused)
    alt = alt_runner.run(min(args.steps, 10), 2, first_step=runner.next_step)
    alt_sm = step_summary(layers, alt, mode0)
    alt_rec = {"fused": bool(args.unfused), "ms_per_step": alt["ms_per_step"], "phase_ms_per_step": alt["tot"],
               "value": alt_sm["value"], "fq_frac_hbm": alt_sm["fq_frac_hbm"], "gemm_tflops": alt_sm["gemm_tflops"],
               "steps": min(args.steps, 10),
               "note": ("fq_fwd -> loss GEMM -> weight-gradient GEMM -> fq_bwd with SGD, four passes"
                        if not args.unfused else "loss GEMM -> weight-gradient GEMM -> fq_step (backward + SGD "
                        "+ next forward in one pass)")}
    bcq = bcq_inference(layers)
    progress("per-mode, fused and deployment legs done")
    rel_loss, finite = sm["rel_loss"], sm["finite"]
    out = {
        "metric": "fake-quant fwd+bwd Gweights/s (%HBM peak); recon GEMM TFLOP/s (%MFMA)",
        "value": sm["value"],
        "unit": "Gweights/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": res["ms_per_step"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "bf16",
        "data": "synthetic",
        "config": {"workload": args.workload, "description": wl.description,
                   "matrices": [[l.R, l.C] for l in layers], "T": layers[0].T, "k": [l.k for l in layers],
                   "g": g, "mapping": args.mode, "seed": args.seed, "parallelism": "single GPU",
                   "loss_form": "target" if args.target else "residual"},
        "fq_hbm_gbs": sm["fq_hbm_gbs"],
        "fq_frac_hbm": sm["fq_frac_hbm"],
        "gemm_tflops": sm["gemm_tflops"],
        "gemm_frac_mfma": sm["gemm_frac_mfma"],
        "phase_ms_per_step": tot,
        "per_layer_phase_ms": per_layer,
        "kernels": ks,
        "fq_fwd_us_by_mode": by_mode,
        "roofline": roof,
        "fused_bwd_step": fused,
        "step_form": ("two GEMMs + fq_step (straight-through backward with SGD fused with the next step's "
                      "forward; the first forward is the initial mapping at set-up)") if not args.unfused else
                     "four passes: fq_fwd, loss GEMM, weight-gradient GEMM, fq_bwd with SGD",
        "other_step_form": alt_rec,
        "optimiser": {"rule": "SGD on L / L_init per layer (learning rates 0.005 for s, 0.0005 for alpha and z_B, "
                              "divided by the layer's initial loss)",
                      "rel_loss_after_timed_steps": rel_loss, "state_finite": finite},
        "bcq_inference": {"per_call": bcq,
                          "note": "deployed layer (fold -> bit-planes + binary16 Theta*_B): Y = X What^T for T "
                                  "activation rows; bytes = planes + parameters + X + Y"},
        "counters_src_hash": src_hash(),
        "precision": "quantizer: fp32 arithmetic on bf16 W / fp32 s, bf16 What and dL/dWhat; "
                     "GEMMs: bf16 MFMA with fp32 accumulation",
    }
    if init_ms:
        iw = sum(l.R * l.C for l in layers)
        ops = sum(init_ops_per_weight(l.k, args.init_grid, args.init_rounds) * l.R * l.C for l in layers)
        isec = sum(init_ms) * 1e-3
        ach = ops / isec / 1e12
        out["init"] = {
            "method": "unified", "grid_G": args.init_grid, "alt_T": args.init_rounds, "clip": args.init_clip,
            "ms_per_layer": init_ms, "ms_total": sum(init_ms), "gweights_per_s": iw / isec / 1e9,
            "roofline": {"bound": "alu", "achieved": ach, "peak": VALU_PEAK_TOPS, "unit": "Tops/s",
                         "frac": ach / VALU_PEAK_TOPS, "algorithmic_ops": ops},
        }
    fq_mix = [0.0, 0.0]
    for l in layers:
        wb = 2 if l.W.dtype == torch.bfloat16 else 4
        r_, w_ = fq_read_write_bytes(l.k, l.g, mode0, wb) if args.unfused else fq_step_bytes_per_weight(l.k, l.g, wb)
        fq_mix[0] += r_ * l.R * l.C
        fq_mix[1] += w_ * l.R * l.C
    del layers, runner
    torch.cuda.synchronize()
    torch.cuda.empty_cache()

    if not args.no_ceilings:
        ce = ceilings()
        progress(f"ceilings: {json.dumps({k: round(v, 1) for k, v in ce.items() if k != 'note'})}")
        out["ceilings"] = ce
        ach_fq = sm["fq_hbm_gbs"]
        # the quantizer kernels read more than they write: the ceiling of
        # their mix is time = read bytes / read rate + written bytes / write rate
        rd, wr = fq_mix
        mix = (rd + wr) / (rd / ce["read_gbs"] + wr / ce["write_gbs"])
        out["ceilings"]["fq_mix_ceiling_gbs"] = mix
        out["ceilings"]["fq_frac_of_mix_ceiling"] = ach_fq / mix
        out["ceilings"]["fq_frac_of_copy"] = ach_fq / ce["copy_gbs"]
        out["ceilings"]["fq_frac_of_read"] = ach_fq / ce["read_gbs"]
        out["ceilings"]["gemm_frac_of_mfma_probe"] = sm["gemm_tflops"] / ce["mfma_bf16_tflops"]
        out["ceilings"]["roofline_frac_of_measured"] = roof["achieved"] / (
            ce["mfma_bf16_tflops"] if roof["bound"] == "mfma" else ce["copy_gbs"])

    subs = [w for w in args.sub_workloads.split(",") if w and w != args.workload]
    if subs:
        out["workloads"] = {}
        for w in subs:
            n_steps = args.block7b_steps if w == "block7b" else args.sub_steps
            out["workloads"][w] = sub_record(w, args, n_steps, min(args.warmup, 5))
            progress(f"sub-record {w}: {out['workloads'][w]['ms_per_step']:.3f} ms per step")
        if "block7b" in out["workloads"]:
            out["workloads"]["block7b"]["note"] = (
                f"the 7B block's seven matrices (q, k, v, o, gate, up, down), each a single-layer step; "
                f"{args.block7b_steps} optimisation steps timed")

    if not args.no_block:
        out["block_decoder"] = block_decoder(args.seed, n_kv=args.block_kv)
        progress(f"decoder block: {out['block_decoder']['ms_per_step']:.2f} ms per step")
        # the same block with grouped-query attention (8 key/value heads, as in Mistral 7B and Llama-3 8B)
        if args.block_kv is None:
            out["block_decoder_gqa"] = block_decoder(args.seed, n_kv=8)

    if init_np is not None:
        out["init"]["cpu_baseline"] = cpu_baseline_init(*init_np, args.init_grid, args.init_rounds,
                                                        args.init_clip)
    if want_cpu and host_np:
        progress("cpu baseline (oracle on the host cores)")
        out["cpu_baseline"] = cpu_baseline(host_np, X_np, args.mode)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
