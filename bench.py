"""Benchmark of the rank-compensation hot path on one MI355X.

One step is one pass of the hot path over one batch of synthetic input, in
method precision with every input resident in HBM:
  - factor apply Y = U diag(s) V^T X on the 65536 x 4096 tail-rank stress
    workload (sigma_j = max(exp(-j/40), 1e-6), Haar singular vectors) at
    batch 4096: FP64 at rank k = 512, FP32 and FP16 at the compensated
    rank k + 1 (--matrix square: the 8192 x 8192 workload instead);
  - TT reconstruction of the normalized 512 x 512 x 224 hyperspectral-shaped
    cube from its own fixed-rank TT-SVD: FP64 at ranks (64, 64), FP32 and
    FP16 at (65, 65).
The device certificates of both compensated representations run once after
the timed steps (the paper leaves them out of its timings); their verdicts
and kernel times are reported beside the line.
Prints one JSON line.  `value` is the step's algorithmic GFLOP divided by
its wall time; the `roofline` object describes the apply or TT kernel with
the largest share of the step, timed by the library's HIP-event kernel
timers over the timed steps; `hbm_ceilings_measured_gbps` holds plain
read / write / copy stream rates and `mfma_ceilings_measured_tflops` the
register-only matrix-core rates (`lrc_mfma_ceiling`) measured in the same run;
`cpu_baseline` is the CPU oracle on a bounded sample of the same apply and
TT work (all host threads, with the CPU model and one-thread times of the
small configurations).

  python bench.py [--steps K] [--warmup W] [--k 512] [--matrix tail|square] [--no-cpu-baseline]
  python bench.py --sweep FILE      per-kernel table over the workload grid
  python bench.py --quant FILE      device rounding and TT gauge cells
  python bench.py --grid FILE       the paper's resident timing grid on synthetic stand-ins
  python bench.py --fixed-memory FILE   fixed-memory comparison on hyperspectral-shaped stand-ins
  python bench.py --factor FILE         randomized FP64 SVD / TT-SVD cells
  python bench.py --report FILE.jsonl   markdown tables from the records the sweeps write beside FILE
  python bench.py --apply-cell M N K B PREC [--reps R]   one apply configuration, R calls (for profilers)
  python bench.py --tt-cell DIMS RANKS PREC [--reps R]   one TT reconstruction, R calls (for profilers)
"""
from __future__ import annotations

import argparse
import hashlib
import json
import math
import os
import sys
import time

import numpy as np

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

# MI355X published peaks (dense; no sparsity)
PEAK_HBM_GBS = 8000.0
PEAK_TFLOPS = {"f64": 78.6, "f32": 157.3, "f16": 2500.0}
# FP32 products formed as six bfloat16 products (the split of the large applies)
PEAK_F32_SPLIT = PEAK_TFLOPS["f16"] / 6
EBYTES = {"f64": 8, "f32": 4, "f16": 2}
NPDT = {"f64": np.float64, "f32": np.float32, "f16": np.float16}
METRIC = "GFLOP/s & HBM GB/s (fraction of roofline) for low-rank apply and TT reconstruct"


def log(msg):
    print(msg, file=sys.stderr, flush=True)


def peak_tflops(p, kernel, labels):
    """Matrix-core peak that bounds `kernel` (None: a whole call) among the
    kernels of `labels`: the FP32 apply's where its operands were split into
    bfloat16 planes, else that of the precision's own instruction."""
    split = "apply_planes_f32" in labels and (kernel is None or kernel.startswith("apply_"))
    return PEAK_F32_SPLIT if p == "f32" and split else PEAK_TFLOPS[p]


# ------------------------------------------------------- algorithmic counts --

def apply_counts(m, n, k, b, e):
    """Flops and bytes of Y = U diag(s) V^T X: 2kb(m+n) + kb flops; factors,
    X and Y moved once (T' stays on chip / in cache)."""
    return 2.0 * k * b * (m + n) + k * b, e * (k * (m + n + 1) + b * (m + n))


def apply_phase_counts(m, n, k, b, e):
    p1 = (2.0 * k * b * n + k * b, e * (n * k + n * b + k * b))
    p2 = (2.0 * k * b * m, e * (m * k + m * b + k * b))
    return p1, p2


def tt_counts(dims, ranks, e):
    """Flops of the reshape chain sum_l 2 (prod_{j<l} n_j) r_{l-1} n_l r_l and
    bytes of the cores plus the dense output."""
    f = 0.0
    rows = dims[0]
    for l in range(1, len(dims)):
        f += 2.0 * rows * ranks[l] * dims[l] * ranks[l + 1]
        rows *= dims[l]
    cores = sum(ranks[l] * dims[l] * ranks[l + 1] for l in range(len(dims)))
    return f, e * (rows + cores)


def gram_counts(rows, cols):
    return 2.0 * cols * cols * rows, 8.0 * rows * cols


# ------------------------------------------------------------- workloads ---

def tt_svd_fixed(T, ranks):
    """Fixed-rank TT-SVD of a dense 3-way cube for benchmark inputs (the
    untimed offline factorization): the first unfolding through the
    eigenvectors of its Gram matrix, the second by a thin SVD."""
    n1, n2, n3 = T.shape
    r1, r2 = ranks
    T1 = T.reshape(n1, n2 * n3)
    w, U1 = np.linalg.eigh(T1 @ T1.T)
    U1 = U1[:, ::-1][:, :r1]
    C = (U1.T @ T1).reshape(r1 * n2, n3)
    U2, S2, Vt2 = np.linalg.svd(C, full_matrices=False)
    G1 = np.ascontiguousarray(U1.reshape(1, n1, r1))
    G2 = np.ascontiguousarray(U2[:, :r2].reshape(r1, n2, r2))
    G3 = np.ascontiguousarray((S2[:r2, None] * Vt2[:r2]).reshape(r2, n3, 1))
    return [G1, G2, G3]


class Workload:
    """One benchmark step: the factor apply on the 65536 x 4096 tail-rank
    workload at batch 4096 (FP64 rank k, FP32 / FP16 rank k + 1; or the
    8192 x 8192 workload with --matrix square) and the TT reconstruction of
    the normalized 512 x 512 x 224 cube from its own fixed-rank TT-SVD (FP64
    (64, 64), FP32 / FP16 (65, 65)).  The certificates of both compensated
    representations are run outside the timed steps."""

    def __init__(self, k, dev, matrix="tail"):
        import torch
        from paper_2607_12969_amd import synth
        t0 = time.time()
        self.k = k
        self.matrix = matrix
        w = (synth.matrix_tail(kmax=k, batch=4096) if matrix == "tail"
             else synth.matrix_square(kmax=k, batch=4096))
        self.m, self.n, self.b = w["m"], w["n"], 4096
        self.sigma = w["sigma"]
        r = k + 1
        U, V, s = w["U"][:, :r], w["V"][:, :r], w["sigma"][:r]
        self.f64 = [torch.from_numpy(np.ascontiguousarray(a)).to(dev) for a in (U, s, V)]
        self.apply_in = {}
        for p in ("f64", "f32", "f16"):
            kk = k if p == "f64" else r
            host = [np.ascontiguousarray(a).astype(NPDT[p]) for a in (U[:, :kk], s[:kk], V[:, :kk], w["X"])]
            dv = [torch.from_numpy(a).to(dev) for a in host]
            Y = torch.empty((self.m, self.b), dtype=dv[0].dtype, device=dev)
            self.apply_in[p] = (dv, Y, kk)
        self.cert_h = {p: [torch.from_numpy(np.ascontiguousarray(a).astype(NPDT[p])).to(dev) for a in (U, s, V)]
                       for p in ("f32", "f16")}
        log(f"matrix workload ready ({time.time() - t0:.1f}s)")
        t0 = time.time()
        T = synth.hyperspectral()
        self.dims = list(T.shape)
        base = tt_svd_fixed(T, (64, 64))
        aug = tt_svd_fixed(T, (65, 65))
        self.T = torch.from_numpy(T.reshape(-1)).to(dev)
        self.base = [torch.from_numpy(c).to(dev) for c in base]
        self.aug = [torch.from_numpy(c).to(dev) for c in aug]
        self.tt_in = {}
        for p in ("f64", "f32", "f16"):
            cs = base if p == "f64" else aug
            dv = [torch.from_numpy(c.astype(NPDT[p])).to(dev) for c in cs]
            out = torch.empty(self.dims, dtype=dv[0].dtype, device=dev)
            self.tt_in[p] = (dv, out, [1] + [int(c.shape[2]) for c in cs])
        self.host_tt = {"base": base, "aug": aug}
        self.host_mat = (U, s, V, w["X"])
        log(f"TT workload ready ({time.time() - t0:.1f}s)")

    def describe(self):
        mat = ("65536x4096 sigma_j=max(exp(-j/40),1e-6)" if self.matrix == "tail"
               else "8192x8192 sigma_j=j^-1.5+1e-8 noise")
        return (f"apply {mat} batch 4096 (FP64 k={self.k}, FP32/FP16 k={self.k + 1}) + TT reconstruct "
                "512x512x224 hyperspectral-shaped cube from its own TT-SVD (FP64 (64,64), FP32/FP16 (65,65))")

    def step(self, lrc):
        for p in ("f64", "f32", "f16"):
            dv, Y, _ = self.apply_in[p]
            lrc.matrix_apply(*dv, Y=Y)
        for p in ("f64", "f32", "f16"):
            dv, out, _ = self.tt_in[p]
            lrc.tt_reconstruct(dv, out=out)

    def certify(self, lrc):
        res = {}
        for p in ("f32", "f16"):
            res[("mat", p)] = lrc.certify_matrix(self.sigma, *self.f64, *self.cert_h[p], self.k)
            res[("tt", p)] = lrc.certify_tt(self.T, self.base, self.aug, self.tt_in[p][0])
        return res

    def step_counts(self):
        """(flops, bytes) per labelled piece of one step."""
        m, n, b = self.m, self.n, self.b
        out = {}
        for p in ("f64", "f32", "f16"):
            kk = self.apply_in[p][2]
            out[f"apply_{p}"] = apply_counts(m, n, kk, b, EBYTES[p])
            out[f"tt_{p}"] = tt_counts(self.dims, self.tt_in[p][2] + [1], EBYTES[p])
        return out

    def kernel_counts(self):
        """(flops, bytes, dtype) per kernel launch label of the step."""
        m, n, b = self.m, self.n, self.b
        out = {}
        for p in ("f64", "f32", "f16"):
            kk = self.apply_in[p][2]
            p1, p2 = apply_phase_counts(m, n, kk, b, EBYTES[p])
            out[f"apply_p1_mfma_{p}"] = (*p1, p)
            out[f"apply_p2_mfma_{p}"] = (*p2, p)
            f, by = tt_counts(self.dims, self.tt_in[p][2] + [1], EBYTES[p])
            out[f"tt_fused_{p}"] = (f, by, p)
        return out


# ----------------------------------------------------------------- CPU ---

def cpu_model():
    try:
        with open("/proc/cpuinfo") as fh:
            for ln in fh:
                if ln.startswith("model name"):
                    return ln.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def cpu_baseline(wl, budget_s=12.0):
    """The oracle's FP64 apply and TT reconstruction on a bounded sample of
    the step's work (a fraction of the batch columns and of the cube's first
    mode) on every host thread, scaled to GFLOP/s with the same algorithmic
    flop counts; then single-thread times of the 512 x 256 apply (k = 20,
    batch 64) and of a 256^3 reconstruction at ranks (15, 15)."""
    import oracle as O
    from paper_2607_12969_amd import synth
    names = {"f64": "fp64", "f32": "fp32", "f16": "fp16"}
    U, s, V, X = wl.host_mat
    base, aug = wl.host_tt["base"], wl.host_tt["aug"]
    dims = wl.dims
    threads = len(os.sched_getaffinity(0))
    O.set_num_threads(threads)
    res = None
    stored = {p: [O.stored(a, names[p]) for a in (U[:, :wl.apply_in[p][2]], s[:wl.apply_in[p][2]],
                                                   V[:, :wl.apply_in[p][2]])] for p in names}
    # growing samples; past the whole batch and cube the whole step is repeated
    for frac in (1 / 256, 1 / 64, 1 / 16, 1 / 4, 1, 2, 4, 8):
        reps = max(1, int(frac))
        bs = max(1, int(round(wl.b * min(frac, 1))))
        n1 = max(1, int(round(dims[0] * min(frac, 1))))
        flops = 0.0
        t0 = time.time()
        for p in ("f64", "f32", "f16") * reps:
            kk = wl.apply_in[p][2]
            O.apply(*stored[p], O.stored(X[:, :bs], names[p]))
            flops += apply_counts(wl.m, wl.n, kk, bs, 8)[0]
            cs = base if p == "f64" else aug
            cs = [O.stored(c, names[p]) for c in cs]
            cs[0] = np.ascontiguousarray(cs[0][:, :n1, :])
            O.tt_full(cs)
            ranks = [1, cs[0].shape[2], cs[1].shape[2], 1]
            flops += tt_counts([n1] + dims[1:], ranks, 8)[0]
        el = time.time() - t0
        res = dict(value=round(flops / el / 1e9, 3), unit="GFLOP/s", cores=O.num_threads(), kind="oracle",
                   cpu_model=cpu_model(),
                   sample=(f"FP64 oracle apply (3 methods, batch {bs} of 4096) and TT reconstruction "
                           f"(3 methods, first {n1} of 512 slabs), {reps} pass(es); {flops / 1e9:.1f} GFLOP in "
                           f"{el:.1f}s; certificates not included"))
        if el >= budget_s:
            break
    # one thread: the small configurations
    O.set_num_threads(1)
    try:
        w = synth.matrix_small()
        m1, n1_, k1 = w["m"], w["n"], 20
        Us, ss, Vs = w["U"][:, :k1], w["sigma"][:k1], w["V"][:, :k1]
        t0 = time.perf_counter()
        reps = 0
        while time.perf_counter() - t0 < 1.0 or reps < 3:
            O.apply(Us, ss, Vs, w["X"])
            reps += 1
        c1_ms = (time.perf_counter() - t0) / reps * 1e3
        cores4 = synth.random_tt_cores((256, 256, 256), (1, 15, 15, 1), tag=1)
        t0 = time.perf_counter()
        O.tt_full(cores4)
        c4_ms = (time.perf_counter() - t0) * 1e3
        c1_f = apply_counts(m1, n1_, k1, 64, 8)[0]
        c4_f = tt_counts([256, 256, 256], [1, 15, 15, 1], 8)[0]
        res["one_thread"] = {
            "apply_512x256_k20_b64": {"ms": round(c1_ms, 4), "gflops": round(c1_f / c1_ms / 1e6, 3)},
            "tt_256^3_ranks15": {"ms": round(c4_ms, 2), "gflops": round(c4_f / c4_ms / 1e6, 3)},
        }
    finally:
        O.set_num_threads(threads)
    return res


# ------------------------------------------------------------ HBM ceilings ---

def hbm_ceilings(dev, gib=4):
    """Read, write and copy rates of plain device-wide streams over a `gib`
    GiB buffer (far above the 256 MB Infinity Cache): a sum reduction
    (read), a fill (write) and a copy, each timed with torch's events on the
    current stream (median of 5).  Context for the kernels' fractions; the
    spec peak stays the reference."""
    import torch
    n = (gib << 30) // 8
    a = torch.ones(n, dtype=torch.float64, device=dev)
    b = torch.empty_like(a)
    out = {}
    for name, fn, nbytes in (("read", lambda: a.sum(), 8 * n), ("write", lambda: b.fill_(2.0), 8 * n),
                             ("copy", lambda: b.copy_(a), 16 * n)):
        for _ in range(2):
            fn()
        ts = []
        for _ in range(5):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            fn()
            e1.record()
            e1.synchronize()
            ts.append(e0.elapsed_time(e1))
        out[name] = round(nbytes / (sorted(ts)[2] * 1e-3) / 1e9, 1)
    del a, b
    torch.cuda.empty_cache()
    return out


# ---------------------------------------------------------------- traffic ---

def kernel_source_hash():
    """Hash of the kernel sources and their launch plans (the .hip files and
    the headers); host-only API code does not change HBM traffic."""
    h = hashlib.sha256()
    d = os.path.join(ROOT, "paper_2607_12969_amd", "csrc")
    for f in sorted(os.listdir(d)):
        if f.endswith((".hip", ".h")):
            with open(os.path.join(d, f), "rb") as fh:
                h.update(fh.read())
    return h.hexdigest()[:16]


def measured_traffic(label):
    """HBM bytes per launch of `label` from the committed counter summary,
    or None if the kernel sources changed since the counters were taken."""
    path = os.path.join(ROOT, "profiles", "traffic_counters.md")
    if not os.path.exists(path):
        return None
    src, val = None, None
    with open(path) as fh:
        for ln in fh:
            if ln.startswith("source_hash:"):
                src = ln.split(":", 1)[1].strip()
            if ln.startswith(f"| {label} |"):
                cells = [c.strip() for c in ln.strip().strip("|").split("|")]
                val = float(cells[-1])
    if src != kernel_source_hash() or val is None:
        return None
    return val


def round_counts(count, e):
    """Rounding of `count` binary64 values to e-byte storage: no flops to
    speak of; 8 bytes read and e written per value."""
    return 0.0, float(count * (8 + e))


def gauge_counts(dims, ranks):
    """Left-orthogonal gauge by CholeskyQR2, per unfolding l < d (m = r_{l-1}
    n_l rows, r = r_l columns, c = n_{l+1} r_{l+1} columns of the next
    core): two Gram products counted in full (2 m r^2 each), two triangular
    right products (m r^2 each), one triangular left product (r^2 c).
    Bytes: every core read and written once as Q, the next core read and
    written once for the R product."""
    f = by = 0.0
    for l in range(len(dims) - 1):
        m, r = ranks[l] * dims[l], ranks[l + 1]
        c = dims[l + 1] * ranks[l + 2]
        f += 4.0 * m * r * r + 2.0 * m * r * r + 1.0 * r * r * c
        by += 8.0 * (2 * m * r + 2 * r * c)
    return f, by


# ----------------------------------------------------------------- sweep ---

def _time_cell(lrc, fn, reps, labels):
    """Average per-launch milliseconds of each kernel label over `reps`
    calls of fn(rep) (after 3 warmup calls)."""
    import torch
    for r in range(3):
        fn(r)
    torch.cuda.synchronize()
    lrc.profile_reset()
    lrc.profile_enable(True)
    t0 = time.perf_counter()
    for r in range(reps):
        fn(r)
    torch.cuda.synchronize()
    wall = (time.perf_counter() - t0) / reps * 1e3
    lrc.profile_enable(False)
    kt = lrc.profile_read()
    return wall, {lab: kt[lab][1] / kt[lab][0] for lab in kt}


ENV_KNOBS = ("LRC_APPLY_TILE", "LRC_TT_WAVE", "LRC_TT_WAVE_NPB", "LRC_TT_P", "LRC_TT_WGS", "LRC_TT_CERT_SPLIT",
             "LRC_TT_MERGE")


def env_knobs():
    """The library's tuning overrides as set for this run (None = default)."""
    return {k: os.environ.get(k) for k in ENV_KNOBS}


def write_records(path, records):
    """One JSON object per line: the machine-readable twin of a table."""
    with open(path, "w") as fh:
        for r in records:
            fh.write(json.dumps(r, sort_keys=True) + "\n")


def read_records(path):
    with open(path) as fh:
        return [json.loads(line) for line in fh if line.strip()]


def _record(task, method, p, kernels_ms, wall_ms, f, by, **shape):
    """One sweep cell: algorithmic counts, the roofline of the cell and its
    measured times.  Parity is the tests' business (the bench never calls
    the oracle outside its CPU baseline), so parity_error stays null."""
    ai = f / by
    peak = peak_tflops(p, None, kernels_ms)
    ridge = peak * 1e12 / (PEAK_HBM_GBS * 1e9)
    kern = sum(kernels_ms.values())
    t_star = max(by / (PEAK_HBM_GBS * 1e9), f / (peak * 1e12)) * 1e3
    return dict(task=task, method=method, prec=p, **shape, flop=f, bytes=by, intensity=ai,
                bound="mfma" if ai > ridge else "hbm", t_star_ms=t_star, kernels_ms=kern, call_ms=wall_ms,
                gflops=f / kern / 1e6, gbs=by / kern / 1e6, frac=t_star / kern,
                per_kernel_ms=dict(kernels_ms), counter_bytes=None, parity_error=None, certificate=None,
                env=env_knobs())


SWEEP_HEAD = ["| cell | prec | GFLOP | MB | flop/B | bound | t* us | kernels us | call us | GFLOP/s | GB/s | "
              "frac of bound | per kernel (us) |", "|" + "---|" * 13]


def render_sweep_row(r):
    ks = ", ".join(f"{k} {v * 1e3:.1f}" for k, v in r["per_kernel_ms"].items())
    return (f"| {r['task']} | {r['prec']} | {r['flop'] / 1e9:.3f} | {r['bytes'] / 1e6:.1f} | {r['intensity']:.1f} | "
            f"{r['bound']} | {r['t_star_ms'] * 1e3:.1f} | {r['kernels_ms'] * 1e3:.1f} | {r['call_ms'] * 1e3:.1f} | "
            f"{r['gflops']:.0f} | {r['gbs']:.0f} | {r['frac']:.3f} | {ks} |")


def sweep(path, dev, lrc):
    """Every apply and TT cell of the workload grid, one at a time: kernel
    times from the library's HIP-event timers; inputs rotated over enough
    copies that consecutive calls do not hit the 256 MB Infinity Cache."""
    import torch
    from paper_2607_12969_amd import synth
    records = []

    def rotated(host_arrays, out_shape, dtype, bytes_per_call):
        copies = max(1, min(8, math.ceil(512e6 / max(bytes_per_call, 1))))
        sets = []
        for _ in range(copies):
            ins = [torch.from_numpy(a).to(dev) for a in host_arrays]
            out = torch.empty(out_shape, dtype=dtype, device=dev)
            sets.append((ins, out))
        return sets

    mats = [("512x256", synth.matrix_small(), [20], [64]),
            ("8192x8192", synth.matrix_square(kmax=256, batch=4096), [64, 128, 256], [1, 64, 4096]),
            ("65536x4096", synth.matrix_tail(kmax=512, batch=4096), [64, 256, 512], [4096])]
    for name, w, ks, bs in mats:
        m, n = w["m"], w["n"]
        U = w["U"]
        V = w["V"]
        sig = w["sigma"]
        for k in ks:
            for b in bs:
                for p in ("f64", "f32", "f16"):
                    kk = k if p == "f64" else k + 1
                    host = [np.ascontiguousarray(a).astype(NPDT[p]) for a in
                            (U[:, :kk], sig[:kk], V[:, :kk], w["X"][:, :b])]
                    f, by = apply_counts(m, n, kk, b, EBYTES[p])
                    sets = rotated(host, (m, b), torch.from_numpy(host[0][:1]).dtype, by)
                    reps = max(10, min(200, int(2e10 / max(f, 1))))
                    wall, km = _time_cell(lrc, lambda r: lrc.matrix_apply(*sets[r % len(sets)][0],
                                                                          Y=sets[r % len(sets)][1]), reps, None)
                    records.append(_record(f"apply {name} k={kk} b={b}", "apply", p, km, wall, f, by,
                                           config=name, m=m, n=n, k=kk, batch=b))
                    log(render_sweep_row(records[-1]))
                    del sets
                    torch.cuda.empty_cache()
    tts = [("256^3 r(15,15)", (256, 256, 256), (15, 15), (15, 15)),
           ("256^3 r(24,24)", (256, 256, 256), (24, 24), (25, 25)),
           ("16^6 r(8,16,24,16,8)", (16,) * 6, (8, 16, 24, 16, 8), (9, 17, 25, 17, 9)),
           ("512x512x224 r(64,64)", (512, 512, 224), (64, 64), (65, 65)),
           ("512x512x224 r(32,32)", (512, 512, 224), (32, 32), (33, 33)),
           ("512x512x224 r(32,32)->(36,36)", (512, 512, 224), (32, 32), (36, 36))]
    for name, dims, rb, ra in tts:
        for p in ("f64", "f32", "f16"):
            ranks = [1] + list(rb if p == "f64" else ra) + [1]
            cores = [c.astype(NPDT[p]) for c in synth.random_tt_cores(dims, ranks, tag=1)]
            f, by = tt_counts(list(dims), ranks, EBYTES[p])
            sets = rotated(cores, dims, torch.from_numpy(cores[0][:1, :1, :1]).dtype, by)
            reps = max(10, min(200, int(5e9 / max(f, 1))))
            wall, km = _time_cell(lrc, lambda r: lrc.tt_reconstruct(sets[r % len(sets)][0], out=sets[r % len(sets)][1]),
                                  reps, None)
            records.append(_record(f"tt {name} ranks={ranks[1:-1]}", "tt", p, km, wall, f, by,
                                   config=name, dims=list(dims), ranks=ranks))
            log(render_sweep_row(records[-1]))
            del sets
            torch.cuda.empty_cache()
    write_records(os.path.splitext(path)[0] + ".jsonl", records)
    with open(path, "w") as fh:
        fh.write("\n".join(SWEEP_HEAD + [render_sweep_row(r) for r in records]) + "\n")


def quant_sweep(path, dev, lrc):
    """Device rounding of the stored factors / cores and the FP64 gauge of
    the TT workloads, each against its own bound (kernel time from the
    library's event timers; the gauge's calls synchronize, so its wall time
    is the call's)."""
    import torch
    from paper_2607_12969_amd import synth
    records = []
    rng = np.random.default_rng([12969, 98])
    for name, (m, n, k) in (("factors 8192x8192 k=257", (8192, 8192, 257)),
                            ("factors 65536x4096 k=513", (65536, 4096, 513))):
        host = [rng.standard_normal((m, k)), rng.standard_normal((n, k))]
        for p, dt in (("f32", torch.float32), ("f16", torch.float16)):
            f, by = round_counts(sum(a.size for a in host), EBYTES[p])
            copies = max(1, min(4, math.ceil(512e6 / by)))
            sets = [([torch.from_numpy(a).to(dev) for a in host],
                     [torch.empty(a.shape, dtype=dt, device=dev) for a in host]) for _ in range(copies)]

            def call(r):
                xs, ys = sets[r % copies]
                for x, y in zip(xs, ys):
                    lrc.round_to(x, p.replace("f", "fp"), out=y)
            wall, km = _time_cell(lrc, call, 50, None)
            km = {k2: v * 2 for k2, v in km.items()}   # two launches (U and V) per call
            records.append(_record(f"round {name}", "round", p, km, wall, max(f, 1.0), by,
                                   config=name, m=m, n=n, k=k))
            log(render_sweep_row(records[-1]))
            del sets
            torch.cuda.empty_cache()
    for name, dims, ranks in (("256^3 r(15,15)", (256, 256, 256), (1, 15, 15, 1)),
                              ("256^3 r(25,25)", (256, 256, 256), (1, 25, 25, 1)),
                              ("16^6 r(9,17,25,17,9)", (16,) * 6, (1, 9, 17, 25, 17, 9, 1)),
                              ("512x512x224 r(33,33)", (512, 512, 224), (1, 33, 33, 1)),
                              ("512x512x224 r(65,65)", (512, 512, 224), (1, 65, 65, 1))):
        cores = [torch.from_numpy(c).to(dev) for c in synth.random_tt_cores(dims, ranks, tag=2)]
        f, by = gauge_counts(dims, ranks)
        wall, km = _time_cell(lrc, lambda r: lrc.tt_left_orthogonalize(cores), 10, None)
        km = {"gauge_qr_f64": km["gauge_qr_f64"] * (len(dims) - 1)}   # one timed span per unfolding
        records.append(_record(f"gauge {name}", "gauge", "f64", km, wall, f, by, config=name, dims=list(dims),
                               ranks=list(ranks)))
        log(render_sweep_row(records[-1]))
    # quality measures of a reconstruction against its reference: two passes
    # over the FP64 pair (band sums, spectral angles), 32 bytes per entry
    for name, dims in (("512x512x224", (512, 512, 224)), ("512x217x204", (512, 217, 204))):
        N = int(np.prod(dims))
        rng = np.random.default_rng([12969, 99])
        Xh_ = rng.standard_normal(N).reshape(dims)
        X = torch.from_numpy(Xh_).to(dev)
        Y = X * 1.001
        wall, km = _time_cell(lrc, lambda r: lrc.band_quality(X, Y), 10, None)
        records.append(_record(f"quality {name} (dense FP64 pair)", "quality", "f64", km, wall, 10.0 * N, 32.0 * N,
                               config=name, dims=list(dims)))
        log(render_sweep_row(records[-1]))
        del X, Y
        torch.cuda.empty_cache()
    # quality of stored TT cores against the reference, fused into the FP64
    # reconstruction: reads the reference once (8 bytes per entry) and the cores
    for name, dims, ranks in (("512x512x224 r(32,32)", (512, 512, 224), (1, 32, 32, 1)),
                              ("512x512x224 r(65,65)", (512, 512, 224), (1, 65, 65, 1))):
        N = int(np.prod(dims))
        X = torch.from_numpy(synth.hyperspectral(shape=dims)).to(dev)
        cores = [torch.from_numpy(c.astype(np.float16)).to(dev) for c in synth.random_tt_cores(dims, ranks, tag=3)]
        f, _ = tt_counts(list(dims), list(ranks), 8)
        by = 8.0 * N + sum(2.0 * c.numel() for c in cores)
        wall, km = _time_cell(lrc, lambda r: lrc.tt_quality(cores, X), 10, None)
        records.append(_record(f"tt quality {name} fused (FP16 cores)", "tt_quality", "f64", km, wall, f + 10.0 * N, by,
                               config=name, dims=list(dims), ranks=list(ranks)))
        log(render_sweep_row(records[-1]))
        del X, cores
        torch.cuda.empty_cache()
    write_records(os.path.splitext(path)[0] + ".jsonl", records)
    with open(path, "w") as fh:
        fh.write("\n".join(SWEEP_HEAD + [render_sweep_row(r) for r in records]) + "\n")


def factor_sweep(path, dev, lrc):
    """Randomized FP64 factorizations (lrc_rsvd, lrc_tt_rsvd): wall time per
    call (the calls synchronize) and the library's event spans per stage,
    summed per call.  Algorithmic flop: the sketch and projection GEMMs over
    the matrix (2 m n l each, (1 + q) of each), the Gram products of the two
    or more CholeskyQR2 runs (2 rows l^2 each), the forward substitutions
    (rows l^2 each) and the singular-vector products (2 (m + n) l k).  The
    dominant kernel is the sketch GEMM (one read of the matrix per pass,
    l / 4 flop per byte: above the FP64 ridge for l > 40)."""
    import torch
    from paper_2607_12969_amd import synth
    PK = PEAK_TFLOPS["f64"]
    rows = ["| cell | GFLOP | call us | stages us (sum) | GFLOP/s | sketch GEMM us | sketch TFLOP/s | "
            "frac of FP64 MFMA | per stage (us per call) |", "|" + "---|" * 9]

    def flops(m, n, l, k, q):
        qr = 0.0
        for it in range(1 + q):
            qr += 2 * (2.0 * m * l * l + m * l * l)   # range finder: two Grams, two substitutions
            qr += 2 * (2.0 * n * l * l + n * l * l)   # projection (or its iteration counterpart)
        return 4.0 * m * n * l * (1 + q) + qr + 2.0 * (m + n) * l * k

    def run(name, fn, f, sketch_flop, reps):
        for _ in range(2):
            fn()
        torch.cuda.synchronize()
        lrc.profile_reset()
        lrc.profile_enable(True)
        t0 = time.perf_counter()
        for _ in range(reps):
            fn()
        torch.cuda.synchronize()
        wall = (time.perf_counter() - t0) / reps * 1e3
        lrc.profile_enable(False)
        kt = lrc.profile_read()
        # CholeskyQR2 spans contain the Gram launches' own spans: those are left out of the sum
        per = {lab: kt[lab][1] / reps for lab in kt if lab.startswith("factor_")}
        tot = sum(per.values())
        sk = per.get("factor_sketch_f64", float("nan"))
        sk_tf = sketch_flop / (sk * 1e-3) / 1e12
        stages = ", ".join(f"{k} {v * 1e3:.0f}" for k, v in sorted(per.items(), key=lambda kv: -kv[1]))
        rows.append(f"| {name} | {f / 1e9:.2f} | {wall * 1e3:.0f} | {tot * 1e3:.0f} | {f / (wall * 1e-3) / 1e9:.0f} | "
                    f"{sk * 1e3:.0f} | {sk_tf:.1f} | {sk_tf / PK:.3f} | {stages} |")
        log(rows[-1])

    for (m, n), l, k, q in (((8192, 8192), 75, 65, 0), ((8192, 8192), 75, 65, 1), ((8192, 8192), 96, 65, 0),
                            ((65536, 4096), 75, 65, 0)):
        sigma = np.arange(1, 601, dtype=np.float64) ** -1.5
        A = torch.from_numpy(synth.spectral_matrix(m, n, sigma, tag=m + n)).to(dev)
        Om = torch.from_numpy(synth.test_vectors(l, n, m)).to(dev)
        f = flops(m, n, l, k, q)
        run(f"rsvd {m}x{n} k={k} l={l} q={q}", lambda: lrc.rsvd(A, Om, k, q), f, 2.0 * m * n * l * (1 + q), 5)
        del A, Om
        torch.cuda.empty_cache()
    for dims, r, l in (((512, 512, 224), 65, 75), ((512, 512, 224), 33, 43), ((145, 145, 200), 36, 46)):
        T = synth.hyperspectral(shape=dims)
        Td = torch.from_numpy(T).to(dev)
        oms, f, skf, rp, cols = [], 0.0, 0.0, 1, int(np.prod(dims[1:]))
        for step in range(2):
            oms.append(torch.from_numpy(synth.test_vectors(l, cols, 60 + step)).to(dev))
            rows_ = rp * dims[step]
            f += flops(rows_, cols, l, r, 0)
            skf += 2.0 * rows_ * cols * l
            rp = r
            cols //= dims[step + 1]
        run(f"tt_rsvd {'x'.join(map(str, dims))} ranks=({r},{r}) l={l}",
            lambda: lrc.tt_rsvd(Td, (r, r), oms, 0), f, skf, 5)
        del Td, oms
        torch.cuda.empty_cache()
    with open(path, "w") as fh:
        fh.write("\n".join(rows) + "\n")


# ------------------------------------------------------------ timing grid ---
# The paper's resident timing protocol (Sec. 4.4 matrix application, Sec. 7.5
# TT reconstruction; its timing paragraph): per task, warmups, then rounds of
# blocks in which every method is sampled in a seeded shuffled order; per
# task the median time per method; the speedup of a method is the median of
# its paired (FP64 / method) block-median ratios; across tasks, geometric
# means with 10,000-resample bootstrap percentile intervals.

# synthetic stand-ins for the ten matrices of the matrix timing grid: square
# and rectangular sizes spanning the small-to-medium range, one of them the
# 494 x 494 size the paper quotes
GRID_MATRICES = [(96, 96), (160, 160), (256, 256), (320, 96), (384, 384), (494, 494), (640, 192), (768, 768),
                 (1024, 1024), (1536, 1536)]
GRID_BATCHES = [256, 2048, 8192]
# TT grid: the four hyperspectral cube shapes the paper lists (ranks 32 -> 36),
# two four-way stand-ins for the dense FROSTT subtensors (16 -> 20) and the
# six-way stress shape (8 -> 12)
GRID_TENSORS = [("hyperspectral 145x145x200", (145, 145, 200), 32, 36),
                ("hyperspectral 83x86x204", (83, 86, 204), 32, 36),
                ("hyperspectral 512x217x204", (512, 217, 204), 32, 36),
                ("hyperspectral 610x340x103", (610, 340, 103), 32, 36),
                ("four-way 128x24x64x64", (128, 24, 64, 64), 16, 20),
                ("four-way 192x24x64x16", (192, 24, 64, 16), 16, 20),
                ("six-way 16^6", (16,) * 6, 8, 12)]
GRID_METHODS = [("FP64 base", "f64", 0), ("FP32 same rank", "f32", 0), ("FP16 same rank", "f16", 0),
                ("FP32 compensated", "f32", 1), ("FP16 compensated", "f16", 1)]


def capped_ranks(dims, nominal):
    """Uniform nominal TT ranks capped by the unfolding dimensions (reading R8)."""
    d = len(dims)
    ranks = [1]
    for l in range(d - 1):
        left = ranks[-1] * dims[l]
        right = int(np.prod(dims[l + 1:]))
        ranks.append(int(min(nominal, left, right)))
    return ranks + [1]


def _grid_task(lrc, calls, rounds=3, blocks=5, samples=20, warmup=30, seed=0):
    """Times of every method of one task: calls[i]() launches method i.
    Each sample is one event pair around `reps` back-to-back calls, reps
    calibrated per method so that a sample lasts about 2 ms (at most 256).
    Returns per-method medians (ms per call) and the block medians."""
    import torch
    nm = len(calls)
    for _ in range(warmup):
        for c in calls:
            c()
    torch.cuda.synchronize()
    st = torch.cuda.current_stream()
    reps = []
    for c in calls:
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record(st)
        for _ in range(8):
            c()
        b.record(st)
        torch.cuda.synchronize()
        t1 = a.elapsed_time(b) / 8
        reps.append(int(max(1, min(256, round(2.0 / max(t1, 1e-4))))))
    rng = np.random.default_rng([12969, 77, seed])
    allt = [[] for _ in range(nm)]
    bmed = [[] for _ in range(nm)]
    for _ in range(rounds):
        for _ in range(blocks):
            order = rng.permutation(nm)
            ev = {i: [] for i in range(nm)}
            for _ in range(samples):
                for i in order:
                    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                    a.record(st)
                    for _ in range(reps[i]):
                        calls[i]()
                    b.record(st)
                    ev[i].append((a, b))
            torch.cuda.synchronize()
            for i in range(nm):
                ts = [a.elapsed_time(b) / reps[i] for a, b in ev[i]]
                allt[i] += ts
                bmed[i].append(float(np.median(ts)))
    return [float(np.median(t)) for t in allt], bmed


def _geo_ci(values, n_boot=10000, seed=0):
    v = np.log(np.asarray(values, dtype=np.float64))
    rng = np.random.default_rng([12969, 78, seed])
    boots = np.exp(v[rng.integers(0, v.size, (n_boot, v.size))].mean(axis=1))
    return float(np.exp(v.mean())), float(np.percentile(boots, 2.5)), float(np.percentile(boots, 97.5))


def _median_ci(values, n_boot=2000, seed=0):
    """Bootstrap 95% interval of the median of a task's block medians."""
    v = np.asarray(values, dtype=np.float64)
    rng = np.random.default_rng([12969, 79, seed])
    meds = np.median(v[rng.integers(0, v.size, (n_boot, v.size))], axis=1)
    return [float(np.percentile(meds, 2.5)), float(np.percentile(meds, 97.5))]


def _grid_record(task, method, p, med, bmed, ratio, storage, f, by, **shape):
    # no kernel names here: FP32 is priced by its own instruction throughout
    t_star = max(by / (PEAK_HBM_GBS * 1e9), f / (PEAK_TFLOPS[p] * 1e12)) * 1e3
    return dict(task=task, method=method, prec=p, **shape, median_ms=med, ci95_ms=_median_ci(bmed),
                speedup_vs_fp64=ratio, storage_vs_fp64=storage, flop=f, bytes=by, t_star_ms=t_star,
                gflops=f / med / 1e6, gbs=by / med / 1e6, frac=t_star / med, counter_bytes=None,
                parity_error=None, certificate=None, env=env_knobs())


def grid(path, dev, lrc):
    import torch
    from paper_2607_12969_amd import synth
    records = []
    out = ["# The paper's resident timing grid on one MI355X (synthetic stand-ins)", "",
           "Command: `python -u bench.py --grid FILE`. Inputs resident in HBM and reused across calls (the",
           "paper's resident protocol, so small tasks run from the Infinity Cache); per task 30 warmups, then",
           "3 rounds x 5 blocks x 20 samples per method in a seeded shuffled order (the paper's protocol),",
           "each sample one HIP event pair around back-to-back calls",
           "calibrated to about 2 ms (at most 256 calls); time = geometric mean over tasks of the per-task",
           "medians per call; speedup = geometric mean over tasks",
           "of the median paired (FP64 / method) block-median ratio, with a 10,000-resample bootstrap interval",
           "over tasks; storage = stored bytes relative to the FP64 base.", ""]
    # ---- matrix application
    for b in GRID_BATCHES:
        per_method = {name: ([], [], []) for name, _, _ in GRID_METHODS}
        rows = []
        for t, (m, n) in enumerate(GRID_MATRICES):
            k0 = 40
            w = synth.random_factors(m, n, k0 + 1, b, tag=20 + t)
            X = w["X"] / np.linalg.norm(w["X"], axis=0, keepdims=True)   # unit-norm samples
            calls = []
            bufs = []
            for name, p, inc in GRID_METHODS:
                k = k0 + inc
                ins = [torch.from_numpy(np.ascontiguousarray(a).astype(NPDT[p])).to(dev)
                       for a in (w["U"][:, :k], w["s"][:k], w["V"][:, :k], X)]
                Y = torch.empty((m, b), dtype=ins[0].dtype, device=dev)
                bufs.append((ins, Y))
                calls.append(lambda ins=ins, Y=Y: lrc.matrix_apply(*ins, Y=Y))
            med, bm = _grid_task(lrc, calls, seed=t)
            base_bytes = (k0) * (m + n + 1) * 8
            for i, (name, p, inc) in enumerate(GRID_METHODS):
                ratio = float(np.median(np.array(bm[0]) / np.array(bm[i])))
                per_method[name][0].append(med[i])
                per_method[name][1].append(ratio)
                per_method[name][2].append((k0 + inc) * (m + n + 1) * EBYTES[p] / base_bytes)
                f, by = apply_counts(m, n, k0 + inc, b, EBYTES[p])
                records.append(_grid_record(f"apply {m}x{n} b={b}", name, p, med[i], bm[i], ratio,
                                            per_method[name][2][-1], f, by, m=m, n=n, k=k0 + inc, batch=b))
            rows.append(f"| {m}x{n} | " + " | ".join(f"{med[i] * 1e3:.1f}" for i in range(len(GRID_METHODS))) + " |")
            log(f"grid apply b={b} {m}x{n}: " + rows[-1])
            del bufs, calls
        out += [f"## Matrix application, base rank 40, compensated rank 41, batch {b}", "",
                "| Method | Time (ms) | Speedup [95% CI] | Storage |", "|---|---|---|---|"]
        for name, _, _ in GRID_METHODS:
            tm, sp, sto = per_method[name]
            g, lo, hi = _geo_ci(sp)
            out.append(f"| {name} | {_geo_ci(tm)[0]:.4f} | {g:.2f} [{lo:.2f}, {hi:.2f}] | {np.mean(sto):.4f} |")
        out += ["", "Per task medians (us): " + ", ".join(n for n, _, _ in GRID_METHODS), "",
                "| task | " + " | ".join(n for n, _, _ in GRID_METHODS) + " |",
                "|---|" + "---|" * len(GRID_METHODS)] + rows + [""]
        torch.cuda.empty_cache()
    # ---- TT reconstruction
    per_method = {name: ([], [], []) for name, _, _ in GRID_METHODS}
    rows = []
    for t, (label, dims, rb, ra) in enumerate(GRID_TENSORS):
        calls = []
        bufs = []
        base = capped_ranks(dims, rb)
        for name, p, inc in GRID_METHODS:
            ranks = capped_ranks(dims, ra if inc else rb)
            cores = [torch.from_numpy(c.astype(NPDT[p])).to(dev) for c in synth.random_tt_cores(dims, ranks, tag=30 + t)]
            outb = torch.empty(dims, dtype=cores[0].dtype, device=dev)
            bufs.append((cores, outb))
            calls.append(lambda cores=cores, outb=outb: lrc.tt_reconstruct(cores, out=outb))
        med, bm = _grid_task(lrc, calls, seed=100 + t)
        base_bytes = sum(base[l] * dims[l] * base[l + 1] for l in range(len(dims))) * 8
        for i, (name, p, inc) in enumerate(GRID_METHODS):
            ranks = capped_ranks(dims, ra if inc else rb)
            ratio = float(np.median(np.array(bm[0]) / np.array(bm[i])))
            per_method[name][0].append(med[i])
            per_method[name][1].append(ratio)
            per_method[name][2].append(sum(ranks[l] * dims[l] * ranks[l + 1] for l in range(len(dims)))
                                       * EBYTES[p] / base_bytes)
            f, by = tt_counts(list(dims), ranks, EBYTES[p])
            records.append(_grid_record(f"tt {label}", name, p, med[i], bm[i], ratio, per_method[name][2][-1],
                                        f, by, dims=list(dims), ranks=ranks))
        rows.append(f"| {label} {rb}->{ra} | " + " | ".join(f"{med[i] * 1e3:.1f}" for i in range(len(GRID_METHODS)))
                    + " |")
        log("grid tt: " + rows[-1])
        del bufs, calls
        torch.cuda.empty_cache()
    out += ["## TT reconstruction (hyperspectral shapes 32 -> 36, four-way 16 -> 20, six-way 8 -> 12)", "",
            "The summary covers the six tensors of the paper's aggregate (the six-way stress shape is listed but",
            "left out of the geometric means, as in the paper).", "",
            "| Method | Time (ms) | Speedup [95% CI] | Storage |", "|---|---|---|---|"]
    for name, _, _ in GRID_METHODS:
        tm, sp, sto = (v[:6] for v in per_method[name])
        g, lo, hi = _geo_ci(sp)
        out.append(f"| {name} | {_geo_ci(tm)[0]:.4f} | {g:.2f} [{lo:.2f}, {hi:.2f}] | {np.mean(sto):.4f} |")
    out += ["", "| task | " + " | ".join(n for n, _, _ in GRID_METHODS) + " |",
            "|---|" + "---|" * len(GRID_METHODS)] + rows + [""]
    write_records(os.path.splitext(path)[0] + ".jsonl", records)
    with open(path, "w") as fh:
        fh.write("\n".join(out) + "\n")


# ---------------------------------------------------- fixed-memory study ---
FM_CUBES = [("145x145x200", (145, 145, 200)), ("610x340x103", (610, 340, 103)), ("83x86x204", (83, 86, 204)),
            ("512x217x204", (512, 217, 204))]


def fixed_memory(path, dev, lrc):
    """The fixed-memory comparison (Sec. sec:hyperspectral_application) on
    hyperspectral-shaped stand-ins of the four cube shapes: FP64 TT-SVD at
    rank R, its cores rounded to FP32 / FP16, the rank-(R + delta) cores
    left-orthogonalized and rounded on the device, and the memory-matched
    FP64 rank for the FP16 compensated budget; quality measured on the
    device.  TT-SVD itself (host, numpy) is the untimed offline step."""
    import torch
    from paper_2607_12969_amd import synth
    R, delta = 32, 4
    out = ["# Fixed-memory comparison on hyperspectral-shaped stand-ins (one MI355X)", "",
           "Command: `python -u bench.py --fixed-memory FILE`. Per cube shape: a synthetic hyperspectral stand-in",
           "(smooth nonnegative endmember spectra times softmax abundance maps, 1e-3 noise, unit Frobenius norm);",
           f"FP64 TT-SVD (host) at rank R = {R} and R + delta = {R + delta}; the augmented cores left-orthogonalized",
           "(`lrc_tt_left_orthogonalize`) and every low-precision core rounded on the device (`lrc_round`); the",
           "FP64 memory-matched rank for the FP16 compensated budget from `lrc_tt_memory_matched_rank`; every",
           "measure from `lrc_tt_quality` (FP64 contraction of the stored cores against the FP64 cube). PSNR,",
           "SSIM and SAM do not depend on the cube's overall scale, so the normalization needs no undoing here.", "",
           "| cube | method | ranks | storage MiB | compression | rel. error | PSNR dB | SSIM | SAM rad |",
           "|---|---|---|---|---|---|---|---|---|"]
    for name, dims in FM_CUBES:
        T = synth.hyperspectral(shape=dims)
        Td = torch.from_numpy(T).to(dev)
        rb, ra = capped_ranks(dims, R), capped_ranks(dims, R + delta)
        budget = lrc.tt_storage_bytes(dims, ra, "fp16")
        Rmm, rmm = lrc.memory_matched_rank(dims, budget)
        base = [torch.from_numpy(c).to(dev) for c in tt_svd_fixed(T, rb[1:3])]
        aug = lrc.tt_left_orthogonalize([torch.from_numpy(c).to(dev) for c in tt_svd_fixed(T, ra[1:3])])
        mm = [torch.from_numpy(c).to(dev) for c in tt_svd_fixed(T, rmm[1:3])]
        methods = [("FP64, R", base, rb, "fp64"),
                   ("FP32, R", [lrc.round_to(c, "fp32") for c in base], rb, "fp32"),
                   ("FP16, R", [lrc.round_to(c, "fp16") for c in base], rb, "fp16"),
                   ("FP32, R + delta", [lrc.round_to(c, "fp32") for c in aug], ra, "fp32"),
                   ("FP16, R + delta", [lrc.round_to(c, "fp16") for c in aug], ra, "fp16"),
                   (f"FP64 memory-matched (R = {Rmm})", mm, rmm, "fp64")]
        dense = 8 * int(np.prod(dims))
        for label, cores, ranks, p in methods:
            q = lrc.tt_quality(cores, Td)
            sb = lrc.tt_storage_bytes(dims, ranks, p)
            out.append(f"| {name} | {label} | {tuple(ranks[1:-1])} | {sb / 2 ** 20:.3f} | {dense / sb:.1f} | "
                       f"{q['rel_err']:.3e} | {q['psnr']:.2f} | {q['ssim']:.5f} | {q['sam']:.4e} |")
            log(out[-1])
        del Td, base, aug, mm
        torch.cuda.empty_cache()
    with open(path, "w") as fh:
        fh.write("\n".join(out) + "\n")


# ------------------------------------------------------------ single cells ---

def run_cell(args, dev, lrc):
    """One apply or TT configuration, --reps calls back to back on seeded
    synthetic inputs (the kernels a profiler then sees are that cell's)."""
    import torch
    from paper_2607_12969_amd import synth
    dt = {"fp64": np.float64, "fp32": np.float32, "fp16": np.float16}
    if args.apply_cell:
        m, n, k, b = (int(v) for v in args.apply_cell[:4])
        p = args.apply_cell[4]
        w = synth.random_factors(m, n, k, b, tag=77)
        ins = [torch.from_numpy(np.ascontiguousarray(w[key]).astype(dt[p])).to(dev) for key in ("U", "s", "V", "X")]
        Y = torch.empty((m, b), dtype=ins[0].dtype, device=dev)
        log(f"apply cell {m}x{n} k={k} b={b} {p}, {args.reps} calls")
        for _ in range(args.reps):
            lrc.matrix_apply(*ins, Y=Y)
    else:
        dims = tuple(int(v) for v in args.tt_cell[0].split("x"))
        ranks = [1] + [int(v) for v in args.tt_cell[1].split(",")] + [1]
        p = args.tt_cell[2]
        cores = [torch.from_numpy(c.astype(dt[p])).to(dev) for c in synth.random_tt_cores(dims, ranks, tag=1)]
        out = torch.empty(dims, dtype=cores[0].dtype, device=dev)
        log(f"tt cell {dims} ranks {ranks[1:-1]} {p}, {args.reps} calls")
        for _ in range(args.reps):
            lrc.tt_reconstruct(cores, out=out)
    torch.cuda.synchronize()
    print(json.dumps({"cell": args.apply_cell or args.tt_cell, "reps": args.reps}))


# ---------------------------------------------------------------- report ---

def render_report(records):
    """Markdown tables from JSONL records: sweep cells (kernel-timed) and
    grid cells (median per call with its interval) each in their own table."""
    cells = [r for r in records if "kernels_ms" in r]
    grid_rows = [r for r in records if "median_ms" in r]
    out = []
    if cells:
        out += SWEEP_HEAD + [render_sweep_row(r) for r in cells] + [""]
    if grid_rows:
        out += ["| task | method | prec | median us [95% CI] | speedup vs FP64 | storage | GFLOP/s | GB/s | "
                "frac of bound |", "|" + "---|" * 9]
        for r in grid_rows:
            lo, hi = r["ci95_ms"]
            out.append(f"| {r['task']} | {r['method']} | {r['prec']} | {r['median_ms'] * 1e3:.1f} "
                       f"[{lo * 1e3:.1f}, {hi * 1e3:.1f}] | {r['speedup_vs_fp64']:.2f} | {r['storage_vs_fp64']:.4f} | "
                       f"{r['gflops']:.0f} | {r['gbs']:.0f} | {r['frac']:.3f} |")
        out.append("")
    knobs = sorted({json.dumps(r.get("env", {}), sort_keys=True) for r in records})
    out += ["Tuning overrides in effect: " + "; ".join(knobs)]
    return "\n".join(out) + "\n"


# ------------------------------------------------------------------ main ---

def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--k", type=int, default=512, help="FP64 rank of the apply (compensated rank k+1)")
    ap.add_argument("--matrix", choices=("tail", "square"), default="tail",
                    help="apply workload: 65536 x 4096 tail-rank stress matrix or 8192 x 8192")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--sweep", default=None, help="write a per-kernel table over the workload grid")
    ap.add_argument("--quant", default=None, help="write the device rounding and TT gauge cells")
    ap.add_argument("--grid", default=None, help="write the paper's resident timing grid (synthetic stand-ins)")
    ap.add_argument("--fixed-memory", default=None, help="write the fixed-memory comparison (synthetic stand-ins)")
    ap.add_argument("--factor", default=None, help="write the randomized FP64 factorization cells")
    ap.add_argument("--copy-calibration", action="store_true", help="run a plain 1 GiB device copy (counter scale)")
    ap.add_argument("--report", default=None, help="render the markdown tables of a .jsonl record file (no GPU)")
    ap.add_argument("--apply-cell", nargs=5, default=None, metavar=("M", "N", "K", "B", "PREC"),
                    help="run one apply configuration --reps times (for profilers)")
    ap.add_argument("--tt-cell", nargs=3, default=None, metavar=("DIMS", "RANKS", "PREC"),
                    help="run one TT reconstruction (e.g. 512x512x224 65,65 fp16) --reps times (for profilers)")
    ap.add_argument("--reps", type=int, default=20)
    args = ap.parse_args()
    if args.report:
        sys.stdout.write(render_report(read_records(args.report)))
        return
    if args.gpus != 1:
        print(json.dumps({"error": "bench.py runs on one GPU only; --gpus must be 1"}))
        sys.exit(2)

    import torch
    from paper_2607_12969_amd import lrc

    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    lrc.lib()

    if args.copy_calibration:
        a = torch.empty(1 << 27, dtype=torch.float64, device=dev).fill_(1.0)
        bb = torch.empty_like(a)
        for _ in range(5):
            bb.copy_(a)
        torch.cuda.synchronize()
        print(json.dumps({"copy_bytes": a.numel() * 8, "launches": 5}))
        return

    if args.apply_cell or args.tt_cell:
        run_cell(args, dev, lrc)
        return
    if args.sweep:
        sweep(args.sweep, dev, lrc)
        return
    if args.quant:
        quant_sweep(args.quant, dev, lrc)
        return
    if args.grid:
        grid(args.grid, dev, lrc)
        return
    if args.fixed_memory:
        fixed_memory(args.fixed_memory, dev, lrc)
        return
    if args.factor:
        factor_sweep(args.factor, dev, lrc)
        return

    wl = Workload(args.k, dev, args.matrix)
    log("warmup")
    for _ in range(args.warmup):
        wl.step(lrc)
    torch.cuda.synchronize()

    # per-kernel table: an untimed pass with every kernel's event timers on
    kc = wl.kernel_counts()
    prof_steps = max(3, min(args.steps, 5))
    lrc.profile_reset()
    lrc.profile_filter(None)
    lrc.profile_enable(True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(prof_steps):
        wl.step(lrc)
    torch.cuda.synchronize()
    prof_ms = (time.perf_counter() - t0) / prof_steps * 1e3
    lrc.profile_enable(False)
    ktimes = lrc.profile_read()
    cells = []
    for lab, (cnt, tot) in sorted(ktimes.items(), key=lambda kv: -kv[1][1]):
        avg_ms = tot / max(cnt, 1)
        row = {"kernel": lab, "launches_per_step": round(cnt / prof_steps, 2), "avg_ms": round(avg_ms, 5),
               "share": round(tot / (prof_ms * prof_steps), 4)}
        if lab in kc:
            f, by, p = kc[lab]
            ai = f / by
            peak = peak_tflops(p, lab, ktimes)
            ridge = peak * 1e12 / (PEAK_HBM_GBS * 1e9)
            row.update(gflops=round(f / avg_ms / 1e6, 1), gbs=round(by / avg_ms / 1e6, 1),
                       bound="mfma" if ai > ridge else "hbm")
            row["frac"] = round((row["gflops"] / 1e3 / peak) if ai > ridge
                                else row["gbs"] / PEAK_HBM_GBS, 4)
        cells.append(row)
    dom = next((c for c in cells if c["kernel"] in kc), None)

    # timed steps: only the dominant kernel's launches carry event pairs
    lrc.profile_reset()
    if dom is not None:
        lrc.profile_filter(dom["kernel"])
        lrc.profile_enable(True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(args.steps):
        wl.step(lrc)
    torch.cuda.synchronize()
    elapsed = time.perf_counter() - t0
    lrc.profile_enable(False)
    lrc.profile_filter(None)
    timed = lrc.profile_read()
    ms = elapsed / args.steps * 1e3
    log(f"timed {args.steps} steps: {ms:.3f} ms/step")

    counts = wl.step_counts()
    flops = sum(f for f, _ in counts.values())
    byts = sum(b for _, b in counts.values())
    value = flops / (ms * 1e-3) / 1e9

    ceil = hbm_ceilings(dev)
    log(f"measured HBM ceilings (GB/s): {ceil}")
    mceil = {p: round(lrc.mfma_ceiling({"f64": "fp64", "f32": "fp32", "f16": "fp16"}[p]), 1) for p in PEAK_TFLOPS}
    log(f"measured matrix-core ceilings (TFLOP/s): {mceil}")

    def measured_peak(lab):
        p_ = kc[lab][2]
        return mceil["f16"] / 6 if peak_tflops(p_, lab, ktimes) == PEAK_F32_SPLIT else mceil[p_]

    for c in cells:
        if c.get("bound") == "hbm":
            c["frac_of_measured"] = round(c["gbs"] / ceil["copy"], 4)
        elif c.get("bound") == "mfma":
            c["frac_of_measured"] = round(c["gflops"] / 1e3 / measured_peak(c["kernel"]), 4)

    roofline = None
    if dom is not None:
        f, by, p = kc[dom["kernel"]]
        cnt, tot = timed.get(dom["kernel"], (0, 0.0))
        avg_ms = tot / max(cnt, 1)
        if dom["bound"] == "mfma":
            ach = f / avg_ms / 1e9
            peak = peak_tflops(p, dom["kernel"], ktimes)
            roofline = {"bound": "mfma", "achieved": round(ach, 3), "peak": peak, "unit": "TFLOP/s",
                        "frac": round(ach / peak, 4),
                        "frac_of_measured_peak": round(ach / measured_peak(dom["kernel"]), 4)}
        else:
            ach = by / avg_ms / 1e6
            roofline = {"bound": "hbm", "achieved": round(ach, 1), "peak": PEAK_HBM_GBS, "unit": "GB/s",
                        "frac": round(ach / PEAK_HBM_GBS, 4), "frac_of_measured_copy": round(ach / ceil["copy"], 4)}
        roofline["kernel"] = dom["kernel"]
        roofline["avg_ms"] = round(avg_ms, 5)
        roofline["launches_timed"] = cnt
        roofline["algorithmic_per_launch"] = {"flop": f, "bytes": by}
        roofline["traffic"] = measured_traffic(dom["kernel"])

    # certificates of both compensated representations, outside the timed steps
    lrc.profile_reset()
    lrc.profile_enable(True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    res = wl.certify(lrc)
    cert_ms = (time.perf_counter() - t0) * 1e3
    lrc.profile_enable(False)
    cert_kernels = {lab: round(tot, 4) for lab, (cnt, tot) in lrc.profile_read().items()}
    verdicts = {f"{a}_{p}": {"certified": r["certified"], "outcome": r["outcome"], "eta": r["eta"],
                             "E_base": r["E_base"], "E_aug": r["E_aug"]} for (a, p), r in res.items()}

    cpu = None
    if not args.no_cpu_baseline:
        log("cpu baseline (oracle)")
        cpu = cpu_baseline(wl)

    line = {
        "metric": METRIC, "value": round(value, 2), "unit": "GFLOP/s", "n_gpus": 1,
        "steps": args.steps, "warmup": args.warmup, "ms_per_step": round(ms, 4),
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "f64/f32/f16(f32-accumulate)", "data": "synthetic",
        "config": {"workload": wl.describe(), "parallelism": "single GPU"},
        "hbm_gbps": round(byts / (ms * 1e-3) / 1e9, 2),
        "hbm_ceilings_measured_gbps": ceil, "mfma_ceilings_measured_tflops": mceil,
        "roofline": roofline,
        "cpu_baseline": cpu,
        "step_parts": {k: {"gflop": round(f / 1e9, 4), "mb": round(b / 1e6, 2)} for k, (f, b) in counts.items()},
        "kernels": cells,
        "certificates": {"untimed_wall_ms": round(cert_ms, 2), "kernel_ms": cert_kernels, "verdicts": verdicts},
    }
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
