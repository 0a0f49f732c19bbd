"""GPU parity of the factor apply Y = U diag(s) V^T X (Sec. 4.4 eq.
gpu_matrix_apply) against the oracle on the same stored values.

Tolerances (relative Frobenius error vs the oracle's FP64 evaluation of the
stored factors): 1e-12 FP64, 1e-5 FP32, 2e-3 FP16 with FP32 accumulation.
Every output is compared, the 8192 x 8192 and 65536 x 4096 workloads
included; those also pass a per-tile Frobenius check and the componentwise
bound of Lemma lem:dot (Sec. 5.2) on every entry."""
import numpy as np
import pytest

import oracle as O
from paper_2607_12969_amd import synth
from parity import PRECS, TOL, apply_bound, componentwise_ratio, rel_fro, stored_pair, tile_rel_fro_max, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lrc():
    import torch
    from paper_2607_12969_amd import lrc as mod
    assert torch.cuda.is_available()
    mod.lib()
    yield mod
    mod.set_apply_path(mod.PATH_AUTO)


def _run(lrc, U, s, V, X, prec, path=0):
    import torch
    hs = [stored_pair(a, prec) for a in (U, s, V, X)]
    lrc.set_apply_path(path)
    try:
        Y = lrc.matrix_apply(*[to_dev(h) for h, _ in hs])
        torch.cuda.synchronize()
    finally:
        lrc.set_apply_path(0)
    return Y.cpu().numpy().astype(np.float64), [o for _, o in hs]


def _assert_parity(Y, u, s, v, x, prec):
    ref = O.apply(u, s, v, x)
    assert rel_fro(Y, ref) <= TOL[prec]
    assert componentwise_ratio(Y, ref, apply_bound(u, s, v, x, prec, ref)) <= 1.0


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("path", [1, 2])
def test_small_workload(lrc, prec, path):
    """512 x 256 matrix, base rank 20 (FP64) / compensated 21, batch 64
    (MFMA path) or the first 5 columns (streaming path)."""
    w = synth.matrix_small()
    U, S, Vt = O.svd(w["A"])
    k = 20 if prec == "fp64" else 21
    X = w["X"] if path == 2 else w["X"][:, :5]
    print(f"apply small prec={prec} path={path}", flush=True)
    Y, (u, s, v, x) = _run(lrc, U[:, :k], S[:k], Vt[:k].T, X, prec, path)
    _assert_parity(Y, u, s, v, x, prec)


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("m,n,k,b", [
    (1, 1, 1, 1), (37, 53, 5, 3), (53, 37, 37, 17), (300, 200, 129, 70),
    (1000, 700, 65, 129), (129, 4100, 100, 8), (64, 64, 64, 64), (2000, 3000, 33, 1),
])
def test_ragged_shapes_both_paths(lrc, prec, m, n, k, b):
    d = synth.random_factors(m, n, k, b, tag=m * 7 + n * 3 + k + b)
    for path in (0, 1, 2):
        if path == 1 and b > 8:
            continue
        print(f"apply ragged prec={prec} m={m} n={n} k={k} b={b} path={path}", flush=True)
        Y, (u, s, v, x) = _run(lrc, d["U"], d["s"], d["V"], d["X"], prec, path)
        _assert_parity(Y, u, s, v, x, prec)


@pytest.mark.parametrize("tile", ["64", "128"])
def test_forced_tile_edges(tile):
    """The matrix-core tiles pinned to 64 or 128 rows (LRC_APPLY_TILE, read
    once per process, so the cases run in a child process): shapes whose
    tiles are mostly edges, every precision, against the oracle."""
    import os
    import subprocess
    import sys
    script = os.path.join(os.path.dirname(os.path.abspath(__file__)), "forced_tile_case.py")
    print(f"apply forced tile {tile}", flush=True)
    r = subprocess.run([sys.executable, "-u", script], env=dict(os.environ, LRC_APPLY_TILE=tile),
                       capture_output=True, text=True, timeout=110)
    print(r.stdout[-4000:], r.stderr[-2000:], flush=True)
    assert r.returncode == 0
    assert r.stdout.count(" ok") == 18


def test_stream_and_mfma_paths_agree(lrc):
    d = synth.random_factors(800, 600, 41, 8, tag=3)
    for prec in PRECS:
        y1, _ = _run(lrc, d["U"], d["s"], d["V"], d["X"], prec, 1)
        y2, _ = _run(lrc, d["U"], d["s"], d["V"], d["X"], prec, 2)
        assert rel_fro(y1, y2) <= 2 * TOL[prec]


@pytest.mark.parametrize("b", [1, 8, 256])
def test_deterministic(lrc, b):
    """Bitwise equal results on repeated calls: the split sums are added in a
    fixed order whatever order the workgroups run in (for the streaming path,
    whichever workgroup finishes a column block last)."""
    d = synth.random_factors(3000, 9000, 65, b, tag=4)
    for prec in PRECS:
        y1, _ = _run(lrc, d["U"], d["s"], d["V"], d["X"], prec, 0)
        for _ in range(3):
            y2, _ = _run(lrc, d["U"], d["s"], d["V"], d["X"], prec, 0)
            assert np.array_equal(y1, y2), prec


def _full(lrc, U, s, V, X, prec, label):
    """Every output of the apply against the oracle on the same stored values:
    the relative Frobenius tolerance over the whole output and over every
    64 x 64 tile, and the componentwise bound of Lemma lem:dot on every
    entry."""
    import torch
    hs = [stored_pair(a, prec) for a in (U, s, V, X)]
    print(f"apply {label} prec={prec} shape={hs[0][0].shape[0]}x{hs[3][0].shape[1]} k={hs[0][0].shape[1]}",
          flush=True)
    Y = lrc.matrix_apply(*[to_dev(h) for h, _ in hs])
    torch.cuda.synchronize()
    got = Y.cpu().numpy().astype(np.float64)
    del Y
    u, s_, v, x = [o for _, o in hs]
    ref = O.apply(u, s_, v, x)
    err = rel_fro(got, ref)
    assert err <= TOL[prec], (label, prec, err)
    tile = tile_rel_fro_max(got, ref)
    assert tile <= TOL[prec], (label, prec, "worst 64 x 64 tile", tile)
    ratio = componentwise_ratio(got, ref, apply_bound(u, s_, v, x, prec, ref))
    assert ratio <= 1.0, (label, prec, "componentwise bound exceeded", ratio)
    return err


@pytest.fixture(scope="module")
def square():
    return synth.matrix_square(kmax=256, batch=4096)


@pytest.mark.parametrize("k", [64, 128, 256])
@pytest.mark.parametrize("b", [1, 64, 4096])
def test_square_workload_full(lrc, square, k, b):
    """8192 x 8192, sigma_j = j^-1.5 (+1e-8 noise): FP64 at rank k, FP32 and
    FP16 at rank k + 1, batches 1, 64 and 4096; every output compared."""
    X = square["X"][:, :b]
    for prec in PRECS:
        r = k if prec == "fp64" else k + 1
        _full(lrc, square["U"][:, :r], square["sigma"][:r], square["V"][:, :r], X, prec, "8192^2")


@pytest.fixture(scope="module")
def tail():
    return synth.matrix_tail(kmax=512, batch=4096)


@pytest.mark.parametrize("k", [64, 256, 512])
@pytest.mark.parametrize("prec", PRECS)
def test_tail_workload_full(lrc, tail, k, prec):
    """65536 x 4096, sigma_j = max(exp(-j/40), 1e-6), batch 4096: FP64 at
    rank k, FP32/FP16 at k + 1; every one of the 268M outputs compared."""
    w = tail
    r = k if prec == "fp64" else k + 1
    _full(lrc, w["U"][:, :r], w["sigma"][:r], w["V"][:, :r], w["X"], prec, "65536x4096")


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("shift", [1, 3])
@pytest.mark.parametrize("b", [37, 129])
def test_unaligned_operands(lrc, prec, shift, b):
    """Operands whose base address is not 16-byte aligned (views `shift`
    elements into a buffer), with odd rank and batch so that every row is
    misaligned too: at batch 37 phase 2 reads U in place (one column tile),
    at batch 129 the operands go through the padded copy; both match the
    oracle."""
    import torch
    m, n, k = 300, 500, 65
    d = synth.random_factors(m, n, k, b, tag=9 + shift + b)
    hs = [stored_pair(a, prec) for a in (d["U"], d["s"], d["V"], d["X"])]
    views = []
    for h, _ in hs:
        buf = torch.zeros(h.size + shift, dtype=torch.from_numpy(h).dtype, device="cuda")
        v = buf[shift:].view(h.shape)
        v.copy_(torch.from_numpy(np.ascontiguousarray(h)))
        views.append(v)
    lrc.set_apply_path(2)
    try:
        Y = lrc.matrix_apply(*views)
        torch.cuda.synchronize()
    finally:
        lrc.set_apply_path(0)
    u, s, v, x = [o for _, o in hs]
    _assert_parity(Y.cpu().numpy().astype(np.float64), u, s, v, x, prec)


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("m,n,b", [(494, 494, 256), (494, 494, 8192), (640, 192, 2048), (96, 96, 8192),
                                   (1536, 1536, 2048)])
@pytest.mark.parametrize("inc", [0, 1])
def test_timing_grid_shapes(lrc, prec, m, n, b, inc):
    """Shapes of the paper's matrix timing grid (base rank 40, compensated
    rank 41, batches 256 / 2048 / 8192, unit-norm samples), same-rank
    controls included; every output compared."""
    k = 40 + inc
    d = synth.random_factors(m, n, k, b, tag=900 + m + b + inc)
    X = d["X"] / np.linalg.norm(d["X"], axis=0, keepdims=True)
    print(f"apply grid prec={prec} m={m} n={n} k={k} b={b}", flush=True)
    Y, (u, s, v, x) = _run(lrc, d["U"], d["s"], d["V"], X, prec)
    assert rel_fro(Y, O.apply(u, s, v, x)) <= TOL[prec]


def test_large_rank_small_batch(lrc):
    """A rank whose T' does not fit the streaming path's 64 KB of LDS at
    batch 1 (FP64, k = 8200) takes the matrix-core path and is applied
    correctly."""
    m, n, k = 8300, 8250, 8200
    rng = synth.rng_for(synth.W_RANDOM, 30, k)
    U = synth.gaussian(rng, (m, k)) / np.sqrt(m)
    V = synth.gaussian(rng, (n, k)) / np.sqrt(n)
    s = 0.999 ** np.arange(k)
    X = synth.gaussian(rng, (n, 1))
    print("apply 8300x8250 k=8200 b=1 fp64", flush=True)
    Y, (u, s, v, x) = _run(lrc, U, s, V, X, "fp64")
    _assert_parity(Y, u, s, v, x, "fp64")


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("m,n,k,b", [
    (300, 2111, 48, 77), (300, 2100, 33, 131),     # one rank tile, even and odd rank, several splits
    (520, 900, 130, 259), (256, 1000, 200, 257),   # 64- and 128-row tiles, read several times
    (700, 1501, 257, 35), (300, 33, 17, 2051),     # five rank tiles, one split
    (9001, 1030, 65, 1025),                        # U copied, X by size
])
def test_odd_batches(lrc, m, n, k, b, shift, prec):
    """X at a pitch (and, shifted, a base) that rules out 16-byte moves: in place or copied."""
    import torch
    d = synth.random_factors(m, n, k, b, tag=m + n + k + b)
    hs = [stored_pair(d[f], prec) for f in ("U", "s", "V", "X")]
    dev = [to_dev(h) for h, _ in hs]
    buf = torch.empty(n * b + shift, dtype=dev[3].dtype, device="cuda")
    x = buf[shift:].view(n, b)
    x.copy_(dev[3])
    print(f"apply odd batch prec={prec} m={m} n={n} k={k} b={b} shift={shift}", flush=True)
    Y = lrc.matrix_apply(dev[0], dev[1], dev[2], x)
    torch.cuda.synchronize()
    _assert_parity(Y.cpu().numpy().astype(np.float64), *[o for _, o in hs], prec)


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("m,n,k,b", [
    (65, 9, 9, 17),         # one row and column past a tile, waves without rows
    (512, 256, 20, 64),     # whole batches of rows
    (130, 257, 33, 31),     # a second block of one rank index, a second batch of one row per wave
    (500, 250, 128, 9),     # the largest rank, four blocks
    (70, 1000, 31, 10),     # four batches
    (2, 3, 1, 4000),        # a tiny factor and many columns
])
def test_one_launch_small(lrc, m, n, k, b, prec):
    """Sizes that take the single launch: edges of its tiles, batches and
    rank blocks against the oracle."""
    d = synth.random_factors(m, n, k, b, tag=m + n + k + b)
    print(f"apply small launch {prec} m={m} n={n} k={k} b={b}", flush=True)
    Y, (u, s, v, x) = _run(lrc, d["U"], d["s"], d["V"], d["X"], prec)
    _assert_parity(Y, u, s, v, x, prec)


@pytest.mark.parametrize("m,n,k,b", [
    (16129, 300, 8, 1024),      # one K step, mostly zero columns past k; one row in the last tile
    (16384, 400, 33, 1032),     # copied factor, one column past a K step; eight columns in the last tile
    (13000, 700, 104, 1283),    # aligned rank that ends inside a K step, odd batch
    (4100, 600, 256, 4096),     # whole K steps
])
def test_fp16_wide_tiles(lrc, m, n, k, b):
    """Phase 2 on 256 x 128 tiles (at least 512 of them): edges in every
    dimension against the oracle, with a huge value past the last row's rank
    range in the neighbouring row (columns past k must not leak)."""
    d = synth.random_factors(m, n, k, b, tag=k + b)
    print(f"apply wide m={m} n={n} k={k} b={b}", flush=True)
    U = np.array(d["U"])
    U[5, 0] = np.inf
    Y, (u, s, v, x) = _run(lrc, U, d["s"], d["V"], d["X"], "fp16")
    assert not np.isfinite(Y[5]).any() and np.isfinite(np.delete(Y, 5, 0)).all()
    u[5, 0], Y[5] = 0.0, 0.0
    Y[5] = O.apply(u[5:6], s, v, x)[0]
    _assert_parity(Y, u, s, v, x, "fp16")


# ---- FP32 by split products on the bfloat16 matrix cores (large batches) ----

@pytest.mark.parametrize("m,n,k,b", [
    (129, 8200, 97, 2049),     # one row past a tile, odd rank and batch, a short last K step
    (4100, 4111, 17, 2047),    # two fragments, odd everything
    (2050, 6200, 273, 2048),   # two rank tiles, the second one padded
    (16385, 257, 256, 1025),   # few rows of V, whole K steps
])
def test_fp32_split_products(lrc, m, n, k, b):
    """Edges of the split path's tiles against the oracle at the FP32
    tolerance and the componentwise FP32 bound."""
    d = synth.random_factors(m, n, k, b, tag=k + b)
    print(f"apply split m={m} n={n} k={k} b={b}", flush=True)
    Y, (u, s, v, x) = _run(lrc, d["U"], d["s"], d["V"], d["X"], "fp32")
    _assert_parity(Y, u, s, v, x, "fp32")


def test_fp32_split_panels_same_bits(lrc):
    """8192 x 8192, rank 257, batch 4096: the planes and partial sums of one
    pass (about 120 MB) exceed the allocation-free entry's scratch, which cuts
    them to panels; every output bit agrees."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(3)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")   # noqa: E731
    args = rnd(8192, 257) / 90, torch.rand(257, generator=g, device="cuda"), rnd(8192, 257) / 90, rnd(8192, 4096)
    out = torch.full((8192, 4096), float("nan"), device="cuda")
    lrc.matrix_apply_noalloc(*args, out)
    assert torch.equal(out, lrc.matrix_apply(*args))


@pytest.mark.parametrize("what", ["inf", "nan", "tiny", "huge"])
def test_fp32_split_special_values(lrc, what):
    """Values outside the split's range (2^-100 to 2^62): their K steps run on
    the FP32 instruction, so infinities and NaN land where the FP64 product
    has them, and tiny or huge columns keep the FP32 tolerance by themselves."""
    m, n, k, b = 1030, 1500, 70, 8200
    d = synth.random_factors(m, n, k, b, tag=9)
    U, s, V, X = (np.array(d[q], dtype=np.float32) for q in ("U", "s", "V", "X"))
    if what == "inf":
        X[7, 5000] = np.inf
        U[9, 3] = -np.inf
    elif what == "nan":
        X[1400, 17] = np.nan
        U[1029, 69] = np.nan
    elif what == "tiny":
        X[:, 3000:] *= np.float32(1e-36)
    else:
        V[5] *= np.float32(1e30)
        X[5] *= np.float32(1e6)
    Y = lrc.matrix_apply(*[to_dev(a) for a in (U, s, V, X)]).cpu().numpy()
    with np.errstate(all="ignore"):
        ref = U.astype(np.float64) @ (s.astype(np.float64)[:, None] * (V.astype(np.float64).T @ X.astype(np.float64)))
    assert np.array_equal(np.isnan(Y), np.isnan(ref))
    assert np.array_equal(np.isinf(Y), np.isinf(ref))
    for cols in (slice(0, 3000), slice(3000, b)):
        ok = np.isfinite(ref[:, cols])
        assert rel_fro(np.where(ok, Y[:, cols], 0), np.where(ok, ref[:, cols], 0)) <= TOL["fp32"]


def test_fp32_split_subnormal_columns(lrc):
    """Columns of X below 2^-134, whose bfloat16 part is zero, against V and U
    large enough to carry them to ordinary outputs, beside normal columns."""
    m, n, k, b = 1030, 1500, 70, 8200
    d = synth.random_factors(m, n, k, b, tag=10)
    U, s, V, X = (np.array(d[q], dtype=np.float32) for q in ("U", "s", "V", "X"))
    U *= np.float32(2.0 ** 60)
    V *= np.float32(2.0 ** 40)
    tiny = slice(4000, 4300)
    X[:, tiny] = np.float32(2.0 ** -140) * np.sign(X[:, tiny])
    X[:, 4100] = 0
    X[11, 4100] = np.float32(2.0 ** -149)
    Y = lrc.matrix_apply(*[to_dev(a) for a in (U, s, V, X)]).cpu().numpy()
    ref = U.astype(np.float64) @ (s.astype(np.float64)[:, None] * (V.astype(np.float64).T @ X.astype(np.float64)))
    for cols in (slice(0, 4000), tiny, slice(4100, 4101), slice(4300, b)):
        assert rel_fro(Y[:, cols], ref[:, cols]) <= TOL["fp32"]


def test_fp32_split_panels_at_the_scratch_limit(lrc):
    """A size whose smallest piece of V's planes is just above a quarter of the
    allocation-free scratch: accepted by both entries, with equal bits."""
    import torch
    m, n, k, b = 8194, 47657, 332, 5388
    g = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")   # noqa: E731
    args = rnd(m, k) / 90, torch.rand(k, generator=g, device="cuda"), rnd(n, k) / 200, rnd(n, b)
    out = torch.full((m, b), float("nan"), device="cuda")
    lrc.matrix_apply_noalloc(*args, out)
    assert torch.equal(out, lrc.matrix_apply(*args))


def _scatter(a, rng, density, values):
    """Sets about density * size entries of a to values in turn."""
    at = rng.integers(0, a.size, max(1, int(a.size * density)))
    a.reshape(-1)[at] = np.resize(np.asarray(values, dtype=a.dtype), at.size)


@pytest.mark.parametrize("m,n,k,b,density", [
    (1030, 1500, 70, 8200, 1e-5),      # few steps and tiles on the FP32 instruction
    (1030, 1501, 97, 8199, 1e-3),      # most of them
    (2050, 6200, 273, 2048, 1e-5),     # two rank tiles
])
def test_fp32_split_scattered_values(lrc, m, n, k, b, density):
    """Values outside the split's range scattered over X, V, U and s: their steps
    run on the FP32 instruction, beside the split's; the componentwise FP32 bound
    holds for every entry."""
    d = synth.random_factors(m, n, k, b, tag=31)
    U, s, V, X = (np.array(d[q], dtype=np.float32) for q in ("U", "s", "V", "X"))
    rng = np.random.default_rng(7)
    for a in (U, V):
        _scatter(a, rng, density, [1e-33, -3e-42, 0.0, 1e-31])
    _scatter(X, rng, density, [-1e-33, 2e-45, 0.0, 1e20])
    s[[3, k - 1]] = 1e-36, 0
    Y = lrc.matrix_apply(*[to_dev(a) for a in (U, s, V, X)]).cpu().numpy().astype(np.float64)
    u, s, v, x = (a.astype(np.float64) for a in (U, s, V, X))
    ref = O.apply(u, s, v, x)
    assert componentwise_ratio(Y, ref, apply_bound(u, s, v, x, "fp32", ref)) <= 1.0


def test_fp32_split_panels_same_bits_outside_the_range(lrc):
    """As test_fp32_split_panels_same_bits with values outside the split's range:
    the steps left to the FP32 instruction do not depend on the panels.  Rank
    2100 has more K steps than a tile marks one by one."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(4)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")   # noqa: E731
    for m, n, k, b in ((8192, 8192, 257, 4096), (33000, 2200, 2100, 1024)):
        args = [rnd(m, k) / 90, torch.rand(k, generator=g, device="cuda"), rnd(n, k) / 90, rnd(n, b)]
        for a in (args[0], args[2], args[3]):
            a.masked_fill_(torch.rand(a.shape, generator=g, device="cuda") < 1e-6, 1e-33)
        Y = lrc.matrix_apply(*args)
        out = torch.full((m, b), float("nan"), device="cuda")
        lrc.matrix_apply_noalloc(*args, out)
        assert torch.equal(out, Y)
        u, s, v, x = (a.double() for a in args)
        ref = u @ (s[:, None] * (v.T.contiguous() @ x))
        assert float((Y - ref).norm() / ref.norm()) <= TOL["fp32"]


def test_fp32_split_time_outside_the_range(lrc):
    """A few values outside the split's range cost little: 8192 x 8192, rank 257,
    batch 4096 with 10 to 300 of them in one operand stays below 1.4 times the
    time without (1.0 to 1.15 seen; 3.1 to 3.4 when a tile started over)."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(6)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")   # noqa: E731
    clean = [rnd(8192, 257) / 90, torch.rand(257, generator=g, device="cuda"), rnd(8192, 257) / 90, rnd(8192, 4096)]
    out = torch.empty(8192, 4096, device="cuda")

    def time_of(args):
        ms = []
        for _ in range(12):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            lrc.matrix_apply(*args, out)
            b.record()
            b.synchronize()
            ms.append(a.elapsed_time(b))
        return sorted(ms)[3]

    base = time_of(clean)
    for i in (0, 2, 3):
        args = list(clean)
        args[i] = clean[i].masked_fill(torch.rand(clean[i].shape, generator=g, device="cuda") < 1e-5, 1e-33)
        t = time_of(args)
        print(f"operand {i}: {t:.3f} ms, without {base:.3f} ms", flush=True)
        assert t <= 1.4 * base
