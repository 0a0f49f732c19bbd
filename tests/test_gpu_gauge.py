"""GPU parity of the left-orthogonal TT gauge (lrc_tt_left_orthogonalize;
Sec. 6.1, Algorithm alg:tt_compensation gauge step) against the oracle's
Householder sweep on the same FP64 cores.  With diag(R) > 0 the thin QR of
a full-rank unfolding is unique, so every core is compared entry by entry
(relative Frobenius error 1e-12, the FP64 tolerance); the properties that
hold at any size (orthonormal unfoldings, unchanged tensor) are checked at
the workload sizes too."""
import numpy as np
import pytest

import oracle as O
from paper_2607_12969_amd import synth
from parity import rel_fro, to_dev

pytestmark = pytest.mark.gpu

TOL = 1e-12


@pytest.fixture(scope="module")
def lrc():
    import torch
    from paper_2607_12969_amd import lrc as mod
    assert torch.cuda.is_available()
    mod.lib()
    return mod


def _gaussian_cores(dims, ranks, tag, growth=1.0):
    rng = np.random.default_rng([12969, 93, tag])
    return [rng.standard_normal((ranks[l], dims[l], ranks[l + 1])) * growth ** l for l in range(len(dims))]


def _gauge(lrc, cores, label):
    import torch
    print(f"gauge {label} ranks={O.tt_shape(cores)[1]}", flush=True)
    dev = [to_dev(c) for c in cores]
    lrc.tt_left_orthogonalize(dev)
    torch.cuda.synchronize()
    return [c.cpu().numpy() for c in dev]


def _compare(got, cores, label):
    ref = O.left_orthogonalize(cores)
    for l, (g, r) in enumerate(zip(got, ref)):
        err = rel_fro(g, r)
        assert err <= TOL, (label, l, err)


SMALL = [
    ("d2", (30, 20), (1, 7, 1)),
    ("square unfolding", (4, 4), (1, 4, 1)),
    ("rank one", (8, 9, 10), (1, 1, 1, 1)),
    ("odd ranks", (6, 5, 7), (1, 5, 3, 1)),
    ("d4 growing scale", (5, 6, 7, 4), (1, 4, 5, 3, 1)),
    ("d6", (4, 5, 3, 6, 2, 5), (1, 3, 7, 9, 8, 4, 1)),
    ("rank 96", (100, 97, 3), (1, 96, 2, 1)),
    ("rank 65 ragged rows", (70, 33, 11), (1, 65, 65, 1)),
]


@pytest.mark.parametrize("case", range(len(SMALL)), ids=[c[0] for c in SMALL])
def test_small_shapes_match_oracle(lrc, case):
    label, dims, ranks = SMALL[case]
    cores = _gaussian_cores(dims, ranks, case, growth=3.0)
    _compare(_gauge(lrc, cores, label), cores, label)


@pytest.mark.parametrize("rank", [15, 16, 17, 32, 33, 47, 48, 49, 64, 80, 81, 95])
def test_every_block_count_of_the_triangular_kernels(lrc, rank):
    """Ranks at the edges of the Cholesky's and the triangular solve's blocks of 16."""
    dims, ranks = (rank + 3, 19, 2), (1, rank, 2, 1)
    cores = _gaussian_cores(dims, ranks, rank)
    _compare(_gauge(lrc, cores, f"rank {rank}"), cores, rank)


@pytest.mark.parametrize("rows,rank", [(32767, 7), (32768, 18), (65573, 33)])
def test_tall_unfoldings(lrc, rows, rank):
    """Both row tilings of the triangular solve, a ragged last tile, several tiles per workgroup."""
    cores = _gaussian_cores((rows, 3), (1, rank, 1), rows)
    _compare(_gauge(lrc, cores, f"{rows} rows"), cores, rows)


WORKLOADS = [
    ("cube 256^3 r15", (256, 256, 256), (1, 15, 15, 1)),
    ("six-way 16^6", (16,) * 6, (1, 9, 17, 25, 17, 9, 1)),
    ("hyperspectral 512x512x224 r65", (512, 512, 224), (1, 65, 65, 1)),
]


@pytest.mark.parametrize("label,dims,ranks", WORKLOADS)
def test_workload_shapes_match_oracle(lrc, label, dims, ranks):
    cores = _gaussian_cores(dims, ranks, 7)
    got = _gauge(lrc, cores, label)
    _compare(got, cores, label)
    # orthonormal left unfoldings of every core but the last
    for l in range(len(dims) - 1):
        M = got[l].reshape(-1, got[l].shape[2])
        assert np.linalg.norm(M.T @ M - np.eye(M.shape[1])) <= 1e-13 * M.shape[1], (label, l)
    # the represented tensor is unchanged: sampled entries against the oracle's slice products
    rng = np.random.default_rng([12969, 97])
    idx = [tuple(int(rng.integers(0, n)) for n in dims) for _ in range(64)]
    before = np.array([O.tt_entry(cores, i) for i in idx])
    after = np.array([O.tt_entry(got, i) for i in idx])
    assert np.max(np.abs(after - before)) <= 1e-12 * np.max(np.abs(before))


def test_tt_svd_cores_change_only_by_rounding(lrc):
    """TT-SVD output is already left-orthogonal: the gauge only fixes the
    signs (diag(R) > 0), and agrees with the oracle's."""
    cores = O.tt_svd(synth.decay_3d(24), ranks=[7, 7])
    _compare(_gauge(lrc, cores, "tt-svd decay 24^3"), cores, "tt-svd")


def test_repeated_calls_are_bitwise_equal(lrc):
    cores = _gaussian_cores((40, 30, 20), (1, 12, 9, 1), 11)
    a = _gauge(lrc, cores, "repeat 1")
    b = _gauge(lrc, cores, "repeat 2")
    for x, y in zip(a, b):
        np.testing.assert_array_equal(x, y)


def test_rank_deficient_unfolding_is_reported(lrc):
    cores = _gaussian_cores((10, 8, 6), (1, 4, 5, 1), 12)
    cores[1][:, :, 4] = cores[1][:, :, 0]          # two equal columns in core 1's unfolding
    with pytest.raises(lrc.LrcError) as ei:
        _gauge(lrc, cores, "rank deficient")
    assert ei.value.code == -6
    assert "core 1" in str(ei.value)
