"""GPU parity: lpp_build_neighbours against the brute-force float64 oracle.
Neighbour indices must be bit-exact (order included)."""
import itertools

import numpy as np
import pytest

import paper_2502_06352_amd as lpp
from oracle import build_neighbours
from workloads import CONFIGS, make_codebook
from gpu_common import run_knn

pytestmark = pytest.mark.gpu


def _check_rows(E, k, got, rows):
    want = build_neighbours(E, k, rows=rows)
    bad = np.flatnonzero((got[rows] != want).any(axis=1))
    assert bad.size == 0, f"{bad.size} of {len(rows)} rows differ; first row {rows[bad[0]]}: " \
                          f"got {got[rows[bad[0]]][:12]} want {want[bad[0]][:12]}"


def test_knn_tiny_full():
    cfg = CONFIGS[1]
    E = make_codebook(cfg)
    got = run_knn(E, cfg.k)
    _check_rows(E, cfg.k, got, np.arange(cfg.V))


def _check_every_row(E, k, got, block=512, workers=8):
    """The brute-force oracle for every row, in row blocks spread over a few worker processes
    (spawned: they import the oracle only)."""
    import multiprocessing as mp
    from concurrent.futures import ProcessPoolExecutor
    from oracle_pool import oracle_rows
    V = E.shape[0]
    jobs = [(E, k, lo, min(lo + block, V)) for lo in range(0, V, block)]
    bad_rows = 0
    first = None
    with ProcessPoolExecutor(max_workers=workers, mp_context=mp.get_context("spawn")) as pool:
        for lo, want in pool.map(oracle_rows, jobs):
            bad = np.flatnonzero((got[lo:lo + len(want)] != want).any(axis=1))
            bad_rows += bad.size
            if bad.size and first is None:
                first = (lo + int(bad[0]), got[lo + bad[0]][:12], want[bad[0]][:12])
    assert bad_rows == 0, f"{bad_rows} of {V} rows differ; first {first}"


@pytest.mark.parametrize("idx", [2, 3, 4, 5])
def test_knn_full_size_every_row(idx):
    # every row of the table at the full size of every workload config (config 5 has the shape
    # of config 3 and a codebook of its own)
    cfg = CONFIGS[idx]
    E = make_codebook(cfg)
    got = run_knn(E, cfg.k)
    assert np.array_equal(got[:, 0], np.arange(cfg.V))
    assert got.min() >= 0 and got.max() < cfg.V
    # every row is a set of k distinct codes
    srt = np.sort(got, axis=1)
    assert np.all(srt[:, 1:] != srt[:, :-1])
    _check_every_row(E, cfg.k, got)


def test_knn_ragged_shapes():
    g = np.random.default_rng(0)
    for V, D, k in [(1000, 6, 33), (77, 3, 77), (130, 20, 1), (4100, 50, 500), (65, 256, 64)]:
        E = g.standard_normal((V, D))
        E = (E / np.linalg.norm(E, axis=1, keepdims=True)).astype(np.float32)
        got = run_knn(E, k)
        _check_rows(E, k, got, np.arange(V))


def test_knn_ties_and_duplicates_take_the_exact_path():
    # exactly-unit rows with many exact ties, duplicated 12 times: > k + 1024 codes tie
    rows = [np.array(s) * 0.5 for s in itertools.product([-1, 1], repeat=4)]
    rows += [s * np.eye(4)[i] for i in range(4) for s in (1, -1)]
    E = np.tile(np.array(rows, dtype=np.float32), (120, 1))          # V = 2880
    got = run_knn(E, 40)
    _check_rows(E, 40, got, np.arange(0, E.shape[0], 7))
    E1 = np.tile(np.array([[0.6, 0.8]], dtype=np.float32), (1500, 1))  # all codes identical
    got = run_knn(E1, 1300)
    _check_rows(E1, 1300, got, np.arange(0, 1500, 31))


def test_knn_unnormalised_rows_still_exact():
    g = np.random.default_rng(1)
    E = (g.standard_normal((900, 8)) * g.uniform(0.2, 3.0, size=(900, 1))).astype(np.float32)
    got = run_knn(E, 100)
    _check_rows(E, 100, got, np.arange(900))
    # rows of more than 16 floats go through the fixed-point filter, whose unit is the largest entry's
    # (short rows of larger codebooks: test_knn_rows_of_other_lengths)
    E = g.standard_normal((700, 40))
    E = (E / np.linalg.norm(E, axis=1, keepdims=True) * g.uniform(0.5, 1.6, size=(700, 1))).astype(np.float32)
    got = run_knn(E, 60)
    _check_rows(E, 60, got, np.arange(700))


def test_knn_long_rows_near_ties_below_bfloat16_resolution():
    # Codes that differ from each other by far less than a bfloat16 rounding (1e-4 against 4e-3), which the
    # sample's 8-bit image cannot tell apart.  Clusters of 12 around 150 centres.
    g = np.random.default_rng(7)
    centres = g.standard_normal((150, 64))
    E = np.repeat(centres, 12, axis=0) + 1e-4 * g.standard_normal((1800, 64))
    E = (E / np.linalg.norm(E, axis=1, keepdims=True)).astype(np.float32)
    for k in (8, 100):
        got = run_knn(E, k)
        _check_rows(E, k, got, np.arange(1800))


def test_knn_deterministic_and_errors():
    cfg = CONFIGS[1]
    E = make_codebook(cfg)
    assert np.array_equal(run_knn(E, 16), run_knn(E, 16))
    assert lpp.lpp_build_neighbours_workspace(1024, 8, 2000) == 0       # k > V
    assert lpp.lpp_build_neighbours_workspace(1024, 300, 16) == 0       # D unsupported
