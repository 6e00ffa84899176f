"""GPU parity of lpp_build_neighbours where its paths change: the one-kernel path for small codebooks of
short rows, every number of contraction steps, the sample's strides, one wave / four / sixteen per ranked
row, lists that take every code, rows that fall through to the exact path.  Bit-exact against the oracle."""
import numpy as np
import pytest
import torch

import paper_2502_06352_amd as lpp
from oracle import build_neighbours
from gpu_common import DEV, dev, run_knn

pytestmark = pytest.mark.gpu


def _unit(g, V, D):
    E = g.standard_normal((V, D))
    return (E / np.linalg.norm(E, axis=1, keepdims=True)).astype(np.float32)


def _check(E, k, rows=None):
    got = run_knn(E, k)
    rows = np.arange(E.shape[0]) if rows is None else rows
    want = build_neighbours(E, k, rows=rows)
    bad = np.flatnonzero((got[rows] != want).any(axis=1))
    assert bad.size == 0, f"{bad.size} of {len(rows)} rows differ; row {rows[bad[0]]}: {got[rows[bad[0]]][:8]} want {want[bad[0]][:8]}"


@pytest.mark.parametrize("V,D,k", [
    (2, 1, 2), (5, 16, 3), (255, 3, 255), (1023, 5, 1), (1024, 16, 1024), (1024, 8, 16), (1000, 13, 900),   # one kernel
    (1025, 8, 16), (1040, 4, 700), (2049, 12, 65), (3000, 16, 300), (4095, 1, 50), (8200, 7, 9), (20000, 8, 40),
    (129, 17, 5), (1024, 64, 16), (513, 65, 200), (1100, 128, 70), (700, 129, 700), (2600, 192, 31),
    (1300, 193, 1000), (300, 255, 8), (9000, 32, 500), (5000, 96, 2500)])
def test_knn_path_edges(V, D, k):
    g = np.random.default_rng(V * 7 + D)
    E = _unit(g, V, D)
    _check(E, k, None if V <= 3000 else np.unique(np.concatenate([[0, V - 1], g.choice(V, size=150)])))


@pytest.mark.parametrize("D", [8, 48])
def test_knn_codebook_with_an_order_of_its_own(D):
    # neighbouring codes close together (a sorted codebook), unused codes all zero, a spread of norms
    g = np.random.default_rng(D)
    E = np.cumsum(g.standard_normal((6000, D)) * 0.05, axis=0)
    E = (E / np.linalg.norm(E, axis=1, keepdims=True)).astype(np.float32)
    E[1000:1400] = 0.0
    E[2000:2100] *= 3.0
    _check(E, 120, np.unique(np.concatenate([[1000, 2050, 5999], g.choice(6000, size=150)])))


@pytest.mark.parametrize("D", [6, 40])
def test_knn_near_ties_inside_the_rounding_of_the_similarities(D):
    # clusters whose members differ by less than the approximate similarities resolve
    g = np.random.default_rng(D)
    E = np.repeat(_unit(g, 250, D).astype(np.float64), 10, axis=0) + 3e-8 * g.standard_normal((2500, D))
    _check((E / np.linalg.norm(E, axis=1, keepdims=True)).astype(np.float32), 25)


@pytest.mark.parametrize("V,D", [(120, 250), (250, 256), (500, 200)])
def test_knn_order_below_the_fixed_point_unit(V, D):
    # flat rows +-c whose entries differ by a few units of the last place of a float: the fixed-point image, and
    # the 24 to 23 value bits of so few codes, cannot tell them apart, the float64 keys must
    g = np.random.default_rng(V + D)
    c = np.float32(1.0 / np.sqrt(D))
    sign = np.where(g.random((4, D)) < 0.5, -1.0, 1.0)[g.integers(0, 4, size=V)]
    E = (sign * c * (1.0 + 2.0 ** -24 * g.integers(-3, 4, size=(V, D)))).astype(np.float32)
    _check(E, V // 2)


@pytest.mark.parametrize("V,D,k", [(1000, 8, 40), (1000, 8, 1000), (1500, 8, 40), (1500, 8, 1500), (700, 40, 30), (700, 40, 700)])
def test_knn_codes_that_hold_a_nan_come_last(V, D, k):
    # on every path: rows of zeros tie everywhere and take the exact one, k = V has to list the NaN codes
    g = np.random.default_rng(V + D)
    E = _unit(g, V, D)
    E[[7, V // 2], D // 2] = np.nan
    E[[3, 11, V - 2]] = 0.0
    _check(E, k, np.unique(np.concatenate([[3, 7, 11, V // 2, V - 2], g.choice(V, size=100)])))


@pytest.mark.parametrize("other", [20.0, 20000.0, 3e38, np.inf, -np.inf])
@pytest.mark.parametrize("V,D,k", [(1030, 8, 40), (1500, 5, 1500), (2500, 2, 300), (1100, 13, 60), (1100, 40, 60)])
def test_knn_large_numbers_beside_a_nan_spoil_no_other_code(V, D, k, other):
    # beyond the halves' range at either scale: the codes that share an operand with such a one (four places before it or
    # behind) are neighbours as ever
    g = np.random.default_rng(V + D)
    E = _unit(g, V, D)
    bad = np.array([3, 9, 127, 128, 500, 503, V - 6, V - 1])
    E[bad] = other
    E[bad, np.arange(len(bad)) % D] = np.nan
    _check(E, k)


@pytest.mark.parametrize("V,D,k", [(1030, 8, 40), (2500, 6, 300), (2047, 13, 64), (1100, 16, 1100), (700, 40, 30)])
def test_knn_does_not_depend_on_what_the_workspace_held(V, D, k):
    # NaN and infinities in every piece of it, and codes that hold a NaN beside others
    g = np.random.default_rng(V)
    E = _unit(g, V, D)
    E[[5, V - 1], 0] = np.nan
    want = build_neighbours(E, k)
    e, ws = dev(E), torch.empty(lpp.lpp_build_neighbours_workspace(V, D, k), dtype=torch.uint8, device=DEV)
    for fill in (0xFF, 0x7C):
        ws.fill_(fill)
        neigh = torch.empty((V, k), dtype=torch.int32, device=DEV)
        lpp.lpp_build_neighbours(e, k, neigh, ws)
        rows = np.setdiff1d(np.arange(V), [5, V - 1])
        assert np.array_equal(neigh.cpu().numpy()[rows], want[rows]), hex(fill)


@pytest.mark.parametrize("V,D,k", [(4096, 65, 20), (4097, 65, 20), (4225, 129, 300), (6001, 250, 60), (8191, 100, 700), (8192, 8, 60),
                                   (8193, 16, 100), (8321, 7, 900), (16383, 3, 50), (16400, 13, 16)])
def test_knn_sample_blocks_of_16_and_32_rows(V, D, k):
    # either side of the sizes at which a block takes 32 rows; strides of one, two and four, a tile of the sample that is not full
    g = np.random.default_rng(V + D)
    E = _unit(g, V, D)
    E[V - 3] *= 40.0 if D <= 16 else 1.0                     # (short rows: the threshold's bin looked at twice)
    rows = np.concatenate([[0, 15, 16, 31, 32, V - 33, V - 17, V - 16, V - 3, V - 2, V - 1], g.choice(V, size=120)])
    _check(E, k, np.unique(rows))


@pytest.mark.parametrize("V,D,k", [(1000, 8, 40), (1100, 8, 40), (1100, 64, 60), (1100, 256, 30)])
def test_knn_codebook_that_starts_off_16_bytes(V, D, k):
    # the same numbers 4 and 16 bytes into a buffer: read through a padded copy, and as they are
    E = _unit(np.random.default_rng(V + D), V, D)
    want = build_neighbours(E, k)
    for off in (1, 4):
        flat = torch.full((V * D + 4,), float("nan"), device=DEV)
        e = flat[off:off + V * D].view(V, D)
        e.copy_(dev(E))
        neigh = torch.empty((V, k), dtype=torch.int32, device=DEV)
        ws = torch.empty(lpp.lpp_build_neighbours_workspace(V, D, k), dtype=torch.uint8, device=DEV)
        lpp.lpp_build_neighbours(e, k, neigh, ws)
        assert np.array_equal(neigh.cpu().numpy(), want), off


@pytest.mark.parametrize("V,D,k", [(16384, 8, 120), (16384, 8, 150), (16384, 8, 480), (16384, 8, 560), (5000, 6, 300), (4096, 64, 300),
                                   (4096, 64, 500), (8192, 256, 240), (3000, 16, 500), (1500, 40, 1500)])
def test_knn_lists_by_one_two_and_four_waves(V, D, k):
    # lists on either side of 512, 1024 and 2048 words, codes four times over among them
    g = np.random.default_rng(V + k)
    E = _unit(g, V, D)
    E[V // 2:V // 2 + 600] = E[np.arange(600) // 4]
    _check(E, k, np.unique(np.concatenate([[0, 1, V // 2, V // 2 + 1, V - 1], g.choice(V, size=100)])))


@pytest.mark.parametrize("order", ["random", "walk"])
@pytest.mark.parametrize("V,D,k", [(120, 20, 9), (128, 64, 128), (129, 65, 40), (256, 33, 20), (257, 130, 257), (384, 17, 15), (500, 256, 60),
                                   (640, 129, 33), (641, 64, 12), (1279, 40, 100), (2047, 24, 31)])
def test_knn_long_rows_each_pair_of_groups_once(V, D, k, order):
    # one group of 128 codes, two that lie opposite, odd and even numbers of them, a last one of a single code, of all
    # but one; neighbours anywhere, or beside each other, so that all of a list comes from one side of the row
    g = np.random.default_rng(V)
    E = _unit(g, V, D)
    if order == "walk":
        E = np.cumsum(0.3 * E + 0.05, axis=0)
        E = (E / np.linalg.norm(E, axis=1, keepdims=True)).astype(np.float32)
    _check(E, k)


def _least_ms(E, k):
    """Least time of one build, device time, of a few."""
    V, D = E.shape
    e = dev(E)
    neigh = torch.empty((V, k), dtype=torch.int32, device=DEV)
    ws = torch.empty(lpp.lpp_build_neighbours_workspace(V, D, k), dtype=torch.uint8, device=DEV)
    best = []
    for _ in range(6):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        lpp.lpp_build_neighbours(e, k, neigh, ws)
        b.record()
        torch.cuda.synchronize()
        best.append(a.elapsed_time(b))
    return min(best)


@pytest.mark.parametrize("V,D,k", [(1024, 8, 16), (16384, 8, 100), (8192, 256, 100), (8192, 256, 1000)])
def test_knn_rows_without_an_order_cost_nothing(V, D, k):
    # a code that holds a NaN, and every twentieth code zeros: 1.0 to 13 ms when such rows took the exact path (or
    # ordered a thousand equal keys: 0.6 ms); as long as any other codebook now
    g = np.random.default_rng(3)
    E = _unit(g, V, D)
    plain = _least_ms(E, k)
    if V > 1024:
        nan = E.copy()
        nan[5, D - 1] = np.nan
        assert _least_ms(nan, k) < 2 * plain
    E[::20] = 0.0
    E[40, 1] = -0.0
    _check(E, k, np.array([0, 1, 20, 40, V - 4, V - 1]))
    assert _least_ms(E, k) < 2.5 * plain


@pytest.mark.parametrize("V,D,k", [(1025, 16, 1025), (2000, 3, 900), (20000, 8, 40), (16384, 8, 1000), (8192, 20, 4096), (3000, 130, 12)])
def test_knn_exact_path_of_every_row(V, D, k):
    # one infinite entry: no bound on any row's similarities.  With the keys kept in LDS, and too many for it.
    g = np.random.default_rng(V + k)
    E = _unit(g, V, D)
    E[V // 3] = E[V // 5]
    E[7, 1] = np.inf
    _check(E, k, np.unique(np.concatenate([[0, 7, V // 3, V - 1], g.choice(V, size=40)])))


@pytest.mark.parametrize("V,D,k,most", [(16384, 8, 100, 7), (8192, 256, 16, 20), (8192, 256, 300, 20), (8192, 256, 1000, 20)])
def test_knn_rows_that_fall_through_share_the_chip(V, D, k, most):
    # 900 codes that are the same: their lists overflow.  1.3 to 28 ms when they took the exact path in the blocks
    # that rank (11, 73, 106 and 50 times a codebook without)
    g = np.random.default_rng(4)
    E = _unit(g, V, D)
    plain = _least_ms(E, k)
    E[g.permutation(V)[:900]] = E[0]
    _check(E, k, g.choice(V, size=60))
    assert _least_ms(E, k) < most * plain


def _uneven(g, V, D, kind):
    E = _unit(g, V, D)
    if kind == "spread":
        E *= g.uniform(0.2, 3.0, size=(V, 1)).astype(np.float32)
    elif kind == "tiny":                                    # the lower halves are denormal
        E *= np.float32(1e-4)
    elif kind == "third":
        E[::3] *= np.float32(0.003)
    elif kind == "few":                                     # 20 codes of length 900: beyond the first scale's 16
        E[g.permutation(V)[:20]] *= np.float32(900)
    else:                                                   # one code with one large entry
        E[5] = 0
        E[5, D - 1] = float(kind)
    return E


# short rows that are not unit vectors: both scales of the halves (entries below and from 16), the second look at a
# crowded bin, and beyond both (20000: the exact path); long rows with entries far below the largest
@pytest.mark.parametrize("kind", ["spread", "tiny", "third", "few", "15.9", "16", "20", "-300", "16376", "20000"])
@pytest.mark.parametrize("V,D,k", [(1500, 8, 40), (9000, 16, 300), (5000, 3, 900), (2000, 64, 60)])
def test_knn_rows_of_other_lengths(V, D, k, kind):
    g = np.random.default_rng(V)
    E = _uneven(g, V, D, kind)
    _check(E, k, np.unique(np.concatenate([[0, 3, 5, V - 1], g.choice(V, size=60)])))


@pytest.mark.parametrize("kind,k", [("20", 16), ("20", 1000), ("300", 100), ("few", 16)])
def test_knn_a_few_large_codes_keep_the_lists(kind, k):
    # 7.2 ms for every row on the exact path where an entry of 16 or more was beyond the halves' range
    g = np.random.default_rng(6)
    assert _least_ms(_uneven(g, 16384, 8, kind), k) < 6 * _least_ms(_unit(g, 16384, 8), k)


@pytest.mark.parametrize("V,D", [(5000, 8), (4200, 256)])
def test_knn_graph_replays_with_and_without_rows_that_fall_through(V, D):
    # the number of rows left to the exact launch is cleared by every build: a captured one, replayed on codebooks
    # with some, with all and with none, and eager builds in between on the same workspace
    k = 20
    g = np.random.default_rng(V)
    some, every, none = _unit(g, V, D), _unit(g, V, D), _unit(g, V, D)
    some[g.permutation(V)[:700]] = some[0]
    every[9, 1] = np.inf
    books = [dev(E) for E in (some, every, none)]
    e = torch.empty_like(books[0])
    neigh = torch.empty((V, k), dtype=torch.int32, device=DEV)
    ws = torch.empty(lpp.lpp_build_neighbours_workspace(V, D, k), dtype=torch.uint8, device=DEV)
    want = []
    for b in books:
        e.copy_(b)
        lpp.lpp_build_neighbours(e, k, neigh, ws)
        torch.cuda.synchronize()
        want.append(neigh.clone())
    rows = np.array([0, 9, V - 1])
    for E, w in zip((some, every, none), want):
        assert np.array_equal(w.cpu().numpy()[rows], build_neighbours(E, k, rows=rows))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        lpp.lpp_build_neighbours(e, k, neigh, ws)
    for i in (0, 2, 1, 1, 2, 0):
        e.copy_(books[i])
        neigh.fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(neigh, want[i]), i
        lpp.lpp_build_neighbours(books[(i + 1) % 3], k, neigh, ws)
        torch.cuda.synchronize()
        assert torch.equal(neigh, want[(i + 1) % 3])


@pytest.mark.parametrize("kind", ["copies", "permuted"])
@pytest.mark.parametrize("V,D,k", [(1200, 17, 90), (1200, 64, 90), (1200, 65, 90), (2000, 128, 300), (1500, 253, 900), (4500, 256, 120),
                                   (5000, 96, 2500), (8192, 256, 2100)])
def test_knn_long_rows_the_same_or_the_same_sum(V, D, k, kind):
    # copies: codes six times over, in any order, some of them one unit of the last place off in one number.
    # permuted: codes of the same numbers in another order, seen from rows of equal numbers: the sums are the same, the
    # keys, added in index order, are not; 17 and 64 floats form keys at once
    g = np.random.default_rng(V + D)
    if kind == "copies":
        E = _unit(g, V // 6 + 1, D)[np.arange(V) // 6]
        i = np.flatnonzero(np.arange(V) % 6 == 5)
        E[i, i % D] = np.nextafter(E[i, i % D], np.float32(2))
        E = E[g.permutation(V)]
    else:
        E = _unit(g, 40, D)[np.arange(V) % 40]
        E = g.permuted(E, axis=1)
        E[::7] = np.float32(1.0 / np.sqrt(D))
        E[3::7] = np.where(np.arange(D) < D // 2, np.float32(0.7), np.float32(0.7) * np.float32(1 + 2.0 ** -23)) / np.float32(np.sqrt(D))
    _check(E, k, None if V <= 2000 else np.unique(np.concatenate([[0, 3, 5, V - 1], g.choice(V, size=200)])))


@pytest.mark.parametrize("V,D,k,most", [(1024, 256, 100, 1.85), (8192, 256, 1000, 2.7)])
def test_knn_every_code_four_times(V, D, k, most):
    # 1.5 and 1.9 times a codebook without copies; 2.2 and 3.5 where a lane in 16 looked for them between the sums
    g = np.random.default_rng(8)
    E = _unit(g, V // 4, D)[g.permutation(V) // 4]
    _check(E, k, g.choice(V, size=60))
    assert _least_ms(E, k) < most * _least_ms(_unit(g, V, D), k)


@pytest.mark.parametrize("k,most", [(100, 1.5), (1000, 3.0)])
def test_knn_copies_among_codes_of_one_norm(k, most):
    # one set of numbers with signs of each code's own, four times over: all 1-norms are the same, bit for bit.  1.2 and
    # 1.8 times a codebook without copies; 1.9 and 6.5 where copies were looked for by 1-norm
    V, D = 8192, 256
    g = np.random.default_rng(9)
    E = _unit(g, 1, D) * np.where(g.random((V // 4, D)) < 0.5, -1, 1).astype(np.float32)
    E = np.ascontiguousarray(E[g.permutation(V) // 4])
    _check(E, k, g.choice(V, size=60))
    assert _least_ms(E, k) < most * _least_ms(_unit(g, V, D), k)
