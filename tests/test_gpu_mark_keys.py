"""Overlap extraction at the edges of what its 32-bit keys hold and of what a lane walks: the number of
nodes, stretches of 640 entries (320 for more than 16 snapshots) and of several times that, tiles with
thousands of rows, and gaps in one list that the other walks over; against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_build_tiles import csr, rand_pairs  # noqa: E402
from test_gpu_parity import pipad, run_case, _reset_options  # noqa: E402,F401


@pytest.mark.parametrize("k,n", [(2, 4_177_982), (2, 4_177_983), (2, 4_177_984), (2, 4_178_100), (2, 4_200_000), (2, 8_400_000),
                                 (2, 16_800_000), (18, 4_200_000), (18, 8_323_579), (18, 8_323_580), (18, 8_400_000)])
def test_numbers_of_nodes_around_what_a_key_holds(pipad, n, k):  # noqa: F811
    rng = np.random.default_rng(n)
    # full rows at both ends, so that the largest keys (last row of a tile, last column) occur
    ends = np.stack([np.repeat([0, 1, n - 2, n - 1], 700), rng.integers(0, n, 2800)], 1)
    ends[::5, 1] = n - 1 - ends[::5, 1] % 40
    pool = np.concatenate([ends, np.stack([rng.integers(0, 700, 3000), rng.integers(n - 3000, n, 3000)], 1)])
    lists = [csr(n, pool[rng.random(len(pool)) < 0.9]) for _ in range(k)]
    run_case(pipad, n, lists, 1, seed=1, validate=False)


@pytest.mark.parametrize("k,n", [(2, 4_177_982), (2, 4_177_983), (18, 8_323_579)])
def test_the_largest_keys(pipad, n, k):  # noqa: F811
    """Tiles of as many rows as entries, all in the last columns: the last row's number times the largest row of
    keys; the other snapshots have some of them, and rows and columns beside them."""
    rng = np.random.default_rng(n)
    rows = np.arange(0, 3000, 2)
    base = np.stack([rows, n - 1 - rows % 5], 1)
    lists = [csr(n, base)]
    for _ in range(k - 1):
        lists.append(csr(n, np.concatenate([base[rng.random(len(base)) < 0.8], [[r, n - 1] for r in rng.integers(0, 3000, 150)]])))
    run_case(pipad, n, lists, 1, seed=1, validate=False)


@pytest.mark.parametrize("k,extra", [(2, 127), (2, 128), (2, 129), (17, 63), (17, 64), (17, 65)])
def test_a_stretch_at_what_a_wave_takes(pipad, k, extra):  # noqa: F811
    """Snapshot 1 has `extra` entries more than the tile between its first entry and the next tile's."""
    n, T = 3000, 512 if k <= 16 else 256
    row = [[7, c] for c in range(100, 100 + 2 * T, 2)]  # the first tile of the base, and more
    base = csr(n, row + [[8, c] for c in range(0, 2 * T)])
    other = csr(n, row[:T] + [[7, c] for c in range(101, 101 + 2 * extra, 2)] + [[8, c] for c in range(0, T, 3)])
    run_case(pipad, n, [base] + [other] * (k - 1), 4, seed=extra)


@pytest.mark.parametrize("rows", [63, 64, 65, 255, 256, 257, 4094, 4095, 4096, 4097])
def test_rows_of_a_tile(pipad, rows):  # noqa: F811
    """Two full rows with empty rows, and rows that only the other snapshots have, in between: in one tile, or in three from
    some 1900 rows on (test_most_rows_of_a_tile keeps more in one)."""
    n, k = 5000, 3
    between = [[r, (r * 7) % 90] for r in range(2, rows, 3)]
    ends = [[0, c] for c in range(1, 200)] + [[rows, c] for c in range(1, 250) if c != rows]
    lists = [csr(n, ends + between[::2]), csr(n, ends[::2] + between[1::2]), csr(n, ends[::3] + between[::3])]
    run_case(pipad, n, lists, 4, seed=rows)


@pytest.mark.parametrize("gap", [1, 5, 6, 7, 8, 9, 60, 400])
def test_gaps_that_are_walked_over(pipad, gap):  # noqa: F811
    """Every other run of `gap` entries of the base is missing in the second snapshot, and the other way round."""
    n = 4000
    cols = np.arange(1, n)
    pairs = np.concatenate([np.stack([np.full(n - 1, r), cols], 1) for r in (0, 3000)])
    keep = (np.arange(len(pairs)) // gap) % 2 == 0
    lists = [csr(n, pairs), csr(n, pairs[keep]), csr(n, pairs[~keep]), csr(n, pairs[(np.arange(len(pairs)) // 3) % 2 == 0])]
    run_case(pipad, n, lists, 4, seed=gap)


@pytest.mark.parametrize("k,mid_max", [(3, 512), (3, 100), (18, 100)])
@pytest.mark.parametrize("rows", [16_381, 16_382, 16_383, 16_384, 70_001])
def test_most_rows_of_a_tile(pipad, rows, k, mid_max):  # noqa: F811
    """The base's first tile begins in row 0 and ends in row `rows`; there are `rows` + 1 of them."""
    rng = np.random.default_rng(rows)
    pipad.set_option("mid_max", mid_max)  # 100: the last row and the first are hub rows
    n = rows + 5
    ends = np.array([[0, c] for c in range(1, 110)] + [[rows, c] for c in range(1, 700)])
    inner = np.stack([rng.integers(1, rows, 90), rng.integers(0, n, 90)], 1)
    lists = [csr(n, np.concatenate([ends, inner[:30]]))]
    lists += [csr(n, np.concatenate([ends[rng.random(len(ends)) < 0.9], inner[20 + t:]])) for t in range(k - 1)]
    run_case(pipad, n, lists, 4, seed=rows)


@pytest.mark.parametrize("k,mid_max", [(2, 512), (2, 100), (17, 100)])
@pytest.mark.parametrize("extra", [313, 639, 640, 641, 1280, 1281, 7001])
def test_stretches_of_several_pieces(pipad, extra, k, mid_max):  # noqa: F811
    """Where the base has row 7 alone, the other snapshots have `extra` entries in front of it, as many behind, and
    some of row 7 in between, so that common and exclusive entries lie in the first, in middle and in last pieces."""
    pipad.set_option("mid_max", mid_max)
    n, T = 9000, 512 if k <= 16 else 256
    row7 = [[7, c] for c in range(100, 100 + 2 * T, 2)]
    base = csr(n, row7 + [[8000, c] for c in range(20, 8000)] + [[8001, c] for c in range(20, 8000)])
    others = [csr(n, [[6, c] for c in range(20, 20 + extra)] + row7[t:T:3] + [[7, c] for c in range(101, 201 + t, 2)]
                  + [[8, c] for c in range(30, 30 + extra)] + [[8000, c] for c in range(20 + t, 500, 2)]) for t in range(k - 1)]
    run_case(pipad, n, [base] + others, 4, seed=extra)


@pytest.mark.parametrize("k", [3, 17])
@pytest.mark.parametrize("eighths,more", [(8, 0), (7, -1), (7, 0), (7, 1), (4, 0), (1, 0), (0, 3), (0, 0)])
def test_stretches_shorter_than_the_tile(pipad, eighths, more, k):  # noqa: F811
    """The other snapshots have that much of every tile of the base, common entries and their own."""
    n, T = 4000, 512 if k <= 16 else 256
    rng = np.random.default_rng(8 * eighths + more)
    count = T * eighths // 8 + more
    cols = 20 + 2 * np.arange(3 * T)
    lists = [csr(n, [[7, c] for c in cols[:T]] + [[3000, c] for c in cols[:2 * T]])]
    for t in range(k - 1):
        pairs = []
        for row, first in ((7, 0), (3000, 0), (3000, T)):
            mine = np.sort(rng.permutation(T)[:count])
            # a tenth of them lies between two entries of the base (behind its first, so that no tile loses them)
            pairs += [[row, cols[first + x] + (x > 0 and x % 10 == t % 10)] for x in mine]
        lists.append(csr(n, pairs))
    run_case(pipad, n, lists, 4, seed=count)
