"""Overlap extraction at the edges of what its 32-bit keys hold and of what a lane walks: the number of
nodes, stretches of 640 entries (320 for more than 16 snapshots), tiles with thousands of rows, and gaps in
one list that the other walks over; against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_build_tiles import csr, rand_pairs  # noqa: E402
from test_gpu_parity import pipad, run_case  # noqa: E402,F401


@pytest.mark.parametrize("k", [2, 18])
@pytest.mark.parametrize("n", [4_177_984, 4_178_100, 4_200_000, 8_400_000, 16_800_000])
def test_numbers_of_nodes_around_what_a_key_holds(pipad, n, k):  # noqa: F811
    if k > 2 and n > 8_400_000:
        pytest.skip("the oracle's time")
    rng = np.random.default_rng(n)
    # full rows at both ends, so that the largest keys (last row of a tile, last column) occur
    ends = np.stack([np.repeat([0, 1, n - 2, n - 1], 700), rng.integers(0, n, 2800)], 1)
    ends[::5, 1] = n - 1 - ends[::5, 1] % 40
    pool = np.concatenate([ends, np.stack([rng.integers(0, 700, 3000), rng.integers(n - 3000, n, 3000)], 1)])
    lists = [csr(n, pool[rng.random(len(pool)) < 0.9]) for _ in range(k)]
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
    """One tile of two full rows with empty rows, and rows that only the other snapshots have, in between."""
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
