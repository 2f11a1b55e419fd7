"""Overlap extraction at the edges of its tiles (512 or 256 entries of the largest snapshot, stretches
of up to a quarter more in the others), against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_parity import pipad, run_case  # noqa: E402,F401


def csr(n, pairs):
    pairs = np.unique(np.asarray(pairs, dtype=np.int64).reshape(-1, 2), axis=0)
    pairs = pairs[pairs[:, 0] != pairs[:, 1]]
    rowptr = np.concatenate([[0], np.cumsum(np.bincount(pairs[:, 0], minlength=n))]).astype(np.int32)
    return rowptr, pairs[:, 1].astype(np.int32)


def rand_pairs(rng, n, count, lo=0, hi=None):
    return np.stack([rng.integers(lo, hi or n, count), rng.integers(0, n, count)], 1)


def head(n, rowptr, col, nnz):
    """The first nnz entries of a pattern."""
    return np.minimum(rowptr, nnz).astype(np.int32), col[:nnz]


@pytest.mark.parametrize("nnz", [1, 255, 256, 257, 511, 512, 513, 1024, 1025])
@pytest.mark.parametrize("k", [2, 17])
def test_entry_counts_around_a_tile(pipad, nnz, k):  # noqa: F811
    rng = np.random.default_rng(nnz + k)
    n = 300
    rowptr, col = csr(n, rand_pairs(rng, n, 4 * nnz + 8))
    lists = [head(n, rowptr, col, nnz - min(t, nnz)) if t % 3 else head(n, rowptr, col, nnz) for t in range(k)]
    run_case(pipad, n, lists, 8, seed=nnz)


@pytest.mark.parametrize("k", [2, 5, 9, 17])
def test_stretches_longer_than_a_window(pipad, k):  # noqa: F811
    """The largest snapshot has its entries in the last rows, the others in the first ones: its tiles
    own hundreds to thousands of their entries."""
    rng = np.random.default_rng(k)
    n = 900
    shared = rand_pairs(rng, n, 400)
    lists = [csr(n, np.concatenate([shared, rand_pairs(rng, n, 9000, 600)]))]
    for t in range(1, k):
        lists.append(csr(n, np.concatenate([shared, rand_pairs(rng, n, 1500 * t % 7000, 0, 40 + t)])))
    run_case(pipad, n, lists, 12, seed=k)


@pytest.mark.parametrize("keep", [0.99, 0.6, 0.05])
def test_rows_that_span_many_tiles(pipad, keep):  # noqa: F811
    """Hub rows of thousands of entries, cut into units, next to rows of a few."""
    rng = np.random.default_rng(int(keep * 100))
    n, k = 6000, 4
    hubs = np.stack([np.repeat([3, 4, 2500, n - 1], n), np.tile(np.arange(n), 4)], 1)
    pool = np.concatenate([hubs, rand_pairs(rng, n, 3000)])
    lists = [csr(n, pool[rng.random(len(pool)) < keep]) for _ in range(k)]
    run_case(pipad, n, lists, 16, seed=1)


def test_more_empty_rows_in_a_tile_than_entries(pipad):  # noqa: F811
    n = 40_000
    ends = [[0, c] for c in range(1, 200)] + [[n - 1, c] for c in range(0, 300, 2)]
    lists = [csr(n, ends), csr(n, ends[::2]), csr(n, ends[:199]), csr(n, [[n // 2, 1]])]
    run_case(pipad, n, lists, 4, seed=2)
