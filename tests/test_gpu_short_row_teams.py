"""Small frames of few columns: several lane groups walk a short row, four entries each at a time.  Rows at the edges of
what a group takes at a time and of what a team fetches at a time, one, two, four and eight groups, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import synth  # noqa: E402
from test_gpu_build_tiles import csr, rand_pairs  # noqa: E402
from test_gpu_parity import pipad, run_case, _reset_options  # noqa: E402,F401

LENGTHS = [1, 3, 4, 5, 7, 8, 9, 12, 15, 16, 17, 24, 31, 32, 33, 47, 48, 49, 63, 64, 65]


def frame_lists(n, k, keep=0.9):
    rng = np.random.default_rng(n + k)
    at = rng.permutation(n)[:3 * len(LENGTHS)]
    rows = np.concatenate([np.stack([np.full(m, at[q]), rng.permutation(n)[:m]], 1) for q, m in enumerate(LENGTHS * 3)])
    # (the last third of the nodes but for these rows has no entries)
    pool = np.concatenate([rows, rand_pairs(rng, n, 4 * n, hi=2 * n // 3)])
    lists = [csr(n, pool[rng.random(len(pool)) < keep ** t]) for t in range(k)]
    return n, lists


# (slices of 2, 4 and 8 lanes; n * k rows: eight groups, four or two, two or one)
@pytest.mark.parametrize("n,k", [(300, 1), (700, 3), (2400, 4), (5000, 2), (9000, 6)])
@pytest.mark.parametrize("F", [1, 2, 4, 5, 8, 9, 16, 17, 32])
def test_rows_of_every_length(pipad, n, k, F):  # noqa: F811
    n, lists = frame_lists(n, k)
    run_case(pipad, n, lists, F, seed=F + k)


@pytest.mark.parametrize("F", [3, 7, 16, 30])
def test_a_subset_gets_the_same_bits(pipad, F):  # noqa: F811
    n, lists = frame_lists(1500, 5)
    frame = pipad.frame_build_overlap([(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists])
    xs = [torch.from_numpy(synth.features(4, t, n, F)).cuda() for t in range(5)]
    Y = pipad.frame_aggregate(frame, xs)
    for chosen in ([3], [4, 0]):
        some = [torch.zeros_like(y) for y in Y]
        pipad.frame_aggregate_subset(frame, chosen, xs, some)
        assert all(torch.equal(some[t], Y[t]) for t in chosen)


@pytest.mark.parametrize("F", [4, 6, 16, 32])
def test_an_infinite_row_without_fillers_stays_infinite(pipad, F):  # noqa: F811
    """What fills the entries of a short row (up to 32 here) up to four is the row itself with weight zero: none is added behind a whole four."""
    n = 400
    rng = np.random.default_rng(F)
    pairs = np.concatenate([np.stack([np.full(m, m), 100 + rng.permutation(n - 100)[:m]], 1) for m in (4, 8, 16, 20, 32)])
    rp, c = csr(n, pairs)
    frame = pipad.frame_build_overlap([(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda())])
    x = torch.from_numpy(synth.features(1, 0, n, F)).cuda()
    x[:100] = float("inf")
    y = pipad.frame_aggregate(frame, [x])[0]
    for m in (4, 8, 16, 20, 32):
        assert bool(torch.isposinf(y[m]).all()), m
    assert bool(torch.isfinite(y[100:]).all())


@pytest.fixture(params=[0, 2])
def scale_codes(pipad, request):  # noqa: F811
    pipad.set_option("scale_codes", request.param)
    yield
    pipad.set_option("scale_codes", 1)


@pytest.mark.parametrize("F", [2, 4, 5, 8, 9, 15])
def test_rows_of_uneven_length_in_many_rows(pipad, F, scale_codes):  # noqa: F811
    """Enough rows in all snapshots (a million for slices of two lanes, 1.75 for four), most entries in long rows: lane groups by the length of the row."""
    n, k = 112_003, 16
    rng = np.random.default_rng(F)
    lengths = np.concatenate([np.tile(LENGTHS, 40), np.full(36, 40_000)])
    at = rng.permutation(n)[:len(lengths)]
    rows = np.concatenate([np.stack([np.full(m, at[q]), rng.integers(0, n, m)], 1) for q, m in enumerate(lengths)])
    pool = np.concatenate([rows, rand_pairs(rng, n, 3 * n)])
    full, less = csr(n, pool), csr(n, pool[rng.random(len(pool)) < 0.9])
    lists = [full if t % 5 else less for t in range(k)]
    run_case(pipad, n, lists, F, seed=F, check_csr=False)
    frame = pipad.frame_build_overlap([(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists])
    xs = [torch.from_numpy(synth.features(4, t, n, F)).cuda() for t in range(k)]
    Y = pipad.frame_aggregate(frame, xs)
    some = [torch.zeros_like(y) for y in Y]
    pipad.frame_aggregate_subset(frame, [7, 2], xs, some)
    assert torch.equal(some[7], Y[7]) and torch.equal(some[2], Y[2])
