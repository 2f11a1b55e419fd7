"""The rows of all slices side by side, a run of slices per XCD: the same bits as the slices in turn and one after
the other, for numbers of slices that do not divide 8, all kinds of rows and none of some."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from _util import check_y, csr_to_coo  # noqa: E402
from test_gpu_build_tiles import csr, rand_pairs  # noqa: E402
from test_gpu_parity import pipad, _reset_options  # noqa: E402,F401


def frames(pipad, lists, **options):  # noqa: F811
    snaps = [(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists]
    got = []
    for order in (2, 0, 1):  # automatic, in turn, one after the other
        pipad.set_option("agg_order", order)
        for key, value in options.items():
            pipad.set_option(key, value)
        got.append(pipad.frame_build_overlap(snaps))
    return got


@pytest.mark.parametrize("k,F,rows", [(3, 64, "all"), (5, 50, "all"), (6, 100, "all"), (9, 64, "all"), (3, 64, "no mid"),
                                      (3, 64, "no short"), (5, 64, "no hub"), (11, 64, "all")])
def test_same_bits_as_the_other_orders(pipad, k, F, rows):  # noqa: F811
    rng = np.random.default_rng(k * F)
    n = 20_500  # matrices of 5 MiB
    hubs = np.stack([np.repeat([3, 900, n - 1], 3000), rng.integers(0, n, 9000)], 1)
    mids = np.stack([np.repeat(rng.integers(0, n, 300), 150), rng.integers(0, n, 45_000)], 1)
    pool = np.concatenate([hubs, mids, rand_pairs(rng, n, 12 * n)])
    lists = [csr(n, pool[rng.random(len(pool)) < 0.95]) for _ in range(k)]
    options = {"no mid": {"mid_max": 64}, "no short": {"short_max": 0}, "no hub": {"mid_max": 1 << 20}}.get(rows, {})
    runs, turn, after = frames(pipad, lists, **options)
    X = [torch.empty((n, F), device="cuda:0").uniform_(-1, 1) for _ in range(k)]
    Y = pipad.frame_aggregate(runs, X)
    for other in (turn, after):
        Z = pipad.frame_aggregate(other, X)
        assert all(torch.equal(a, b) for a, b in zip(Y, Z))
    r, c = csr_to_coo(n, *lists[k - 1])
    _, yd, bound, _ = oracle.aggregate(n, r, c, X[k - 1].cpu().numpy(), threads=8)
    check_y(Y[k - 1].cpu().numpy(), yd, bound)
    # three of the snapshots, and through the fixed scratch
    some = [torch.zeros_like(y) for y in Y]
    pipad.frame_aggregate_subset(runs, [2, 0, 1], X, some)
    assert all(torch.equal(some[t], Y[t]) for t in range(3))
    Z = pipad.frame_aggregate(runs, X, static_scratch=True)
    assert all(torch.equal(a, b) for a, b in zip(Y, Z))
