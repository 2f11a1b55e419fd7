"""Rows of more than 64 columns: one slice or two by where the rows start, the last slice not always full; rows of
one to four columns, lanes of one column each; against the oracle, with rows on cache lines, dense ones and ones
that start anywhere."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
import synth  # noqa: E402
from _util import check_y, csr_to_coo  # noqa: E402
from test_gpu_build_tiles import csr, rand_pairs  # noqa: E402
from test_gpu_parity import pipad, _reset_options  # noqa: E402,F401


def matrices(values, ld, offset):
    """Device copies of the matrices with row stride ld, `offset` floats behind where an allocation starts."""
    got = []
    for v in values:
        n, F = v.shape
        flat = torch.full((offset + n * ld,), float("nan"), device="cuda:0")
        x = flat[offset:].view(n, ld)[:, :F]
        x.copy_(torch.from_numpy(v))
        got.append(x)
    return got


@pytest.mark.parametrize("hubs", [False, True])
@pytest.mark.parametrize("F", [1, 2, 3, 4, 5, 33, 64, 65, 66, 67, 80, 95, 96, 97, 100, 127, 128, 129, 160, 250])
def test_any_start_of_a_row(pipad, F, hubs):  # noqa: F811
    rng = np.random.default_rng(F)
    n, k = 1300, 3 + F % 2
    pool = rand_pairs(rng, n, 9 * n)
    if hubs:
        pool = np.concatenate([pool, np.stack([np.repeat([7, 900], 1250), rng.integers(0, n, 2500)], 1)])
        pipad.set_option("mid_max", 200)  # class parts; else a workgroup per row or a wave
    lists = [csr(n, pool[rng.random(len(pool)) < 0.9]) for _ in range(k)]
    snaps = [(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists]
    frame = pipad.frame_build_overlap(snaps)
    X = [synth.features(F, t, n, F) for t in range(k)]
    ref = [oracle.aggregate(n, *csr_to_coo(n, *lists[t]), X[t], threads=8)[1:3] for t in range(k)]
    lines = (F + 31) // 32 * 32
    for ld, offset in ((lines, 0), (F, 0), (lines, 5), (F + 3, 1)):
        xs = matrices(X, ld, offset)
        Y = pipad.frame_aggregate(frame, xs)
        for t in range(k):
            check_y(Y[t].cpu().numpy(), *ref[t], f"stride {ld}, offset {offset}, snapshot {t}")
        Z = pipad.frame_aggregate(frame, xs, static_scratch=True)
        some = [torch.zeros_like(y) for y in Y]
        pipad.frame_aggregate_subset(frame, [2, 1], xs, some)
        assert all(torch.equal(a, b) for a, b in zip(Y, Z))
        assert torch.equal(some[1], Y[1]) and torch.equal(some[2], Y[2])


@pytest.mark.parametrize("mid_max", [200, 512])
@pytest.mark.parametrize("F", [65, 66, 80, 95, 96, 97, 100, 112, 127, 128])
def test_a_subset_gets_the_bits_of_the_whole_call_wherever_rows_start(pipad, F, mid_max):  # noqa: F811
    """Row strides that are whole lines while the snapshots' matrices start on lines, off them, or some on and
    some off (the concatenated operand: X[t] = base + t * F): every single snapshot gets the bits of the call
    over all of them, and the bits do not depend on where a matrix lies."""
    rng = np.random.default_rng(F)
    n, k = 1300, 8
    pool = np.concatenate([rand_pairs(rng, n, 9 * n), np.stack([np.repeat([7, 900], 1250), rng.integers(0, n, 2500)], 1),
                           np.stack([np.repeat([30, 31, 32], 150), rng.integers(0, n, 450)], 1)])
    pipad.set_option("mid_max", mid_max)  # hub rows by class, or by a workgroup each
    lists = [csr(n, pool[rng.random(len(pool)) < 0.9]) for _ in range(k)]
    frame = pipad.frame_build_overlap([(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists])
    X = [synth.features(F, t, n, F) for t in range(k)]
    beside = torch.stack([torch.from_numpy(x) for x in X], 1).cuda()  # [n, k, F]; k * F is a multiple of 32 where F is one of 4
    placed = {"on lines": matrices(X, 160, 0), "off lines": matrices(X, 160, 5),
              "some": [m for t in range(k) for m in matrices(X[t:t + 1], 160, 4 * (t % 3))],
              "side by side": [beside[:, t, :] for t in range(k)]}
    results = {}
    for what, xs in placed.items():
        Y = results[what] = pipad.frame_aggregate(frame, xs, [torch.empty((n, F), device="cuda:0") for _ in range(k)])
        for t in range(k):
            one = torch.full((n, F), float("nan"), device="cuda:0")
            pipad.frame_aggregate_subset(frame, [t], [xs[t] if u == t else None for u in range(k)],
                                         [one if u == t else None for u in range(k)])
            assert torch.equal(one, Y[t]), f"{what}, snapshot {t}"
    for what in ("off lines", "some"):
        assert all(torch.equal(a, b) for a, b in zip(results[what], results["on lines"])), what
    for t in range(k):
        bounds = oracle.aggregate(n, *csr_to_coo(n, *lists[t]), X[t], threads=8)[1:3]
        check_y(results["on lines"][t].cpu().numpy(), *bounds, f"snapshot {t}")
        check_y(results["side by side"][t].cpu().numpy(), *bounds, f"snapshot {t}, side by side")


@pytest.mark.parametrize("F", [66, 96, 100, 127])
@pytest.mark.parametrize("n,k", [(59_999, 1), (60_000, 1), (16_666, 3), (16_667, 3), (2_499, 4), (2_500, 4)])
def test_rows_of_all_snapshots_around_one_slice_and_two(pipad, n, k, F):  # noqa: F811
    """n * k on both sides of where rows of 65 columns and more go in one slice."""
    rng = np.random.default_rng(n)
    pool = np.concatenate([rand_pairs(rng, n, 3 * n), np.stack([np.repeat([7, 900], 700), rng.integers(0, n, 1400)], 1),
                           np.stack([np.repeat([30, 31, 32], 150), rng.integers(0, n, 450)], 1)])
    lists = [csr(n, pool[rng.random(len(pool)) < 0.9]) for _ in range(k)]
    frame = pipad.frame_build_overlap([(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists])
    X = [synth.features(F, t, n, F) for t in range(k)]
    for xs in (matrices(X, 128, 0), matrices(X, F, 0)):
        Y = pipad.frame_aggregate(frame, xs, [torch.empty((n, F), device="cuda:0") for _ in range(k)])
        one = torch.full((n, F), float("nan"), device="cuda:0")
        pipad.frame_aggregate_subset(frame, [k - 1], xs, [None] * (k - 1) + [one])
        assert torch.equal(one, Y[k - 1])
        for t in range(k):
            check_y(Y[t].cpu().numpy(), *oracle.aggregate(n, *csr_to_coo(n, *lists[t]), X[t], threads=8)[1:3], f"snapshot {t}")
