"""Long rows of small frames: a workgroup walks a unit from the parts' own lists, and finishes the row where no row
is cut into several.  Rows at the edges of what a wave takes of them, with exclusive lists of very different
lengths, against the oracle; both operand layouts, every width of a lane team, the update and the transposed frame."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
import synth  # noqa: E402
from _util import check_y, csr_to_coo  # noqa: E402
from test_gpu_build_tiles import csr, rand_pairs  # noqa: E402
from test_gpu_parity import pipad, run_case, _reset_options  # noqa: E402,F401


def frame_lists(k, keep, lengths, n=5000):
    rng = np.random.default_rng(k + len(lengths))
    hubs = np.concatenate([np.stack([np.full(m, 5 + 7 * q), rng.permutation(n)[:m]], 1) for q, m in enumerate(lengths)])
    pool = np.concatenate([hubs, rand_pairs(rng, n, 2000)])
    # the first snapshot has every entry, the others fewer and fewer
    return n, [csr(n, pool[rng.random(len(pool)) < keep ** t]) for t in range(k)]


DIRECT, CUT = [513, 514, 767, 1023, 1024, 1025, 2040], [513, 1030, 2047, 2100, 4097, 4990]


@pytest.mark.parametrize("lengths", [DIRECT, CUT], ids=["whole", "cut"])
@pytest.mark.parametrize("k,keep", [(1, 1.0), (3, 0.97), (5, 0.2)])
@pytest.mark.parametrize("F,layout", [(1, "list"), (3, "list"), (4, "list"), (7, "list"), (16, "list"), (30, "list"),
                                      (64, "list"), (100, "list"), (1, "wide"), (2, "wide"), (4, "wide"), (9, "wide"),
                                      (27, "wide")])
def test_rows_of_every_length(pipad, lengths, k, keep, F, layout):  # noqa: F811
    pipad.set_option("agg_coalescent", 2)
    n, lists = frame_lists(k, keep, lengths)
    run_case(pipad, n, lists, F, seed=F, layout=layout)


@pytest.mark.parametrize("lengths", [DIRECT, CUT], ids=["whole", "cut"])
def test_other_paths(pipad, lengths):  # noqa: F811
    k, F = 3, 64
    n, lists = frame_lists(k, 0.8, lengths)
    snaps = [(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists]
    frame = pipad.frame_build_overlap(snaps)
    X = [synth.features(9, t, n, F) for t in range(k)]
    xs = [torch.from_numpy(x).cuda() for x in X]
    Y = pipad.frame_aggregate(frame, xs)
    for generic in (0, 1):  # neither the fixed scratch nor 64-bit addresses change a bit
        pipad.set_option("agg_generic", generic)
        other = pipad.frame_build_overlap(snaps)
        Z = pipad.frame_aggregate(other, xs, static_scratch=True)
        assert generic or all(torch.equal(a, b) for a, b in zip(Y, Z))
        coo = csr_to_coo(n, *lists[1])
        check_y(Z[1].cpu().numpy(), *oracle.aggregate(n, *coo, X[1], threads=8)[1:3])
    pipad.set_option("agg_generic", 0)
    some = [torch.zeros_like(y) for y in Y]
    pipad.frame_aggregate_subset(frame, [2, 0], xs, some)
    assert torch.equal(some[2], Y[2]) and torch.equal(some[0], Y[0])
    # the update, inside the kernel (Fo = 48) and behind it (Fo = 50)
    for Fo in (48, 50):
        W = torch.empty((F, Fo), device="cuda:0").uniform_(-1, 1)
        A = [torch.zeros_like(y) for y in Y]
        H = pipad.frame_aggregate_update(frame, xs, W, None, A=A)
        for t in range(k):
            assert torch.equal(A[t], Y[t])
            exact = A[t].double() @ W.double()
            bound = A[t].double().abs() @ W.double().abs()
            assert bool(((H[t].double() - exact).abs() <= (F + 2) * 2.0 ** -24 * bound).all())
    # columns of the transposed frame: the same lengths as rows of this one
    back = pipad.frame_transpose(pipad.frame_build_overlap([
        (torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda())
        for rp, c in (csr(n, np.stack(csr_to_coo(n, *part)[::-1], 1)) for part in lists)]))
    Z = pipad.frame_aggregate(back, xs)
    for t in range(k):
        rows, cols = csr_to_coo(n, *lists[t])
        z, bound = oracle.aggregate_transposed(n, cols, rows, X[t])
        check_y(Z[t].cpu().numpy(), z, bound, f"transposed, snapshot {t}")


@pytest.mark.parametrize("k", [1, 4, 5])
@pytest.mark.parametrize("F,layout", [(4, "list"), (16, "list"), (64, "list"), (3, "wide")])
def test_longest_row_of_a_lane_team(pipad, k, F, layout):  # noqa: F811
    """Small frames leave rows of more than 32 or 48 entries to a whole wave."""
    n, lists = frame_lists(k, 0.98, [31, 32, 33, 34, 47, 48, 49, 50, 63, 64, 65, 66], n=700)
    run_case(pipad, n, lists, F, seed=k, layout=layout)
