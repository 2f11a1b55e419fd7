"""The per-entry scales and the class-grouped copies of the hub rows, against the oracle: numbers of
snapshots that no 16-byte piece of scales fits, and hub units at the edges of the pieces (512 entries of a
wave, 2048 of a workgroup) that are put in class order at a time."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
import synth  # noqa: E402
from _util import check_y, csr_to_coo  # noqa: E402
from test_gpu_build_tiles import csr, rand_pairs  # noqa: E402
from test_gpu_parity import pipad, run_case, _reset_options  # noqa: E402,F401


@pytest.mark.parametrize("k", [1, 2, 3, 5, 6, 7, 11, 13, 17])
def test_scales_of_any_number_of_snapshots(pipad, k):  # noqa: F811
    rng = np.random.default_rng(k)
    n, F = 500, 8
    pool = rand_pairs(rng, n, 6000)
    lists = [csr(n, pool[rng.random(len(pool)) < 0.9]) for _ in range(k)]
    pipad.set_option("short_max", 4)
    pipad.set_option("mid_max", 11)
    run_case(pipad, n, lists, F, seed=k)
    # the transposed frame writes them again
    snaps = [(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists]
    back = pipad.frame_transpose(pipad.frame_build_overlap(snaps))
    X = [synth.features(k, t, n, F) for t in range(k)]
    Z = pipad.frame_aggregate(back, [torch.from_numpy(x).cuda() for x in X])
    for t in range(k):
        rows, cols = csr_to_coo(n, *lists[t])
        z, bound = oracle.aggregate_transposed(n, rows, cols, X[t])
        check_y(Z[t].cpu().numpy(), z, bound, f"transposed, snapshot {t}")


@pytest.mark.parametrize("segment", [2048, 1 << 20])
@pytest.mark.parametrize("keep", [0.97, 0.2])
@pytest.mark.parametrize("sub", [1, 4])
def test_units_at_the_edges_of_a_piece(pipad, segment, keep, sub):  # noqa: F811
    """Mostly common (a workgroup per unit of the common part, a wave elsewhere) and mostly exclusive."""
    rng = np.random.default_rng(segment + sub)
    n, k = 9000, 3
    lengths = [511, 512, 513, 2047, 2048, 2049, 4100, n - 1]
    hubs = np.concatenate([np.stack([np.full(m, 5 + 7 * q), rng.permutation(n)[:m]], 1)
                           for q, m in enumerate(lengths)])
    pool = np.concatenate([hubs, rand_pairs(rng, n, 2000)])
    whole = csr(n, pool)
    lists = [whole] + [csr(n, pool[rng.random(len(pool)) < keep]) for _ in range(k - 1)]
    pipad.set_option("mid_max", 300)
    pipad.set_option("hub_threshold", segment)
    pipad.set_option("hub_segment", segment)
    pipad.set_option("sub_classes", sub)
    run_case(pipad, n, lists, 16, seed=1)


@pytest.mark.parametrize("units", [1, 3, 64, 301])
@pytest.mark.parametrize("k", [1, 2, 4, 9])
@pytest.mark.parametrize("sizes", ["first", "last", "growing", "one empty", "disjoint"])
def test_parts_of_very_different_sizes(pipad, sizes, k, units):  # noqa: F811
    """The exclusive parts' units are dealt to the XCDs by the parts' sizes: one part has everything, or each
    twice what the one before has, or one has nothing, or all have as much and the common part nothing."""
    rng = np.random.default_rng(k * units)
    n = 1500
    pool = np.concatenate([np.stack([np.full(m, 2 * q), rng.permutation(n)[:m]], 1)
                           for q, m in enumerate(rng.integers(210, 700, units))] + [rand_pairs(rng, n, 800)])
    pool = pool[rng.permutation(len(pool))]
    m = len(pool)
    share = {"first": lambda t: slice(0, m if t == 0 else m // 50), "last": lambda t: slice(0, m if t == k - 1 else m // 50),
             "growing": lambda t: slice(0, m >> (k - 1 - t)), "one empty": lambda t: slice(0, 0 if t == k // 2 else m),
             "disjoint": lambda t: slice(m * t // k, m * (t + 1) // k)}[sizes]
    pipad.set_option("mid_max", 40)
    pipad.set_option("short_max", 20)
    run_case(pipad, n, [csr(n, pool[share(t)]) for t in range(k)], 8, seed=units)
