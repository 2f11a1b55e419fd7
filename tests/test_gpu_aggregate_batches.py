"""The aggregation at the sizes where it changes how rows are dealt to waves, against the oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import synth  # noqa: E402
from test_gpu_parity import pipad, run_case, run_update_case, churned, _reset_options  # noqa: E402,F401


def power_law(n, edges, k, seed):
    edges = min(edges, n * (n - 1) // 8)
    s = synth.graphs(n, edges, k, 0.1, "chung-lu", (2.1, 2.0 * edges / n), seed)
    return [(s.rowptr[t], s.col[t]) for t in range(k)]


@pytest.mark.parametrize("n,k", [(15, 2), (16, 1), (17, 3), (1029, 1), (8191, 2), (30_003, 3)])
def test_fused_update_batches(pipad, n, k):  # noqa: F811
    """Rows per wave of the fused update: fewer than a tile, a tile, several."""
    run_update_case(pipad, n, power_law(n, 4 * n, k, n), 32, 16, seed=n, with_a=n % 2 == 0)


@pytest.mark.parametrize("F", [4, 5, 6, 7, 9, 15, 17, 30, 63, 65, 66, 67, 127, 130])
@pytest.mark.parametrize("layout", ["list", "wide"])
def test_widths_that_are_no_multiple_of_a_vector(pipad, F, layout):  # noqa: F811
    """Rows at any multiple of 4 bytes; the last lane of a slice shares columns with its neighbour."""
    run_case(pipad, 1500, power_law(1500, 30_000, 3, F), F, seed=F, layout=layout)


@pytest.mark.parametrize("n,edges,k", [(700, 3000, 1), (9000, 40_000, 5), (40_000, 400_000, 2)])
def test_batches_of_short_rows(pipad, n, edges, k):  # noqa: F811
    run_case(pipad, n, power_law(n, edges, k, n), 20, seed=n)


@pytest.mark.parametrize("n,k,F,Fo", [(1, 1, 1, 1), (15, 2, 3, 15), (17, 1, 4, 17), (33, 3, 15, 33), (530, 2, 16, 112),
                                      (1000, 2, 17, 66), (47, 4, 63, 49), (300, 1, 65, 129), (2049, 3, 130, 5),
                                      (45_000, 3, 66, 80)])
def test_update_behind_the_aggregation(pipad, n, k, F, Fo):  # noqa: F811
    """Remainders of rows, of K and of output columns, one and several row tiles per wave."""
    lists = power_law(n, 4 * n, k, n) if n > 2000 else churned(np.random.default_rng(n), n, k, 0.03, 0.8)
    run_update_case(pipad, n, lists, F, Fo, seed=n, with_bias=n % 2 == 1)
