"""The update for widths of H that fill neither a tile of 16 columns nor a 16-byte piece, inside the aggregation
kernel and behind it (one block of columns, or several of equal width); nothing is written behind a row."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_build_tiles import csr, rand_pairs  # noqa: E402
from test_gpu_parity import pipad, _reset_options  # noqa: E402,F401

INSIDE = [(F, Fo) for F in (16, 20, 64) for Fo in (1, 7, 8, 15, 17, 30, 33, 48, 50, 63, 64)]
BEHIND = [(128, 65), (128, 80), (128, 81), (128, 112), (128, 113), (128, 128), (96, 128), (100, 128), (30, 129), (7, 300),
          (300, 20), (1100, 16)]


@pytest.mark.parametrize("bias", [True, False])
@pytest.mark.parametrize("F,Fo", INSIDE + BEHIND)
def test_every_width(pipad, F, Fo, bias):  # noqa: F811
    rng = np.random.default_rng(F + Fo)
    n, k = (1003, 2) if F <= 32 or Fo % 16 == 0 or F > 64 else (50_003, 8)  # (inside from 400k rows on)
    pool = np.concatenate([rand_pairs(rng, n, 8 * n), np.stack([np.full(900, 17), rng.integers(0, n, 900)], 1)])
    lists = [csr(n, pool[rng.random(len(pool)) < 0.9]) for _ in range(k)]
    snaps = [(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists]
    for mid_max in (512, 300):  # a workgroup per long row, or its class parts
        pipad.set_option("mid_max", mid_max)
        frame = pipad.frame_build_overlap(snaps)
        X = [torch.empty((n, F), device="cuda:0").uniform_(-1, 1) for _ in range(k)]
        W = torch.empty((F, Fo), device="cuda:0").uniform_(-1, 1)
        b = torch.empty(Fo, device="cuda:0").uniform_(-1, 1) if bias else None
        wide = [torch.full((n, Fo + 5), 77.0, device="cuda:0") for _ in range(k)]
        A = [torch.zeros((n, F), device="cuda:0") for _ in range(k)]
        pipad.frame_aggregate_update(frame, X, W, b, H=[h[:, :Fo] for h in wide], A=A)
        Y = pipad.frame_aggregate(frame, X)
        for t in range(k):
            assert torch.equal(A[t], Y[t])
            exact = Y[t].double() @ W.double() + (b.double() if bias else 0.0)
            bound = Y[t].double().abs() @ W.double().abs() + (b.double().abs() if bias else 0.0)
            assert bool(((wide[t][:, :Fo].double() - exact).abs() <= (F + 2) * 2.0 ** -24 * bound).all())
            assert bool((wide[t][:, Fo:] == 77.0).all())


@pytest.mark.parametrize("Fo", [8, 20, 50])
def test_odd_widths_without_room_for_the_aggregation_stay_refused(pipad, Fo):  # noqa: F811
    n, F = 300, 32
    rng = np.random.default_rng(1)
    rp, c = csr(n, rand_pairs(rng, n, 900))
    frame = pipad.frame_build_overlap([(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda())])
    X, W = [torch.zeros((n, F), device="cuda:0")], torch.zeros((F, Fo), device="cuda:0")
    with pytest.raises(Exception):
        pipad.frame_aggregate_update(frame, X, W, H=[torch.zeros((n, Fo), device="cuda:0")])


@pytest.mark.parametrize("n,k,F,Fo", [(32_735, 2, 128, 112), (32_800, 2, 128, 112), (32_800, 2, 200, 64), (16_300, 2, 300, 40),
                                      (16_400, 2, 300, 40), (40_003, 2, 90, 127), (270_001, 2, 128, 112), (260_001, 2, 128, 112)])
def test_blocks_of_columns_by_the_size_of_the_frame(pipad, n, k, F, Fo):  # noqa: F811
    """Both sides of 4096 and 2048 tiles of 16 rows, and of results past 256 MB: other blocks of columns, the same values."""
    rng = np.random.default_rng(F + Fo)
    snaps = [(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in [csr(n, rand_pairs(rng, n, 2 * n)) for _ in range(k)]]
    frame = pipad.frame_build_overlap(snaps)
    X = [torch.empty((n, F), device="cuda:0").uniform_(-1, 1) for _ in range(k)]
    W, b = torch.empty((F, Fo), device="cuda:0").uniform_(-1, 1), torch.empty(Fo, device="cuda:0").uniform_(-1, 1)
    A, H = [torch.zeros((n, F), device="cuda:0") for _ in range(k)], [torch.full((n, Fo), 77.0, device="cuda:0") for _ in range(k)]
    pipad.frame_aggregate_update(frame, X, W, b, H=H, A=A)
    for t in range(k):
        exact = A[t].double() @ W.double() + b.double()
        bound = A[t].double().abs() @ W.double().abs() + b.double().abs()
        assert bool(((H[t].double() - exact).abs() <= (F + 2) * 2.0 ** -24 * bound).all())


@pytest.mark.parametrize("n,k,F,Fo,per_row", [(7_249, 2, 48, 48, 3), (7_251, 2, 48, 48, 3), (1_499, 10, 64, 64, 3), (1_501, 10, 36, 64, 3),
                                              (11_999, 2, 64, 32, 25), (12_001, 2, 64, 32, 25),
                                              (12_001, 2, 36, 16, 8), (28_990, 2, 64, 64, 12), (29_010, 2, 64, 64, 12)])
def test_few_rows_and_whole_tiles_of_columns(pipad, n, k, F, Fo, per_row):  # noqa: F811
    """Both sides of the numbers of rows from and up to which widths of whole tiles are multiplied behind the aggregation, where it
    is kept; without room for it they stay inside.  Eager and recorded, at the scratch the aggregation leaves."""
    rng = np.random.default_rng(n + Fo)
    pool = np.concatenate([rand_pairs(rng, n, per_row * n), np.stack([np.full(900, 17), rng.integers(0, n, 900)], 1)])
    lists = [csr(n, pool[rng.random(len(pool)) < 0.9]) for _ in range(k)]
    snaps = [(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists]
    X = [torch.empty((n, F), device="cuda:0").uniform_(-1, 1) for _ in range(k)]
    W, b = torch.empty((F, Fo), device="cuda:0").uniform_(-1, 1), torch.empty(Fo, device="cuda:0").uniform_(-1, 1)
    for segment in (700, 300):  # hub rows in parts, too
        pipad.set_option("mid_max", segment)
        pipad.set_option("hub_segment", segment)
        pipad.set_option("hub_threshold", segment)
        frame = pipad.frame_build_overlap(snaps)
        Y = pipad.frame_aggregate(frame, X)

        def check(H, A):
            for t in range(k):
                assert A is None or torch.equal(A[t], Y[t])
                exact = Y[t].double() @ W.double() + b.double()
                bound = Y[t].double().abs() @ W.double().abs() + b.double().abs()
                # (F products, F sums and the bias, each rounded once)
                assert bool(((H[t][:, :Fo].double() - exact).abs() <= (F + 2) * 2.0 ** -24 * bound).all())
                assert bool((H[t][:, Fo:] == 77.0).all())

        for keep in (True, False):
            wide = [torch.full((n, Fo + 4), 77.0, device="cuda:0") for _ in range(k)]
            H = [h[:, :Fo] for h in wide]
            A = [torch.zeros((n, F), device="cuda:0") for _ in range(k)] if keep else None
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                pipad.frame_aggregate_update(frame, X, W, b, H=H, A=A)
            for _ in range(2):
                for m in H + (A or []):
                    m.fill_(float("nan"))
                graph.replay()
                torch.cuda.synchronize()
                check(wide, A)
            for m in H + (A or []):
                m.fill_(float("nan"))
            pipad.frame_aggregate_update(frame, X, W, b, H=H, A=A)
            check(wide, A)
        frame.close()


@pytest.mark.parametrize("n,k,F,Fo,bias", [(7_251, 2, 48, 48, True), (1_501, 10, 36, 64, False), (12_001, 2, 64, 32, True), (12_001, 2, 40, 16, True),
                                           (28_990, 2, 64, 64, True), (15_003, 3, 60, 48, False), (15_003, 3, 44, 16, True)])
def test_same_bits_with_and_without_the_aggregation(pipad, n, k, F, Fo, bias):  # noqa: F811
    """Shapes that are multiplied behind the aggregation where it is kept, inside where it is not."""
    rng = np.random.default_rng(n + Fo)
    pool = np.concatenate([rand_pairs(rng, n, 25 * n), np.stack([np.full(900, 17), rng.integers(0, n, 900)], 1)])
    snaps = [(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in
             [csr(n, pool[rng.random(len(pool)) < 0.9]) for _ in range(k)]]
    frame = pipad.frame_build_overlap(snaps)
    X = [torch.empty((n, F), device="cuda:0").uniform_(-1, 1) for _ in range(k)]
    X[0][5, F - 1] = float("inf")  # (columns past the last one take no part)
    W = torch.empty((F, Fo), device="cuda:0").uniform_(-1, 1)
    b = torch.empty(Fo, device="cuda:0").uniform_(-1, 1) if bias else None
    H, A = [[torch.full((n, Fo), 77.0, device="cuda:0") for _ in range(k)] for _ in range(2)], [torch.empty((n, F), device="cuda:0") for _ in range(k)]
    pipad.frame_aggregate_update(frame, X, W, b, H=H[0], A=A)
    pipad.frame_aggregate_update(frame, X, W, b, H=H[1])
    for t in range(k):
        assert torch.equal(H[0][t].view(torch.int32), H[1][t].view(torch.int32)), t
    frame.close()


@pytest.mark.parametrize("options", [{}, {"mid_max": 300}, {"mid_max": 600, "hub_segment": 300, "hub_threshold": 700}])
@pytest.mark.parametrize("n,k,F,Fo,bias", [(7_251, 2, 48, 48, True), (1_501, 10, 36, 64, False), (28_990, 2, 64, 64, True),
                                           (15_003, 3, 60, 48, False), (15_003, 3, 44, 16, True)])
def test_same_bits_where_hub_rows_end_in_partial_sums(pipad, options, n, k, F, Fo, bias):  # noqa: F811
    """The same shapes with rows that are summed in parts: longer than hub_threshold, or by column class."""
    rng = np.random.default_rng(n + F)
    hubs = [np.stack([np.full(length, row), rng.permutation(n)[:length]], 1) for row, length in ((17, min(n - 1, 5000)), (n - 1, 1400))]
    pool = np.concatenate([rand_pairs(rng, n, 25 * n), *hubs])
    lists = [csr(n, pool[rng.random(len(pool)) < 0.95]) for _ in range(k)]
    assert min(np.diff(rp).max() for rp, _ in lists) > (2048 if n > 2048 and not options else 700)
    for key, value in options.items():
        pipad.set_option(key, value)
    frame = pipad.frame_build_overlap([(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists])
    X = [torch.empty((n, F), device="cuda:0").uniform_(-1, 1) for _ in range(k)]
    W = torch.empty((F, Fo), device="cuda:0").uniform_(-1, 1)
    b = torch.empty(Fo, device="cuda:0").uniform_(-1, 1) if bias else None
    H, A = [[torch.full((n, Fo), 77.0, device="cuda:0") for _ in range(k)] for _ in range(2)], [torch.empty((n, F), device="cuda:0") for _ in range(k)]
    pipad.frame_aggregate_update(frame, X, W, b, H=H[0], A=A)
    pipad.frame_aggregate_update(frame, X, W, b, H=H[1])
    for t in range(k):
        assert torch.equal(H[0][t].view(torch.int32), H[1][t].view(torch.int32)), t
        exact = A[t].double() @ W.double() + (b.double() if bias else 0.0)
        bound = A[t].double().abs() @ W.double().abs() + (b.double().abs() if bias else 0.0)
        assert bool(((H[1][t].double() - exact).abs() <= (F + 2) * 2.0 ** -24 * bound).all())  # (F products, F sums, the bias)
    frame.close()
