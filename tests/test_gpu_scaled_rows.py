"""Concatenated operands whose rows are multiplied by their scales first (k_scale_rows): lane layouts and strides, and the
same bits where there is no room for the products."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
import synth  # noqa: E402
from _util import check_y, csr_to_coo  # noqa: E402
from test_gpu_aggregate_batches import power_law  # noqa: E402
from test_gpu_parity import pipad, _reset_options  # noqa: E402,F401


# frames just past the rule 3 k entries > 10^7 + k n (4 F + 1)
@pytest.mark.parametrize("n,entries,k,F,pad,plain", [(6000, 260_000, 16, 1, 0, True), (6000, 700_000, 7, 2, 0, False), (6000, 1_000_000, 4, 3, 1, True),
                                                     (6000, 1_100_000, 4, 4, 3, False), (6000, 1_400_000, 3, 3, 0, False),
                                                     (6000, 300_000, 16, 5, 0, True), (6000, 700_000, 6, 8, 1, False),
                                                     (6000, 700_000, 7, 13, 0, False), (6000, 1_950_000, 2, 31, 0, True)])
@pytest.mark.parametrize("codes", [0, 2])  # (2: scales as codes, hub rows by class)
def test_against_the_oracle_and_without_room(pipad, n, entries, k, F, pad, plain, codes):  # noqa: F811
    pipad.set_option("agg_coalescent", 2)
    pipad.set_option("scale_codes", codes)
    if not plain:  # hub rows by class, several units each
        pipad.set_option("mid_max", 300)
        pipad.set_option("hub_segment", 700)
        pipad.set_option("hub_threshold", 700)
    lists = power_law(n, entries // 2, k, F)
    shared = min(len(c) for _, c in lists)
    assert 3 * k * shared > 10_000_000 + k * n * (4 * F + 1)
    snaps = [(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists]
    frame, fresh = pipad.frame_build_overlap(snaps), pipad.frame_build_overlap(snaps)
    store = torch.zeros((n, k * F + pad), device="cuda:0")
    X = [store[:, pad + t * F:pad + (t + 1) * F] for t in range(k)]
    for t in range(k):
        X[t].copy_(torch.from_numpy(synth.features(3, t, n, F)))
    out = torch.full_like(store, float("nan"))
    Y = [out[:, pad + t * F:pad + (t + 1) * F] for t in range(k)]
    pipad.frame_aggregate(frame, X, Y)
    want = out.clone()
    for t in (0, k - 1):
        _, yd, bound, _ = oracle.aggregate(n, *csr_to_coo(n, *lists[t]), synth.features(3, t, n, F), threads=8)
        check_y(Y[t].cpu().numpy(), yd, bound, f"snapshot {t}")
    out.fill_(float("nan"))
    pipad.frame_aggregate(frame, X, Y, static_scratch=True)
    assert torch.equal(out[:, pad:], want[:, pad:])
    # recorded on a frame whose scratch holds the partial sums and no more
    parts = [torch.zeros((n, F), device="cuda:0") for _ in range(k)]
    pipad.frame_aggregate(fresh, parts, [torch.empty_like(p) for p in parts])
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pipad.frame_aggregate(fresh, X, Y)
    for _ in range(3):
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out[:, pad:], want[:, pad:])
    frame.close()
    fresh.close()


@pytest.mark.parametrize("k,F,products", [(16, 1, False), (16, 2, False), (16, 4, False), (16, 2, True)])
def test_short_rows_longest_first(pipad, k, F, products):  # noqa: F811
    """Batches of several steps: 600,000 rows, most of them short, of very different lengths."""
    n = 600_000
    s = synth.graphs(n, 2_400_000 if products else 600_000, k, 0.01, "rmat", (0.57, 0.19, 0.19, 0.05), 5)
    assert (3 * k * min(len(s.col[t]) for t in range(k)) > 10_000_000 + k * n * (4 * F + 1)) == products
    frame = pipad.frame_build_overlap([(torch.from_numpy(s.rowptr[t]).cuda(), torch.from_numpy(s.col[t]).cuda()) for t in range(k)])
    x = torch.empty((n, k, F), device="cuda:0").uniform_(-1, 1)
    y = pipad.frame_aggregate(frame, x)
    for t in (0, k - 1):
        _, yd, bound, _ = oracle.aggregate(n, *csr_to_coo(n, s.rowptr[t], s.col[t]), x[:, t].cpu().numpy(), threads=8)
        check_y(y[:, t].cpu().numpy(), yd, bound, f"snapshot {t}")
    frame.close()


@pytest.mark.parametrize("k,F,classes", [(3, 1, False), (4, 4, True), (5, 2, True), (7, 1, False), (16, 2, True), (16, 4, False)])
def test_entries_shared_by_a_quad(pipad, k, F, classes):  # noqa: F811
    """Rows whose common entries are fetched once for a team's snapshots: teams of 4 to 64 lanes, idle lanes among them, short,
    mid and hub rows; the products that the kernel makes itself are summed up without that."""
    n = 20_000 if classes else 70_000
    pipad.set_option("agg_coalescent", 2)
    if classes:  # hub rows by column class in a small frame, too
        pipad.set_option("mid_max", 300)
    s = synth.graphs(n, 1_300_000, k, 0.02, "rmat", (0.57, 0.19, 0.19, 0.05), 9)
    frame = pipad.frame_build_overlap([(torch.from_numpy(s.rowptr[t]).cuda(), torch.from_numpy(s.col[t]).cuda()) for t in range(k)])
    assert frame.common()[1].numel() >= 10 * n
    assert 3 * k * min(len(s.col[t]) for t in range(k)) > 10_000_000 + k * n * (4 * F + 1)
    x = torch.empty((n, k, F), device="cuda:0").uniform_(-1, 1)
    y = pipad.frame_aggregate(frame, x)
    for t in (0, k - 1):
        _, yd, bound, _ = oracle.aggregate(n, *csr_to_coo(n, s.rowptr[t], s.col[t]), x[:, t].cpu().numpy(), threads=8)
        check_y(y[:, t].cpu().numpy(), yd, bound, f"snapshot {t}")
    # recorded on a frame whose scratch holds the partial sums and no more: no room for the products
    fresh = pipad.frame_build_overlap([(torch.from_numpy(s.rowptr[t]).cuda(), torch.from_numpy(s.col[t]).cuda()) for t in range(k)])
    parts = [torch.zeros((n, F), device="cuda:0") for _ in range(k)]
    pipad.frame_aggregate(fresh, parts, [torch.empty_like(p) for p in parts])
    torch.cuda.synchronize()
    out = torch.full_like(y, float("nan"))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pipad.frame_aggregate(fresh, x, out)
    for _ in range(2):
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, y)
    frame.close()
    fresh.close()


@pytest.mark.parametrize("codes", [0, 2])
@pytest.mark.parametrize("F", [2, 5])
def test_infinite_rows_are_infinite_either_way(pipad, F, codes):  # noqa: F811
    """What fills up a step of four entries is the row itself with weight 0 where the kernel makes the products: it takes no part."""
    n, k = 6000, 7
    pipad.set_option("scale_codes", codes)
    pipad.set_option("agg_coalescent", 2)
    lists = power_law(n, 350_000, k, F)
    assert 3 * k * min(len(c) for _, c in lists) > 10_000_000 + k * n * (4 * F + 1)
    frame = pipad.frame_build_overlap([(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists])
    x = torch.empty((n, k, F), device="cuda:0").uniform_(-1, 1)
    x[::50] = float("inf")
    y = pipad.frame_aggregate(frame, x)
    assert not y.isnan().any() and y[::50].isinf().all()
    assert torch.equal(pipad.frame_aggregate(frame, x, static_scratch=True), y)
    # recorded with room for the partial sums and no more
    fresh = pipad.frame_build_overlap([(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists])
    parts = [torch.zeros((n, F), device="cuda:0") for _ in range(k)]
    pipad.frame_aggregate(fresh, parts, [torch.empty_like(p) for p in parts])
    torch.cuda.synchronize()
    out = torch.full_like(y, float("nan"))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pipad.frame_aggregate(fresh, x, out)
    for _ in range(2):
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, y)
    frame.close()
    fresh.close()


def test_recorded_calls_outlive_later_products(pipad):  # noqa: F811
    """Calls recorded before one that needs (more) room for products still find theirs, with the library's own allocator, too."""
    n, k = 6000, 7
    pipad.set_option("agg_coalescent", 2)
    pipad.set_option("mid_max", 300)
    pipad.set_option("hub_segment", 700)
    pipad.set_option("hub_threshold", 700)
    lists = power_law(n, 350_000, k, 4)
    snaps = [(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists]
    frame = pipad.frame_build_overlap(snaps, allocator="library")
    x = {F: torch.empty((n, k, F), device="cuda:0").uniform_(-1, 1) for F in (2, 4, 5)}
    shared = [x[5][:, t].contiguous() for t in range(k)]
    lists_out = [torch.empty_like(m) for m in shared]
    pipad.frame_aggregate(frame, shared, lists_out)
    torch.cuda.synchronize()
    recorded = []

    def record(operand, out):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            pipad.frame_aggregate(frame, operand, out)
        recorded.append((graph, out))

    record(shared, lists_out)
    for F in (2, 4, 5):  # the list's scratch is large enough for all of them, their products take more and more
        assert 3 * k * min(len(c) for _, c in lists) > 10_000_000 + k * n * (4 * F + 1)
        out = torch.empty_like(x[F])
        pipad.frame_aggregate(frame, x[F], out)
        torch.cuda.synchronize()
        record(x[F], out)
    fresh = pipad.frame_build_overlap(snaps)
    want = [pipad.frame_aggregate(fresh, shared)] + [pipad.frame_aggregate(fresh, x[F]) for F in (2, 4, 5)]
    for _ in range(2):
        for (graph, out), expected in zip(recorded, want):
            outs, expected = (out, expected) if isinstance(out, list) else ([out], [expected])
            for o in outs:
                o.fill_(float("nan"))
            graph.replay()
            torch.cuda.synchronize()
            assert all(torch.equal(o, e) for o, e in zip(outs, expected))
    frame.close()
    fresh.close()


@pytest.mark.parametrize("hubs,length,classes,F", [(600, 1500, True, 4), (600, 1500, True, 7), (190, 5000, False, 2), (190, 5000, False, 12)])
def test_rows_in_parts_are_finished_in_64_bits(pipad, hubs, length, classes, F):  # noqa: F811
    """Sums without a rounding (scales of 1/2, features of few bits): what is left is the finish of the rows, summed by column class
    or in units, which has to be that of 64 bits rounded once."""
    n, k = 8000, 4
    pipad.set_option("agg_coalescent", 2)
    if classes:
        pipad.set_option("mid_max", 500)
    rng = np.random.default_rng(hubs + F)
    rows = [np.sort(rng.choice(n - hubs, length, replace=False) + hubs) for _ in range(hubs)]
    few = (np.arange(n - hubs)[:, None] + np.arange(1, 4)) % (n - hubs) + hubs  # three entries each: scales of 1/2
    rowptr = np.concatenate([[0], np.cumsum([length] * hubs + [3] * (n - hubs))]).astype(np.int32)
    col = np.concatenate(rows + [np.sort(few, axis=1).ravel()]).astype(np.int32)
    assert 3 * k * len(col) > 10_000_000 + k * n * (4 * F + 1)
    snap = (torch.from_numpy(rowptr).cuda(), torch.from_numpy(col).cuda())
    frame = pipad.frame_build_overlap([snap] * k, validate=True)
    x = torch.from_numpy(rng.integers(-512, 513, (n, k, F)).astype(np.float32) / 512).cuda()
    d = frame.dinv()[0].double().cpu().numpy()
    xd = x.double().cpu().numpy()
    want = np.stack([d[i] * ((d[rows[i], None, None] * xd[rows[i]]).sum(0) + d[i] * xd[i]) for i in range(hubs)]).astype(np.float32)
    y = pipad.frame_aggregate(frame, x)
    assert np.array_equal(y[:hubs].cpu().numpy(), want)
    assert torch.equal(pipad.frame_aggregate(frame, x, static_scratch=True), y)
    frame.close()


def test_calls_without_partial_sums_share_no_scratch(pipad):  # noqa: F811
    """Calls that allocate nothing, side by side on two streams: where no row is summed up in parts there is nothing they share,
    the products among it."""
    n, k, F = 20_000, 4, 4
    pipad.set_option("agg_coalescent", 2)
    rng = np.random.default_rng(11)
    pairs = np.unique(rng.integers(0, n * n, 1_200_000))
    pairs = np.stack([pairs // n, pairs % n], 1)
    pairs = pairs[pairs[:, 0] != pairs[:, 1]]
    counts = np.bincount(pairs[:, 0], minlength=n)
    assert counts.max() <= 500 and 3 * k * len(pairs) > 10_000_000 + k * n * (4 * F + 1)
    snap = (torch.from_numpy(np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)).cuda(),
            torch.from_numpy(pairs[:, 1].astype(np.int32)).cuda())
    frame = pipad.frame_build_overlap([snap] * k, validate=True)
    x = [torch.empty((n, k, F), device="cuda:0").uniform_(-1, 1) for _ in range(2)]
    want = [pipad.frame_aggregate(frame, m) for m in x]
    got = [[torch.full_like(w, float("nan")) for _ in range(20)] for w in want]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    for i in range(20):
        for m, outs, stream in zip(x, got, streams):
            pipad.frame_aggregate(frame, m, outs[i], stream=stream, static_scratch=True)
    torch.cuda.synchronize()
    for outs, w in zip(got, want):
        assert all(torch.equal(y, w) for y in outs)
    frame.close()


def test_products_that_cannot_be_had_are_asked_for_once(pipad):  # noqa: F811
    """Behind the partial sums, which a call cannot do without; then the kernel makes the products itself, with the same bits."""
    import ctypes

    from paper_2301_00391_amd import binding
    n, k = 6000, 7
    pipad.set_option("agg_coalescent", 2)
    pipad.set_option("mid_max", 300)
    lists = power_law(n, 350_000, k, 4)
    snaps = [(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists]
    arr = (binding._Csr * k)()
    for t, (rp, c) in enumerate(snaps):
        arr[t].n, arr[t].nnz, arr[t].rowptr, arr[t].colidx = n, c.numel(), rp.data_ptr(), c.data_ptr()
    kept, requests, refuse = [], [], set()

    def alloc(nbytes, _ctx):
        requests.append(nbytes)
        if len(requests) in refuse:
            return None
        kept.append(torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device="cuda:0"))
        return kept[-1].data_ptr()

    lib, cb, out = pipad.load_library(), binding.ALLOC_FN(alloc), ctypes.c_void_p()
    assert lib.pipad_frame_build_overlap(n, k, arr, 0, ctypes.cast(cb, ctypes.c_void_p), None,
                                         torch.cuda.current_stream().cuda_stream, ctypes.byref(out)) == 0
    frame, usual = binding.Frame(out.value, n, k, snaps[0][0].device, {}), pipad.frame_build_overlap(snaps)
    x = {F: torch.empty((n, k, F), device="cuda:0").uniform_(-1, 1) for F in (2, 5)}
    want = {F: pipad.frame_aggregate(usual, x[F]) for F in x}
    requests.clear()
    refuse.add(2)
    for F, asked in ((5, 2), (5, 2), (5, 2), (2, 3), (2, 3), (5, 3)):  # the sums and the products; nothing; fewer products
        assert 3 * k * min(len(c) for _, c in lists) > 10_000_000 + k * n * (4 * F + 1)
        assert torch.equal(pipad.frame_aggregate(frame, x[F]), want[F])
        assert len(requests) == asked
    assert requests[1] > 4 * n * k * 5 > requests[2] > 4 * n * k * 2
    torch.cuda.synchronize()
    frame.close()
    usual.close()
