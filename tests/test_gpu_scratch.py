"""Calls that find a scratch which cannot grow: recorded into a HIP graph, or in the fixed array."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
import synth  # noqa: E402
from _util import check_y, csr_to_coo  # noqa: E402
from test_gpu_parity import pipad, churned, _reset_options  # noqa: E402,F401


def operand(n, k, F, seed, layout):
    x = torch.from_numpy(np.stack([synth.features(seed, t, n, F) for t in range(k)], axis=1)).cuda()
    return x if layout == "wide" else [x[:, t].contiguous() for t in range(k)]


def results(n, k, F, layout):
    if layout == "wide":
        return torch.full((n, k, F), float("nan"), device="cuda:0")
    return [torch.full((n, F), float("nan"), device="cuda:0") for _ in range(k)]


def call(pipad, frame, x, weights, y, h):  # noqa: F811
    if weights is None:
        pipad.frame_aggregate(frame, x, y)
    else:
        pipad.frame_aggregate_update(frame, x, weights, H=h, A=y)


# the call that sizes the scratch, the recorded one (with the update where Fo is given)
@pytest.mark.parametrize("k,sized,recorded,Fo,slice_cols", [
    (3, (9, "list"), (9, "wide"), 0, 0),       # groups of snapshots with idle lanes
    (21, (3, "list"), (3, "wide"), 0, 0),
    (12, (6, "wide"), (5, "wide"), 0, 0),      # the narrower call has the wider teams
    (8, (9, "wide"), (9, "list"), 0, 0),       # rows padded to the slice: several launches
    (5, (20, "wide"), (20, "list"), 24, 0),    # ... and the update behind the last of them
    (5, (20, "wide"), (20, "list"), 32, 0),    # ... and fused in
    (1, (36, "list"), (36, "list"), 16, 4),    # slices narrower than those of the fused update
])
def test_recorded_after_another_form_has_sized_the_scratch(pipad, k, sized, recorded, Fo, slice_cols):  # noqa: F811
    n = 700
    for key, value in (("short_max", 2), ("mid_max", 5), ("hub_threshold", 16), ("hub_segment", 8),
                       ("agg_coalescent", 2), ("slice_cols", slice_cols)):
        pipad.set_option(key, value)
    lists = churned(np.random.default_rng(k), n, k, 0.03, 0.8)
    snaps = [(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists]
    frame, other = pipad.frame_build_overlap(snaps), pipad.frame_build_overlap(snaps)
    pipad.frame_aggregate(frame, operand(n, k, sized[0], 1, sized[1]))
    F, layout = recorded
    x, y = operand(n, k, F, 2, layout), results(n, k, F, layout)
    W = torch.randn((F, Fo), device="cuda:0") if Fo else None
    h = results(n, k, Fo, "list") if Fo else None
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(pipad, frame, x, W, y, h)
    for replay in range(3):
        fresh = operand(n, k, F, 10 + replay, layout)
        for t in range(k):
            (x[:, t] if layout == "wide" else x[t]).copy_(fresh[:, t] if layout == "wide" else fresh[t])
        want, want_h = results(n, k, F, layout), results(n, k, Fo, "list") if Fo else []
        call(pipad, other, x, W, want, want_h)
        torch.cuda.synchronize()
        for out in [*y, *(h or [])]:
            out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for got, expected in zip([*y, *(h or [])], [*want, *want_h]):
            assert torch.equal(got, expected), f"replay {replay}"
    rows, cols = csr_to_coo(n, *lists[k - 1])
    _, yd, bound, _ = oracle.aggregate(n, rows, cols, synth.features(12, k - 1, n, F), threads=4)
    check_y((y[:, k - 1] if layout == "wide" else y[k - 1]).cpu().numpy(), yd, bound, "last snapshot")
    frame.close()
    other.close()


@pytest.mark.parametrize("layout", ["list", "wide"])
def test_recorded_with_more_columns_than_any_eager_call(pipad, layout):  # noqa: F811
    """Refused with nothing enqueued; the recording goes on."""
    n, k = 500, 3
    for key, value in (("short_max", 2), ("mid_max", 5), ("agg_coalescent", 2)):
        pipad.set_option(key, value)
    lists = churned(np.random.default_rng(8), n, k, 0.03, 0.8)
    frame = pipad.frame_build_overlap([(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists])
    x, y = operand(n, k, 8, 1, layout), results(n, k, 8, layout)
    wider, y_wider = operand(n, k, 17, 1, layout), results(n, k, 17, layout)
    want = pipad.frame_aggregate(frame, x)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        with pytest.raises(pipad.PipadError) as info:
            pipad.frame_aggregate(frame, wider, y_wider)
        pipad.frame_aggregate(frame, x, y)
    assert info.value.status == -6
    graph.replay()
    torch.cuda.synchronize()
    for t in range(k):
        assert torch.equal(*((a[:, t] if layout == "wide" else a[t]) for a in (y, want)))
    assert all(torch.isnan(out).all() for out in y_wider)
    frame.close()


@pytest.mark.parametrize("k,F,rows", [(12, 9, 100_000), (21, 3, 150_000)])
def test_fixed_array_and_many_units_on_the_concatenated_operand(pipad, k, F, rows):  # noqa: F811
    """Every row a unit: no room for the class parts, and room for one sum per unit only without the
    idle lanes of the snapshots' teams."""
    pipad.set_option("short_max", 0)
    pipad.set_option("mid_max", 0)
    ahead = (np.arange(rows, dtype=np.int64)[:, None] + [1, 2, 7]) % rows
    lists = []
    for t in range(k):
        keep = np.ones((rows, 3), dtype=bool)
        keep[t::k, 2] = False
        cols = np.sort(np.where(keep, ahead, rows), axis=1)
        lists.append((np.concatenate([[0], np.cumsum(keep.sum(axis=1))]).astype(np.int32),
                      cols[cols < rows].astype(np.int32)))
    assert rows * 8 * k * F * 4 > 64 << 20 >= rows * k * F * 4
    frame = pipad.frame_build_overlap([(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists])
    x = operand(rows, k, F, 4, "wide")
    y = pipad.frame_aggregate(frame, x, static_scratch=True)
    assert torch.equal(y, pipad.frame_aggregate(frame, x))
    for t in (0, k - 1):
        r, c = csr_to_coo(rows, *lists[t])
        _, yd, bound, _ = oracle.aggregate(rows, r, c, synth.features(4, t, rows, F), threads=8)
        check_y(y[:, t].cpu().numpy(), yd, bound, f"snapshot {t}")
    frame.close()


def test_scratch_taken_under_another_stream(pipad):  # noqa: F811
    """PyTorch's allocator may give memory out again, in the order of the stream it was asked for under, as soon as the frame is
    closed: the frame's own stream must be done with it by then."""
    rng = np.random.default_rng(7)
    n, k = 500, 3
    pipad.set_option("short_max", 2)
    pipad.set_option("mid_max", 4)
    pipad.set_option("hub_threshold", 6)  # rows in several parts: the first aggregation asks for scratch
    pipad.set_option("hub_segment", 4)
    snaps = [(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in churned(rng, n, k, 0.05, 0.8)]
    X = [torch.empty((n, 8), device="cuda:0").uniform_(-1, 1) for _ in range(k)]
    own, other = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    for first, then in ((own, other), (torch.cuda.default_stream(), other)):
        with torch.cuda.stream(first):
            frame = pipad.frame_build_overlap(snaps)
        first.synchronize()
        with torch.cuda.stream(then):
            want = pipad.frame_aggregate(frame, X)
        then.synchronize()
        with torch.cuda.stream(first):
            torch.cuda._sleep(20_000_000)
            got = pipad.frame_aggregate(frame, X)
        frame.close()
        assert first.query()
        assert all(torch.equal(a, b) for a, b in zip(got, want))
