"""The native half of the binding: the results of the long way, whose business whatever is not a plain argument stays."""
import ctypes

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def pipad():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2301_00391_amd as p
    p.load_library()
    return p


class Long:
    """Stands in for the native half: what it makes is None, but for the memory."""

    def __init__(self, host):
        self.Buffers, self.ALLOCATE = host.Buffers, host.ALLOCATE
        self.build = self.transpose = self.aggregate = self.subset = self.update = lambda *args: None


class Seen:
    """The native half, and what it made of its calls."""

    def __init__(self, host):
        self.Buffers, self.ALLOCATE, self.made = host.Buffers, host.ALLOCATE, []
        for name in ("build", "transpose", "aggregate", "subset", "update"):
            setattr(self, name, lambda *args, fn=getattr(host, name): self.made.append(fn(*args)) or self.made[-1])


def graph(n, k, seed):
    rng = np.random.default_rng(seed)
    got = []
    for _ in range(k):
        a = np.triu(rng.random((n, n)) < 0.1, 1)
        a = a | a.T
        got.append((torch.from_numpy(np.concatenate([[0], a.sum(1).cumsum()]).astype(np.int32)).cuda(),
                    torch.from_numpy(np.nonzero(a)[1].astype(np.int32)).cuda()))
    return got


@pytest.mark.parametrize("n,k", [(1, 1), (40, 1), (40, 3), (301, 16), (60, 32)])
@pytest.mark.parametrize("layout", ["list", "tuple", "padded", "wide", "wide padded", "one column"])
def test_same_results_both_ways(pipad, monkeypatch, n, k, layout):
    from paper_2301_00391_amd import binding
    F = 1 if layout == "one column" else 12
    gen = torch.Generator(device="cuda").manual_seed(n + k)

    def matrices(cols, fill=True):
        if layout.startswith("wide"):
            x = torch.zeros((n, k, cols + (4 if layout == "wide padded" else 0)), device="cuda")
            return x.uniform_(-1, 1, generator=gen)[:, :, :cols] if fill else x[:, :, :cols]
        got = [torch.zeros((n, cols + (4 if layout == "padded" else 0)), device="cuda") for _ in range(k)]
        got = [(x.uniform_(-1, 1, generator=gen) if fill else x)[:, :cols] for x in got]
        return tuple(got) if layout == "tuple" else got

    snaps, X, W, bias = graph(n, k, n * k), matrices(F), torch.randn((F, 8), device="cuda"), torch.randn(8, device="cuda")
    results = []
    host = binding._host
    for half in (Seen(host), Long(host), None):  # (None: it could not be loaded)
        monkeypatch.setattr(binding, "_host", half)
        Y, Z, A, H = matrices(F, False), matrices(F, False), matrices(F, False), matrices(8, False)
        frame = pipad.frame_build_overlap(snaps, validate=True)
        pipad.frame_aggregate(frame, X, Y)
        pipad.frame_aggregate(frame, X, Z, static_scratch=True)
        pipad.frame_aggregate_update(frame, X, W, bias, H=H, A=A)
        mats = [Y, Z, A, H]
        if not layout.startswith("wide"):
            some = matrices(F, False)
            pipad.frame_aggregate_subset(frame, [k - 1], X, some)
            mats.append(some)
        back = pipad.frame_transpose(frame)
        results.append([frame.common(), back.common(), *[m if isinstance(m, torch.Tensor) else torch.stack(list(m)) for m in mats]])
        if isinstance(half, Seen):
            assert len(half.made) == 1 + len(mats) and None not in half.made
            assert all(m == 0 if isinstance(m, int) else m[0] == 0 for m in half.made)
        back.close()
        frame.close()
    for other in results[1:]:
        for a, b in zip(results[0], other):
            assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]) if isinstance(a, tuple) else torch.equal(a, b)


def test_what_is_not_plain_goes_the_long_way(pipad, monkeypatch):
    from paper_2301_00391_amd import binding
    n, k, F = 50, 3, 8
    snaps = graph(n, k, 5)
    X = [torch.randn((n, F), device="cuda") for _ in range(k)]
    Y = [torch.empty_like(x) for x in X]

    class Sub(torch.Tensor):
        pass

    seen = Seen(binding._host)
    monkeypatch.setattr(binding, "_host", seen)
    frame = pipad.frame_build_overlap(snaps)
    pipad.frame_aggregate(frame, X, Y)
    want = torch.stack(Y)
    W = torch.randn((F, 4), device="cuda")
    H = [torch.empty((n, 4), device="cuda") for _ in range(k)]
    half = [x.half() for x in X]
    for call, error in [
            (lambda: pipad.frame_build_overlap(s for s in snaps), TypeError),
            (lambda: pipad.frame_build_overlap([(rp.long(), c) for rp, c in snaps]), ValueError),
            (lambda: pipad.frame_build_overlap([(rp, c.cpu()) for rp, c in snaps]), ValueError),
            (lambda: pipad.frame_aggregate(frame, X[:2], Y), ValueError),
            (lambda: pipad.frame_aggregate(frame, X, Y[:2]), ValueError),
            (lambda: pipad.frame_aggregate(frame, half, Y), ValueError),
            (lambda: pipad.frame_aggregate(frame, [x.cpu() for x in X], Y), ValueError),
            (lambda: pipad.frame_aggregate(frame, [x.t() for x in X], Y), ValueError),
            (lambda: pipad.frame_aggregate(frame, [x[:-1] for x in X], Y), ValueError),
            (lambda: pipad.frame_aggregate(frame, [x[:, ::2] for x in X], [y[:, :4] for y in Y]), ValueError),
            (lambda: pipad.frame_aggregate(frame, X, [y[:, :4] for y in Y]), ValueError),
            (lambda: pipad.frame_aggregate(frame, [X[0], X[1], torch.randn((n, F + 4), device="cuda")[:, :F]], Y), ValueError),
            (lambda: pipad.frame_aggregate_subset(frame, [0], X[:2], Y), ValueError),
            (lambda: pipad.frame_aggregate_subset(frame, [1], [X[0], None, X[2]], Y), ValueError),
            (lambda: pipad.frame_aggregate_subset(frame, [1, 1], X, Y), pipad.PipadError),
            (lambda: pipad.frame_aggregate_update(frame, X, W[:-1], H=H), ValueError),
            (lambda: pipad.frame_aggregate_update(frame, X, W.t().contiguous().t(), H=H), ValueError),
            (lambda: pipad.frame_aggregate_update(frame, X, W, torch.randn(5, device="cuda"), H=H, A=Y), ValueError),
            (lambda: pipad.frame_aggregate_update(frame, X, W, H=Y, A=Y), ValueError)]:
        with pytest.raises(error):
            call()
    for other in ([x.as_subclass(Sub) for x in X], iter(X), [torch.nn.Parameter(x) for x in X]):
        for y in Y:
            y.fill_(float("nan"))
        pipad.frame_aggregate(frame, other, Y)
        assert torch.equal(torch.stack(Y), want)
    assert torch.equal(torch.stack(pipad.frame_aggregate(frame, X)), want)
    frame.close()
    for call in (lambda: pipad.frame_aggregate(frame, X, Y), lambda: pipad.frame_transpose(frame)):
        with pytest.raises(pipad.PipadError):
            call()


def test_memory_without_the_native_half(pipad, monkeypatch):
    """Taken from torch's allocator and given back with the frame; more than there is ends the build with an error."""
    from paper_2301_00391_amd import binding
    monkeypatch.setattr(binding, "_host", None)
    graphs, before = graph(200, 4, 1), torch.cuda.memory_allocated()
    pipad.set_option("mid_max", 8)  # (rows in parts: scratch for the aggregation)
    try:
        frame = pipad.frame_build_overlap(graphs)
    finally:
        pipad.set_option("mid_max", 512)
    built = torch.cuda.memory_allocated()
    x = [torch.ones((200, 8), device="cuda") for _ in range(4)]
    y = [torch.empty_like(m) for m in x]
    pipad.frame_aggregate(frame, x, y)
    assert before < built and torch.cuda.memory_allocated() > built and len(frame._buffers) >= 2
    frame.close()
    del frame, x, y
    assert torch.cuda.memory_allocated() == before and not binding._owners
    monkeypatch.setattr(binding.torch, "empty", lambda *a, **b: (_ for _ in ()).throw(RuntimeError("no memory")))
    with pytest.raises(pipad.PipadError):
        pipad.frame_build_overlap(graphs)
    monkeypatch.undo()
    assert torch.cuda.memory_allocated() == before and not binding._owners


def test_memory_of_a_frame(pipad):
    """In one piece for a small frame, given back with it; scratch that a call asks for lies with it; none left at the end."""
    from paper_2301_00391_amd import binding
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    frame = pipad.frame_build_overlap(graph(200, 4, 1))
    assert len(frame._buffers) == 1 and torch.cuda.memory_allocated() > before
    frame.close()
    assert len(frame._buffers) == 0
    buffers = binding._host.Buffers()
    allocate = binding.ALLOC_FN(binding._host.ALLOCATE)
    at = [allocate(size, buffers.context()) for size in (0, 1000, 1 << 20)]
    assert len(buffers) == 3 and len(set(at)) == 3 and not any(p % 256 for p in at)
    assert allocate(1 << 60, buffers.context()) is None and len(buffers) == 3
    buffers.pop(at[1], None)
    buffers.pop(at[1], None)
    assert len(buffers) == 2
    buffers.clear()
    assert len(buffers) == 0
    assert torch.cuda.memory_allocated() <= before
