"""Frames whose entries' scales are stored as 16-bit codes: the same bits as with floats, wherever they are read."""
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


@pytest.fixture
def option(pipad):
    before = {key: pipad.get_option(key) for key in ("scale_codes", "mid_max", "short_max", "agg_generic")}
    yield pipad.set_option
    for key, value in before.items():
        pipad.set_option(key, value)


def csr(key, n):
    rows = torch.arange(n + 1, device="cuda:0") * n
    return torch.searchsorted(key, rows).to(torch.int32), (key % n).to(torch.int32)


def snapshots(n, entries, k, seed):
    """Directed, some rows long, one empty; most entries in all snapshots."""
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(seed)
    rows = (torch.rand(entries, device="cuda:0", generator=gen) ** 3 * n).long().clamp_(max=n - 2)
    pool = torch.unique(rows * n + torch.randint(0, n, (entries,), device="cuda:0", generator=gen))
    return [csr(pool[torch.rand(pool.numel(), device="cuda:0", generator=gen) < 0.9], n) for _ in range(k)]


def results(pipad, snaps, n, F, wide):
    """What every reader of the scales makes of them: whole calls, a part of the snapshots, the update, the transposed frame."""
    k = len(snaps)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(1)
    shape = (n, k, F) if wide else (k, n, F)
    x = torch.empty(shape, device="cuda:0").uniform_(-1, 1, generator=gen)
    X = x if wide else list(x)

    def fresh():
        return torch.zeros_like(x) if wide else [torch.zeros_like(X[0]) for _ in X]

    frame = pipad.frame_build_overlap(snaps)
    got = [frame.dinv()]
    for f in (frame, pipad.frame_transpose(frame)):
        y = fresh()
        pipad.frame_aggregate(f, X, y)
        got += [y] if wide else y
        if not wide:
            y = fresh()
            pipad.frame_aggregate_subset(f, [k - 1], X, y)
            got.append(y[k - 1])
            w = torch.empty((F, 16), device="cuda:0").uniform_(-1, 1, generator=gen)
            h = [torch.zeros((n, 16), device="cuda:0") for _ in X]
            y = fresh()
            pipad.frame_aggregate_update(f, X, w, None, H=h, A=y)
            got += h + y
        f.close()
    return got


# every instance by number of snapshots; widths of one, two and four columns per lane, one lane to a whole wave per row
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 8, 9, 12, 13, 16, 18])
@pytest.mark.parametrize("F,wide", [(1, False), (6, False), (16, False), (64, False), (100, False), (1, True), (3, True), (12, True)])
def test_same_bits_as_floats(pipad, option, k, F, wide):
    n, entries = 3001, 90_000 if k <= 9 else 40_000
    snaps = snapshots(n, entries, k, k)
    option("mid_max", 100)  # (hub rows with their copies by class in either frame)
    got = []
    for codes in (0, 2):
        option("scale_codes", codes)
        got.append(results(pipad, snaps, n, F, wide))
    for a, b in zip(*got):
        assert torch.equal(a, b)


@pytest.mark.parametrize("F", [3, 64])
def test_generic_kernel(pipad, option, F):
    n = 2000
    snaps = snapshots(n, 60_000, 3, 5)
    option("mid_max", 100)
    option("agg_generic", 1)
    got = []
    for codes in (0, 2):
        option("scale_codes", codes)
        got.append(results(pipad, snaps, n, F, False))
    for a, b in zip(*got):
        assert torch.equal(a, b)


# the longest row that has a code, and rows without one: floats then
@pytest.mark.parametrize("k", [1, 2, 3, 8])
@pytest.mark.parametrize("longest", [65_533, 65_534, 65_535, 70_000])
def test_long_rows(pipad, option, longest, k):
    n, F = 70_001, 4
    hub = torch.arange(1, longest + 1, device="cuda:0")
    few = torch.arange(1, n - 1, device="cuda:0") * n
    snaps = [csr(torch.unique(torch.cat([hub, few + t, few + n - 1])), n) for t in range(k)]
    x = torch.rand((n, F), device="cuda:0")
    got = []
    option("mid_max", 500)
    for codes in (0, 2):
        option("scale_codes", codes)
        frame = pipad.frame_build_overlap(snaps)
        y = [torch.empty_like(x) for _ in range(k)]
        pipad.frame_aggregate(frame, [x] * k, y)
        got.append(y + [frame.dinv()])
        frame.close()
    for a, b in zip(*got):
        assert torch.equal(a, b)


def test_scales_of_all_lengths(pipad, option):
    """D^-1/2 is 1 / sqrt(1 + length) rounded once."""
    n = 70_000
    rng = np.random.default_rng(3)
    length = np.zeros(n, dtype=np.int64)
    length[:4000] = np.arange(4000)
    length[4000:4150] = rng.integers(4000, 65_533, 150)
    length[4150:4155] = [65_532, 65_533, 65_534, 65_535, 69_999]
    length = torch.from_numpy(length).cuda()
    rowptr = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda:0"), length.cumsum(0)])
    col = torch.arange(int(rowptr[-1]), device="cuda:0") - torch.repeat_interleave(rowptr[:-1], length)
    want = (1.0 / (length + 1).double().sqrt()).float()
    for codes in (0, 2):
        option("scale_codes", codes)
        frame = pipad.frame_build_overlap([(rowptr.int(), col.int())])
        assert torch.equal(frame.dinv().reshape(-1), want)
        frame.close()
