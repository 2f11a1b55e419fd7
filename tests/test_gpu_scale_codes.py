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


def requests(pipad, snaps):
    """What a build asks its allocator for: bytes, in order; and the entries of the parts."""
    import ctypes
    from paper_2301_00391_amd import binding
    kept, sizes = [], []

    def give(nbytes, _):
        sizes.append(nbytes)
        kept.append(torch.empty(nbytes, dtype=torch.uint8, device="cuda:0"))
        return kept[-1].data_ptr()

    lib, n, k = pipad.load_library(), snaps[0][0].numel() - 1, len(snaps)
    csr_of = (binding._Csr * k)(*[binding._Csr(n, col.numel(), rp.data_ptr(), col.data_ptr()) for rp, col in snaps])
    callback, out = binding.ALLOC_FN(give), ctypes.c_void_p()
    assert lib.pipad_frame_build_overlap(n, k, csr_of, 0, callback, None, torch.cuda.current_stream().cuda_stream, ctypes.byref(out)) == 0
    views = [binding._Csr() for _ in range(k + 1)]
    lib.pipad_frame_common(out, ctypes.byref(views[0]))
    for t in range(k):
        lib.pipad_frame_delta(out, t, ctypes.byref(views[t + 1]))
    torch.cuda.synchronize()
    lib.pipad_frame_destroy(out)
    return sizes, [v.nnz for v in views]


def parts_bytes(nnz, scale):
    """Columns and scales of all parts, and the arrays of no hub rows, each from a multiple of 256 bytes on."""
    k, up = len(nnz) - 1, lambda x: max(x + 255, 256) // 256 * 256
    return (4 + k) * 256 + up(4 * nnz[0]) + k * up(scale * nnz[0]) + sum(up(4 * x) + up(scale * x) for x in nnz[1:])


# codes from 24 million entries in all snapshots on, or 2^23 in one; up to 2^25 entries, and fewer than 2^23 in one, floats get room
# before the sizes are known
@pytest.mark.parametrize("k,entries,codes,room", [(1, 8_300_000, False, True), (1, 9_000_000, True, False), (2, 8_300_000, False, True),
                                                  (2, 8_600_000, True, False), (2, 12_200_000, True, False), (3, 7_900_000, False, True),
                                                  (3, 8_100_000, True, True), (5, 6_000_000, True, True), (4, 8_388_000, True, True),
                                                  (4, 8_500_000, True, False)])
def test_form_of_the_scales(pipad, option, k, entries, codes, room):
    n = 200_000
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(entries)
    keys = torch.unique(torch.randint(0, n * n, (int(1.02 * entries) + 1000,), device="cuda:0", generator=gen))
    keys = keys[torch.randperm(keys.numel(), device="cuda:0", generator=gen)[:entries + k]]
    snaps = [csr(torch.cat([keys[:entries - 1], keys[entries - 1 + t:entries + t]]).sort().values, n) for t in range(k)]
    assert all(c.numel() == entries for _, c in snaps)
    option("mid_max", 1 << 30)  # (no hub rows: nothing else is asked for)
    for setting in (0, 1):
        option("scale_codes", setting)
        sizes, nnz = requests(pipad, snaps)
        coded = setting == 1 and codes
        if room and not coded:
            assert len(sizes) == 2
        else:
            assert len(sizes) == 3 and sizes[2] == parts_bytes(nnz, 2 if coded else 4)


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
@pytest.mark.parametrize("k", [1, 2, 3, 5, 8, 9, 18])
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


def test_scales_of_lengths_past_the_codes(pipad, option):
    """D^-1/2 is 1 / sqrt(1 + length) rounded once, in a frame that keeps floats as well."""
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


@pytest.mark.parametrize("first", range(0, 65_534, 5000))
def test_scale_of_every_code(pipad, option, first):
    """A node of every length that has a code, and a row with an entry for each: what the aggregation makes of the code comes out as
    the scale of the entry's column, bit for bit the one of D^-1/2, through lists of scales and the codes next to the rows."""
    lengths = torch.arange(first, min(first + 5000, 65_534), device="cuda:0")
    m = lengths.numel()
    n = 2 * m + 65_534
    # nodes [0, m): rows with one entry, column m + their number; nodes [m, 2 m): rows of the lengths, whose columns lie behind
    rows = torch.cat([torch.ones(m, dtype=torch.int64, device="cuda:0"), lengths, torch.zeros(n - 2 * m, dtype=torch.int64, device="cuda:0")])
    rowptr = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda:0"), rows.cumsum(0)])
    assert int(rowptr[-1]) < 2 ** 31
    at = torch.arange(int(rowptr[-1]) - m, device="cuda:0") - torch.repeat_interleave(rowptr[m:2 * m] - m, lengths) + 2 * m
    col = torch.cat([m + torch.arange(m, device="cuda:0"), at]).int()
    del at
    snaps = [(rowptr.int(), col)]
    option("scale_codes", 2)
    option("mid_max", 1 << 30)
    sizes, nnz = requests(pipad, snaps)
    assert sizes[2:] == [parts_bytes(nnz, 2)]
    frame = pipad.frame_build_overlap(snaps)
    want = (1.0 / (1 + lengths).double().sqrt()).float()
    dinv = frame.dinv().reshape(-1)
    assert torch.equal(dinv[m:2 * m], want)
    x = torch.zeros((n, 1), device="cuda:0")
    x[m:2 * m] = 1.0
    y = pipad.frame_aggregate(frame, [x])[0].reshape(-1)[:m]
    own = dinv[0]  # of a row of one entry, whose own feature is 0
    assert torch.equal(y, own * want)
    frame.close()
