"""Frames that are built in two launches (a tile finds its bounds itself, rows and entries are made in one kernel), at the
edges of that form's range and of its searches."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_build_tiles import csr  # noqa: E402
from test_gpu_parity import pipad, run_case  # noqa: E402,F401


# 2048 tiles of 512 entries, 262,144 rows and 20,000 waves are the last ones (k > 16: tiles of 256 entries)
@pytest.mark.parametrize("n,tiles,over,k", [(3000, 2048, 0, 2), (3000, 2048, 1, 2), (262_144, 500, 0, 2), (262_145, 500, 0, 2),
                                            (2000, 1250, 0, 16), (2000, 1250, 1, 16), (1500, 1176, 0, 17), (1500, 1176, 1, 17),
                                            (700, 0, 1, 1), (300, 0, 0, 3)])
def test_edges(pipad, n, tiles, over, k):  # noqa: F811
    rng = np.random.default_rng(n + tiles + k)
    entries = tiles * (512 if k <= 16 else 256) + over
    keys = np.unique(rng.integers(0, n * n, 2 * entries + 4000))
    keys = keys[keys // n != keys % n]
    keys = np.sort(rng.permutation(keys)[:entries])
    assert len(keys) == entries
    pairs = np.stack([keys // n, keys % n], 1)
    run_case(pipad, n, [csr(n, pairs)] + [csr(n, pairs[rng.random(len(pairs)) < 0.9]) for _ in range(k - 1)], 3, seed=k)


# A tile starts in a long row; the other snapshot has so many entries of that row, all of them in front of the tile's first
# column, or all behind it (the search looks at 32 places at a time).
@pytest.mark.parametrize("behind", [False, True])
@pytest.mark.parametrize("length", [0, 1, 31, 32, 33, 34, 65, 66, 99, 1055, 1056, 1088, 1089, 1090, 1122])
def test_row_lengths(pipad, length, behind):  # noqa: F811
    def row(i, first, count):
        return np.stack([np.full(count, i), np.arange(first, first + count)], 1)

    n = 6000
    lead, rest = row(2, 700, 16), row(9, 100, 40)
    base = np.concatenate([lead, row(5, 2500, 800), rest, row(11, 12, 600)])  # the second tile starts at (5, 2996)
    other = np.concatenate([lead[::2], row(5, 3000 if behind else 2996 - length, length), rest[1::2]])
    run_case(pipad, n, [csr(n, base), csr(n, other)], 4, seed=length)


@pytest.mark.parametrize("entries", [3000, 600_000, 2048 * 512 + 1])
@pytest.mark.parametrize("which", ["largest", "another"])
def test_column_twice(pipad, entries, which):  # noqa: F811
    """Noticed without validation, with nothing written past the room of the parts, which is there before the sizes are known."""
    import ctypes

    from paper_2301_00391_amd import binding
    n = 3000
    rng = np.random.default_rng(entries)
    keys = np.unique(rng.integers(0, n * n, 2 * entries + 4000))
    keys = keys[keys // n != keys % n]
    keys = np.sort(rng.permutation(keys)[:entries])
    pairs = np.stack([keys // n, keys % n], 1)
    good, fewer = csr(n, pairs), csr(n, pairs[:-1])
    rowptr, col = good if which == "largest" else fewer
    at = int(rowptr[np.flatnonzero(np.diff(rowptr) > 1)[len(rowptr) // 9]])
    bad = rowptr, np.concatenate([col[:at + 1], col[at:at + 1], col[at + 2:]])
    lists = [bad, fewer, fewer] if which == "largest" else [fewer, bad, good]
    snaps = [(torch.from_numpy(rp).cuda(), torch.from_numpy(c.astype(np.int32)).cuda()) for rp, c in lists]
    arr = (binding._Csr * len(snaps))()
    for t, (rp, c) in enumerate(snaps):
        arr[t].n, arr[t].nnz, arr[t].rowptr, arr[t].colidx = n, c.numel(), rp.data_ptr(), c.data_ptr()
    kept, guard = [], 4096

    def alloc(nbytes, _ctx):
        kept.append(torch.full((int(nbytes) + guard,), 0x5a, dtype=torch.uint8, device="cuda:0"))
        return kept[-1].data_ptr()

    cb, out = binding.ALLOC_FN(alloc), ctypes.c_void_p()
    status = pipad.load_library().pipad_frame_build_overlap(n, len(snaps), arr, 0, ctypes.cast(cb, ctypes.c_void_p), None,
                                                            torch.cuda.current_stream().cuda_stream, ctypes.byref(out))
    assert status == -2 and out.value is None
    torch.cuda.synchronize()
    for buf in kept:
        assert bool((buf[-guard:] == 0x5a).all())


@pytest.mark.parametrize("n,edges,k,requests", [(500, 3000, 3, 1), (60_000, 300_000, 2, 1), (60_000, 900_000, 2, 2), (70_000, 300_000, 2, 2)])
def test_temporaries_in_one_request(pipad, n, edges, k, requests):  # noqa: F811
    """Small frames and their transposes, with nothing to hand back, and frames past either line."""
    import ctypes

    from paper_2301_00391_amd import binding
    rng = np.random.default_rng(n + edges)
    lists = []
    for _ in range(k):
        keys = np.unique(rng.integers(0, n * n, edges))
        keys = keys[keys // n != keys % n]
        lists.append(csr(n, np.stack([keys // n, keys % n], 1)))
    snaps = [(torch.from_numpy(rp).cuda(), torch.from_numpy(c.astype(np.int32)).cuda()) for rp, c in lists]
    arr = (binding._Csr * k)()
    for t, (rp, c) in enumerate(snaps):
        arr[t].n, arr[t].nnz, arr[t].rowptr, arr[t].colidx = n, c.numel(), rp.data_ptr(), c.data_ptr()
    kept = []

    def alloc(nbytes, _ctx):
        kept.append(torch.full((int(nbytes),), 0x5a, dtype=torch.uint8, device="cuda:0"))
        return kept[-1].data_ptr()

    lib, cb = pipad.load_library(), binding.ALLOC_FN(alloc)
    stream = torch.cuda.current_stream().cuda_stream
    made = []
    for back in (False, True):
        out, ptr, size = ctypes.c_void_p(), ctypes.c_void_p(), ctypes.c_size_t(1)
        before = len(kept)
        ctx = (ctypes.cast(cb, ctypes.c_void_p), None, stream, ctypes.byref(out))
        assert (lib.pipad_frame_transpose(made[0], *ctx) if back else lib.pipad_frame_build_overlap(n, k, arr, 0, *ctx)) == 0
        made.append(out)
        assert len(kept) - before == requests
        assert lib.pipad_frame_temporaries(out, ctypes.byref(ptr), ctypes.byref(size)) == 0
        assert bool(ptr.value) == (requests > 1) and bool(size.value) == (requests > 1)
    torch.cuda.synchronize()
    for h in made:
        lib.pipad_frame_destroy(h)
    run_case(pipad, n, lists, 4, seed=n)


@pytest.mark.parametrize("n,entries,k,kept", [(3000, 1_000_000, 2, 0.95), (3000, 1_300_000, 4, 0.95), (3000, 1_300_000, 5, 0.3), (40_000, 1_300_000, 8, 0.99),
                                              (3000, 700_000, 17, 0.99), (5000, 1_200_000, 1, 1.0)])
def test_room_for_parts(pipad, n, entries, k, kept):  # noqa: F811
    """What a frame holds whose parts are written before their sizes are known: less than 4 bytes per input entry more than they
    need, and all of it there (the last one of every part as well)."""
    import ctypes

    from paper_2301_00391_amd import binding
    rng = np.random.default_rng(n + k)
    keys = np.unique(rng.integers(0, n * n, entries + entries // 4))
    keys = np.sort(rng.permutation(keys[keys // n != keys % n])[:entries])
    pairs = np.stack([keys // n, keys % n], 1)
    lists = [csr(n, pairs[rng.random(len(pairs)) <= kept]) for _ in range(k)]
    snaps = [(torch.from_numpy(rp).cuda(), torch.from_numpy(c.astype(np.int32)).cuda()) for rp, c in lists]
    arr = (binding._Csr * k)()
    for t, (rp, c) in enumerate(snaps):
        arr[t].n, arr[t].nnz, arr[t].rowptr, arr[t].colidx = n, c.numel(), rp.data_ptr(), c.data_ptr()
    buffers, guard = [], 4096

    def alloc(nbytes, _ctx):
        buffers.append((int(nbytes), torch.full((int(nbytes) + guard,), 0x5a, dtype=torch.uint8, device="cuda:0")))
        return buffers[-1][1].data_ptr()

    lib, cb, out = pipad.load_library(), binding.ALLOC_FN(alloc), ctypes.c_void_p()
    pipad.set_option("mid_max", 1 << 20)  # no copies of long rows
    assert lib.pipad_frame_build_overlap(n, k, arr, 0, ctypes.cast(cb, ctypes.c_void_p), None,
                                         torch.cuda.current_stream().cuda_stream, ctypes.byref(out)) == 0
    pipad.set_option("mid_max", 512)
    ptr, size = ctypes.c_void_p(), ctypes.c_size_t()
    assert lib.pipad_frame_temporaries(out, ctypes.byref(ptr), ctypes.byref(size)) == 0 and ptr.value
    held = sum(b for b, _ in buffers) - size.value
    torch.cuda.synchronize()
    for b, buf in buffers:
        assert bool((buf[b:] == 0x5a).all())
    frame = binding.Frame(out.value, n, k, snaps[0][0].device, {})
    common = frame.common()[1].numel()
    assert common >= 100
    total = sum(c.numel() for _, c in snaps)
    parts = 4 * common * (1 + k) + 8 * (total - k * common)
    nodes = 4 * n * (3 * k + 8) + 65_536  # row pointers, scales, row lists
    assert parts <= held < parts + 4 * total + nodes
    assert held < 2 * parts + nodes
    x = [torch.empty((n, 4), device="cuda:0").uniform_(-1, 1) for _ in range(k)]
    want = pipad.frame_build_overlap(snaps)
    for t in [None, *range(k)]:
        for a, b in zip(frame.common() if t is None else frame.delta(t), want.common() if t is None else want.delta(t)):
            assert torch.equal(a, b), t
    dinv = want.dinv().double()
    for t, (a, (rp, c)) in enumerate(zip(pipad.frame_aggregate(frame, x), snaps)):
        row = torch.repeat_interleave(torch.arange(n, device="cuda:0"), torch.diff(rp.long()))
        scaled = x[t].double() * dinv[t][:, None]
        full = scaled.clone().index_add_(0, row, scaled[c.long()]) * dinv[t][:, None]
        size_of = scaled.abs().index_add_(0, row, scaled.abs()[c.long()]) * dinv[t][:, None]
        assert bool(((a.double() - full).abs() <= 1e-5 * size_of).all()), t
    frame.close()
    want.close()
