"""A build that fails gives its memory back at once, so nothing of it may still be running when it returns; one that gets no room
for what its parts can hold at most is made with what they do hold."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_build_tiles import csr  # noqa: E402
from test_gpu_parity import pipad, churned, _reset_options  # noqa: E402,F401


def descriptors(binding, lists):
    snaps = [(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists]
    arr = (binding._Csr * len(snaps))()
    for t, (rp, col) in enumerate(snaps):
        arr[t].n, arr[t].nnz, arr[t].rowptr, arr[t].colidx = rp.numel() - 1, col.numel(), rp.data_ptr(), col.data_ptr()
    return arr, snaps


def allocator(binding, kept, refuse_at, stream):
    """Serves all requests but number `refuse_at`, before which it puts 10 ms of work on the stream."""
    def alloc(nbytes, _ctx):
        if len(kept) + 1 == refuse_at:
            with torch.cuda.stream(stream):
                torch.cuda._sleep(20_000_000)
            return None
        kept.append(torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device="cuda:0"))
        return kept[-1].data_ptr()
    return binding.ALLOC_FN(alloc)


def test_out_of_memory_behind_the_first_kernels(pipad):  # noqa: F811
    from paper_2301_00391_amd import binding
    lib = pipad.load_library()
    n, k = 300, 3
    pipad.set_option("short_max", 2)
    pipad.set_option("mid_max", 4)
    arr, _snaps = descriptors(binding, churned(np.random.default_rng(3), n, k, 0.05, 0.8))
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    frame = ctypes.c_void_p()
    assert lib.pipad_frame_build_overlap(n, k, arr, 0, None, None, side.cuda_stream, ctypes.byref(frame)) == 0
    calls = {"build": lambda cb, out: lib.pipad_frame_build_overlap(n, k, arr, 0, cb, None, side.cuda_stream, out),
             "transpose": lambda cb, out: lib.pipad_frame_transpose(frame, cb, None, side.cuda_stream, out)}
    for name, call in calls.items():
        kept, out = [], ctypes.c_void_p()
        cb = allocator(binding, kept, 3, side)  # the request for what is sized by the data
        assert call(ctypes.cast(cb, ctypes.c_void_p), ctypes.byref(out)) == -3, name
        assert side.query(), f"{name}: work is left on the stream"
        assert out.value is None and len(kept) == 2
    lib.pipad_frame_destroy(frame)


def test_snapshots_that_turn_out_not_to_be_canonical(pipad):  # noqa: F811
    """A column twice in a row of the largest snapshot: noticed without validation, while the kernel
    behind the sizes has the row pointers of two million rows to write."""
    n, k = 2_000_000, 4
    rowptr = torch.zeros(n + 1, dtype=torch.int32, device="cuda:0")
    rowptr[1:] = 2
    good = torch.tensor([5, 9], dtype=torch.int32, device="cuda:0")
    longer = rowptr.clone()
    longer[1:] = 3
    twice = torch.tensor([5, 9, 9], dtype=torch.int32, device="cuda:0")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with pytest.raises(pipad.PipadError) as info:
        pipad.frame_build_overlap([(rowptr, good)] * (k - 1) + [(longer, twice)], stream=side)
    assert info.value.status == -2
    assert side.query(), "work is left on the stream"


# in one request with the temporaries; two launches, requests of their own; two launches, k > 16; entries behind a scan, for every
# instance that writes them
@pytest.mark.parametrize("n,entries,k,refused", [(5000, 200_000, 3, 1), (60_000, 1_000_000, 2, 2), (3000, 50_000, 17, 1),
                                                 (70_000, 1_300_000, 1, 2), (70_000, 1_300_000, 2, 2), (70_000, 1_300_000, 3, 2),
                                                 (70_000, 1_300_000, 4, 2), (70_000, 1_300_000, 5, 2), (70_000, 1_300_000, 8, 2),
                                                 (70_000, 600_000, 17, 2)])
def test_room_refused(pipad, n, entries, k, refused):  # noqa: F811
    from paper_2301_00391_amd import binding
    lib = pipad.load_library()
    rng = np.random.default_rng(n + k)
    keys = np.unique(rng.integers(0, n * n, entries + entries // 8))
    keys = np.sort(rng.permutation(keys[keys // n != keys % n])[:entries])
    pairs = np.stack([keys // n, keys % n], 1)
    arr, snaps = descriptors(binding, [csr(n, pairs[rng.random(len(pairs)) < 0.9]) for _ in range(k)])
    stream = torch.cuda.current_stream()
    want = pipad.frame_build_overlap(snaps)
    x = [torch.empty((n, 8), device="cuda:0").uniform_(-1, 1) for _ in range(k)]
    kept, sizes, refuse = [], [], {refused}

    def alloc(nbytes, _ctx):
        sizes.append(nbytes)
        if len(sizes) in refuse:
            return None
        kept.append(torch.full((max(int(nbytes), 256),), 0x5a, dtype=torch.uint8, device="cuda:0"))
        return kept[-1].data_ptr()

    cb, out = binding.ALLOC_FN(alloc), ctypes.c_void_p()

    def build():
        return lib.pipad_frame_build_overlap(n, k, arr, 0, ctypes.cast(cb, ctypes.c_void_p), None, stream.cuda_stream, ctypes.byref(out))

    assert build() == 0
    again = refused + 1
    assert sizes[2] < sizes[refused - 1]
    frame = binding.Frame(out.value, n, k, want.device, {})
    for t in [None, *range(k)]:
        for a, b in zip(frame.common() if t is None else frame.delta(t), want.common() if t is None else want.delta(t)):
            assert torch.equal(a, b), t
    for a, b in zip(pipad.frame_aggregate(frame, x), pipad.frame_aggregate(want, x)):
        assert torch.equal(a, b)
    torch.cuda.synchronize()
    frame.close()
    want.close()
    sizes.clear()
    out.value = None
    refuse.add(again)
    assert build() == -3 and out.value is None
