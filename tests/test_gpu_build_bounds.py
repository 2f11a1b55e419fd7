"""The tiles' bounds by 8 or 16 lanes each, in builds that find them in a launch of their own."""
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


# the last number of snapshots with 8 lanes, the first with 16, one per lane, more than lanes, two tiles' sizes
@pytest.mark.parametrize("k", [8, 9, 16, 17, 32])
def test_parts_of_a_frame_with_many_tiles(pipad, k):
    n, entries = 40_000, 1_100_000 if k <= 16 else 600_000
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(k)
    pool = torch.randint(0, n * n, (entries + entries // 4,), device="cuda:0", generator=gen)
    pool = torch.unique(pool)
    pool = pool[pool // n != pool % n]
    rows = torch.arange(n + 1, device="cuda:0") * n
    keys, snaps = [], []
    for t in range(k):
        key = pool[torch.rand(pool.numel(), device="cuda:0", generator=gen) < (0.99 if t % 5 else 0.7)]
        keys.append(key)
        snaps.append((torch.searchsorted(key, rows).to(torch.int32), (key % n).to(torch.int32)))
    common = keys[0]
    for key in keys[1:]:
        common = common[torch.isin(common, key)]
    frame = pipad.frame_build_overlap(snaps)
    for t in [None, *range(k)]:
        want = common if t is None else keys[t][~torch.isin(keys[t], common)]
        rowptr, col = frame.common() if t is None else frame.delta(t)
        assert torch.equal(rowptr, torch.searchsorted(want, rows).to(torch.int32)), t
        assert torch.equal(col, (want % n).to(torch.int32)), t
    frame.close()
