"""The transposition's first pass: a wave's share of 256, 512 or 1024 entries spans so many rows that it goes
through them (up to 4096) or searches, with empty rows in front, in between and behind; parts of every
size beside each other; D^-1/2 copied along."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_build_tiles import csr  # noqa: E402
from test_gpu_parity import pipad  # noqa: E402,F401
from test_gpu_transpose_sizes import transposed  # noqa: E402


@pytest.mark.parametrize("n,every,per_row", [(9000, 1, 1), (9000, 7, 3), (9000, 16, 1), (40_000, 17, 2), (40_000, 900, 300),
                                             (600_000, 1200, 1), (600_000, 1, 4), (200_000, 50_000, 5000)])
def test_rows_of_a_share(pipad, n, every, per_row):  # noqa: F811
    rng = np.random.default_rng(n + every)
    rows = np.repeat(np.arange(every // 2, n, every), per_row)
    pairs = np.stack([rows, rng.integers(0, n, len(rows))], 1)
    k = 3
    lists = [csr(n, pairs), csr(n, pairs[rng.random(len(pairs)) < 0.8]), csr(n, pairs[:1])]
    frame = pipad.frame_build_overlap([(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists])
    back = pipad.frame_transpose(frame)
    for part in [None, *range(k)]:
        rp, col = frame.common() if part is None else frame.delta(part)
        key = torch.repeat_interleave(torch.arange(n, device="cuda:0"), torch.diff(rp.long())) * n + col.long()
        want = transposed(n, key)
        got = back.common() if part is None else back.delta(part)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), part
    assert torch.equal(frame.dinv(), back.dinv())


@pytest.mark.parametrize("n", [700, 5000, 65_536, 65_537, 262_144, 262_145])
@pytest.mark.parametrize("entries", [2049, 64 * 2048, 64 * 2048 + 1])
def test_sums_without_a_launch(pipad, n, entries):  # noqa: F811
    """Up to 64 tiles of 2048 entries in a part, and up to 1024 blocks of 256 rows, are added up where they are needed (a
    thread takes a second block from 65,537 rows on)."""
    rng = np.random.default_rng(n + entries)
    keys = np.unique(rng.integers(0, n * n, entries + entries // 2 + 5000))
    keys = np.sort(rng.permutation(keys[keys // n != keys % n])[:entries])
    assert len(keys) == entries
    pairs = np.stack([keys // n, keys % n], 1)
    lists = [csr(n, pairs), csr(n, pairs), csr(n, pairs[rng.random(entries) < 0.999])]
    pipad.set_option("short_max", 3)  # mid rows and, where there are any, hub rows
    pipad.set_option("mid_max", 40)
    try:
        frame = pipad.frame_build_overlap([(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists])
    finally:
        pipad.set_option("short_max", 64)
        pipad.set_option("mid_max", 512)
    back = pipad.frame_transpose(frame)
    for part in [None, 0, 1, 2]:
        rp, col = frame.common() if part is None else frame.delta(part)
        key = torch.repeat_interleave(torch.arange(n, device="cuda:0"), torch.diff(rp.long())) * n + col.long()
        want = transposed(n, key)
        got = back.common() if part is None else back.delta(part)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), part
    X = [torch.empty((n, 8), device="cuda:0").uniform_(-1, 1) for _ in lists]
    Z = pipad.frame_aggregate(back, X)
    d = frame.dinv().double()
    for t, (rp, c) in enumerate(lists):
        x = X[t].double() * d[t][:, None]
        at = torch.from_numpy(np.repeat(np.arange(n), np.diff(rp))).cuda()
        col = torch.from_numpy(c.astype(np.int64)).cuda()
        z = x.clone().index_add_(0, col, x[at]) * d[t][:, None]
        size = x.abs().index_add_(0, col, x.abs()[at]) * d[t][:, None]
        assert bool(((Z[t].double() - z).abs() <= 1e-5 * size).all())
