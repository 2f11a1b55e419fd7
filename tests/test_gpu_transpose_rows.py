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
