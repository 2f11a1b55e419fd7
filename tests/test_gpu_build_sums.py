"""Frames at the edges of what k_rows_scatter adds up itself: 2048 tiles of the base (512 entries each, 256 with more than 16
snapshots), 1024 blocks of rows and 20,000 waves of tiles; hub rows, whose places depend on the sums, among them, and sizes at which
the lanes that add up take one more tile or block each."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from _util import check_overlap, check_y, csr_to_coo  # noqa: E402
from test_gpu_build_tiles import csr, head  # noqa: E402
from test_gpu_parity import pipad, _reset_options  # noqa: E402,F401


@pytest.mark.parametrize("n,tiles,over,k", [(3000, 3, 1, 2), (5000, 1024, 0, 2), (5000, 1024, 1, 2), (65_536, 700, 0, 3),
                                            (65_537, 700, 0, 3), (4000, 1024, 0, 17), (4000, 1024, 1, 17),
                                            (5000, 2048, 0, 2), (5000, 2048, 1, 2), (262_144, 700, 0, 3), (262_145, 700, 0, 3),
                                            (4000, 1176, 0, 17), (4000, 1176, 1, 17), (5000, 1250, 0, 16), (5000, 1250, 1, 16)])
def test_edges(pipad, n, tiles, over, k):  # noqa: F811
    rng = np.random.default_rng(n + tiles + over)
    entries = tiles * (512 if k <= 16 else 256) + over
    hubs = np.concatenate([r * n + rng.permutation(n)[:2500] for r in (3, n // 2, n - 1)])
    keys = np.unique(np.concatenate([hubs, rng.integers(0, n * n, 2 * entries + 20_000)]))
    keys = keys[keys // n != keys % n]
    drop = rng.permutation(len(keys))[:max(len(keys) - entries, 0)]
    keys = np.delete(keys, drop)[:entries]
    base = csr(n, np.stack([keys // n, keys % n], 1))
    assert len(base[1]) == min(entries, len(keys))
    lists = [base] + [csr(n, np.stack([keys // n, keys % n], 1)[rng.random(len(keys)) < 0.9]) for _ in range(k - 1)]
    lists[1] = head(n, *lists[1], 1000) if k == 3 else lists[1]
    pipad.set_option("short_max", 8)
    pipad.set_option("mid_max", 300)  # class-grouped copies of longer rows
    snaps = [(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists]
    frame = pipad.frame_build_overlap(snaps, validate=True)
    coo = [csr_to_coo(n, *part) for part in lists]
    check_overlap(frame, oracle.overlap(n, coo))
    X = [torch.empty((n, 8), device="cuda:0").uniform_(-1, 1) for _ in range(k)]
    Y = pipad.frame_aggregate(frame, X)
    for t in (0, k - 1):
        _, yd, bound, _ = oracle.aggregate(n, *coo[t], X[t].cpu().numpy(), threads=8)
        check_y(Y[t].cpu().numpy(), yd, bound, f"snapshot {t}")
