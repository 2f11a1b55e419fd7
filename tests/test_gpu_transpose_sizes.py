"""pipad_frame_transpose at the sizes where its sort changes: number of digits, length of the tiles."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_parity import pipad  # noqa: E402,F401


def random_csr(n, nnz, seed):
    """A random directed pattern on the GPU, made and transposed with torch."""
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(seed)
    key = torch.unique(torch.randint(0, n * n, (nnz,), device="cuda:0", generator=gen))
    key = key[key // n != key % n]
    return key


def csr_of(n, key):
    rows = torch.arange(n + 1, device="cuda:0") * n
    return torch.searchsorted(key, rows).to(torch.int32), (key % n).to(torch.int32)


def transposed(n, key):
    return csr_of(n, torch.sort(key % n * n + key // n).values)


@pytest.mark.parametrize("n,nnz,k", [
    (2, 3, 1), (512, 2047, 2), (513, 4097, 3),             # one digit, then two
    (3000, 2049, 2), (3000, 300_000, 5),
    (40_000, 1_200_000, 2),                                # tiles of 4096 entries
    (1_100_000, 400_000, 2),                               # three digits, mostly empty rows
    (700_000, 34_000_000, 1),                              # tiles of 8192 entries, an empty part
])
def test_parts_against_a_sort(pipad, n, nnz, k):  # noqa: F811
    base = random_csr(n, nnz, n)
    keys = [base] + [base[torch.arange(len(base), device="cuda:0") % (7 + t) != 0] for t in range(1, k)]
    frame = pipad.frame_build_overlap([csr_of(n, key) for key in keys])
    back = pipad.frame_transpose(frame)
    for part in [None, *range(k)]:
        rp, col = frame.common() if part is None else frame.delta(part)
        key = torch.repeat_interleave(torch.arange(n, device="cuda:0"), torch.diff(rp.long())) * n + col.long()
        want = transposed(n, key)
        got = back.common() if part is None else back.delta(part)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), part
    assert torch.equal(frame.dinv(), back.dinv())
    back.close()
    frame.close()


# 8 and 32 tiles of 2048 entries are the last whose digits are counted by the sort itself (10 bits and more nodes than 4096, up to
# 4096 nodes); digits of 10, 11 and 12 bits, then two
@pytest.mark.parametrize("n,entries", [(1024, 8 * 2048), (1025, 32 * 2048), (1025, 32 * 2048 + 1), (2048, 2047), (2049, 2049), (4096, 32 * 2048),
                                       (4096, 32 * 2048 + 1), (4097, 8 * 2048), (4097, 8 * 2048 + 1), (60_000, 8 * 2048 - 1)])
@pytest.mark.parametrize("skewed", [False, True])
def test_digits_counted_by_the_sort(pipad, n, entries, skewed):  # noqa: F811
    rng = np.random.default_rng(n + entries)
    cols = (n * rng.random(4 * entries) ** (3 if skewed else 1)).astype(np.int64)
    key = np.unique(rng.integers(0, n, 4 * entries) * n + cols)
    key = rng.permutation(key[key // n != key % n])[:entries]
    key = torch.from_numpy(np.sort(key)).cuda()
    assert len(key) == entries
    half = key[torch.arange(entries, device="cuda:0") % 2 == 0]
    for keys in ([key], [key, half, half]):
        frame = pipad.frame_build_overlap([csr_of(n, q) for q in keys])
        back = pipad.frame_transpose(frame)
        for part in [None, *range(len(keys))]:
            rp, col = frame.common() if part is None else frame.delta(part)
            want = transposed(n, torch.repeat_interleave(torch.arange(n, device="cuda:0"), torch.diff(rp.long())) * n + col.long())
            got = back.common() if part is None else back.delta(part)
            assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), part
        assert torch.equal(frame.dinv(), back.dinv())
        back.close()
        frame.close()
