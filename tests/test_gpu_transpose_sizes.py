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
