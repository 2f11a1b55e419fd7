"""The coalescent kernel at the widths, groups and alignments where its lanes are dealt differently."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
import synth  # noqa: E402
from _util import check_y, csr_to_coo  # noqa: E402
from test_gpu_parity import pipad, run_case, churned, _reset_options  # noqa: E402,F401
from test_gpu_aggregate_batches import power_law  # noqa: E402


@pytest.mark.parametrize("k,F", [(2, 1), (16, 1), (5, 2), (7, 3), (8, 4), (16, 5), (12, 9), (5, 13), (5, 16),
                                 (3, 21), (3, 27), (2, 31)])
@pytest.mark.parametrize("mid_max,sub", [(512, 1), (12, 1), (12, 4)])
def test_groups_of_snapshots(pipad, k, F, mid_max, sub):  # noqa: F811
    """Even and uneven groups, idle lanes, hub units by class and by sub class."""
    pipad.set_option("agg_coalescent", 2)
    pipad.set_option("short_max", 6)
    pipad.set_option("mid_max", mid_max)
    pipad.set_option("sub_classes", sub)
    pipad.set_option("hub_threshold", 64)
    pipad.set_option("hub_segment", 32)
    run_case(pipad, 1200, power_law(1200, 20_000, k, 7 * k + F), F, seed=F, layout="wide", check_csr=False)


@pytest.mark.parametrize("k,F,pad", [(4, 16, 1), (8, 2, 3), (3, 5, 2), (6, 4, 1)])
def test_operand_at_any_multiple_of_four_bytes(pipad, k, F, pad):  # noqa: F811
    n = 900
    lists = churned(np.random.default_rng(k * F), n, k, 0.02, 0.8)
    pipad.set_option("agg_coalescent", 2)
    frame = pipad.frame_build_overlap([(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists])
    store = torch.zeros(n, k * F + pad, device="cuda")
    X = [store[:, pad + t * F:pad + (t + 1) * F] for t in range(k)]
    for t in range(k):
        X[t].copy_(torch.from_numpy(synth.features(3, t, n, F)))
    out = torch.zeros_like(store)
    Y = [out[:, pad + t * F:pad + (t + 1) * F] for t in range(k)]
    pipad.frame_aggregate(frame, X, Y)
    frame.close()
    for t in range(k):
        rows, cols = csr_to_coo(n, *lists[t])
        _, yd, bound, _ = oracle.aggregate(n, rows, cols, synth.features(3, t, n, F), threads=4)
        check_y(Y[t].cpu().numpy(), yd, bound, f"snapshot {t}")
    assert not out[:, :pad].any()


def test_static_scratch_without_room_for_the_class_parts(pipad):  # noqa: F811
    """More partial sums than the fixed scratch holds: one per hub unit, with the same bits."""
    n, k, F = 60_000, 2, 31
    pipad.set_option("short_max", 0)
    pipad.set_option("mid_max", 0)
    pipad.set_option("hub_threshold", 64)
    pipad.set_option("hub_segment", 32)
    lists = power_law(n, 300_000, k, 5)
    assert (np.diff(lists[0][0]) > 0).sum() * 8 * 64 * 4 > 64 << 20
    frame = pipad.frame_build_overlap([(torch.from_numpy(rp).cuda(), torch.from_numpy(c).cuda()) for rp, c in lists])
    x = torch.from_numpy(np.stack([synth.features(9, t, n, F) for t in range(k)], axis=1)).cuda()
    y = pipad.frame_aggregate(frame, x)
    y_static = pipad.frame_aggregate(frame, x, static_scratch=True)
    assert torch.equal(y, y_static)
    frame.close()
