"""The decoder where its partitions span hundreds of groups of Index words: listed by a kernel of
their own (little can be set), and walked by the decoder's waves beyond the groups they request
ahead (little is set although the plan has room for much), with empty stretches, full words and
non-zeros at the edges of groups and chunks.  Every form, against the oracle; small integers, so
values must agree bit for bit."""
import numpy as np
import pytest
import torch

from synth import gradients as G
from tests.helpers import run_both, compare_all

pytestmark = pytest.mark.gpu

_N = (1 << 22) + 4001


def _positions(rng):
    """About 2000 positions: spread over the first half, a full stretch, edges, the very end."""
    at = set(rng.choice(_N // 2, 1500, replace=False).tolist())
    at.update(range(_N // 2 + 2040, _N // 2 + 2040 + 300))
    for edge in (2048, 32768, 64 * 32768):
        at.update([edge - 1, edge, edge + 2047, edge + 2048])
    at.update([0, _N - 1, _N - 33])
    return np.array(sorted(at))


@pytest.mark.parametrize("listed", [True, False])
@pytest.mark.parametrize("ranks,fused,workgroups,P,T", [
    (2, False, 0, 0, 0), (2, False, 0, 9000, 12288), (2, True, 0, 0, 0), (6, True, 0, 0, 0),
    (6, True, 1, 0, 0), (3, False, 1, 100, 150), (6, True, 2, 100, 150)])
def test_long_partitions(listed, ranks, fused, workgroups, P, T):
    print("\n[case] sparse index listed=%d ranks=%d fused=%d grid=%d P=%d" %
          (listed, ranks, fused, workgroups, P), flush=True)
    # (room: the plan's partitions, of P unknowns each, are counted from what may be kept)
    keep = 500 if listed else 12_000
    if P == 100 and listed:
        keep = 10
    b = G.Bucket("sparse", G.F32, ranks, [G.Seg(0, _N, keep, 1, "w")], _N, 1500)
    rng = np.random.default_rng(8)
    at = _positions(rng)[:: 60 if P == 100 and listed else 1]
    grads = []
    for r in range(ranks):
        g = torch.zeros(_N)
        g[torch.from_numpy(at)] = torch.from_numpy(
            (rng.integers(1, 1001, at.size) * rng.choice([-1, 1], at.size)).astype(np.float32))
        grads.append(g)
    ores, tb = run_both(b, grads, seed=6, P=P, T=T, fused=fused, decode_workgroups=workgroups)
    groups = -(-_N // 32768) * 16
    assert (groups > 256 * tb.sizes.partition_capacity) == listed
    assert ores.U <= at.size and ores.A >= 1
    compare_all(b, ores, tb, exact_values=True)
