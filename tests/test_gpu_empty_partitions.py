"""Fewer non-zeros than sketch partitions (fixed ratio: the number of cells does not depend on how
much was kept), so that partitions without an unknown stand between the others.  Where c-index 0 is
a non-zero the first of them have the bounds [0, 0), else [i, i).  Every form of the decoder,
against the oracle; small integers, so values must agree bit for bit."""
import numpy as np
import pytest
import torch

from oracle import tagc_oracle as O
from synth import gradients as G
from tests.helpers import run_both, compare_all

pytestmark = pytest.mark.gpu

_N = 1 << 20
# non-zeros of every rank; the last has them all at the Index's end
_AT = {"first": [0], "first and others": [0, 1, 77, 2048 * 7 + 31, _N - 1],
       "not the first": [5, 2047, 2048, 400_000], "end": [_N - 2, _N - 1]}


@pytest.mark.parametrize("at", list(_AT))
@pytest.mark.parametrize("ranks,fused,workgroups,P,T", [
    (2, False, 0, 0, 0),        # one summed sketch, a workgroup per partition
    (2, False, 3, 0, 0),        # ... and many partitions per workgroup
    (2, False, 0, 9000, 12288),  # c-indices hashed anew
    (2, True, 0, 0, 0), (2, True, 3, 0, 0),    # ranks held in registers
    (6, True, 0, 0, 0),         # added up as they come
    (6, True, 3, 0, 0),         # summed beside the rounds
])
def test_more_partitions_than_non_zeros(at, ranks, fused, workgroups, P, T):
    print("\n[case] empty partitions %s ranks=%d fused=%d grid=%d P=%d" %
          (at, ranks, fused, workgroups, P), flush=True)
    b = G.Bucket("sparse", G.F32, ranks, [G.Seg(0, _N, 10_000, 1, "w")], _N, 4000)
    grads = []
    for r in range(ranks):
        g = torch.zeros(_N)
        g[_AT[at]] = torch.arange(1.0, len(_AT[at]) + 1.0) * (r + 1)
        grads.append(g)
    ores, tb = run_both(b, grads, seed=2, P=P, T=T, sizing=O.SIZE_FIXED_RATIO, fused=fused,
                        decode_workgroups=workgroups)
    assert ores.A > 2 * ores.U == 2 * len(_AT[at])
    if at.startswith("first"):
        assert ores.bnd[0] == ores.bnd[1] == 0
    compare_all(b, ores, tb, exact_values=True)
