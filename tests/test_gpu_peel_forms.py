"""The decoder's two forms of keeping an unknown in LDS: packed slots (partitions of up to 8192
unknowns and 12288 cells) and c-indices hashed anew (larger ones), at the edges of both, against
the oracle.  Small integers: every sum is exact in float32, so the order of the adds is free and
values must agree bit for bit."""
import numpy as np
import pytest
import torch

from synth import gradients as G
from oracle import tagc_oracle as O
from tests.helpers import run_both, compare_all

pytestmark = pytest.mark.gpu

_PACKED = [(8192, 12288), (8191, 12285), (8192, 12282), (1000, 1500), (33, 48)]
_HASHED = [(8192, 12291), (8193, 12288), (9000, 12291), (16384, 9000), (300, 14997)]


def _bucket(milli):
    n, ranks = 200_000, 2
    segs = [G.Seg(0, 120_001, 110_000, 1, "a"), G.Seg(120_008, 79_992, 90_000, 1, "b")]
    b = G.Bucket("peel_forms", G.F32, ranks, segs, n, milli)
    rng = np.random.default_rng(4)
    return b, [torch.from_numpy(rng.integers(-1000, 1001, n).astype(np.float32)) for _ in range(ranks)]


@pytest.mark.parametrize("P,T", _PACKED + _HASHED)
@pytest.mark.parametrize("milli,mode", [(1500, O.DECODE_PEEL), (1150, O.DECODE_PEEL_ESTIMATE)])
def test_forms_of_an_unknown(P, T, milli, mode):
    print("\n[case] peel forms P=%d T=%d milli=%d" % (P, T, milli), flush=True)
    b, grads = _bucket(milli)
    ores, tb = run_both(b, grads, seed=3, P=P, T=T, decode_mode=mode)
    compare_all(b, ores, tb, exact_values=True)


@pytest.mark.parametrize("P,T", _PACKED)
def test_fused_decode_at_the_same_sizes(P, T):
    print("\n[case] peel forms fused P=%d T=%d" % (P, T), flush=True)
    b, grads = _bucket(1500)
    ores, tb = run_both(b, grads, seed=3, P=P, T=T, fused=True)
    compare_all(b, ores, tb, exact_values=True)
