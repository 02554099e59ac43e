"""Rounds of up to 64 queue entries, which the decoder leaves to one wave: partitions whose first rounds
have about that many, so that a peel begins with them, goes over to them and comes back, against the
oracle.  Small integers: every sum is exact in float32, so values must agree bit for bit, and the
number of rounds is the oracle's."""
import numpy as np
import pytest
import torch

from synth import gradients as G
from tests.helpers import run_both, compare_all

pytestmark = pytest.mark.gpu


# (three cells per unknown: about three quarters are alone in one of theirs at the start, so 80 to
# 92 unknowns queue 64 give or take a few; at 1.3 about a quarter are, and later rounds grow again)
@pytest.mark.parametrize("milli,sizes", [(3000, (1, 2, 63, 64, 65, 80, 83, 86, 89, 92, 130)),
                                         (1300, (3, 64, 230, 250, 270, 290, 700, 1500))])
@pytest.mark.parametrize("ranks,P,T,fused", [(1, 8192, 12288, False), (6, 8192, 12288, True),
                                             (1, 9000, 12291, False)])
def test_rounds_of_about_a_wave(milli, sizes, ranks, P, T, fused):
    for n in sizes:
        print("\n[case] peel tail n=%d milli=%d ranks=%d P=%d" % (n, milli, ranks, P), flush=True)
        b = G.Bucket("peel_tail", G.F32, ranks, [G.Seg(0, n, 1_000_000, 1, "a")], n, milli)
        rng = np.random.default_rng(n)
        grads = [torch.from_numpy(rng.integers(1, 1001, n).astype(np.float32)) for _ in range(ranks)]
        for seed in (1, 2, 3):
            ores, tb = run_both(b, grads, seed=seed, P=P, T=T, fused=fused)
            compare_all(b, ores, tb, exact_values=True)
            tb.close()
