"""The encoder takes a partition's pairs 2048 at a time: one partition of a pair list that ends just
before, at and just behind a batch, from one rank and from three, against the oracle.  Small integers, so
cells and values must agree bit for bit."""
import numpy as np
import pytest
import torch

from synth import gradients as G
from tests.helpers import run_both, compare_all

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pairs", [1, 2047, 2048, 2049, 4096, 4097, 8192])
@pytest.mark.parametrize("ranks", [1, 3])
def test_pairs_of_a_partition(pairs, ranks):
    print("\n[case] encode pairs=%d ranks=%d" % (pairs, ranks), flush=True)
    n = 10_000
    b = G.Bucket("encode", G.F32, ranks, [G.Seg(0, n, 1_000_000 * pairs // n, 1, "w")], n, 1500)
    rng = np.random.default_rng(pairs)
    at = np.sort(rng.permutation(n)[:pairs])  # the same entries of every rank: one partition
    grads = []
    for _ in range(ranks):
        g = torch.zeros(n)
        g[at] = torch.from_numpy((rng.integers(1, 1000, pairs) * rng.choice([-1, 1], pairs)).astype(np.float32))
        grads.append(g)
    ores, tb = run_both(b, grads, seed=1, fused=False)
    assert ores.A == 1 and ores.ranks[0].cnt == b.segments[0].length * b.segments[0].keep_ppm // 1_000_000
    compare_all(b, ores, tb, exact_values=True)
