"""fp32: the threshold's low 16 key bits, at the edges of the kernel that counts them: ties across
waves, chunks with more candidates than one read of 64, tables of more segments than lanes,
segments that share a workgroup's span, and the dense route (an odd offset).  Called twice: the
second call selects from counters that the first left."""
import numpy as np
import pytest
import torch

from synth import gradients as G
from tests.helpers import run_both, compare_all

pytestmark = pytest.mark.gpu


def _case(name):
    rng = np.random.default_rng(17)
    if name == "ties":          # a few hundred distinct values: thousands of equal keys
        n, segs = 600_000, [(0, 600_000, 10_000)]
        g = np.round(rng.standard_normal(n) * 64).astype(np.float32) / 64
    elif name == "one_value":   # every candidate ties
        n, segs = 300_000, [(0, 300_000, 20_000)]
        g = np.where(rng.random(n) < 0.1, 0.375, 0.001).astype(np.float32)
    elif name == "crowded":     # chunks of 1024 with some 130 candidates
        n, segs = 500_000, [(0, 500_000, 100_000)]
        g = rng.standard_normal(n).astype(np.float32)
    elif name == "many_segments":
        length = 132_000
        segs = [(i * length, length - 4 * (i % 3), 1_000 + 100 * i) for i in range(70)]
        n = 70 * length
        g = rng.standard_normal(n).astype(np.float32)
    else:                       # "dense": an odd offset, beside one on the candidate route
        n, segs = 700_003, [(0, 300_000, 10_000), (300_001, 400_002, 30_000)]
        g = rng.standard_normal(n).astype(np.float32)
    return G.Bucket(name, G.F32, 1, [G.Seg(o, m, k, 1, "w%d" % i) for i, (o, m, k) in enumerate(segs)],
                    n, 1600), [torch.from_numpy(g)]


@pytest.mark.parametrize("name", ["ties", "one_value", "crowded", "many_segments", "dense"])
def test_low_key_bits(name):
    print("\n[case] refine %s" % name, flush=True)
    b, grads = _case(name)
    ores, tb = run_both(b, grads, seed=1, P=1024, T=3072)
    compare_all(b, ores, tb)
    tb.run([g.cuda() for g in grads])
    torch.cuda.synchronize()
    compare_all(b, ores, tb)
