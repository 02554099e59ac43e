"""The Index aggregation where it takes three launches (layout and bounds, pair ranges, salts: many
partitions times ranks, in a plan whose decoder leaves room for other buckets): one launch of ranks and two, partitions without an unknown among them,
an Index without a bit; against the oracle, with values whose sums are exact."""
import numpy as np
import pytest
import torch

from oracle import tagc_oracle as O
from synth import gradients as G
from tests.helpers import run_both, compare_all

pytestmark = pytest.mark.gpu

_SPLIT = 32768   # (partition, rank) pairs from which on


@pytest.mark.parametrize("n,keep_ppm,ranks,P,T,sizing,milli,nonzeros", [
    (200_000, 300_000, 4, 16, 24, O.SIZE_LOAD_FACTOR, 1600, None),
    (200_000, 50_000, 35, 64, 96, O.SIZE_LOAD_FACTOR, 1600, None),
    (300_001, 100_000, 35, 100, 150, O.SIZE_FIXED_RATIO, 2000, 40),    # fewer non-zeros than partitions
    (300_001, 100_000, 17, 100, 150, O.SIZE_FIXED_RATIO, 2000, 0),
])
def test_split_layout(n, keep_ppm, ranks, P, T, sizing, milli, nonzeros):
    print("\n[case] split layout n=%d ranks=%d P=%d %s" % (n, ranks, P, nonzeros), flush=True)
    b = G.Bucket("split", G.F32, ranks, [G.Seg(0, n, keep_ppm, 1, "w")], n, milli)
    rng = np.random.default_rng(7)
    at = np.arange(0, n, n // nonzeros) if nonzeros else None
    grads = []
    for r in range(ranks):
        g = rng.integers(-1000, 1001, n).astype(np.float32)
        if nonzeros is not None:
            keep = np.zeros(n, bool)
            keep[at if nonzeros else []] = True
            g = np.where(keep, np.abs(g) + 1, 0).astype(np.float32)
        grads.append(torch.from_numpy(g))
    ores, tb = run_both(b, grads, seed=2, P=P, T=T, sizing=sizing, dense=False,
                        decode_workgroups=32)
    assert tb.sizes.partition_capacity * ranks > _SPLIT
    # (16 unknowns to 24 cells leave residues, whose rounds differ by rounding order)
    hdr, _ = compare_all(b, ores, tb, exact_values=P != 16)
    bounds = tb.bounds()
    first = (5 + tb.sizes.n_seg_compressed + 3) // 4 * 4
    for r in range(ranks):
        got = tb._np(tb._rk_tensors[r]["cnt"], np.uint32)[first:first + hdr["A"] + 1]
        idx, _ = tb.rank_pairs(r)
        assert np.array_equal(got, np.searchsorted(idx, bounds))
