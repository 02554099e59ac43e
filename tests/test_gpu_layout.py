"""Layout, bounds, salts and pair ranges at the edges of the kernel that derives them from the
merged Index: one partition and several thousand (more than one batch of bounds per workgroup),
one Index chunk and more than one per thread, more ranks than one launch takes, nothing kept."""
import numpy as np
import pytest
import torch

from synth import gradients as G
from tests.helpers import run_both, compare_all

pytestmark = pytest.mark.gpu


def _ints(n, ranks, seed):
    rng = np.random.default_rng(seed)
    return [torch.from_numpy(rng.integers(-1000, 1001, n).astype(np.float32)) for _ in range(ranks)]


@pytest.mark.parametrize("n,keep_ppm,ranks,P,T,least", [
    (4096, 100_000, 1, 0, 0, 1),              # one partition, one chunk
    (32_769, 100_000, 3, 0, 0, 1),            # a chunk and one bit
    (300_000, 300_000, 2, 16, 24, 4097),      # more than 8 partitions for each of 512 workgroups
    (200_000, 50_000, 33, 512, 768, 200),     # ranks beyond the first launch's
    (40_000_003, 2_000, 2, 1024, 1536, 100),  # 1221 chunks: two per thread
])
def test_layout_and_ranges(n, keep_ppm, ranks, P, T, least):
    print("\n[case] layout n=%d ranks=%d P=%d" % (n, ranks, P), flush=True)
    b = G.Bucket("layout", G.F32, ranks, [G.Seg(0, n, keep_ppm, 1, "w")], n, 1600)
    ores, tb = run_both(b, _ints(n, ranks, 7), seed=2, P=P, T=T, dense=False)
    hdr, _ = compare_all(b, ores, tb, exact_values=P != 16)
    assert hdr["A"] >= least
    _check_ranges(tb, ranks, hdr["A"])


# All workgroups do both, searches and salts: as many partitions as the device holds workgroups, nearly; many small
# ones.  Apart: nearly as many as the device holds under a plan for twice as many, which are two turns of the salts; more
# than eight ranks, which have more searchers.
@pytest.mark.parametrize("n,keep_ppm,ranks,shared,P,T,cap,least,most", [
    (4_000_000, 15_000, 4, False, 512, 768, (456, 512), 456, 512),
    (4_000_000, 4_000, 16, False, 256, 384, (1024, 2000), 1000, 2000),
    (8_000_000, 77_500, 4, True, 2500, 4002, (513, 2000), 449, 512),
    (8_000_000, 16_000, 16, False, 2500, 4002, (768, 2000), 700, 2000),
])
def test_who_searches(n, keep_ppm, ranks, shared, P, T, cap, least, most):
    print("\n[case] who searches, ranks=%d P=%d ppm=%d" % (ranks, P, keep_ppm), flush=True)
    b = G.Bucket("layout", G.F32, ranks, [G.Seg(0, n, keep_ppm, 1, "w")], n, 1600)
    grads = _ints(n, ranks, 11)
    if shared:
        grads = grads[:2] * 2
    ores, tb = run_both(b, grads, seed=2, P=P, T=T, dense=False)
    assert torch.cuda.get_device_properties(0).multi_processor_count == 256  # (two workgroups each)
    assert cap[0] <= tb.sizes.partition_capacity <= cap[1]
    hdr, _ = compare_all(b, ores, tb, exact_values=True)
    assert least <= hdr["A"] <= most
    assert (tb.sizes.union_capacity >= 2048 * tb.sizes.partition_capacity) == (P == 2500)  # the line between them
    _check_ranges(tb, ranks, hdr["A"])


def _check_ranges(tb, ranks, A):
    """A rank's ranges: where its sorted pairs cross the partition bounds."""
    bounds = tb.bounds()
    first = (5 + tb.sizes.n_seg_compressed + 3) // 4 * 4
    for r in range(ranks):
        got = tb._np(tb._rk_tensors[r]["cnt"], np.uint32)[first:first + A + 1]
        idx, _ = tb.rank_pairs(r)
        assert np.array_equal(got, np.searchsorted(idx, bounds))


def test_an_index_without_a_bit():
    print("\n[case] layout of nothing", flush=True)
    n = 70_000
    b = G.Bucket("nothing", G.F32, 2, [G.Seg(0, n, 10_000, 1, "w")], n, 1500)
    ores, tb = run_both(b, [torch.zeros(n) for _ in range(2)], seed=1)
    hdr, _ = compare_all(b, ores, tb)
    assert hdr == dict(U=0, A=0, m_sub=0, m=0) and tb.bounds().tolist() == [tb.sizes.n_c]
