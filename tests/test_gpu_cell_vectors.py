"""The decoder reads a partition's cells four at a time from wherever the partition starts: partitions
of every remainder mod 4, at every alignment, the last one at the end of the sketch, in every form of the
decoder, against the oracle.  Small integers: sums are exact in float32, so values agree bit for bit."""
import numpy as np
import pytest
import torch

from paper_2504_05638_amd import binding as B
from synth import gradients as G
from tests.helpers import run_both, compare_all

pytestmark = pytest.mark.gpu


# (ranks, P, T, sum inside the decoder, partitions at least): one summed sketch, up to four ranks, a workgroup per partition,
# more partitions than workgroups, partitions beyond the default size.  A workgroup per partition: the plan has room for
# no more of them than the device has compute units, 256, and zeros beside the peel stand for that form in the profile
@pytest.mark.parametrize("ranks,P,T,fused,partitions", [(2, 40, 75, False, 257), (3, 40, 75, True, 257), (6, 256, 600, True, 100),
                                                        (6, 40, 75, True, 257), (2, 9000, 12291, False, 2)])
def test_cells_of_every_remainder(ranks, P, T, fused, partitions):
    n, seen = 60_000, set()
    rng = np.random.default_rng(8)
    grads = [torch.from_numpy(rng.integers(-500, 501, n).astype(np.float32)) for _ in range(ranks)]
    for milli in range(1500, 1860, 17):
        print("\n[case] cell vectors ranks=%d P=%d fused=%d milli=%d" % (ranks, P, fused, milli), flush=True)
        b = G.Bucket("cells", G.F32, ranks, [G.Seg(0, n, 100_000, 1, "a")], n, milli)
        ores, tb = run_both(b, grads, seed=2, P=P, T=T, fused=fused)
        compare_all(b, ores, tb, exact_values=True)
        assert ores.A >= partitions and (tb.sizes.partition_capacity <= 256) == (partitions < 257)
        B.tagc_profile_enable(True)
        try:
            (tb.reduce_decompress if fused else tb.decompress)()
            torch.cuda.synchronize()
        finally:
            B.tagc_profile_enable(False)
        assert ("dense" in B.tagc_profile_read()) == (partitions != 100)
        seen.add(3 * ores.m_sub % 4)
        tb.close()
        if len(seen) == 4:
            return
    pytest.fail("remainders seen: %s" % seen)
