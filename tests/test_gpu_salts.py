"""The choice of the partitions' hash salts where it is not salt 0: sub-tables so small for their
unknowns that pairs with the same three cells are common under every salt, some or none, with few, many and
more suspects than the kernel lists, against the oracle."""
import numpy as np
import pytest
import torch

from synth import gradients as G
from oracle import tagc_oracle as O
from tests.helpers import run_both, compare_all

pytestmark = pytest.mark.gpu


# (unknowns, cells per sub-table, partition size; smallest and largest salt over the seeds): pairs over triples of
# cells 0.02 to 1000.  64 filter bits a cell, so under salt 0 the filter finds 19 to 4600 of the unknowns suspect;
# they are listed if they are no more than 2048 (at the default size), 512, 4096 and 16 (at the others): the third
# and the last three have more, 1024 unknowns at 40 cells about as many.  12000 are more than the eight unknowns
# that a thread keeps in registers.
@pytest.mark.parametrize("unknowns,m_sub,P,T,lowest,highest", [
    (1200, 330, 8192, 12288, 0, 0), (2000, 126, 8192, 12288, 0, 2), (8192, 322, 8192, 12288, 0, 9),
    (8192, 600, 8192, 12288, 0, 1), (900, 70, 1024, 3072, 0, 4), (1024, 40, 1024, 3072, 15, 15),
    (12000, 400, 16384, 9000, 0, 6), (64, 12, 64, 48, 1, 2), (500, 5, 8192, 12288, 15, 15)])
def test_salts_of_crowded_partitions(unknowns, m_sub, P, T, lowest, highest):
    print("\n[case] salts U=%d m_sub=%d P=%d" % (unknowns, m_sub, P), flush=True)
    n = 131_072
    # floor(ceil(n * 1000 / milli) / 3) cells per sub-table
    milli = n * 1000 // (3 * m_sub + 1)
    seen = set()
    for seed in range(6):
        rng = np.random.default_rng(seed)
        g = np.zeros(n, np.float32)
        g[rng.choice(n, unknowns, replace=False)] = rng.integers(1, 1000, unknowns)
        b = G.Bucket("salts", G.F32, 1, [G.Seg(0, n, 1_000_000, 1, "a")], n, milli)
        ores, tb = run_both(b, [torch.from_numpy(g)], seed=seed, P=P, T=T, sizing=O.SIZE_FIXED_RATIO,
                            dense=False)
        assert tb.header()["A"] == 1 and abs(tb.header()["m_sub"] - m_sub) <= 1
        compare_all(b, ores, tb, exact_values=True)
        seen.update(int(s) for s in tb.salts())
        tb.close()
    assert (min(seen), max(seen)) == (lowest, highest), seen
