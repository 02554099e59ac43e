"""TagcBucket's and the binding's host side, without a device."""
import pytest

from paper_2504_05638_amd.bucket import TagcBucket


def test_number_of_workspaces():
    mib, n = 1 << 20, TagcBucket._workspaces
    assert n(16, 40 * mib, 0) == 16              # as many as ranks, where they fit a GiB,
    assert n(64, mib, 0) == 32                   # up to what one launch takes
    assert n(16, 400 * mib, 0) == 2
    assert n(16, 4096 * mib, 0) == 1             # one at least
    assert n(16, 40 * mib, 1) == 1               # or as many as the caller asks for
    assert n(16, 400 * mib, 4) == 4 and n(3, mib, 8) == 3 and n(3, 0, 0) == 3
    with pytest.raises(ValueError):
        n(16, mib, -1)


@pytest.mark.gpu
@pytest.mark.parametrize("together,min_bytes,want", [(0, {}, 5), (2, {}, 2), (1, {}, 1), (8, {}, 5),
                                                     (0, {"rank_ws": 300 << 20}, 3)])
def test_ranks_together(together, min_bytes, want):
    import torch
    from synth import gradients as G
    from tests.helpers import compare_all, oracle_config, oracle_segments
    from oracle import tagc_oracle as O
    b = G.small_mixed_bucket(seed=3, dtype=G.BF16, n_ranks=5, sizing_milli=1500)
    grads = [G.rank_gradient(b, r, "cpu") for r in range(5)]
    ores = O.run_bucket([G.to_numpy_raw(g) for g in grads], oracle_config(b), oracle_segments(b))
    tb = TagcBucket(b.segments, b.dtype, 5, sizing_milli=1500, dense=True, ranks_together=together,
                    min_bytes=min_bytes)
    assert len({rk.workspace for rk in tb.rk}) == len(tb.rank_ws) == want
    for _ in range(2):
        tb.run([g.cuda() for g in grads])
        torch.cuda.synchronize()
        compare_all(b, ores, tb)
