"""The sparsifier's dense route at the sizes where it changes form: segments one workgroup holds in
its registers and those just too long for it, one entry to a few tiles, off every alignment; and
values that leave its histogram window (40 octaves in one segment, an outlier, ties).  Pairs and
Index bit for bit against the oracle, which has one form for all of them; twice, so that what the
first call leaves behind is seen."""
import numpy as np
import pytest
import torch

from oracle import tagc_oracle as O
from synth import gradients as G
from tests.helpers import oracle_config, oracle_segments

pytestmark = pytest.mark.gpu


def _values(kind, rng, n):
    v = rng.standard_normal(n).astype(np.float32)
    if kind == "octaves":       # magnitudes over 40 octaves
        v *= np.exp2(rng.uniform(-30, 10, n)).astype(np.float32)
    elif kind == "outlier":     # one entry 60 octaves above the rest, some far below
        v[rng.integers(0, n)] = 2.0 ** 60
        v[rng.random(n) < 0.3] *= np.float32(2.0 ** -50)
    elif kind == "ties":        # a few values, a third of them zero
        v = rng.integers(-1, 2, n).astype(np.float32) * rng.integers(1, 4, n).astype(np.float32)
    return v


@pytest.mark.parametrize("dtype", [G.F32, G.BF16])
@pytest.mark.parametrize("kind", ["normal", "octaves", "outlier", "ties"])
def test_dense_route_edges(dtype, kind):
    from paper_2504_05638_amd.bucket import TagcBucket
    print("\n[case] dense route edges %s dtype=%d" % (kind, dtype), flush=True)
    limit = 32768 if dtype == G.F32 else 65535          # longest segment of one workgroup
    tile = 4096 if dtype == G.F32 else 8192             # compaction tile
    lens = [1, 7, limit, limit + 1, tile, 3 * tile + 1, limit - 1, 130_003, 2 * limit + 5]
    keep = [1_000_000, 400_000, 10_000, 300_000, 1_000_000, 5_000, 999_999, 400_000, 500_000]
    for skew in (0, 1):     # (segments that start on 16-byte boundaries, and off them)
        segs, off = [], skew
        for i, (n, ppm) in enumerate(zip(lens, keep)):
            segs.append(G.Seg(off, n, ppm, 1, "s%d" % i))
            off += n if skew else (n + 7) // 8 * 8
        b = G.Bucket("edges", dtype, 2, segs, off, 1500)
        rng = np.random.default_rng(11 + skew)
        td = torch.float32 if dtype == G.F32 else torch.bfloat16
        tb = TagcBucket(b.segments, b.dtype, 2, sizing_milli=1500, seed=3)
        for step in range(2):
            grads = [torch.from_numpy(_values(kind, rng, off)).to(td) for _ in range(2)]
            tb.compress_index_all([g.cuda() for g in grads])
            torch.cuda.synchronize()
            for r in range(2):
                want = O.sparsify(G.to_numpy_raw(grads[r]), oracle_config(b), oracle_segments(b))
                cnt = tb.rank_counts(r)
                assert cnt["total"] == want.cnt and cnt["flags"] == 0 and cnt["nonfinite"] == 0
                assert cnt["seg"] == list(want.seg_cnt)
                assert cnt["dense_segments"] == len(segs)
                idx, val = tb.rank_pairs(r)
                assert np.array_equal(idx, want.idx)
                assert np.array_equal(val.view(np.uint32), want.val.view(np.uint32))
                assert np.array_equal(tb.rank_bitmap(r), want.bitmap[:tb.sizes.bitmap_words])
        tb.close()
