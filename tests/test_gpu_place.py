"""The survivors' ordered output: a wave takes a super-chunk (32 chunks of 2048 bf16 or 1024 fp32 entries), 256
slots to a step, and collects the Index words of 16 chunks at a time.  Lengths that end inside a chunk, a window and
a super-chunk; fewer slots than a step, several steps, halves without any slot; ties cut off by the quota; a
second segment whose Index words start off a 16-byte boundary.  Selections are whole numbers: exact."""
import pytest
import torch

from synth import gradients as G
from tests.helpers import run_both, compare_all

pytestmark = pytest.mark.gpu

_SC = {G.F32: 32 * 1024, G.BF16: 32 * 2048}


def _check(what, segs, dtype, values):
    print("\n[case] place %s" % (what,), flush=True)
    n = segs[-1].offset + segs[-1].length
    b = G.Bucket("place", dtype, 2, segs, n, 3000)
    # rounded to bf16 in fp32 too: there are ties at every threshold
    grads = [values(r, n).to(torch.bfloat16).to(b.torch_dtype) for r in range(2)]
    ores, tb = run_both(b, grads, seed=5)
    dev = [g.cuda() for g in grads]
    for _ in range(2):  # (the second time with a pre-threshold that the first left)
        tb.run(dev)
        torch.cuda.synchronize()
        compare_all(b, ores, tb)
        assert all(tb.rank_counts(r)["dense_segments"] == 0 for r in range(2))


def _normal(r, n):
    return torch.randn(n, generator=torch.Generator().manual_seed(100 + r)).mul_(1e-3)


# slots per chunk, fp32 / bf16: 3 / 5, 13 / 27, 133 / 266
@pytest.mark.parametrize("ppm", [2_000, 10_000, 100_000])
@pytest.mark.parametrize("length", [(1, 1), (3, -31), (2.5, 5), (4.5, -1), (5, 0)])
@pytest.mark.parametrize("dtype", [G.F32, G.BF16])
def test_lengths_and_fractions(dtype, length, ppm):
    n = 131072 + int(length[0] * _SC[dtype]) + length[1]
    off = (n + 7) // 8 * 8
    segs = [G.Seg(0, n, ppm, 1, "a"), G.Seg(off, 200_003, 3 * ppm // 2, 1, "b")]
    _check(("lengths", dtype, n, ppm), segs, dtype, _normal)


@pytest.mark.parametrize("first", [True, False])
@pytest.mark.parametrize("dtype", [G.F32, G.BF16])
def test_windows_without_a_slot(dtype, first):
    n, half = 7 * _SC[dtype] + 777, _SC[dtype] // 2

    def values(r, n):
        x = _normal(r, n)
        empty = (torch.arange(n) // half) % 2 == (0 if first else 1)
        x[empty] *= 1e-3
        return x
    _check(("windows", dtype, first), [G.Seg(0, n, 4_000, 1, "a")], dtype, values)


def test_more_segments_than_lanes():
    segs, off = [], 0
    for i in range(67):
        n = 131_080 + 8 * i
        segs.append(G.Seg(off, n, 12_000 + 100 * i, 1, "s%d" % i))
        off += n
    _check("segments", segs, G.BF16, _normal)


@pytest.mark.parametrize("dtype,n", [(G.BF16, 26_000_021), (G.F32, 13_000_013)])
def test_counts_from_memory(dtype, n):
    """16 ranks in one launch have more slots than the last cache holds, and count has a form of its own for
    that; a rank at a time has not.  The same selections, whole and to the bit."""
    from paper_2504_05638_amd.bucket import TagcBucket
    ranks, ppm = 16, 150_000
    print("\n[case] count from memory dtype=%d" % dtype, flush=True)
    slots = 1.3 * ranks * (n * ppm // 10**6) * (8 if dtype == G.F32 else 4)
    assert slots > 244e6 > slots / ranks
    segs = [G.Seg(0, n, ppm, 1, "a")]
    td = torch.float32 if dtype == G.F32 else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(4)
    grads = [torch.randn(n, generator=gen, device="cuda").to(td) for _ in range(ranks)]
    apart = TagcBucket(segs, dtype, ranks, seed=3, ranks_together=1, dense=False)
    whole = TagcBucket(segs, dtype, ranks, seed=3, ranks_together=ranks, dense=False)
    assert len(whole.rank_ws) == ranks
    for tb in (apart, whole):
        tb.compress_index_all(grads)
    torch.cuda.synchronize()
    for r in range(ranks):
        a, w = apart.rank_counts(r), whole.rank_counts(r)
        assert a["dense_segments"] == w["dense_segments"] == 0 and a["total"] == n * ppm // 10**6
        assert a == w
        for name in ("idx", "val", "bitmap"):
            used = 4 * a["total"] if name != "bitmap" else 4 * whole.sizes.bitmap_words
            assert torch.equal(apart._rk_tensors[r][name][:used], whole._rk_tensors[r][name][:used]), (r, name)
    apart.close()
    whole.close()
