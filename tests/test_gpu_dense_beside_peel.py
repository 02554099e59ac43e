"""The dense output where partitions are fewer than compute units: workgroups without one write the zeros, by the
merged Index, while the others peel and put their values among them.  Every entry of it is written, whatever was
there, at sizes around a wave's 16 Index words and a workgroup's, and where nothing is kept."""
import numpy as np
import pytest
import torch

from synth import gradients as G
from tests.helpers import run_both, compare_all

pytestmark = pytest.mark.gpu


def _took(tb, fused):
    """The kernels of a decode into a filled output, which is then what the unknowns and their values say."""
    from paper_2504_05638_amd import binding as B
    tb.out_dense.view(torch.int32).fill_(-1)
    torch.cuda.synchronize()
    B.tagc_profile_enable(True)
    try:
        (tb.reduce_decompress if fused else tb.decompress)()
        torch.cuda.synchronize()
    finally:
        B.tagc_profile_enable(False)
    idx, val = tb.outputs()
    want = np.zeros(tb.sizes.n_c, np.float32)
    want[idx] = val
    assert np.array_equal(tb.dense().view(np.uint32), want.view(np.uint32))
    return set(B.tagc_profile_read())


@pytest.mark.parametrize("n", [1, 33, 511, 513, 8191, 8193, 100_003])
@pytest.mark.parametrize("ranks,fused", [(1, False), (3, True), (31, True), (32, True)])
def test_every_entry_is_written(n, ranks, fused):
    print("\n[case] dense beside peel n=%d ranks=%d fused=%d" % (n, ranks, fused), flush=True)
    rng = np.random.default_rng(n)
    segs = [G.Seg(0, n, 50_000, 1, "a"), G.Seg(n, n, 1_000_000, 1, "b"), G.Seg(2 * n, n, 0, 1, "c")]
    b = G.Bucket("beside", G.F32, ranks, segs, 3 * n, 1500)
    grads = [torch.from_numpy(rng.integers(-9, 10, 3 * n).astype(np.float32)) for _ in range(ranks)]
    for g in grads:  # (of the second segment little is kept all the same: zeros never are)
        g[n:2 * n][torch.from_numpy(rng.random(n) < 0.9)] = 0
    ores, tb = run_both(b, grads, seed=5, fused=fused)
    assert ("dense" in _took(tb, fused)) == (ranks > 31)  # (32 ranks leave no room for the output's address)
    tb.run([g.cuda() for g in grads], fused=fused)
    torch.cuda.synchronize()
    compare_all(b, ores, tb, exact_values=True)
    tb.close()


def test_nothing_kept():
    from paper_2504_05638_amd.bucket import TagcBucket
    print("\n[case] dense beside peel, nothing kept", flush=True)
    tb = TagcBucket([(0, 300_000, 20_000, 1)], G.F32, 2, dense=True)
    tb.out_dense.view(torch.int32).fill_(-1)
    tb.run([torch.zeros(300_000, device="cuda")] * 2, fused=True)
    torch.cuda.synchronize()
    assert tb.header()["U"] == 0 and not tb.dense().view(np.uint32).any()
    assert "dense" not in _took(tb, True)
    tb.close()


# The launch that writes all of it (a plan that limits the decoder's workgroups has it): 256 words to a workgroup, of which
# a quarter's values are staged
@pytest.mark.parametrize("words", [255, 256, 257, 1023, 1025, 2300])
@pytest.mark.parametrize("ppm", [100_000, 700_000])
def test_a_launch_of_its_own(words, ppm):
    print("\n[case] dense kernel words=%d ppm=%d" % (words, ppm), flush=True)
    n = 32 * words - 3
    b = G.Bucket("dense", G.F32, 1, [G.Seg(0, n, ppm, 1, "a")], n, 1500)
    g = torch.from_numpy(np.random.default_rng(words).integers(1, 100, n).astype(np.float32))
    ores, tb = run_both(b, [g], seed=5, P=256, T=384, decode_workgroups=200)
    tb.out_dense.view(torch.int32).fill_(-1)
    tb.run([g.cuda()])
    torch.cuda.synchronize()
    compare_all(b, ores, tb, exact_values=True)
    assert "dense" in _took(tb, False)
    tb.close()


# The decoder takes what the merged Index holds at the moment, whatever the bounds were made from: with fewer set bits
# than there were unknowns, the others' c-indices are what the local memory held.
@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("n", [100_003, 3_000_000])
def test_nothing_lands_outside(n, fused):
    from paper_2504_05638_amd import binding as B
    from paper_2504_05638_amd.bucket import TagcBucket
    print("\n[case] dense beside peel, Index cleared, n=%d fused=%d" % (n, fused), flush=True)
    tb = TagcBucket([(0, n, 50_000, 1)], G.F32, 2)
    grads = [torch.randn(n, generator=torch.Generator().manual_seed(r)).cuda() for r in range(2)]
    for _ in range(2):
        tb.run(grads, fused=fused)
    room, guard = int(tb.sizes.n_c), 1 << 28
    out = torch.full((room + 2 * guard,), -1, dtype=torch.int32, device="cuda")
    at, s = out.data_ptr() + 4 * guard, torch.cuda.current_stream().cuda_stream
    tb.sh_bitmap.zero_()
    if fused:
        B.tagc_reduce_decompress(tb.plan, tb.rk, tb.shared, tb.out_idx.data_ptr(), tb.out_val.data_ptr(), at, s, 2)
    else:
        B.tagc_decompress(tb.plan, tb.shared, tb.out_idx.data_ptr(), tb.out_val.data_ptr(), at, s)
    torch.cuda.synchronize()
    assert bool((out[:guard] == -1).all()) and bool((out[guard + room:] == -1).all())
    # (no bit is set: all is zero but for the few entries that such a c-index may name)
    assert int((out[guard:guard + room] != 0).sum()) <= tb.header()["U"]
    tb.close()


# Three ranks keep the one entry of every segment: their 1-bit Indexes add up to two set bits each, more than the plan
# has room for.  No partition is decoded then, and the dense output is zeros.
@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("segments", [1, 40])
def test_zeros_after_an_overflow(segments, fused):
    from paper_2504_05638_amd import binding as B
    from paper_2504_05638_amd.bucket import TagcBucket
    print("\n[case] dense beside peel, overflow segments=%d fused=%d" % (segments, fused), flush=True)
    tb = TagcBucket([(i, 1, 1_000_000, 1) for i in range(segments)], G.F32, 3, index_mode=B.TAGC_INDEX_ADD1, dense=True)
    tb.out_dense.view(torch.int32).fill_(-1)
    tb.run([torch.full((segments,), 5.0, device="cuda")] * 3, fused=fused)
    torch.cuda.synchronize()
    assert tb.status()["flags"] == B.TAGC_FLAG_OVERFLOW and tb.header()["A"] == 0
    assert np.array_equal(tb.shared_bitmap(), np.full(segments, 3, np.uint32))
    assert not tb.dense().view(np.uint32).any()
    tb.close()


# A dense output in the place of a sketch, which nobody needs behind the decoder: by the launch behind it
@pytest.mark.parametrize("fused,where", [(False, "sum"), (True, "sketch0"), (True, "sketch2"), (True, "idx"), (True, "bounds")])
@pytest.mark.parametrize("n,P,T", [(2_000, 0, 0), (30_000, 32, 48)])
def test_in_the_place_of_what_was_read(fused, where, n, P, T):
    from paper_2504_05638_amd import binding as B
    print("\n[case] dense over %s n=%d" % (where, n), flush=True)
    b = G.Bucket("beside", G.F32, 3, [G.Seg(0, n, 900_000, 1, "a")], n, 3000)
    rng = np.random.default_rng(n)
    grads = [torch.from_numpy(rng.integers(-9, 10, n).astype(np.float32)) for _ in range(3)]
    ores, tb = run_both(b, grads, seed=5, P=P, T=T, fused=fused)
    want = tb.dense()
    out = {"sum": tb.sh_sketch, "idx": tb.out_idx, "bounds": tb.sh_bounds}.get(where)
    if out is None:
        out = tb._rk_tensors[int(where[-1])]["sketch"]
    elif where in ("idx", "bounds"):  # (at the end of a buffer that begins as that one)
        big = torch.zeros(out.numel() + 4 * n + 4096, dtype=torch.uint8, device="cuda")
        big[:out.numel()] = out
        out = big
        if where == "idx":
            tb.out_idx = big
        else:
            tb.shared.bounds = big.data_ptr()
    assert out.numel() >= 4 * int(tb.sizes.n_c)
    tb.out_dense = out
    B.tagc_profile_enable(True)
    try:
        (tb.reduce_decompress if fused else tb.decompress)()
        torch.cuda.synchronize()
    finally:
        B.tagc_profile_enable(False)
    assert "dense" in B.tagc_profile_read()
    assert np.array_equal(tb.dense(), want)  # (an entry that cancels may be a zero of either sign)
    tb.close()


# Where the lines lie: what a writing workgroup may have (partitions of 32 unknowns, 200 of them, 56 workgroups left, some
# eighteen turns of 16 words a wave each; 8192 unknowns, 30 partitions), and the sum of more than four ranks into 16 to 64 MB
@pytest.mark.parametrize("n,ppm,ranks,P,T,fused,beside", [
    (8_364_000, 765, 1, 32, 48, True, True), (8_367_000, 765, 1, 32, 48, True, False), (8_364_033, 765, 1, 32, 48, False, True),
    (3_999_969, 15_000, 4, 0, 0, True, True),
    ((4 << 20) - 32, 9500, 5, 0, 0, True, True), (4 << 20, 9500, 5, 0, 0, True, False), (4 << 20, 9500, 5, 0, 0, False, True),
    (4 << 20, 9500, 4, 0, 0, True, True), ((16 << 20) - 32, 3500, 5, 0, 0, True, False), (16 << 20, 3500, 5, 0, 0, True, True)])
def test_who_writes_it(n, ppm, ranks, P, T, fused, beside):
    from paper_2504_05638_amd.bucket import TagcBucket
    print("\n[case] dense beside peel or behind n=%d ranks=%d P=%d fused=%d" % (n, ranks, P, fused), flush=True)
    tb = TagcBucket([(0, n, ppm, 1)], G.F32, ranks, part_unknowns=P, part_cells=T, dense=True,
                    sizing_milli=1500)
    assert tb.sizes.partition_capacity == 200 if P else tb.sizes.partition_capacity < 60
    gen = torch.Generator(device="cuda").manual_seed(n)
    tb.run([torch.randn(n, device="cuda", generator=gen) for _ in range(ranks)], fused=fused)
    assert ("dense" in _took(tb, fused)) != beside
    tb.close()
