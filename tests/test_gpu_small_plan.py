"""Plans whose segments are all held by one workgroup's registers: one launch from the gradient to pairs, Index and
counts.  Segments that fall short of what they are to keep (fewer non-zeros than that), at the front and in the middle,
move the pairs of all behind them; the most segments such a plan has, and more; entries that are not finite; ties; segments that keep nothing or are empty; the
largest such segment and one entry more; odd offsets; repeated calls, the state left behind included; against the oracle."""
import numpy as np
import pytest
import torch

from oracle import tagc_oracle as O
from paper_2504_05638_amd import binding as B
from synth import gradients as G
from tests.helpers import run_both, compare_all, oracle_config, oracle_segments

pytestmark = pytest.mark.gpu


def _run(segs, n, dtype, zeros, ranks=2, ties=False, one=True):
    """`zeros`: segments left with three non-zeros, by rank; `one`: whether one launch takes them."""
    b = G.Bucket("small", dtype, ranks, segs, n, 1500)
    rng = np.random.default_rng(n)
    td = torch.float32 if dtype == G.F32 else torch.bfloat16
    grads = []
    for r in range(ranks):
        x = rng.integers(-3, 4, n) if ties else rng.integers(-120, 121, n)
        for i in zeros[r % len(zeros)]:
            s = segs[i]
            x[s.offset + 3:s.offset + s.length] = 0
        grads.append(torch.from_numpy(x.astype(np.float32)).to(td))
    ores, tb = run_both(b, grads, seed=6)
    compare_all(b, ores, tb, exact_values=True)
    for _ in range(2):  # the counters are back where they were
        B.tagc_profile_enable(True)
        try:
            tb.run([g.cuda() for g in grads])
            torch.cuda.synchronize()
        finally:
            B.tagc_profile_enable(False)
        took = B.tagc_profile_read()
        assert ("small" in took, "place" in took) == (one, not one), took
        compare_all(b, ores, tb, exact_values=True)
    tb.close()


def _segments(lengths, ppm, gap=0):
    segs, at = [], 0
    for i, n in enumerate(lengths):
        segs.append(G.Seg(at, n, ppm[i % len(ppm)], 1, "s%d" % i))
        at += n + gap
    return segs, at


@pytest.mark.parametrize("dtype", [G.F32, G.BF16])
@pytest.mark.parametrize("zeros", [((),), ((0,), ()), ((2,), (3,)), ((0, 1, 2, 3, 4),), ((4,),)])
@pytest.mark.parametrize("ties", [False, True])
def test_segments_that_fall_short(dtype, zeros, ties):
    print("\n[case] small plan dtype=%d zeros=%s ties=%d" % (dtype, zeros, ties), flush=True)
    segs, n = _segments([4097, 1023, 30_001, 8192, 777], [20_000, 300_000, 50_000])
    _run(segs, n, dtype, zeros, ties=ties)


@pytest.mark.parametrize("dtype", [G.F32, G.BF16])
@pytest.mark.parametrize("count,zeros", [(1, ((0,),)), (64, ((),)), (64, ((3,),)), (64, ((50,), (60, 62))), (65, ((20,),)), (130, ((63, 128), ()))])
def test_many_segments(dtype, zeros, count):
    print("\n[case] small plan, %d segments dtype=%d zeros=%s" % (count, dtype, zeros), flush=True)
    segs, n = _segments([33 + 7 * (i % 5) for i in range(count)], [200_000, 400_000], gap=1)
    _run(segs, n, dtype, zeros, one=count <= 64)


# As many workgroups as the rule allows, a compute unit for a half or a quarter of them at once
@pytest.mark.parametrize("dtype,count,ranks", [(G.F32, 64, 16), (G.BF16, 64, 8), (G.BF16, 16, 32)])
def test_several_turns_of_workgroups(dtype, count, ranks):
    print("\n[case] small plan, %d segments of %d ranks dtype=%d" % (count, ranks, dtype), flush=True)
    segs, n = _segments([33 + 700 * (i % 5) for i in range(count)], [20_000, 400_000], gap=1)
    _run(segs, n, dtype, ((), (5, 6), (count - 1,)), ranks=ranks)


@pytest.mark.parametrize("dtype,most", [(G.F32, 32768), (G.BF16, 65535)])
@pytest.mark.parametrize("more", [0, 1])
def test_the_largest_segment_and_one_more(dtype, most, more):
    print("\n[case] small plan dtype=%d n=%d" % (dtype, most + more), flush=True)
    segs = [G.Seg(1, most + more, 30_000, 1, "a"), G.Seg(most + 5, 0, 30_000, 1, "b"), G.Seg(most + 5, 999, 0, 1, "c"),
            G.Seg(most + 1007, 31, 1_000_000, 1, "d")]
    _run(segs, most + 1038, dtype, ((0,), ()), one=not more)


@pytest.mark.parametrize("dtype", [G.F32, G.BF16])
def test_not_finite(dtype):
    from paper_2504_05638_amd.bucket import TagcBucket
    print("\n[case] small plan, not finite dtype=%d" % dtype, flush=True)
    segs, n = _segments([5000, 300, 7000], [50_000])
    tb = TagcBucket(segs, dtype, 1)
    for bad in ([], [7, 5100, 11_000, 11_001], []):  # (counted anew in every call)
        g = torch.randn(n, generator=torch.Generator().manual_seed(1))
        g[bad] = torch.tensor([float("inf"), float("nan"), -float("inf"), float("inf")])[:len(bad)]
        tb.run([g.to(torch.float32 if dtype == G.F32 else torch.bfloat16).cuda()])
        torch.cuda.synchronize()
        cnt = tb.rank_counts(0)
        assert cnt["nonfinite"] == len(bad) and cnt["dense_segments"] == 3 and cnt["total"] == sum(cnt["seg"])
    tb.close()


def _took(segs, n, dtype, ranks):
    """The sparsifier's kernels in the second call on a plan."""
    from paper_2504_05638_amd.bucket import TagcBucket
    tb = TagcBucket(segs, dtype, ranks)
    g = [torch.ones(n, device="cuda", dtype=torch.float32 if dtype == G.F32 else torch.bfloat16)] * ranks
    tb.compress_index_all(g)
    torch.cuda.synchronize()
    B.tagc_profile_enable(True)
    try:
        tb.compress_index_all(g)
        torch.cuda.synchronize()
    finally:
        B.tagc_profile_enable(False)
    tb.close()
    return set(B.tagc_profile_read())


# Lengths, kept (ppm), ranks; whether one launch takes them.  What a workgroup would be slower over than the device
# is left to the device: too many pairs of a segment, more than two turns of workgroups (fp32: four); and a plan that keeps nothing.
@pytest.mark.parametrize("dtype,lengths,ppm,ranks,one", [
    (G.F32, [32768], 375_000, 1, True), (G.F32, [32768], 376_000, 1, False),
    (G.BF16, [65535], 62_000, 1, True), (G.BF16, [65535], 63_000, 1, False),
    (G.BF16, [8192], 1_000_000, 1, True), (G.BF16, [8193], 1_000_000, 1, False), (G.BF16, [8700], 945_000, 1, True),
    (G.F32, [32768] * 64, 20_000, 2, True), (G.BF16, [65535] * 64, 20_000, 2, True), (G.F32, [32768] * 64, 20_000, 16, True),
    (G.F32, [700] * 32, 20_000, 32, True), (G.F32, [700] * 33, 20_000, 32, False),
    (G.BF16, [700] * 16, 20_000, 32, True), (G.BF16, [700] * 17, 20_000, 32, False),
    (G.F32, [700] * 64, 20_000, 4, True), (G.F32, [700] * 65, 20_000, 1, False), (G.BF16, [40] * 7, 20_000, 2, False)])
def test_which_plans_take_one_launch(dtype, lengths, ppm, ranks, one):
    print("\n[case] small plan, route dtype=%d lengths=%s ppm=%d ranks=%d" % (dtype, lengths[:3], ppm, ranks), flush=True)
    segs, n = _segments(lengths, [ppm])
    took = _took(segs, n, dtype, ranks)
    assert ("small" in took, "place" in took) == (one, not one), took


# What the workgroups of a launch tell each other, a word a segment behind the table's rows, is there long before anybody
# looks.  Below zero before the launch, it counts as not there, as if that workgroup had not started yet: a wave of each of the
# others counts the segment then, 64 16-byte vectors at a time, and all words are zero behind the launch.
_WIN_WORDS = 1544  # per segment, of the candidate histograms in front of the counters


def _untold(tb, n_seg, which):
    """Marks the words of the segments `which`, of every rank; returns a view of all words."""
    slot = n_seg * _WIN_WORDS + 8 + (7 * n_seg + 7) // 8 * 8
    state = tb.table.view(torch.int32)[8 + 8 * n_seg:][:slot * min(tb.n_ranks, 32)].view(-1, slot)
    words = state[:, n_seg * _WIN_WORDS + 8 + 4 * n_seg:][:, :n_seg]
    assert not words.any().item()
    words[:, which] = -1 << 31
    return words


@pytest.mark.parametrize("dtype", [G.F32, G.BF16])
@pytest.mark.parametrize("at", ["spread", "end", "none", "dense"])
@pytest.mark.parametrize("which", [[], [0], [1, 3, 4], [0, 1, 2, 3, 4, 5, 6]])
def test_segments_nobody_has_told_of(dtype, at, which):
    print("\n[case] small plan, untold dtype=%d at=%s which=%s" % (dtype, at, which), flush=True)
    turn = 256 if dtype == G.F32 else 512  # entries of a wave's turn
    lengths = [turn, 32_768 if dtype == G.F32 else 65_535, turn + 1, 3 * turn - 5, 77, 70 * turn + 3, 901]
    for kept in (60, 700):
        segs, at0 = [], 0
        for i, n in enumerate(lengths):
            segs.append(G.Seg(at0, n, 1_000_000 * min(kept, n) // n, 1, "s%d" % i))
            at0 += n
        b = G.Bucket("small", dtype, 3, segs, at0, 1500)
        rng = np.random.default_rng(kept)
        grads = []
        for r in range(3):  # one non-zero fewer than are kept, as many, one more
            x = np.zeros(at0)
            for s in segs:
                k = s.length * s.keep_ppm // 1_000_000
                n = {"none": 0, "dense": s.length}.get(at, min(k - 1 + r, s.length))
                lo = s.length - n if at == "end" else 0
                x[s.offset + rng.choice(np.arange(lo, s.length), n, replace=False)] = rng.integers(1, 120, n)
            grads.append(torch.from_numpy(x.astype(np.float32)).to(torch.float32 if dtype == G.F32 else torch.bfloat16))
        ores, tb = run_both(b, grads, seed=6)
        for _ in range(2):
            words = _untold(tb, len(segs), which)
            for t in tb._rk_tensors:
                t["idx"].fill_(0xFF)
            B.tagc_profile_enable(True)
            try:
                tb.run([g.cuda() for g in grads])
                torch.cuda.synchronize()
            finally:
                B.tagc_profile_enable(False)
            assert "small" in B.tagc_profile_read()
            assert not words.any().item()
            compare_all(b, ores, tb, exact_values=True)
        tb.close()


# Words that say more than a segment can emit, as nobody but the library should write them: the pairs are in the wrong
# place, but in the list, and the next call is right again.
@pytest.mark.parametrize("dtype", [G.F32, G.BF16])
def test_nothing_lands_outside_the_list(dtype):
    print("\n[case] small plan, words too large dtype=%d" % dtype, flush=True)
    segs, n = _segments([4097, 1023, 9_001, 777], [20_000, 300_000])
    b = G.Bucket("small", dtype, 2, segs, n, 1500)
    rng = np.random.default_rng(3)
    td = torch.float32 if dtype == G.F32 else torch.bfloat16
    grads = [torch.from_numpy(rng.integers(-120, 121, n).astype(np.float32)).to(td) for _ in range(2)]
    ores, tb = run_both(b, grads, seed=6)
    room, guard = int(tb.sizes.pair_capacity), 1 << 22
    own = [(r.idx, r.val) for r in tb.rk]
    out = torch.full((4, room + 2 * guard), -1, dtype=torch.int32, device="cuda")
    for r in range(2):
        tb.rk[r].idx, tb.rk[r].val = (out[2 * r + i].data_ptr() + 4 * guard for i in range(2))
    words = _untold(tb, len(segs), [])
    words[:, :3] = 1 << 20
    tb.compress_index_all([g.cuda() for g in grads])
    torch.cuda.synchronize()
    assert not words.any().item()
    assert bool((out[:, :guard] == -1).all()) and bool((out[:, guard + room:] == -1).all())
    for r in range(2):
        tb.rk[r].idx, tb.rk[r].val = own[r]
    tb.run([g.cuda() for g in grads])
    torch.cuda.synchronize()
    compare_all(b, ores, tb, exact_values=True)
    tb.close()


# With an accumulator: the launch before replaces the gradient by the sum, read through the Index that this one then writes
# anew; bit for bit the oracle's over a few steps, the scale changing between them
@pytest.mark.parametrize("dtype", [G.F32, G.BF16])
@pytest.mark.parametrize("index_mode", [O.INDEX_OR1, O.INDEX_ADD4])
def test_with_an_accumulator(dtype, index_mode):
    from paper_2504_05638_amd.bucket import TagcBucket
    print("\n[case] small plan, accumulator dtype=%d mode=%d" % (dtype, index_mode), flush=True)
    segs, n = _segments([4097, 1023, 20_001, 777, 31], [20_000, 300_000, 50_000, 0], gap=3)
    n = segs[-1].offset + segs[-1].length
    ranks, td = 2, torch.float32 if dtype == G.F32 else torch.bfloat16
    b = G.Bucket("small", dtype, ranks, segs, n, 1500)
    cfg, osegs = oracle_config(b, seed=3, index_mode=index_mode), oracle_segments(b)
    tb = TagcBucket(segs, dtype, ranks, sizing_milli=1500, seed=3, error_feedback=True, index_mode=index_mode)
    acc = [np.zeros(n, np.uint16 if dtype == G.BF16 else np.float32) for _ in range(ranks)]
    B.tagc_profile_enable(True)
    try:
        for step, scale in enumerate([1.0, 1.0, 100.0, 1e-3, 1.0]):
            gen = torch.Generator().manual_seed(step)
            grads = [(torch.randn(n, generator=gen) * scale).to(td) for _ in range(ranks)]
            states = []
            for r in range(ranks):
                state, acc[r] = O.error_feedback_step(G.to_numpy_raw(grads[r]), acc[r], cfg, osegs)
                states.append(state)
            tb.run([g.cuda() for g in grads])
            torch.cuda.synchronize()
            for r in range(ranks):
                idx, val = tb.rank_pairs(r)
                assert np.array_equal(idx, states[r].idx), (step, r)
                assert np.array_equal(val.view(np.uint32), states[r].val.view(np.uint32)), (step, r)
                local = states[r].bitmap[:tb.sizes.bitmap_words]
                assert np.array_equal(tb.rank_bitmap(r), O.index_widen4(local) if index_mode == O.INDEX_ADD4 else local)
                if step % 2:  # (the next step does not depend on it)
                    tb.feedback_apply(r)
                    torch.cuda.synchronize()
                    got = tb.rank_acc(r)[:n]
                    keep = np.zeros(n, bool)
                    for s in segs:
                        keep[s.offset:s.offset + s.length] = True
                    assert np.array_equal(got[keep], acc[r].view(got.dtype)[keep]), (step, r)
    finally:
        B.tagc_profile_enable(False)
    took = B.tagc_profile_read()
    assert {"accumulate", "small"} <= set(took) and "place" not in took, took
    tb.close()
