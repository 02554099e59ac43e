"""The dense output written by the decoder's workgroups, partition by partition (there are three
turns of partitions or more), and what is left of it for the launch behind: ranges that start and end anywhere,
ranges longer than what is put together at once, ranges much longer than the others, partitions without an
unknown, nothing kept at all, against the oracle.  Small integers, so values must agree bit for bit.  The
output is filled with something else before the call that is looked at, and the call's kernels are those of
this form."""
import numpy as np
import pytest
import torch

from oracle import tagc_oracle as O
from paper_2504_05638_amd import binding as B
from synth import gradients as G
from tests.helpers import run_both, compare_all

pytestmark = pytest.mark.gpu


def _check(b, grads, kernels=("dense_rest",), **kw):
    """Returns the oracle's result and the kernels of the call: {name: (ms, launches)}."""
    fused = kw.get("fused", False)
    ores, tb = run_both(b, grads, seed=5, **kw)
    dev = [g.cuda() for g in grads]
    tb.out_dense.fill_(0x55)
    torch.cuda.synchronize()
    B.tagc_profile_enable(True)
    try:
        tb.run(dev, fused=fused)
        torch.cuda.synchronize()
    finally:
        B.tagc_profile_enable(False)
    took = B.tagc_profile_read()
    assert {"dense_rest", "dense"} & set(took) == set(kernels), took
    compare_all(b, ores, tb, exact_values=True)
    return ores, took


# Whose output the decoder writes itself: partitions of at most four even shares, if there are three turns
# of them on a device of 256 compute units.
def _own(ores):
    length = np.diff(np.append(0, ores.bnd[1:]).astype(np.int64))
    return length[length // 4 <= ores.n_c // ores.A] if ores.A >= 3 * 256 else length[:0]


@pytest.mark.parametrize("P,T", [(32, 48), (33, 48), (24, 39)])
@pytest.mark.parametrize("ranks,fused", [(1, False), (2, True), (4, True), (3, False)])
@pytest.mark.parametrize("milli,mode", [(1500, O.DECODE_PEEL), (1150, O.DECODE_PEEL_ESTIMATE)])
def test_ranges_of_any_length(P, T, ranks, fused, milli, mode):
    print("\n[case] dense in decoder P=%d ranks=%d fused=%d milli=%d" % (P, ranks, fused, milli), flush=True)
    # a quarter kept; one entry in ten thousand over four pieces' length; two fifths kept
    segs = [G.Seg(0, 100_003, 250_000, 1, "a"), G.Seg(100_008, 149_997, 100, 1, "b"),
            G.Seg(250_008, 3001, 400_000, 1, "c")]
    n = 253_009
    b = G.Bucket("dense_in_decoder", G.F32, ranks, segs, n, milli)
    rng = np.random.default_rng(ranks)
    grads = [torch.from_numpy(rng.integers(-1000, 1001, n).astype(np.float32)) for _ in range(ranks)]
    ores, _ = _check(b, grads, P=P, T=T, fused=fused, decode_mode=mode)
    # (the second layer's few partitions are not for the decoder)
    assert 0.9 * ores.A < _own(ores).size < ores.A


# One rank: 91 thousand c-indices a partition in the first layer, 30 thousand in the second (three pieces, and one); two: half of that
@pytest.mark.parametrize("ranks,fused", [(1, False), (2, True)])
def test_ranges_of_several_pieces(ranks, fused):
    print("\n[case] dense in decoder, several pieces, ranks=%d" % ranks, flush=True)
    n = 40_000_037
    segs = [G.Seg(0, 20_000_001, 350, 1, "a"), G.Seg(20_000_008, 20_000_029, 1050, 1, "b")]
    b = G.Bucket("dense_in_decoder", G.F32, ranks, segs, n, 1500)
    rng = np.random.default_rng(ranks)
    # (up to 32 values and a second rank's in a partition: sums below 2^24 unless half of them share a cell)
    grads = [torch.from_numpy(rng.integers(-500_000, 500_001, n).astype(np.float32)) for _ in range(ranks)]
    ores, _ = _check(b, grads, P=32, T=48, fused=fused)
    own = _own(ores)
    assert own.size >= 3 * 256 and own.min() <= 36_864 and own.max() > 36_864 * (3 - ranks)


@pytest.mark.parametrize("kept", [0, 1, 3])
@pytest.mark.parametrize("fused", [False, True])
def test_hardly_anything_kept(kept, fused):
    print("\n[case] dense in decoder kept=%d fused=%d" % (kept, fused), flush=True)
    n = 200_001
    b = G.Bucket("dense_in_decoder", G.F32, 2, [G.Seg(0, n, 250_000, 1, "w")], n, 4000)
    grads = [torch.zeros(n) for _ in range(2)]
    for r, g in enumerate(grads):
        g[[0, 77, n - 1][:kept]] = float(r + 1)
    ores, _ = _check(b, grads, P=32, T=48, sizing=O.SIZE_FIXED_RATIO, fused=fused)
    assert ores.A >= 3 * 256 if kept else ores.A == 0


def test_default_partitions():
    print("\n[case] dense in decoder, default partitions", flush=True)
    n = 7_200_001
    b = G.Bucket("dense_in_decoder", G.BF16, 1, [G.Seg(0, n, 900_000, 1, "w")], n, 1500)
    g = torch.randint(-200, 201, (n,), generator=torch.Generator().manual_seed(3)).to(torch.bfloat16)
    ores, _ = _check(b, [g], fused=True)
    assert _own(ores).size == ores.A


def test_a_plan_of_one_turn():
    print("\n[case] dense in decoder, one turn", flush=True)
    n = 20_001
    b = G.Bucket("dense_in_decoder", G.F32, 1, [G.Seg(0, n, 250_000, 1, "w")], n, 1500)
    g = torch.from_numpy(np.random.default_rng(0).integers(-1000, 1001, n).astype(np.float32))
    _check(b, [g], P=32, T=48, kernels=())  # (its zeros come from workgroups without a partition)
    _check(b, [g], P=32, T=48, kernels=("dense",), decode_workgroups=157)


# Ranges far longer than the others', or far fewer partitions than the plan has room for: one workgroup
# stores some 30 GB/s, which is 2 ms for the 64 MB of such a range.
@pytest.mark.parametrize("what", ["one segment keeps little", "a plan's few partitions", "mostly zeros, fixed ratio"])
@pytest.mark.parametrize("ranks,fused", [(1, False), (2, True)])
def test_long_ranges_go_to_the_whole_device(what, ranks, fused):
    print("\n[case] dense in decoder, %s, ranks=%d" % (what, ranks), flush=True)
    n, sizing, milli = 16_000_000, O.SIZE_LOAD_FACTOR, 1500
    segs = [G.Seg(0, n, 8000, 1, "a")]
    if what == "one segment keeps little":
        segs = [G.Seg(0, n, 5, 1, "a"), G.Seg(n, 256_000, 250_000, 1, "b"), G.Seg(n + 256_000, n, 5, 1, "c")]
        n = 2 * n + 256_000
    elif what.endswith("ratio"):
        sizing, milli = O.SIZE_FIXED_RATIO, 100_000
    b = G.Bucket("dense_in_decoder", G.F32, ranks, segs, n, milli)
    rng = np.random.default_rng(ranks)
    grads = []
    for _ in range(ranks):
        if len(segs) == 3:
            g = rng.integers(1, 1001, n).astype(np.float32)
        else:  # (all within the first thousandth: the last partitions' range is the rest)
            g = np.zeros(n, np.float32)
            g[rng.choice(n // 1000, 3000, replace=False)] = rng.integers(1, 1001, 3000)
        grads.append(torch.from_numpy(g))
    ores, took = _check(b, grads, P=32, T=48, sizing=sizing, fused=fused)
    # (12 us a turn of rounds, 14 turns in the largest case; 30 GB/s for what lies between two ends)
    longest = 4 * np.diff(ores.bnd.astype(np.int64)).max() / 30e6
    assert took["sum_peel" if fused else "peel"][0] + took["dense_rest"][0] < 0.5 < longest
