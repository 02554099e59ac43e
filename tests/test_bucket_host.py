"""TagcBucket's and the binding's host side, without a device."""
import types

import pytest
import torch

from paper_2504_05638_amd import binding as B
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


class _Grad:
    """Stands in for a gradient on the device."""
    dtype, is_cuda = torch.float32, True

    def __init__(self, at):
        self.at = at

    def data_ptr(self):
        return self.at

    def is_contiguous(self):
        return True

    def numel(self):
        return 1000


class _Stacked:
    """A tensor with a row per rank, as far as a caller of run() can tell: it has a length and rows,
    and no truth value."""
    def __init__(self, rows):
        self.rows = rows

    def __len__(self):
        return len(self.rows)

    def __getitem__(self, r):
        return self.rows[r]

    def __bool__(self):
        raise RuntimeError("Boolean value of Tensor with more than one value is ambiguous")


def _bucket(n_ranks):
    tb = TagcBucket.__new__(TagcBucket)
    tb.plan = tb.plan_whole = tb.shared = None
    tb.cfg, tb.n_ranks, tb._ranks_together = B.tagc_config(dtype=B.TAGC_F32), n_ranks, 0
    tb.sizes = types.SimpleNamespace(grad_elems=1000)
    tb.rk = (B.tagc_rank_buffers * n_ranks)()
    return tb


def test_rows_of_one_tensor_as_gradients(monkeypatch):
    """run() takes whatever has a length and rank r's buffer at [r]."""
    calls = []
    monkeypatch.setattr(B, "tagc_compress_ranks",
                        lambda plan, phase, grads, ranks, shared, stream, n: calls.append((grads, n)))
    tb, stream = _bucket(3), types.SimpleNamespace(cuda_stream=0)
    for kind in (list, tuple, _Stacked, lambda rows: dict(enumerate(rows))):
        calls.clear()
        tb.compress_index_all(kind([_Grad(256 * (r + 1)) for r in range(3)]), stream)
        assert calls == [([256, 512, 768], 3)]
    calls.clear()
    tb.compress_index_all([], stream)
    tb.compress_index_all(torch.empty(0, 1000), stream)
    assert not calls


def test_no_more_ranks_than_there_are():
    """A number of ranks beyond the buffers given never reaches the library, which would read
    past them; a bucket's n_ranks is the end of a slice, as of its list of ranks."""
    tb = _bucket(4)
    assert [tb._n(n) for n in (None, 0, 1, 4, 9, -1, -9)] == [4, 4, 1, 4, 4, 3, 0]
    plan = B.tagc_plan(B.tagc_config(dtype=0, n_ranks=8, n_hash=3, sizing_milli=1500),
                       [(0, 1000, 10_000, 1)])
    sh, ranks = B.tagc_shared_buffers(), [B.tagc_rank_buffers()] * 2
    for arr in (ranks, (B.tagc_rank_buffers * 2)(*ranks)):
        for n in (3, 8, -1):
            with pytest.raises(ValueError):
                B.tagc_compress_ranks(plan, B.TAGC_PHASE_INDEX, [256] * max(n, 0), arr, sh, 0, n)
            with pytest.raises(ValueError):
                B.tagc_aggregate(plan, B.TAGC_PHASE_INDEX, arr, sh, 0, n)
            with pytest.raises(ValueError):
                B.tagc_reduce_decompress(plan, arr, sh, 256, 256, None, 0, n)
        for grads in ([256], [256] * 3):
            with pytest.raises(ValueError):
                B.tagc_compress_ranks(plan, B.TAGC_PHASE_INDEX, grads, arr, sh)
        with pytest.raises(B.TagcError):     # (null buffers: the library's own refusal)
            B.tagc_aggregate(plan, B.TAGC_PHASE_INDEX, arr, sh, 0, 2)
        with pytest.raises(B.TagcError):
            B.tagc_aggregate(plan, B.TAGC_PHASE_INDEX, arr, sh, 0, 0)
    B.tagc_plan_destroy(plan)


def test_ranks_together_holds_for_the_sketches(monkeypatch):
    """Every rank once, in order, as many to a call as the bucket was asked for."""
    calls = []
    monkeypatch.setattr(B, "tagc_compress_ranks",
                        lambda plan, phase, grads, ranks, shared, stream, n:
                        calls.append([ranks[r].idx for r in range(n)]))
    tb, stream = _bucket(5), types.SimpleNamespace(cuda_stream=0)
    for r in range(5):
        tb.rk[r].idx = 4096 + 16 * r
    every = [4096 + 16 * r for r in range(5)]
    for together, n, want in ((0, None, [every]), (1, None, [[i] for i in every]),
                              (2, None, [every[:2], every[2:4], every[4:]]), (8, None, [every]),
                              (2, 3, [every[:2], every[2:3]])):
        calls.clear()
        tb._ranks_together = together
        tb.compress_sketch_all(n, stream)
        assert calls == want
