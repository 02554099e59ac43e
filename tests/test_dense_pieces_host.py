"""The pieces in which the decoder writes a partition's dense output: they follow each other, cover its
range and end, also where the range ends just below 2^32 (the largest c-index space a plan accepts has
2^32 - 32 entries) and a step behind the last piece would wrap."""
import pytest

from paper_2504_05638_amd import binding as B

END = 2 ** 32 - 32


@pytest.mark.parametrize("hi", [1, 5, 36_864, 36_865, 250_003, 2 ** 31, END - 36_864, END - 4096, END])
@pytest.mark.parametrize("length", [1, 3, 4, 36_863, 36_864, 36_865, 100_001, 3_000_000])
def test_pieces_cover_a_range(hi, length):
    lo = max(0, hi - length)
    pieces = B.tagc_dense_pieces_host(lo, hi)
    assert pieces is not None
    at = lo & ~3
    for first, n in pieces:
        assert first == at and n % 4 == 0 and 0 < n <= 36_864
        at += n
    assert hi <= at < hi + 4 and len(pieces) == -(-(hi - (lo & ~3)) // 36_864)
