"""Sizes of the workspace queries (CPU)."""
import pytest


def _up(n):
    return (n + 255) // 256 * 256


def _equal_splits(S, Hq, Hkv, D, max_blocks, bs):
    """Partial results of equal splits: one round of waves, of four 32-slot tiles of the table at least."""
    waves = 1024 if D == 128 else 2048
    rows = S * Hq * min(-(-waves // (S * Hkv)), max(1, max_blocks * bs // 128))
    return _up(rows * D * 4) + _up(rows * 8)


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Hq,Hkv", [(32, 8), (40, 8), (16, 1), (12, 12), (24, 3)])
def test_decode_query_follows_equal_splits(Hq, Hkv, D):
    """A wide table's decode asks for no more than equal splits take and what its units are looked up in, a narrow
    one's for at most three times that (five to seven tiles make one split of four or more, but three of two)."""
    from paper_2609_35750_amd.kvs import lib

    for S in (1, 2, 7, 24, 64, 128, 200, 257, 600, 4096):
        for max_blocks in (1, 4, 20, 100, 700, 5000):
            got = lib.kvs_paged_decode_workspace(S, Hq, Hkv, D, max_blocks, 16)
            equal = _equal_splits(S, Hq, Hkv, D, max_blocks, 16)
            assert got >= equal
            waves = 1024 if D == 128 else 2048
            wide = max_blocks * 16 >= 128 * -(-waves // (S * Hkv))
            assert got <= (1 if wide else 3) * equal + 32 * waves + 16 * S + 4096, (S, max_blocks)
