"""Sizes just below the format's 2^32 elements: planned for as long as every count of
its own can be indexed (host only, no device work)."""
import pytest

from paper_2105_12912_amd import ebc


@pytest.mark.parametrize("rank,dims,options", [
    (2, (1, 4_294_000_000), {}), (2, (1, 4_294_000_000), dict(codec="huffman")),
    (2, (1, 4_294_000_000), dict(codec="rle_vle")), (2, (1, 4_294_000_000), dict(n_bins=65536)),
    (2, (1, 4_230_000_000), dict(huff_chunk=64)), (3, (1, 65535, 65535), {}), (1, ((1 << 32) - 1,), {}),
    (2, (65536, 65535), dict(huff_chunk=64, dtype=ebc.EBC_F64)),
])
def test_large_fields_are_planned(rank, dims, options):
    n = 1
    for d in dims:
        n *= d
    assert ebc.ebc_compress_workspace_size(rank, dims, ebc.make_params(1e-3, **options)) > 6 * n
