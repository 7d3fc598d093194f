"""What the library decides on the host before a product: K splits, routes, and what hac_dot_noalloc takes.

Headers are made up here (no blob behind them): the decisions read the header, the batch and the launch settings only.
"""
import ctypes as C

import pytest

import paper_2108_12704_amd as hac


def header(fmt, n, m, nnz, k, chunk=64):
    return hac.Desc(magic=0x31434148, version=2, format=fmt, header_bytes=256, n=n, m=m, nnz=nnz, k_sym=k, lut_bits=10, lmax=12,
                    chunk=chunk, n_chunks=max(1, nnz // chunk), ent_bits=8 if fmt == hac.HAC_FORMAT_IM else 32,
                    max_col_nnz=max(1, 2 * nnz // m), max_col_bits=max(1, 20 * nnz // m), has_zero=1,
                    idx_pitch=(m + 15) // 16 * 16)


# maps around 8 MB (8-bit pointers: as much as the 16 MB of hac_dot_noalloc hold twice) and a smaller one; few output tiles
@pytest.mark.parametrize("B,n,ms,least", [(64, 4608, range(1600, 2000, 16), 8), (64, 4096, range(3900, 4200, 16), 8),
                                          (64, 4096, range(1936, 2144, 16), 8), (200, 4608, range(3500, 3760, 16), 4),
                                          (784, 4608, [512], 9)])
def test_index_map_product_splits_k_whatever_the_map_takes(B, n, ms, least):
    """im_dot keeps its map in the blob: its K splits (workspace / (B m floats)) do not depend on the map's size."""
    for m in ms:
        parts = hac.hac_workspace_bytes(header(hac.HAC_FORMAT_IM, n, m, n * m, 64), B) / (4 * B * m)
        assert parts == int(parts) and parts >= least, (m, parts)
