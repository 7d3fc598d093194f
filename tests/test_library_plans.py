"""What the library decides on the host before a product: K splits, routes, and what hac_dot_noalloc takes.

Headers are made up here (no blob behind them): the decisions read the header, the batch and the launch settings only.
"""
import ctypes as C
import random

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
                                          (784, 4608, [512], 8)])
def test_index_map_product_splits_k_whatever_the_map_takes(B, n, ms, least):
    """im_dot keeps its map in the blob: its K splits (workspace / (B m floats)) do not depend on the map's size."""
    for m in ms:
        parts = hac.hac_workspace_bytes(header(hac.HAC_FORMAT_IM, n, m, n * m, 64), B) / (4 * B * m)
        assert parts == int(parts) and parts >= least, (m, parts)


def products():
    """2000 products on both sides of the array's size, most on the library's own choice of route."""
    rng = random.Random(16)

    def spread(lo, hi):
        return round(lo * (hi / lo) ** rng.random())
    for _ in range(2000):
        n, m, B = spread(1000, 30000), spread(100, 6000), spread(24, 4000)
        nnz = int(n * m * rng.uniform(0.005, 0.6))
        yield rng.choice((hac.HAC_FORMAT_HAC, hac.HAC_FORMAT_SHAC)), n, m, nnz, rng.choice((16, 64, 255, 256, 300)), B, rng.choice((0, 0, 0, 0, 0x400, 0x800))


def takes(fmt, n, m, nnz, k, B, variant):
    """hac_dot_noalloc's answer without a product: a missing X is refused after the size."""
    launch = C.byref(hac.Launch(variant=variant)) if variant else None
    return hac.load_library().hac_dot_noalloc(C.byref(header(fmt, n, m, nnz, k)), C.c_void_p(256), None, B, n, None, m, launch, None) != -6


# a bit per product: 1 where a product of its size was taken when the call was introduced (the first digit only marks the start)
TAKEN = (
    "1ee75d591f4fdff7deffdaa9f67bdcfc05eff55b8cf42bcf8efe8d0f798fbfc1fc6947bddfd44e3ffe3bf70e9efdefbfdfdb9fcb13ebecbb5be87fdd"
    "d6a1fb7ed5f4c8f749ed7fbaf7c6f77f5bdfe757cb4afaeae1e4dfbe7f59ddde3e49bf7df2cafaafcf4b9f4ed9f6f3db7ffc9f7ffefbf3def1f96fab"
    "b9d79796f175dd65bf86ff2ddd5f8fd0d87dff7d73f9f3a76c6d466fc77eeccf90d76fb6f323adf1d59ca7f675b3ef5b8becfef1cf6fb5af7b4efb9e"
    "7bcaffe779159f3f7bea337efddf60f76f3606a41cffd2fe64dd509733ef9ef73fc4897ffae9bcfafba17a8dfffed5bcdeb91efaeebdc241dfdd734c"
    "f97b5e57d835df7bfcffe")


def test_noalloc_takes_what_it_always_took():
    """A caller that sizes its batches by what the fixed array takes finds the same answers whatever the kernels' plans are."""
    want = bin(int(TAKEN, 16))[3:]
    got = "".join("1" if takes(*p) else "0" for p in products())
    assert len(want) == len(got) and [p for p, a, b in zip(products(), got, want) if a != b] == []


@pytest.mark.parametrize("n,m,prune,B", [(16269, 1661, 0.73, 170), (4772, 421, 0.85, 1997)])
def test_noalloc_takes_products_that_want_more_on_the_quicker_route(n, m, prune, B):
    """The route that is quicker in a workspace of its own needs more than the array here; the other one fits."""
    assert takes(hac.HAC_FORMAT_HAC, n, m, int(n * m * (1 - prune)), 64, B, 0)


# times of both routes, us (sparse, dense), as measured while the sparse route passed over its lists 32 columns at a time with one
# wavefront per column of W: the data that the rule of that time was fitted to, not what the routes take now (the last shape, sparse: 13 to 14)
@pytest.mark.parametrize("n,m,prune,B,sparse_us,dense_us",
                         [(15097, 501, 0.57, 246, 457, 106), (17139, 478, 0.57, 244, 430, 139), (25088, 1000, 0.90, 512, 397, 183),
                          (4608, 512, 0.60, 784, 156, 75), (25088, 4096, 0.90, 300, 812, 423), (2000, 2000, 0.80, 2048, 287, 124),
                          (4096, 4096, 0.96, 256, 54, 84), (25088, 4096, 0.98, 256, 111, 294), (512, 4096, 0.70, 64, 18, 28),
                          (9973, 1511, 0.93, 100, 45, 69), (25088, 4096, 0.98, 2048, 848, 1756), (4096, 1000, 0.90, 64, 17, 40)])
def test_the_quicker_route_is_taken(n, m, prune, B, sparse_us, dense_us):
    nnz = int(n * m * (1 - prune))
    d = header(hac.HAC_FORMAT_HAC, n, m, nnz, 32, max(4, nnz // m // 64))
    assert hac.hac_dot_route(d, B) == (1 if dense_us < sparse_us else 0)


# the same with the kernels that run now, longest column and its bits as they were: several wavefronts per column with X as it is or
# from its copy, one wavefront per column with wide and narrow passes, lists in several windows
@pytest.mark.parametrize("n,m,prune,B,k,most,bits,sparse_us,dense_us",
                         [(497, 908, 0.814, 61, 118, 121, 1333, 10, 19), (929, 11, 0.85, 285, 86, 170, 1800, 7, 18), (1424, 1275, 0.874, 36, 25, 223, 1923, 11, 23),
                          (3181, 1825, 0.86, 51, 102, 509, 4419, 17, 39), (529, 243, 0.95, 417, 219, 41, 465, 10, 20), (24391, 100, 0.5, 46, 24, 12300, 60000, 51, 153),
                          (362, 4012, 0.671, 341, 26, 158, 890, 44, 29), (6818, 765, 0.555, 333, 65, 3148, 20747, 366, 75),
                          (4962, 123, 0.617, 3884, 150, 1971, 19240, 160, 59), (22466, 1346, 0.867, 183, 58, 3147, 25129, 338, 140)])
def test_the_quicker_route_with_several_wavefronts_per_column(n, m, prune, B, k, most, bits, sparse_us, dense_us):
    nnz = int(n * m * (1 - prune))
    d = header(hac.HAC_FORMAT_HAC, n, m, nnz, k, max(4, -(-most // 64)))
    d.max_col_nnz, d.max_col_bits = most, bits
    assert hac.hac_dot_route(d, B) == (1 if dense_us < sparse_us else 0)


# columns from full to 5 or 20 % of that, headers and times as measured: where the longest column is most of a launch, where a HAC stream's emptiest
# columns leave no room for their words in the decode's LDS, and where both are as on equal columns
@pytest.mark.parametrize("fmt,n,m,B,nnz,k,lmax,chunk,n_chunks,most,bits,total,ri_bits,sparse_us,dense_us",
                         [("hac", 22082, 184, 50, 754108, 62, 21, 146, 5251, 9334, 63633, 7528560, 0, 112, 495),
                          ("hac", 19745, 706, 51, 1882098, 118, 21, 90, 21257, 5703, 50669, 24346516, 0, 158, 540),
                          ("hac", 23642, 675, 63, 2236407, 165, 22, 111, 20484, 7042, 64661, 29372980, 0, 206, 700),
                          ("hac", 16082, 3057, 41, 14845442, 15, 13, 112, 134085, 7160, 32774, 84228019, 0, 552, 208),
                          ("rice", 3709, 1965, 258, 894425, 151, 20, 16, 56823, 998, 9166, 9266475, 0, 139, 56),
                          ("rice", 2807, 3390, 314, 1036713, 25, 17, 11, 95773, 662, 4916, 8349408, 0, 159, 69),
                          ("rice", 24298, 1743, 51, 3973801, 31, 20, 88, 46021, 5569, 41873, 32768001, 0, 231, 104),
                          ("shac", 17418, 750, 48, 3352411, 35, 19, 118, 28786, 7491, 28022, 12536962, 15, 161, 73),
                          ("shac", 19166, 1839, 106, 1942956, 130, 21, 41, 48293, 2620, 14409, 10646447, 15, 208, 96),
                          ("shac", 20457, 982, 49, 4123786, 69, 21, 127, 32968, 8065, 37009, 18940005, 15, 176, 87),
                          ("hac", 2118, 3763, 165, 1763568, 193, 22, 16, 112003, 962, 8130, 19190048, 0, 114, 58),
                          ("hac", 5787, 1372, 259, 814517, 20, 17, 14, 58834, 852, 8241, 10281253, 0, 113, 61),
                          ("rice", 24157, 280, 39, 895433, 181, 20, 104, 8748, 6615, 62604, 9440111, 0, 94, 168)])
def test_the_quicker_route_with_uneven_columns(fmt, n, m, B, nnz, k, lmax, chunk, n_chunks, most, bits, total, ri_bits, sparse_us, dense_us):
    d = header(hac.HAC_FORMAT_HAC if fmt == "hac" else hac.HAC_FORMAT_SHAC, n, m, nnz, k, chunk)
    d.lmax, d.n_chunks, d.max_col_nnz, d.max_col_bits, d.total_bits, d.ri_bits = lmax, n_chunks, most, bits, total, ri_bits
    if fmt == "hac":
        d.zero_len = 1
    else:
        d.has_zero, d.ri_coding = 0, hac.RI_RICE if fmt == "rice" else hac.RI_FIELDS
    assert hac.hac_dot_route(d, B) == (1 if dense_us < sparse_us else 0)


@pytest.mark.parametrize("n,m", [(1_000_000, 1), (67_000_000, 1), (300_000, 65), (4096, 10), (25088, 4096), (100_000, 129)])
def test_device_encoder_workspace_follows_the_matrix(n, m):
    """At most as much as W beside the fixed tables (about 4 MB), whatever the matrix's shape."""
    assert hac.load_library().hac_encode_dev_workspace_bytes(n, m) <= 4_200_000 + 4 * n * m
