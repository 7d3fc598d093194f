"""GPU parity of the matrix-core paths: im_dot (index map, Sect. III-C1) and the dense
route of hac_dot / shac_dot (decode to an index map, then MFMA tiles).

Same bar as the vector path: |Y - Yref|_ij <= 1e-5 (|X| . |W|)_ij and
max |Y - Yref| <= 1e-5 max |Yref|, Yref the dense fp64 product of the oracle.
"""
import numpy as np
import pytest

import workloads
from oracle import dot as odot
from oracle import indexmap

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-5
SPARSE, DENSE = 0x400, 0x800


@pytest.fixture(scope="module")
def hac():
    import paper_2108_12704_amd as lib
    lib.load_library()
    assert torch.cuda.is_available(), "GPU tests need a device"
    return lib


def dev():
    return torch.device("cuda:0")


def check_y(Y, X, W, what=""):
    ref = odot.dense_dot(X, W)
    scale = odot.abs_dot(X, W)
    got = Y.detach().cpu().numpy().astype(np.float64)
    assert got.shape == ref.shape, what
    err = np.abs(got - ref)
    bad = err > TOL * scale + 1e-37
    assert not bad.any(), f"{what}: {int(bad.sum())} entries off, worst {float((err / (scale + 1e-300)).max()):.3e}"
    if ref.size and np.abs(ref).max() > 0:
        assert err.max() <= TOL * np.abs(ref).max(), what


def dense_layers():
    yield "cfg5-640x33", workloads.scaled(5, 640, 33)
    yield "cfg5-300x129", workloads.scaled(5, 300, 129)
    yield "cfg5-97x200", workloads.scaled(5, 97, 200)
    yield "cfg5-2100x40", workloads.scaled(5, 2100, 40)                                # K loop split into 8
    yield "unpruned-257x256", workloads.make_layer(257, 256, 0.02, 0.0, 64, "kmeans", 5)
    yield "cfg1", workloads.layer(1)
    yield "no_repeats_40x30", workloads.stress_cases()["no_repeats_40x30"]             # 16-bit pointers
    rng = np.random.default_rng(8)
    yield "distinct-100x60", rng.permutation(np.arange(1, 6001, dtype=np.float32)).reshape(100, 60) / np.float32(64)
    for name, W in workloads.edge_cases().items():
        yield name, W


LAYERS = list(dense_layers())
IDS = [c[0] for c in LAYERS]
BATCHES = [1, 2, 5, 8, 9, 64, 127, 128, 129, 300]


@pytest.mark.parametrize("name,W", LAYERS, ids=IDS)
def test_im_dot_parity(hac, name, W):
    n, m = W.shape
    blob = hac.im_encode(W)
    im = indexmap.im_encode(W)
    assert int(blob.desc.ent_bits) == im.bbar and int(blob.desc.k_sym) == im.c.size
    db = blob.to_device(dev())
    for B in BATCHES:
        print(f"[case] im_dot {name} {W.shape} B={B}", flush=True)
        X = workloads.make_batch(B, n, 31 + B) - np.float32(0.125)
        Y = hac.im_dot(db, torch.from_numpy(X).to(dev()))
        torch.cuda.synchronize()
        check_y(Y, X, W, f"im {name} B={B}")


def test_im_dot_small_batch_on_a_tall_map_with_a_long_value_list(hac):
    """At most 32 rows of X against a tall index map: the blocks of the small-batch kernel then hold
    close to a thousand rows of X, the partial sums of their row groups and the representatives in
    LDS, more than a kernel gets without asking for it."""
    W = workloads.make_layer(25088, 64, 0.02, 0.0, 256, "kmeans", 77)
    blob = hac.im_encode(W)
    assert int(blob.desc.k_sym) >= 200
    db = blob.to_device(dev())
    for B in (32, 9):
        print(f"[case] im_dot tall map B={B}", flush=True)
        X = workloads.make_batch(B, W.shape[0], 12 + B)
        Y = hac.im_dot(db, torch.from_numpy(X).to(dev()))
        torch.cuda.synchronize()
        check_y(Y, X, W, f"tall map B={B}")
    # the same shape as the dense route of a pruned layer forced at a small batch
    Wp = workloads.make_layer(25088, 64, 0.02, 0.6, 256, "kmeans", 78)
    dbp = hac.hac_encode(Wp).to_device(dev())
    X = workloads.make_batch(32, Wp.shape[0], 5)
    print("[case] dense route forced at B=32 on a tall layer", flush=True)
    Y = hac.hac_dot(dbp, torch.from_numpy(X).to(dev()), launch=hac.Launch(variant=DENSE))
    torch.cuda.synchronize()
    check_y(Y, X, Wp, "dense route tall")


def test_im_dot_strided_and_unaligned(hac):
    W = workloads.scaled(5, 301, 70)
    db = hac.im_encode(W).to_device(dev())
    for rows in (40, 6):                                          # the matrix-core kernel, and the one for small batches
        Xbig = torch.from_numpy(workloads.make_batch(rows, 310, 2)).to(dev())
        Ybig = torch.full((rows, 90), 3.0, device=dev())
        for shift in (0, 1, 4):
            X = Xbig[:, shift:shift + 301]                       # ldx = 310, pointer offset by `shift` floats
            Y = Ybig[:, 7:77]
            hac.im_dot(db, X, Y=Y)
            torch.cuda.synchronize()
            check_y(Y, X.cpu().numpy(), W, f"rows {rows} shift {shift}")
            assert torch.all(Ybig[:, :7] == 3.0) and torch.all(Ybig[:, 77:] == 3.0)


@pytest.mark.parametrize("name,W", LAYERS, ids=IDS)
def test_dense_route_matches_the_oracle(hac, name, W):
    n, m = W.shape
    blobs = [("hac", hac.hac_dot, hac.hac_encode(W)), ("shac", hac.shac_dot, hac.shac_encode(W)),
             ("shac/rice", hac.shac_dot, hac.shac_encode(W, ri_coding=1)),
             ("hac c=3", hac.hac_dot, hac.hac_encode(W, chunk_nnz=3))]
    for what, f, blob in blobs:
        db = blob.to_device(dev())
        for B in (1, 3, 8, 9, 33, 128, 200):
            print(f"[case] dense route {what} {name} {W.shape} B={B}", flush=True)
            X = workloads.make_batch(B, n, 3 + B) - np.float32(0.2)
            Y = f(db, torch.from_numpy(X).to(dev()), launch=hac.Launch(variant=DENSE))
            torch.cuda.synchronize()
            check_y(Y, X, W, f"{what} dense {name} B={B}")


def test_dense_route_decode_without_its_lds_copies(hac):
    # the decode kernel keeps a block's stream words, ri fields and the column index in LDS when
    # they fit; these layers do not fit: 256 chunks of a very sparse, tall HAC layer span more
    # stream words than the staging area ever has (20480), 256 chunks of 500 non-zeros carry more ri bits than
    # there is ever room for (28672 words), 256 chunks of 700 with Rice-coded gaps more words again, and a layer with more
    # than 8191 columns has too long an index
    tall = workloads.make_layer(30000, 24, 0.02, 0.999, 8, "uniform", 71)
    fat = workloads.make_layer(8000, 300, 0.02, 0.5, 16, "uniform", 72)
    wide = workloads.make_layer(24, 9000, 0.02, 0.7, 8, "uniform", 73)
    cases = [("tall", tall, hac.hac_encode(tall), hac.hac_dot), ("tall/rice", tall, hac.shac_encode(tall, ri_coding=1), hac.shac_dot),
             ("fat ri", fat, hac.shac_encode(fat, chunk_nnz=500), hac.shac_dot),
             ("fat rice", fat, hac.shac_encode(fat, ri_coding=1, chunk_nnz=700), hac.shac_dot),
             ("wide", wide, hac.hac_encode(wide), hac.hac_dot), ("wide", wide, hac.shac_encode(wide), hac.shac_dot)]
    descs = {what: blob.desc for what, _, blob, _ in cases}
    assert descs["tall"].n_chunks <= 256 and descs["tall"].n_words > 20480                    # one block
    assert 256 * 500 * descs["fat ri"].ri_bits / 32 > 28672 and descs["fat ri"].n_chunks > 256
    assert 0.9 * 256 * 700 * descs["fat rice"].total_bits / descs["fat rice"].nnz / 32 > 20480
    for what, W, blob, f in cases:
        db = blob.to_device(dev())
        for B in (1, 33):
            print(f"[case] dense route, decode from the blob: {what} {W.shape} B={B}", flush=True)
            X = workloads.make_batch(B, W.shape[0], 9 + B) - np.float32(0.2)
            Y = f(db, torch.from_numpy(X).to(dev()), launch=hac.Launch(variant=DENSE))
            torch.cuda.synchronize()
            check_y(Y, X, W, f"{what} B={B}")


def test_route_selection_and_workspace(hac):
    W = workloads.scaled(5, 2100, 70)                        # 40 % non-zero
    n, m = W.shape
    pitch = 80
    for enc, f in ((hac.hac_encode, hac.hac_dot), (hac.shac_encode, hac.shac_dot)):
        b = enc(W)
        bits = 8 if int(b.desc.k_sym) + (0 if enc is hac.hac_encode else 1) <= 256 else 16
        idx_bytes = (n * pitch * bits // 8 + 255) // 256 * 256
        db = b.to_device(dev())
        for B in (40, 256, 700):
            X = workloads.make_batch(B, n, 1)
            Xd = torch.from_numpy(X).to(dev())
            route = hac.hac_dot_route(b.desc, B)
            need = hac.hac_workspace_bytes(b.desc, B)
            if route == 0:
                assert need == 4 * n * (-(-B // 256) * 256 if B > 256 else 1 << (B - 1).bit_length())
            else:
                assert need >= idx_bytes                                       # index map (+ partial tiles)
            dense = hac.Launch(variant=DENSE)
            assert hac.hac_dot_route(b.desc, B, dense) == 1 and hac.hac_dot_route(b.desc, B, hac.Launch(variant=SPARSE)) == 0
            assert hac.hac_workspace_bytes(b.desc, B, dense) >= idx_bytes
            Y0 = f(db, Xd)
            Yd = f(db, Xd, launch=dense)
            Ys = f(db, Xd, launch=hac.Launch(variant=SPARSE))
            torch.cuda.synchronize()
            for Y, what in ((Y0, "default"), (Yd, "dense"), (Ys, "sparse")):
                check_y(Y, X, W, f"{f.__name__} {what} B={B}")
            assert torch.equal(Y0, Yd if route == 1 else Ys)                   # the default is one of the two, bit for bit
            assert torch.equal(Yd, f(db, Xd, launch=dense))                    # split-K parts are added in a fixed order
        Xd = torch.from_numpy(workloads.make_batch(256, n, 1)).to(dev())
        small = torch.empty(256, dtype=torch.uint8, device=dev())
        with pytest.raises(hac.HacError) as e:
            f(db, Xd, workspace=small, launch=hac.Launch(variant=DENSE))
        assert e.value.status == -6
        with pytest.raises(hac.HacError) as e:
            f(db, Xd, launch=hac.Launch(variant=SPARSE | DENSE))
        assert e.value.status == -1


def test_im_dot_argument_checks(hac):
    import ctypes as C
    lib = hac.load_library()
    W = workloads.scaled(5, 100, 20)
    ib = hac.im_encode(W).to_device(dev())
    hb = hac.hac_encode(W).to_device(dev())
    X = torch.zeros((4, 100), device=dev())
    with pytest.raises(hac.HacError) as e:
        hac.im_dot(hb, X)                                    # a HAC blob
    assert e.value.status == -1
    with pytest.raises(hac.HacError) as e:
        hac.hac_dot(ib, X)                                   # an index map given to hac_dot
    assert e.value.status == -1
    Y = torch.empty((4, 20), device=dev())
    assert lib.im_dot(C.byref(ib.desc), ib.tensor.data_ptr(), X.data_ptr(), 4, 50, Y.data_ptr(), 20, None, 0, None, None) == -1
    assert lib.im_dot(C.byref(ib.desc), ib.tensor.data_ptr(), None, 0, 100, None, 20, None, 0, None, None) == 0
    tall = hac.im_encode(workloads.scaled(5, 2100, 20))      # few tiles, long K: partial tiles need a workspace
    assert hac.hac_workspace_bytes(tall.desc, 4) > 0
    td = tall.to_device(dev())
    X = torch.zeros((4, 2100), device=dev())
    assert lib.im_dot(C.byref(td.desc), td.tensor.data_ptr(), X.data_ptr(), 4, 2100, Y.data_ptr(), 20, None, 0, None, None) == -6
    torch.cuda.synchronize()


@pytest.mark.parametrize("B,n,m", [(33, 31, 5), (64, 32, 128), (65, 33, 129), (225, 300, 20), (700, 517, 260)])
@pytest.mark.parametrize("bits", [8, 16])
def test_split_operands(hac, B, n, m, bits):
    """Operands of 24 significant bits over a wide range of magnitudes, strided X; every product needs its
    second- and third-order parts for this bound: fp32 sums of n terms in any order, (n + 8) 2^-24 |X| . |W|."""
    rng = np.random.default_rng(B * 1000 + n + bits)
    k = 100 if bits == 8 else 700
    reps = (rng.standard_normal(k) * np.exp2(rng.integers(-12, 12, k))).astype(np.float32)
    W = rng.choice(reps, (n, m))
    W.flat[:min(k, W.size)] = reps[:min(k, W.size)]
    X = (rng.standard_normal((B, n)) * np.exp2(rng.integers(-12, 12, (B, n)))).astype(np.float32)
    Xd = torch.zeros((B, n + 3), device=dev())[:, :n]
    Xd.copy_(torch.from_numpy(X))
    Y = hac.im_dot(hac.im_encode(W).to_device(dev()), Xd).cpu().numpy().astype(np.float64)
    err = np.abs(Y - X.astype(np.float64) @ W.astype(np.float64))
    bound = (n + 8) * 2.0 ** -24 * (np.abs(X).astype(np.float64) @ np.abs(W).astype(np.float64))
    assert (err <= bound).all(), float((err / bound).max())


# two to four row tiles a block, dealt unevenly (some blocks one less); one to five K steps, a partial last one; one and several
# K splits; a value list that leaves room for fewer row tiles (3000); X at any row length
@pytest.mark.parametrize("B,n,m", [(3130, 33, 1000), (3130, 97, 1000), (3130, 900, 5), (12530, 31, 260), (12530, 65, 260),
                                   (3130, 17, 2000), (3130, 97, 2000), (3130, 130, 2000), (12530, 1000, 5), (33, 65, 5)])
@pytest.mark.parametrize("k", [64, 700, 3000])
def test_row_tiles_dealt_unevenly(hac, B, n, m, k):
    """fp32 sums of n terms in any order: (n + 8) 2^-24 |X| . |W|."""
    rng = np.random.default_rng(B + n + m + k)
    W = rng.standard_normal(k).astype(np.float32)[rng.integers(0, k, (n, m))]
    X = np.maximum(rng.standard_normal((B, n)), 0).astype(np.float32)
    Xd = torch.zeros((B, n + 1 + k % 3), device=dev())[:, :n]
    Xd.copy_(torch.from_numpy(X))
    Y = torch.full((B, m + 2), float("nan"), device=dev())
    hac.im_dot(hac.im_encode(W).to_device(dev()), Xd, Y=Y[:, :m])
    Y = Y.cpu().numpy().astype(np.float64)
    err = np.abs(Y[:, :m] - X.astype(np.float64) @ W.astype(np.float64))
    bound = (n + 8) * 2.0 ** -24 * (X.astype(np.float64) @ np.abs(W).astype(np.float64)) + n * 2.0 ** -149
    assert (err <= bound).all() and np.isnan(Y[:, m:]).all()


def test_not_finite_and_largest(hac):
    """Infinities, NaN and values near the largest float give what fp32 products and sums give."""
    W = workloads.make_layer(257, 130, 0.02, 0.0, 64, "kmeans", 5)
    X = workloads.make_batch(70, 257, 3)
    X[3, 7], X[11, 256], X[40, 0] = np.inf, np.nan, -np.inf
    X[64, 5], X[65, 5] = 3.4e38, -3.4e38
    X[66, 6] = np.array([0x7f800001], np.uint32).view(np.float32)[0]      # a NaN in its lowest bit only
    Y = hac.im_dot(hac.im_encode(W).to_device(dev()), torch.from_numpy(X).to(dev())).cpu().numpy()
    with np.errstate(invalid="ignore"):
        ref = X.astype(np.float64) @ W.astype(np.float64)
    assert np.array_equal(np.isnan(Y), np.isnan(ref)) and np.array_equal(np.isinf(Y), np.isinf(ref))
    ok = np.isfinite(ref)
    scale = np.abs(np.where(np.isfinite(X), X, 0)).astype(np.float64) @ np.abs(W).astype(np.float64)
    assert (np.abs(Y[ok] - ref[ok]) <= TOL * scale[ok]).all()
    assert np.array_equal(Y[~ok & ~np.isnan(ref)], ref[~ok & ~np.isnan(ref)])


def product_bound(X, W, factor):
    """factor 2^-24 |X| . |W|, and what lies below the smallest fp32."""
    return factor * 2.0 ** -24 * (np.abs(X).astype(np.float64) @ np.abs(W).astype(np.float64)) + X.shape[1] * 2.0 ** -149


# every row tile count, one and several K splits, pointers of 8 and 16 bits, a value list that fits LDS and one that does not
@pytest.mark.parametrize("B,n,m,k", [(33, 700, 130, 64), (100, 2100, 40, 300), (300, 96, 1000, 64), (2000, 257, 520, 5000)])
@pytest.mark.parametrize("where", ["first", "last", "all"])
def test_rows_that_are_not_finite(hac, B, n, m, k, where):
    """A tile with infinities or NaN is computed in fp32: those rows are what fp32 gives, the others stay right."""
    rng = np.random.default_rng(B + n)
    reps = rng.standard_normal(k).astype(np.float32)
    W = rng.choice(reps, (n, m))
    X = rng.standard_normal((B, n)).astype(np.float32)
    rows = np.arange(0, B, 7)
    if where == "all":
        X[rows] = np.nan
        X[rows + 1 - (rows + 1) // B] = np.inf
    else:
        X[rows, 0 if where == "first" else n - 1] = np.where(np.arange(rows.size) % 2, np.nan, -np.inf)
    print(f"[case] not finite {where}: {B} x {n} x {m}, k = {k}", flush=True)
    Y = hac.im_dot(hac.im_encode(W).to_device(dev()), torch.from_numpy(X).to(dev())).cpu().numpy()
    with np.errstate(invalid="ignore"):
        ref = X.astype(np.float64) @ W.astype(np.float64)
    assert np.array_equal(np.isnan(Y), np.isnan(ref)) and np.array_equal(np.isinf(Y), np.isinf(ref))
    assert np.array_equal(Y[np.isinf(ref)], ref[np.isinf(ref)])
    ok = np.isfinite(X).all(axis=1)
    assert (np.abs(Y[ok] - ref[ok]) <= product_bound(X[ok], W, n + 8)).all()


def test_a_batch_of_nan_costs_about_as_much(hac):
    """The fp32 tile pass takes about twice the time of the parts (1.6 to 2.7 times as measured); one thread per output took 60 times."""
    B, n, m = 784, 2304, 512
    db = hac.im_encode(np.random.default_rng(1).choice(np.linspace(-1, 1, 50).astype(np.float32), (n, m))).to_device(dev())
    Y = torch.empty((B, m), device=dev())
    ws = torch.empty(hac.hac_workspace_bytes(db.desc, B) + 256, dtype=torch.uint8, device=dev())

    def seconds(X):
        best = float("inf")
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                hac.im_dot(db, X, Y=Y, workspace=ws)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        return best
    X = torch.randn((B, n), device=dev())
    plain = seconds(X)
    X[:, n // 2] = float("nan")
    assert seconds(X) < 8 * plain
    assert seconds(torch.full_like(X, float("inf"))) < 8 * plain


# exponents of X and of W: at and below where a third bf16 part runs out of room, subnormal X, W, and products just above
# the smallest normal number from operands that are not small
@pytest.mark.parametrize("ex,ew", [(-104, 0), (-109, 0), (-111, 0), (-118, 20), (-126, 20), (-135, 30), (0, -109), (0, -118), (20, -126), (-70, -50)])
@pytest.mark.parametrize("B,n,m,k", [(33, 700, 130, 64), (300, 96, 200, 5000)])
def test_small_operands(hac, ex, ew, B, n, m, k):
    """Operands of any size keep all their bits (as products and sums of fp32 do)."""
    rng = np.random.default_rng(B + 200 + ex)
    W = rng.choice((rng.uniform(1, 2, k) * 2.0 ** ew).astype(np.float32), (n, m))        # one sign: bits that are cut add up
    X = (rng.uniform(1, 2, (B, n)) * 2.0 ** ex).astype(np.float32)
    print(f"[case] small operands 2^{ex} x 2^{ew}", flush=True)
    Y = hac.im_dot(hac.im_encode(W).to_device(dev()), torch.from_numpy(X).to(dev())).cpu().numpy().astype(np.float64)
    err = np.abs(Y - X.astype(np.float64) @ W.astype(np.float64))
    assert (err <= product_bound(X, W, n + 8)).all()


def test_small_operands_among_others(hac):
    """One small entry in an otherwise empty row, one representative that is small, each at the end of a long loop."""
    rng = np.random.default_rng(4)
    n, m, B = 1100, 140, 70
    X = rng.standard_normal((B, n)).astype(np.float32)
    X[9], X[9, n - 1] = 0.0, np.float32(1.2345678 * 2.0 ** -118)
    W = rng.choice(rng.standard_normal(50).astype(np.float32), (n, m))
    W[:, 3], W[n - 2, 3] = 0.0, np.float32(1.7654321 * 2.0 ** -115)
    Y = hac.im_dot(hac.im_encode(W).to_device(dev()), torch.from_numpy(X).to(dev())).cpu().numpy().astype(np.float64)
    err = np.abs(Y - X.astype(np.float64) @ W.astype(np.float64))
    assert (err <= product_bound(X, W, n + 8)).all()


@pytest.mark.parametrize("n,terms", [(1, 1), (2, 2), (700, 1), (700, 2), (700, 4), (700, 8), (4608, 1)])
def test_sums_of_few_terms(hac, n, terms):
    """Short sums, and long ones of which few terms are not zero: (terms + 1) 2^-24 |X| . |W|.  That is the
    rounding of the result (2^-24), the products of parts left out (together 2^-24) and terms - 1 roundings on
    the way; the fp32 instruction's own sums come to `terms` roundings.  A product alone (n = 1) is the fp32 product."""
    rng = np.random.default_rng(n + terms)
    B, m = 300, 150
    W = rng.choice(rng.standard_normal(60).astype(np.float32), (n, m))
    X = np.zeros((B, n), np.float32)
    for b in range(B):
        X[b, rng.permutation(n)[:terms]] = rng.standard_normal(terms)
    Y = hac.im_dot(hac.im_encode(W).to_device(dev()), torch.from_numpy(X).to(dev())).cpu().numpy()
    err = np.abs(Y.astype(np.float64) - X.astype(np.float64) @ W.astype(np.float64))
    assert (err <= product_bound(X, W, terms + 1)).all()
    if n == 1:
        assert np.array_equal(Y, X * W)


# products that the sparse route took from the dense one: long columns of dot_split_kernel and of dot_batch_kernel (one pass, several, passes of 32 columns),
# and short ones whose dense sums, in one K split, are closer than any of the sparse kernels'
@pytest.mark.parametrize("n,m,pruned,k,B,fmt", [(2772, 2179, 0.784, 60, 134, "rice"), (1425, 1511, 0.695, 32, 146, "hac"), (3783, 1654, 0.711, 32, 72, "shac"),
                                                (4644, 1247, 0.624, 32, 93, "hac"), (9473, 1555, 0.869, 32, 105, "hac"), (1302, 3332, 0.67, 32, 77, "hac"),
                                                (3481, 3811, 0.773, 32, 116, "shac"), (511, 2009, 0.967, 32, 415, "rice"), (661, 2914, 0.967, 32, 512, "hac")])
def test_a_change_of_route_does_not_round_more(hac, n, m, pruned, k, B, fmt):
    """Relative error against 64 bits of the route that runs, at most that of the dense route that had the product before (the
    two differ by a quarter and more where the sums are not as careful, and by the share of rounding errors that happen to agree, 1 %, where they are)."""
    print(f"[case] route error {fmt} {n} x {m}, {B} rows", flush=True)
    rng = np.random.default_rng(n + m)
    at = np.clip(np.round(rng.standard_normal((n, m)) * k / 6 + k / 2), 0, k - 1).astype(np.int64)
    values = ((np.arange(k) - (k - 1) / 2) * 0.01).astype(np.float32)
    W = np.where(rng.random((n, m)) < pruned, np.float32(0), values[at]).astype(np.float32)
    X = np.maximum(rng.standard_normal((B, n)), 0).astype(np.float32)
    Wd, Xd = torch.from_numpy(W).to(dev()), torch.from_numpy(X).to(dev())
    blob = hac.hac_encode_dev(Wd, hac.HAC_FORMAT_HAC if fmt == "hac" else hac.HAC_FORMAT_SHAC, ri_coding=hac.RI_RICE if fmt == "rice" else hac.RI_FIELDS)
    call = hac.hac_dot if fmt == "hac" else hac.shac_dot
    ref = Xd.double() @ Wd.double()

    def error(Y):
        return float((Y.double() - ref).norm() / ref.norm())
    now, dense = error(call(blob, Xd)), error(call(blob, Xd, launch=hac.Launch(variant=DENSE)))
    assert now <= 1.01 * dense, (now, dense)
