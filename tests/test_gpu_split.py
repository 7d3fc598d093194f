"""dot_split_kernel (several wavefronts per column) against the oracle's dense fp64 product, at the edges of its splits.

Tolerance: |Y - Yref| <= 1e-5 (|X| . |W|) componentwise (fp32 sums of at most a few thousand terms stay below 1e-6 of it).
"""
import numpy as np
import pytest

from oracle import dot as odot

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

ENCODERS = {"hac": ("hac_encode", {}), "shac": ("shac_encode", {}), "rice": ("shac_encode", {"ri_coding": 1})}


@pytest.fixture(scope="module")
def hac():
    import paper_2108_12704_amd as lib
    assert torch.cuda.is_available(), "GPU tests need a device"
    return lib


def matrix(n, m, density, seed, k=24):
    rng = np.random.default_rng(seed)
    values = np.sort(rng.standard_normal(k)).astype(np.float32)
    W = np.where(rng.random((n, m)) < density, values[rng.integers(0, k, (n, m))], np.float32(0)).astype(np.float32)
    if m > 4:
        W[:, 0] = 0                                          # an empty column first, one in the middle, one at the end
        W[:, m // 2] = 0
        W[:, -1] = 0
    if m > 3:
        W[:, 1] = values[rng.integers(0, k, n)]              # a column without a zero: the longest
    assert np.count_nonzero(W) > 0
    return W


def run(hac, fmt, W, X, strided=False):
    enc, kw = ENCODERS[fmt]
    db = getattr(hac, enc)(W, **kw).to_device("cuda:0")
    dot = hac.hac_dot if fmt == "hac" else hac.shac_dot
    B, n = X.shape
    m = W.shape[1]
    if not strided:
        Y = dot(db, torch.from_numpy(X).cuda(), launch=hac.Launch(variant=0x400))
        return Y, hac.hac_last_kernels()
    Xp = torch.full((B, n + 3), float("nan"), device="cuda:0")
    Yp = torch.full((B, m + 5), 7.0, device="cuda:0")
    Xp[:, 1:n + 1] = torch.from_numpy(X)                     # rows of X that start at an odd address
    Y = dot(db, Xp[:, 1:n + 1], Y=Yp[:, :m], launch=hac.Launch(variant=0x400))
    assert bool((Yp[:, m:] == 7.0).all())
    return Y, hac.hac_last_kernels()


def check(Y, X, W):
    ref, scale = odot.dense_dot(X, W), odot.abs_dot(X, W)
    assert bool((np.abs(Y.cpu().numpy().astype(np.float64) - ref) <= 1e-5 * scale + 1e-37).all())


# columns at and around those of a block (1, 2, 4), every width of a tile of X read as it is, one more row than a tile has
@pytest.mark.parametrize("fmt", sorted(ENCODERS))
@pytest.mark.parametrize("n,m,density,B,nbd", [(70, 1, 0.3, 2, 4), (300, 5, 0.3, 4, 4), (500, 300, 0.3, 5, 8), (500, 1025, 0.2, 8, 8),
                                               (257, 2049, 0.1, 9, 16), (900, 33, 0.4, 16, 16), (3001, 10, 0.2, 17, 24),
                                               (640, 65, 0.3, 25, 32), (640, 65, 0.02, 33, 24), (1200, 40, 0.3, 64, 32),
                                               (4100, 21, 0.1, 65, 24), (2000, 3, 0.5, 200, 32)])
def test_x_as_it_is(hac, fmt, n, m, density, B, nbd):
    W = matrix(n, m, density, n + m)
    X = np.random.default_rng(B).standard_normal((B, n)).astype(np.float32)
    print(f"[case] split {fmt} {n}x{m} B={B}", flush=True)
    Y, kernels = run(hac, fmt, W, X)
    assert kernels == [f"dot_split_kernel<{'true' if fmt == 'shac' else 'false'}, {nbd}>"]
    check(Y, X, W)
    Ys, _ = run(hac, fmt, W, X, strided=True)
    assert torch.equal(Ys, Y)


def test_a_matrix_of_zeros(hac):
    for m, B in ((1, 2), (3, 200), (300, 8)):
        print(f"[case] split, zeros {m} B={B}", flush=True)
        X = np.random.default_rng(B).standard_normal((B, 500)).astype(np.float32)
        Y, _ = run(hac, "hac", np.zeros((500, m), np.float32), X)
        assert not bool(Y.any())


# batches whose last panel or quad of batch columns is not full; two, four and sixteen wavefronts per column
@pytest.mark.parametrize("fmt", sorted(ENCODERS))
@pytest.mark.parametrize("n,m,density,B", [(9000, 1500, 0.03, 5), (4000, 1500, 0.03, 31), (9973, 700, 0.05, 37), (9973, 200, 0.05, 70),
                                           (26000, 40, 0.05, 130), (9000, 130, 0.02, 300)])
def test_rows_of_the_copy(hac, fmt, n, m, density, B):
    W = matrix(n, m, density, n + m)
    W[:, 1] *= (np.arange(n) % 5 == 0)                        # (all of a tall column's non-zeros have to fit the list)
    X = np.random.default_rng(B).standard_normal((B, n)).astype(np.float32)
    X[-1] = np.nan                                            # a row of X reaches its own row of Y only
    print(f"[case] split, copy {fmt} {n}x{m} B={B}", flush=True)
    Y, kernels = run(hac, fmt, W, X)
    assert kernels[-1] == f"dot_split_kernel<{'true' if fmt == 'shac' else 'false'}, 0>" and len(kernels) == 2
    check(Y[:-1], X[:-1], W)
    assert bool(torch.isnan(Y[-1][torch.from_numpy((W != 0).any(0)).cuda()]).all())
    Ys, _ = run(hac, fmt, W, X, strided=True)
    assert torch.equal(Ys[:-1], Y[:-1])


def test_a_column_too_long_for_the_list_takes_the_other_kernel(hac):
    W = matrix(24000, 4, 0.9, 3)
    X = np.random.default_rng(1).standard_normal((6, 24000)).astype(np.float32)
    print("[case] split, long column", flush=True)
    Y, kernels = run(hac, "hac", W, X)
    assert not any("split" in k for k in kernels)
    check(Y, X, W)


def test_an_old_copy_of_x_is_only_reused_where_every_call_leaves_one(hac):
    """HAC_LAUNCH_REUSE_XT (0x100) after a call that read X as it is."""
    rng = np.random.default_rng(5)
    narrow, wide = matrix(1200, 20, 0.2, 1), matrix(1200, 4096, 0.05, 2)
    X = rng.standard_normal((40, 1200)).astype(np.float32)
    Xd = torch.from_numpy(X).cuda()
    dn, dw = hac.hac_encode(narrow).to_device("cuda:0"), hac.shac_encode(wide).to_device("cuda:0")
    ws = torch.full((max(hac.hac_workspace_bytes(d.desc, 40) for d in (dn, dw)) // 4,), float("nan"), device="cuda:0").view(torch.uint8)
    print("[case] reuse of the copy", flush=True)
    check(hac.hac_dot(dn, Xd, workspace=ws), X, narrow)
    check(hac.shac_dot(dw, Xd, workspace=ws, launch=hac.Launch(variant=0x500)), X, wide)


# what the first call names and what the one that reuses its copy does; more than 2^19 values of X, passes of 128 columns by default
@pytest.mark.parametrize("left", [{}, {"pass_width": 32}, {"tile_width": 32}, {"pass_width": 256}, {"variant": 0x200}])
@pytest.mark.parametrize("reused", [{}, {"pass_width": 32}, {"tile_width": 64}, {"pass_width": 256}, {"variant": 0x200}])
def test_a_copy_of_x_is_reused_however_it_was_left(hac, left, reused):
    """The copy's layout depends on X alone, not on the widths that either launch names."""
    rng = np.random.default_rng(7)
    B, n = 200, 4096
    first, second = matrix(n, 300, 0.02, 3), matrix(n, 2100, 0.02, 4)
    X = rng.standard_normal((B, n)).astype(np.float32)
    Xd = torch.from_numpy(X).cuda()
    df, ds = hac.hac_encode(first).to_device("cuda:0"), hac.shac_encode(second).to_device("cuda:0")
    ws = torch.full((B * 2 * n,), float("nan"), device="cuda:0").view(torch.uint8)

    def launch(kw, flags):
        return hac.Launch(**{**kw, "variant": kw.get("variant", 0) | flags})

    print(f"[case] copy left by {left}, reused by {reused}", flush=True)
    check(hac.hac_dot(df, Xd, workspace=ws, launch=launch(left, 0x400)), X, first)
    assert any("transpose" in k for k in hac.hac_last_kernels())
    Y = hac.shac_dot(ds, Xd, workspace=ws, launch=launch(reused, 0x500))
    assert not any("transpose" in k for k in hac.hac_last_kernels())
    check(Y, X, second)


# rows of a panel of 2, 4, 8, 16 and 32 columns, full or not; X too short for a second launch, or kept in LDS by other matrices
@pytest.mark.parametrize("B,n", [(2, 4097), (3, 2049), (5, 1025), (8, 1300), (13, 700), (29, 333), (32, 64), (40, 1200), (200, 1111), (8, 500), (2, 4096)])
@pytest.mark.parametrize("fmt", ["hac", "shac"])
def test_a_call_that_reads_x_as_it_is_leaves_the_copy_too(hac, B, n, fmt):
    """HAC_LAUNCH_REUSE_XT after one launch that re-laid nothing out: no pass over X, and the sums of the wide matrix are right."""
    narrow, wide = matrix(n, 20, 0.3, 1), matrix(n, 4096, 0.05, 2)
    wide[:, 1] *= (np.arange(n) % 5 == 0)
    X = np.random.default_rng(B).standard_normal((B, n)).astype(np.float32)
    Xd = torch.full((B, n + 3), float("nan"), device="cuda:0")
    Xd[:, 1:n + 1] = torch.from_numpy(X)
    Xd = Xd[:, 1:n + 1]
    dn, dw = hac.hac_encode(narrow).to_device("cuda:0"), getattr(hac, fmt + "_encode")(wide).to_device("cuda:0")
    reuse = hac.Launch(variant=0x700)                         # reuse the copy, sparse route, the kernel that reads it
    ws = torch.full((B * 2 * n + 64,), float("nan"), device="cuda:0").view(torch.uint8)
    print(f"[case] copy left beside the product {fmt} {n} B={B}", flush=True)
    check(hac.hac_dot(dn, Xd, workspace=ws, launch=hac.Launch(variant=0x400)), X, narrow)
    assert [k.split("<")[0] for k in hac.hac_last_kernels()] == ["dot_split_kernel"]
    Y = (hac.hac_dot if fmt == "hac" else hac.shac_dot)(dw, Xd, workspace=ws, launch=reuse)
    in_lds = B <= 8 and n * (1 << (B - 1).bit_length()) <= 8192
    assert any("transpose" in k for k in hac.hac_last_kernels()) == in_lds
    check(Y, X, wide)


# passes of 64, 128 and 256 batch columns (four, two and one lane group), one wavefront per column and several
@pytest.mark.parametrize("m,kernel", [(3300, "dot_batch_kernel"), (300, "dot_split_kernel")])
@pytest.mark.parametrize("B", [64, 100, 250])
def test_columns_lose_nothing_in_a_wide_pass(hac, B, m, kernel):
    """350 non-zeros a column: sums of five products in fp32, those in 64 bits: (5 + 1 for the result) 2^-24 |X| . |W|."""
    rng = np.random.default_rng(B + m)
    n = 2500
    values = rng.uniform(0.5, 1.0, 16).astype(np.float32)
    W = np.where(rng.random((n, m)) < 0.14, values[rng.integers(0, 16, (n, m))], np.float32(0)).astype(np.float32)
    X = rng.uniform(0.5, 1.0, (B, n)).astype(np.float32)     # all of one sign: partial sums grow, and with them what a chain rounds away
    print(f"[case] wide pass {kernel} B={B}", flush=True)
    Y, kernels = run(hac, "hac", W, X)
    assert kernels[-1].startswith(kernel)
    assert bool((np.abs(Y.cpu().numpy().astype(np.float64) - odot.dense_dot(X, W)) <= 6 * 2.0 ** -24 * odot.abs_dot(X, W)).all())


@pytest.mark.parametrize("fmt", sorted(ENCODERS))
@pytest.mark.parametrize("B", [2, 6, 13, 20, 32, 70])
def test_short_columns_are_rounded_once(hac, B, fmt):
    """Products and sums of two that fp32 holds exactly: what is added after that, in 64 bits, leaves one rounding."""
    rng = np.random.default_rng(B)
    n, m = 600, 150
    values = rng.choice(np.arange(1, 2048), 24, replace=False).astype(np.float32)
    W = np.zeros((n, m), np.float32)
    for j in range(m):                                        # at most one non-zero a lane
        rows = rng.choice(n, rng.integers(1, 65), replace=False)
        W[rows, j] = values[rng.integers(0, 24, rows.size)]
    X = rng.integers(1, 4096, (B, n)).astype(np.float32)
    print(f"[case] short columns {fmt} B={B}", flush=True)
    Y, kernels = run(hac, fmt, W, X)
    assert kernels[0].startswith("dot_split_kernel") and not kernels[0].endswith(" 0>")
    exact = X.astype(np.int64) @ W.astype(np.int64)
    assert exact.max() > 1 << 26
    assert bool((Y.cpu().numpy() == exact.astype(np.float32)).all())


# the last pass of the widest kind full, partly full, mostly padding; a dense and a sparse matrix, two tiles of the batch
@pytest.mark.parametrize("density,kinds", [(0.1, {72: 1, 96: 1, 128: 2, 144: 1, 200: 2, 256: 2, 280: 2}), (0.01, {72: 2, 129: 2, 160: 2, 256: 2})])
def test_passes_that_the_batch_fills(hac, density, kinds):
    """The kernel's last parameter is 2 for passes of 64 columns or more, 1 for several of 32 that were chosen before them."""
    n, m = 4500, 3200
    W = matrix(n, m, density, 11)
    W[:, 1] *= (np.arange(n) % 20 == 0)
    rng = np.random.default_rng(12)
    for B, kind in kinds.items():
        X = rng.standard_normal((B, n)).astype(np.float32)
        print(f"[case] passes {density} B={B}", flush=True)
        Y, kernels = run(hac, "hac", W, X)
        assert kernels[-1].startswith("dot_batch_kernel") and kernels[-1].endswith(f"{kind}>"), (B, kernels)
        check(Y, X, W)


# where the other kernels are the quicker ones: blocks that wait for LDS (few rows of X, and five rounds of them), two rows of many
# columns, dense columns over X as it is, short columns for two wavefronts; and the neighbours that stay
@pytest.mark.parametrize("n,m,density,B,kernel", [
    (10590, 1502, 0.38, 2, "dot_small_kernel<false, 2, false>"), (10590, 400, 0.05, 2, "dot_split_kernel<false, 4>"),
    (770, 2872, 0.33, 2, "dot_small_kernel<false, 2, true>"), (770, 2872, 0.33, 3, "dot_split_kernel<false, 4>"),
    (778, 1963, 0.35, 26, "dot_split_kernel<false, 0>"), (778, 1963, 0.1, 26, "dot_split_kernel<false, 32>"),
    (529, 3100, 0.35, 8, "dot_batch_kernel<false, 4, false, false, 1>"), (16841, 1291, 0.26, 70, "dot_batch_kernel<false, 4, true, false, 0>"),
    (3000, 2000, 0.015, 32, "dot_batch_kernel<false, 4, false, false, 1>"), (3000, 2000, 0.08, 32, "dot_split_kernel<false, 0>")])
def test_which_products_take_it(hac, n, m, density, B, kernel):
    W = matrix(n, m, density, n + B)
    W[:, 1] *= (np.arange(n) % max(1, round(1 / density)) == 0)
    X = np.random.default_rng(B).standard_normal((B, n)).astype(np.float32)
    print(f"[case] which kernel {n}x{m} {density} B={B}", flush=True)
    Y, kernels = run(hac, "hac", W, X)
    assert kernels[-1] == kernel
    check(Y, X, W)
