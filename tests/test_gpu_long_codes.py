"""Codewords longer than the first-level table: all lengths up to the longest, tables of 1 to 12 bits, alphabets whose
values are read from LDS and from the blob, every decode loop of the products."""
import numpy as np
import pytest

from oracle import dot as odot

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DENSE, LIST = 0x800, 0x200


@pytest.fixture(scope="module")
def hac():
    import paper_2108_12704_amd as lib
    lib.load_library()
    assert torch.cuda.is_available(), "GPU tests need a device"
    return lib


def matrix(kind):
    rng = np.random.default_rng(len(kind))
    if kind == "deep":                                      # counts like Fibonacci's numbers: a length per value, up to 24 bits
        n, m, counts = 2500, 100, [int(1.62 ** i) for i in range(24)]
    elif kind == "dense":                                   # 0.0 is rare, so its codeword is a long one
        n, m, counts = 700, 60, [20000, 12000, 6000, 2500, 900, 300, 90, 30, 9, 3, 1]
    else:                                                   # more values than LDS holds
        n, m, counts = 900, 90, [3 + i % 40 for i in range(1500)]
    values = np.unique(rng.standard_normal(4 * len(counts)).astype(np.float32))
    values = rng.permutation(values[values != 0.0])[:len(counts)]
    W = np.zeros(n * m, np.float32)
    W[rng.permutation(n * m)[:sum(counts)]] = np.repeat(values, counts)
    return W.reshape(n, m)


@pytest.mark.parametrize("kind", ["deep", "dense", "many"])
@pytest.mark.parametrize("lut_bits", [1, 4, 9, 10, 12])
def test_long_codewords(hac, kind, lut_bits):
    W = matrix(kind)
    n, m = W.shape
    blobs = {"hac": hac.hac_encode(W, lut_bits=lut_bits), "shac": hac.shac_encode(W, lut_bits=lut_bits),
             "rice": hac.shac_encode(W, lut_bits=lut_bits, ri_coding=hac.RI_RICE)}
    for fmt, blob in blobs.items():
        d = blob.to_device("cuda:0")
        if fmt == "hac":
            assert np.array_equal(hac.hac_decode_dev(d)[0].cpu().numpy().view(np.uint32), W.view(np.uint32))
        for B, variant in ((1, 0), (2, 0), (7, 0), (40, 0), (40, LIST), (40, DENSE)):
            print(f"[case] long codes {kind} {fmt} lut {lut_bits} lmax {blob.desc.lmax} B={B} variant {variant:#x}", flush=True)
            X = np.random.default_rng(B).standard_normal((B, n)).astype(np.float32)
            call = hac.hac_dot if fmt == "hac" else hac.shac_dot
            Y = call(d, torch.from_numpy(X).cuda(), launch=hac.Launch(variant=variant)).cpu().numpy().astype(np.float64)
            # the bar of the other tests: 1e-5 of the sum of the terms' sizes.  Sums of at most 2500 terms (a column of `deep` has 1720 in the mean), whose
            # roundings add up like a random walk: one chain of all of them would be off by about sqrt(2500) 2^-24 = 3e-6 of that
            assert np.all(np.abs(Y - odot.dense_dot(X, W)) <= 1e-5 * odot.abs_dot(X, W) + 1e-37)
