"""The host encoders on several threads write the blob they write on one (byte for byte), and it decodes to W."""
import os

import numpy as np
import pytest

import paper_2108_12704_amd as hac


def layer(n, m, density, k, seed):
    rng = np.random.default_rng(seed)
    W = np.zeros((n, m), dtype=np.float32)
    mask = rng.random((n, m)) < density
    W[mask] = rng.choice(np.arange(1, k + 1, dtype=np.float32) * np.float32(0.25), size=int(mask.sum()))
    return W


# one tall column, one wide row, fewer rows than parts, columns that are empty, dense without zeros, more values than fit a byte
SHAPES = [(200000, 1, 0.3, 7), (1, 200000, 0.3, 7), (9, 30011, 0.5, 40), (4099, 67, 0.0, 1), (517, 523, 1.0, 300),
          (1031, 257, 0.02, 5)]


@pytest.mark.parametrize("n,m,density,k", SHAPES)
@pytest.mark.parametrize("encode", ["hac", "shac", "rice", "rows", "im"])
def test_threads_do_not_change_the_blob(n, m, density, k, encode):
    call = {"hac": lambda W: hac.hac_encode(W), "shac": lambda W: hac.shac_encode(W),
            "rice": lambda W: hac.shac_encode(W, ri_coding=hac.RI_RICE),
            "rows": lambda W: hac.hac_encode(W, chunk_rows=hac.CHUNK_ROWS_AUTO), "im": lambda W: hac.im_encode(W)}[encode]
    W = layer(n, m, density, k, n + m)
    blob = call(W)
    cpus = os.sched_getaffinity(0)
    os.sched_setaffinity(0, {min(cpus)})
    try:
        alone = call(W)
    finally:
        os.sched_setaffinity(0, cpus)
    assert np.array_equal(blob.data, alone.data)
    assert blob.validate(deep=True) == 0
    assert np.array_equal(blob.decode_host()[0], W)
