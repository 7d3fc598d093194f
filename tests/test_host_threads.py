"""The host encoders on several threads write the blob they write on one (byte for byte), and it decodes to W."""
import os
import time

import numpy as np
import pytest

import paper_2108_12704_amd as hac


def layer(n, m, density, k, seed):
    rng = np.random.default_rng(seed)
    W = np.zeros((n, m), dtype=np.float32)
    mask = rng.random((n, m)) < density
    W[mask] = rng.choice(np.arange(1, k + 1, dtype=np.float32) * np.float32(0.25), size=int(mask.sum()))
    return W


# one tall column, one wide row, fewer rows than parts, columns that are empty, dense without zeros, more values than fit a byte;
# the widest matrix whose rows are scanned several at a time, the next one, and a group that does not divide 1024
SHAPES = [(200000, 1, 0.3, 7), (1, 200000, 0.3, 7), (9, 30011, 0.5, 40), (4099, 67, 0.0, 1), (517, 523, 1.0, 300),
          (1031, 257, 0.02, 5), (3001, 64, 0.4, 9), (3001, 65, 0.4, 9), (30011, 7, 0.9, 9), (1, 1, 1.0, 1)]


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


@pytest.mark.parametrize("m", [1, 7, 64])
def test_rows_apart_give_the_same_blob(m):
    """Rows side by side are scanned several at a time, rows with other columns between them one by one."""
    wide = layer(5003, m + 3, 0.3, 9, 11 + m)
    part = wide[:, :m]
    assert np.array_equal(hac.hac_encode(part).data, hac.hac_encode(np.ascontiguousarray(part)).data)


@pytest.mark.parametrize("apart", [0, 1])
def test_time_grows_with_the_size(apart):
    """Less than one non-zero per row on one CPU: the lists that collect them must not be copied over and over.
    Eight times the rows take eight times as long; a list that grows by a fixed amount took 64 to 100 times."""
    def seconds(n):
        W = np.zeros((n, 1 + apart), np.float32)[:, :1]
        W[1:, 0] = np.where(np.random.default_rng(3).random(n - 1) < 0.3, 2.0, 0.0)
        return min(timed(W) for _ in range(2))

    def timed(W):
        start = time.perf_counter()
        hac.hac_encode(W)
        return time.perf_counter() - start
    cpus = os.sched_getaffinity(0)
    os.sched_setaffinity(0, {min(cpus)})
    try:
        small, large = seconds(250_000), seconds(2_000_000)
    finally:
        os.sched_setaffinity(0, cpus)
    assert large < 30 * small, (small, large)
