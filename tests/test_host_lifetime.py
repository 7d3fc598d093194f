"""The arrays an encoder returns stay valid as long as something refers to them, interpreter exit included."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# The handler is registered before the first encode, so it runs after whatever the package registered
# later; the blob is alive then.  It first takes up blocks of the blob's size, so that freed memory shows.
PROGRAM = """
import atexit, os
kept = []
def look():
    junk = [np.full(size, 170, np.uint8) for blob, copy in kept for size in range(len(copy) - 512, len(copy) + 512, 16)]
    same = all(bytes(blob.data) == copy for blob, copy in kept)
    print("intact" if same and kept[0][0].validate(deep=True) == 0 else "damaged", flush=True)
atexit.register(look)
import numpy as np
import paper_2108_12704_amd as hac
rng = np.random.default_rng(1)
W = np.where(rng.random((600, 400)) < 0.3, rng.choice(np.arange(1, 30, dtype=np.float32), (600, 400)), 0).astype(np.float32)
for blob in ({calls}):
    kept.append((blob, bytes(blob.data)))
"""


@pytest.mark.parametrize("calls", ["hac.hac_encode(W),", "hac.shac_encode(W),", "hac.im_encode(W),",
                                   "hac.hac_net_encode([W], [hac.HAC_FORMAT_SHAC]),"])
def test_blob_is_alive_in_an_exit_handler(calls):
    out = subprocess.run([sys.executable, "-c", PROGRAM.replace("{calls}", calls)], cwd=ROOT, capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and out.stdout.split() == ["intact"], (out.returncode, out.stdout, out.stderr)


def test_blob_outlives_what_returned_it():
    """The other end: the buffer goes when the last array on it goes, not before."""
    import gc

    import numpy as np

    import paper_2108_12704_amd as hac
    W = np.where(np.arange(600 * 400).reshape(600, 400) % 5 == 0, 1.5, 0).astype(np.float32)
    blob = hac.hac_encode(W)
    part, copy = blob.data[100:], blob.data[100:].copy()
    del blob
    gc.collect()
    for _ in range(4):
        hac.hac_encode(-W)                                     # would take over the freed block
    assert np.array_equal(part, copy)
