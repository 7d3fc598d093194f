"""What the library launches and waits for, seen without a GPU (tests/native/hip_stub.cpp)."""
import os
import sys

import numpy as np
import pytest

import paper_2108_12704_amd as hac

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import hip_stub

# hac_encode_dev on made-up addresses: fill, scan, code, bits, column sums, columns; the pinned counts are the last one's 11th argument
ENCODE = """
def encode(get_last_error, synchronize):
    stub.stub_reset()
    stub.stub_fail(get_last_error, synchronize)
    stub.stub_copy_arg(5, 10, 8)
    d = hac.Desc()
    n, m = 640, 96
    room = lib.hac_encode_dev_workspace_bytes(n, m)
    lib.hac_encode_dev(hac.HAC_FORMAT_HAC, C.c_void_p(1 << 20), n, m, m, None, C.c_void_p(1 << 30), 1 << 20, C.byref(d), C.c_void_p(1 << 24), room, None)
    seen = events()
    return ["".join(e[0] for e in seen), next(e[3] for e in seen[5:])]
print(json.dumps([encode(*how) for how in {how}]))
"""


def test_pinned_counts_are_kept_until_the_stream_has_been_waited_for(tmp_path):
    """A call that ends with an error behind its launches must not hand the box to the next one while its kernels may still write there;
    where the wait fails too, never."""
    good, failed, after, lost, other, more = hip_stub.run(tmp_path, ENCODE.replace("{how}", "((0, 0), (1, 0), (0, 0), (1, 1), (0, 0), (0, 0))"))
    assert good[0].startswith("LLLLLLS") and good[1]
    assert failed[0] == "LLLLLLS", "the wait is missing"
    assert failed[1] == after[1] == lost[1] == good[1]                     # waited for: the same box again
    assert other[1] not in (0, lost[1]) and more[1] == other[1]            # not waited for: left alone


def test_calls_without_a_pinned_box_copy_the_counts(tmp_path):
    """All boxes lost one after the other: the next call's counts are copied, not waited for in pinned memory."""
    runs = hip_stub.run(tmp_path, ENCODE.replace("{how}", "[(1, 1)] * 16 + [(0, 0)]"))
    assert len({box for _, box in runs[:16]}) == 16 and 0 not in {box for _, box in runs[:16]}
    assert runs[16][1] == 0 and runs[16][0].startswith("LLLLLLMS")


def uneven(n, m, most, least, k):
    """Columns from `most` full to `least` full, values used as equal bins of a Gaussian are."""
    rng = np.random.default_rng(n + m + k)
    at = np.clip(np.round(rng.standard_normal((n, m)) * k / 6 + k / 2), 0, k - 1).astype(np.int64)
    values = ((np.arange(k) - k / 2 + 0.3) * 0.01).astype(np.float32)
    return np.where(rng.random((n, m)) < np.linspace(most, least, m), values[at], np.float32(0))


def words_of_the_fullest_block(blob):
    """Stream words from the first to the last of 256 chunks that follow one another, as decode_to_index_kernel copies them."""
    d, data = blob.desc, blob.data
    section = lambda off, count: data[off:off + 4 * count].view(np.uint32).astype(np.int64)
    first, start = section(d.off_col_chunk, d.m + 1), section(d.off_col_bit, d.m + 1)
    entry = section(d.off_chunk_ent, d.n_chunks)
    assert d.ent_bits == 32
    begin = start[np.searchsorted(first, np.arange(d.n_chunks), side="right") - 1] + (entry >> d.row_bits)
    begin = np.append(begin, start[-1])
    blocks = np.arange(0, d.n_chunks, 256)
    ends = begin[np.minimum(blocks + 256, d.n_chunks)]
    return int(((ends + 31) // 32 - (begin[blocks] // 32 & ~3)).max()) + 8


# (the dense route's launches: the map cleared, the decode, whose fifth argument is the room for stream words, the product)
DECODE = """
d = hac.Desc.from_buffer_copy(bytes.fromhex({head!r}))
launch = hac.Launch(variant=0x800)
stub.stub_copy_arg(1, 4, 4)
at = lambda x: C.c_void_p(x << 32)
rc = lib.{call}(C.byref(d), at(1), at(2), 48, d.n, at(3), d.m, at(4), hac.hac_workspace_bytes(d, 48, launch), C.byref(launch), None)
seen = events()
print(json.dumps([rc, seen[1][2], seen[1][3]]))
"""


@pytest.mark.parametrize("n,m,most,least,k", [(2048, 1024, 0.5, 0.05, 32), (2048, 1024, 0.5, 0.05, 250), (4096, 1000, 0.5, 0.1, 32),
                                              (4608, 512, 0.7, 0.1, 32), (1000, 4000, 0.5, 0.05, 32)])
@pytest.mark.parametrize("fmt", ["hac", "rice"])
def test_decode_of_uneven_columns_runs_on_words_in_lds(tmp_path, fmt, n, m, most, least, k):
    """Chunks have as many non-zeros each, so those of emptier columns are longer than the average; all blocks' words fit all the same."""
    W = uneven(n, m, most, least, k)
    blob = hac.hac_encode(W) if fmt == "hac" else hac.shac_encode(W, ri_coding=hac.RI_RICE)
    rc, lds, room = hip_stub.run(tmp_path, DECODE.format(head=bytes(blob.desc).hex(), call="hac_dot" if fmt == "hac" else "shac_dot"))
    assert rc == 0 and lds <= 160 * 1024
    assert room >= words_of_the_fullest_block(blob)
