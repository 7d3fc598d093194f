"""What the library launches and waits for, seen without a GPU (tests/native/hip_stub.cpp)."""
import os
import sys

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
