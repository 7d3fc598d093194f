"""The native call path of the binding: arguments by position and name, and what it refuses, without a GPU."""
import pytest

import paper_2108_12704_amd as hac

torch = pytest.importorskip("torch")

X = "X must be a 2-D float32 CUDA tensor"


@pytest.mark.parametrize("call,args,kw,error,text", [
    ("hac_dot", (), {}, TypeError, "missing argument 'dblob'"),
    ("hac_dot", (None,), {}, TypeError, "missing argument 'X'"),
    ("hac_dot", (None, torch.zeros(2, 3)), {}, TypeError, X),                       # not on the GPU
    ("shac_dot", (), {"dblob": None, "X": [[1.0]]}, TypeError, X),                  # not a tensor
    ("im_dot", (None, torch.zeros(2, 3), None, None, None, None), {}, TypeError, "too many arguments"),
    ("im_dot", (None, torch.zeros(2, 3)), {"launch": None}, TypeError, "unexpected keyword argument 'launch'"),
    ("hac_dot", (None, torch.zeros(2, 3)), {"X": None}, TypeError, "multiple values for argument 'X'"),
    ("hac_dot_noalloc", (None, torch.zeros(2, 3), None), {}, TypeError, X + " with unit column stride"),
    ("hac_forward", ([], torch.zeros(2, 3, dtype=torch.float64)), {}, TypeError, X),
])
def test_refused_arguments(call, args, kw, error, text):
    with pytest.raises(error, match=text):
        getattr(hac._native(), call)(*args, **kw)


def test_public_calls_go_through_it():
    with pytest.raises(TypeError, match=X):
        hac.hac_dot(None, torch.zeros(2, 3))
    with pytest.raises(TypeError, match=X):
        hac.hac_forward([], torch.zeros(2, 3))


@pytest.mark.gpu
def test_results_buffers_and_errors_on_the_gpu():
    import numpy as np
    W = np.zeros((300, 40), np.float32)
    W[::7, ::3] = 0.5
    db = hac.hac_encode(W).to_device("cuda:0")
    x = torch.rand(6, 300, device="cuda:0")
    y = torch.full((6, 40), -1.0, device="cuda:0")
    ws = torch.empty(max(hac.hac_workspace_bytes(db.desc, 6), 256), dtype=torch.uint8, device="cuda:0")
    print("[case] binding", flush=True)
    ref = x.double().cpu() @ torch.from_numpy(W).double()
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    assert hac.hac_dot(db, x, Y=y, workspace=ws, launch=hac.Launch(), stream=stream) is y
    stream.synchronize()
    assert torch.allclose(y.cpu().double(), ref, rtol=1e-5, atol=1e-5)              # (43 terms of at most 0.5)
    assert torch.equal(hac.hac_dot(db, x.t().contiguous().t()), y)                  # rows of X not contiguous
    assert hac.hac_dot(db, x[:0]).shape == (0, 40)
    assert hac.hac_dot_noalloc(db, x, y) is y
    for bad in (y[:5], y.double(), y.cpu(), torch.empty(40, 6, device="cuda:0").t()):
        with pytest.raises(TypeError, match="Y must be"):
            hac.hac_dot(db, x, Y=bad)
    for bad in (bytes(64), bytearray(64), np.zeros(64, np.uint8), hac.Desc()):                  # bytes are no launch settings
        with pytest.raises(TypeError, match="expected Launch"):
            hac.hac_dot(db, x, launch=bad)
        with pytest.raises(TypeError, match="expected Launch"):
            hac.hac_dot_noalloc(db, x, y, launch=bad)
    class Bytes:
        desc, tensor = bytes(db.desc), db.tensor
    with pytest.raises(TypeError, match="expected Desc"):
        hac.hac_dot(Bytes, x)
    with pytest.raises(ValueError, match="X has the wrong width"):
        hac.hac_dot(db, x[:, 1:])
    with pytest.raises(hac.HacError) as e:
        hac.shac_dot(db, x)
    assert e.value.status == -1 and "shac_dot" in str(e.value)
    with pytest.raises(TypeError, match="bias must be"):
        hac.hac_forward([(db, torch.zeros(39, device="cuda:0"), True)], x)
    assert torch.equal(hac.hac_forward([(db, None, np.bool_(False))], x), hac.hac_dot(db, x))


@pytest.mark.gpu
def test_out_of_memory_is_torchs_exception():
    """The limit is checked before the driver is asked: nothing is allocated."""
    import numpy as np
    W = np.zeros((300, 40), np.float32)
    W[::7, ::3] = 0.5
    db = hac.hac_encode(W).to_device("cuda:0")
    x = torch.rand(1 << 21, 300, device="cuda:0")              # Y: 336 MB
    print("[case] out of memory", flush=True)
    torch.cuda.empty_cache()
    torch.cuda.set_per_process_memory_fraction(1e-6)
    try:
        for call in (lambda: hac.hac_dot(db, x), lambda: hac.hac_forward([(db, None, False)], x),                   # Y
                     lambda: hac.hac_dot(db, x, Y=x[:, :40], launch=hac.Launch(variant=0x400)),                     # the copy of X
                     lambda: hac.hac_dot(db, x.view(300, -1).t(), Y=x[:, :40])):                                    # rows of X
            with pytest.raises(torch.OutOfMemoryError):
                call()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)


@pytest.mark.gpu
@pytest.mark.parametrize("call", ["hac_dot", "hac_forward"])
def test_buffers_made_here_belong_to_the_stream_of_the_call(call):
    """`stream` is not the current one: a copy of X neither waits for the current stream nor is its memory given to it early."""
    import numpy as np
    W = np.zeros((1000, 60), np.float32)
    W[::7, ::3] = 0.5
    db = hac.hac_encode(W).to_device("cuda:0")
    other, busy = torch.cuda.Stream(), 20_000_000                                   # (10 to 200 ms of either stream)

    def product(x):
        return hac.hac_dot(db, x, stream=other) if call == "hac_dot" else hac.hac_forward([(db, None, False)], x, stream=other)

    def nan_in_free_memory():
        blocks = [torch.full((n,), float("nan"), device="cuda:0") for n in (48 * 1000, 48 * 1000, 64 * 1000, 64 * 60)]
        del blocks
    xt = torch.rand(1000, 48, device="cuda:0")                                      # rows of X are columns of it
    ref = (xt.t().double().cpu() @ torch.from_numpy(W).double())
    product(xt.t())
    with torch.cuda.stream(other):
        nan_in_free_memory()
    nan_in_free_memory()
    torch.cuda.synchronize()
    print("[case] streams", flush=True)
    torch.cuda._sleep(busy)                                                         # the current stream is late
    y = product(xt.t())
    other.synchronize()
    with torch.cuda.stream(other):
        got = y.cpu()
    torch.cuda.synchronize()
    assert torch.allclose(got.double(), ref, rtol=1e-5, atol=1e-5)                  # (143 terms of at most 0.5)
    with torch.cuda.stream(other):
        torch.cuda._sleep(busy)                                                     # the stream of the call is late
    y = product(xt.t())
    nan_in_free_memory()
    torch.cuda.synchronize()
    assert torch.allclose(y.cpu().double(), ref, rtol=1e-5, atol=1e-5)
