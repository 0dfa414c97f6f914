"""The native calls of the binding: what they refuse goes through the Python checks and ends in the same error, and what they
take reaches the C entry point with the same arguments."""
import ctypes as C

import pytest
import torch

import paper_2406_11430_amd as l2kv
from paper_2406_11430_amd import binding


def tensors(dtype=torch.bfloat16, device="cpu"):
    Q, O, ws = torch.zeros((1, 4, 64), dtype=dtype), torch.zeros((1, 4, 64)), torch.zeros(1 << 16, dtype=torch.uint8)
    K, V = (torch.zeros((1, 2, 8, 64), dtype=dtype) for _ in range(2))
    return [x.to(device) for x in (Q, K, V, O, ws)]


def test_host_tensors_are_refused():
    args = tensors()
    for call in (l2kv.l2kv_decode_attn, l2kv.l2kv_decode_attn_out):
        with pytest.raises(ValueError, match="device tensors"):
            call(*args)
    Q, K, V, O, ws = args
    with pytest.raises(ValueError, match="device tensors"):
        l2kv.l2kv_compress(K, V, 0.5, torch.zeros((1, 2, 8)), torch.zeros((1, 2, 4), dtype=torch.int32), K, V, ws)


def test_what_is_not_a_tensor_or_a_number_is_left_to_the_checks():
    native = binding.calls()
    assert native.decode_attn(1, 2, 3, 4, 5, 0.0, None, binding._stream) is None
    assert native.decode_attn(*tensors(), "x", None, binding._stream) is None
    assert native.decode_attn() is None and native.decode_attn_out() is None and native.compress() is None


@pytest.fixture
def unloaded():
    before = binding._calls
    binding._calls = None
    yield
    binding._calls = before


def test_library_alone(unloaded, monkeypatch, tmp_path):
    """Without the native calls, or with some for another torch or that do not load, the library is called as well."""
    broken = tmp_path / "l2kv_calls.so"
    broken.write_bytes(b"not a library")
    for path, version, message in ((str(tmp_path / "none.so"), torch.__version__, "missing"), (str(broken), torch.__version__, "l2kv_calls"),
                                   (binding.CALLS_PATH, "0.0", "built for torch")):
        binding._calls = None
        monkeypatch.setattr(binding, "CALLS_PATH", path)
        monkeypatch.setattr(torch, "__version__", version)
        with pytest.warns(RuntimeWarning, match=message), pytest.raises(ValueError, match="device tensors"):
            l2kv.l2kv_decode_attn(*tensors())
        assert binding.calls().decode_attn(*tensors(), 0.0, None, binding._stream) is None


@pytest.mark.gpu
@pytest.mark.parametrize("change", ["none", "stride", "dtype", "shape", "dims", "output", "half", "nan_scale", "workspace", "group"])
def test_decode_errors(change):
    Q, K, V, O, ws = tensors(device="cuda")
    binding.l2kv_decode_workspace_init(ws)
    scale, expected = 0.0, None
    if change == "stride":
        K, expected = torch.zeros((1, 2, 64, 8), dtype=K.dtype, device="cuda").transpose(2, 3), ValueError
    elif change == "dtype":
        V, expected = V.float(), AssertionError
    elif change == "shape":
        V, expected = V[:, :, :7].contiguous(), AssertionError
    elif change == "dims":
        Q, expected = Q[0], ValueError
    elif change == "output":
        O, expected = O[:, :3].contiguous(), AssertionError
    elif change == "half":
        Q, K, V, expected = Q.half(), K.half(), V.half(), TypeError
    elif change == "nan_scale":
        scale, expected = float("nan"), l2kv.L2KVError
    elif change == "workspace":
        ws, expected = ws[:16], l2kv.L2KVError
    elif change == "group":
        Q, O, expected = Q[:, :3].contiguous(), O[:, :3].contiguous(), l2kv.L2KVError
    for call in (l2kv.l2kv_decode_attn, l2kv.l2kv_decode_attn_out):
        if expected is None:
            call(Q, K, V, O, ws, scale=scale, stream=torch.cuda.current_stream())
        else:
            with pytest.raises(expected):
                call(Q, K, V, O, ws, scale=scale)


@pytest.mark.gpu
def test_subclass_of_tensor_takes_the_python_way():
    class Named(torch.Tensor):
        pass
    Q, K, V, O, ws = tensors(device="cuda")
    binding.l2kv_decode_workspace_init(ws)
    V.normal_()
    sub = O.clone().as_subclass(Named)
    assert binding.calls().decode_attn(Q, K, V, sub, ws, 0.0, None, binding._stream) is None
    l2kv.l2kv_decode_attn(Q, K, V, sub, ws)
    l2kv.l2kv_decode_attn(Q, K, V, O, ws)
    assert torch.equal(sub.as_subclass(torch.Tensor), O) and O.abs().sum() > 0


def compress_tensors(dtype=torch.bfloat16):
    K, V = (torch.randn((1, 2, 100, 64), device="cuda").to(dtype) for _ in range(2))
    norms, idx = torch.empty((1, 2, 100), device="cuda"), torch.empty((1, 2, 50), dtype=torch.int32, device="cuda")
    Kc, Vc = (torch.empty((1, 2, 50, 64), dtype=dtype, device="cuda") for _ in range(2))
    return [K, V, norms, idx, Kc, Vc, torch.zeros(256, dtype=torch.uint8, device="cuda")]


@pytest.mark.gpu
@pytest.mark.parametrize("at,change,expected", [
    (0, lambda x: x.transpose(2, 3).contiguous().transpose(2, 3), ValueError), (0, lambda x: x.half(), AssertionError), (0, lambda x: x.cpu(), ValueError),
    (1, lambda x: x[:, :, :99].contiguous(), AssertionError), (1, lambda x: x.float(), AssertionError), (2, lambda x: x.double(), AssertionError),
    (2, lambda x: x[..., :99].contiguous(), AssertionError), (3, lambda x: x.long(), AssertionError), (3, lambda x: x[:, :1].contiguous(), AssertionError),
    (4, lambda x: x[..., :32].contiguous(), AssertionError), (5, lambda x: x.float(), AssertionError), (6, lambda x: x[:16], l2kv.L2KVError),
    (6, lambda x: x[1:], l2kv.L2KVError)])
def test_compress_errors(at, change, expected):
    args = compress_tensors()
    args[at] = change(args[at])
    with pytest.raises(expected):
        l2kv.l2kv_compress(args[0], args[1], 0.5, *args[2:])


@pytest.mark.gpu
def test_same_arguments(monkeypatch):
    """Both ways reach the C entry points with the same arguments."""
    other = torch.cuda.Stream()
    Q, K, V, O, ws = tensors(device="cuda")
    binding.l2kv_decode_workspace_init(ws)
    c, half = compress_tensors(), O.bfloat16()
    calls = [lambda s: l2kv.l2kv_decode_attn(Q, K, V, O, ws, scale=0.25, stream=s), lambda s: l2kv.l2kv_decode_attn_out(Q, K, V, half, ws, stream=s),
             lambda s: l2kv.l2kv_compress(c[0], c[1], 0.5, *c[2:], slab_heads=1, stream=s)]
    seen = []

    def entry(name, argtypes):
        def record(*args):
            seen.append((name,) + args)
            return 0
        return C.CFUNCTYPE(C.c_int, *argtypes)(record)
    names = ("l2kv_decode_attn", "l2kv_decode_attn_out", "l2kv_compress")
    entries = {n: entry(n, binding.SIGNATURES[n][1]) for n in names}

    class Library:
        def __getattr__(self, name):
            return entries[name] if name in entries else getattr(real, name)
    real = binding.lib()
    monkeypatch.setattr(binding, "_lib", Library())
    try:
        for way in (None, binding._PythonCalls):
            binding._calls = way
            for stream in (None, other):
                for call in calls:
                    call(stream)
    finally:
        binding._calls = None                                         # bound to the real library again
    assert len(seen) == 12 and {s[-1] or 0 for s in seen} == {0, other.cuda_stream}
    assert seen[:6] == seen[6:]


@pytest.mark.gpu
def test_work_is_done_on_the_stream_that_is_given():
    """On a stream that is kept busy, so that the call on it comes after a copy made there, whatever the current one does."""
    Q, K, V, O, ws = tensors(device="cuda")
    binding.l2kv_decode_workspace_init(ws)
    c, late = compress_tensors(), torch.randn((1, 2, 100, 64), device="cuda").bfloat16()
    V2, busy = torch.randn_like(V), torch.zeros(1 << 27, device="cuda")
    torch.cuda.synchronize()
    other = torch.cuda.Stream()
    with torch.cuda.stream(other):
        for _ in range(20):
            busy.add_(1.0)                                            # some milliseconds
        V.copy_(V2)
        c[0].copy_(late)
    l2kv.l2kv_decode_attn(Q, K, V, O, ws, stream=other)
    l2kv.l2kv_compress(c[0], c[1], 0.5, *c[2:], stream=other)
    torch.cuda.synchronize()
    want, norms = torch.empty_like(O), torch.empty_like(c[2])
    l2kv.l2kv_decode_attn(Q, K, V2, want, ws)
    l2kv.l2kv_norms(late, norms)
    assert torch.equal(O, want) and O.abs().sum() > 0 and torch.equal(c[2], norms)
