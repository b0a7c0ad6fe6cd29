"""The binding's native calls without a GPU: native/calls.cpp linked with stand-ins for the library that
count calls and return a set status, given tensors that say they are on a GPU (their storage is host
memory nobody reads).

An error of the library is raised once, from the one call that was made: a call that reports an error may
have enqueued its kernels, so running it again could apply an update in place twice.
"""
import ctypes
import importlib.machinery
import importlib.util
import os
import shutil
import subprocess
import sysconfig
import types

import pytest
import torch

import paper_2609_32518_amd as u

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
B, H, GH, GW, C, S, R, W = 1, 2, 2, 3, 2, 0, 4, 1
T = GH * GW
N = C * T


@pytest.fixture(scope="module")
def module(tmp_path_factory):
    if shutil.which("g++") is None or not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"):
        pytest.skip("needs g++ and the HIP headers")
    spec = importlib.util.spec_from_file_location("unstep_build", os.path.join(ROOT, "paper_2609_32518_amd", "build.py"))
    b = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(b)
    d, tl = tmp_path_factory.mktemp("calls"), os.path.join(os.path.dirname(torch.__file__), "lib")
    inc = os.path.join(os.path.dirname(torch.__file__), "include")
    so = str(d / "_calls.so")
    r = subprocess.run(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM", f"-I{ROOT}/include",
                        f"-isystem{inc}", f"-isystem{inc}/torch/csrc/api/include", f"-isystem{b.ROCM}/include",
                        f"-isystem{sysconfig.get_paths()['include']}", b.CALLS_SRC,
                        os.path.join(ROOT, "tests", "c_abi", "stub_unstep.cpp"), "-o", so, f"-L{tl}", "-ltorch_python", "-ltorch",
                        "-ltorch_cpu", "-lc10", "-lc10_hip", f"-Wl,-rpath,{tl}"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    loader = importlib.machinery.ExtensionFileLoader("_calls", so)
    mod = importlib.util.module_from_spec(importlib.util.spec_from_loader("_calls", loader))
    loader.exec_module(mod)
    return mod, so


class Stub:
    """The stand-in library: its counters, and the binding's functions by name."""

    def __init__(self, so):
        self.so = ctypes.CDLL(so)
        for name, (res, args) in u.SIGNATURES.items():
            if hasattr(self.so, name):
                f = getattr(self.so, name)
                f.restype, f.argtypes = res, args
        self.unstep_cache_destroy = u.lib.unstep_cache_destroy
        self.calls = ctypes.c_int.in_dll(self.so, "stub_calls")
        self.fail_next = ctypes.c_int.in_dll(self.so, "stub_fail_next")
        self.handle = ctypes.c_void_p.in_dll(self.so, "stub_handle")
        self.optional = ctypes.c_void_p.in_dll(self.so, "stub_pointer")
        self.scratch = ctypes.c_void_p.in_dll(self.so, "stub_scratch")
        self.workspace = ctypes.c_size_t.in_dll(self.so, "stub_workspace")

    def __getattr__(self, name):
        return getattr(self.so, name)


@pytest.fixture
def stub(module, monkeypatch):
    mod, so = module
    s = Stub(so)
    s.calls.value, s.fail_next.value, s.workspace.value, s.optional.value = 0, u.OK, 0, 1
    monkeypatch.setattr(u, "_calls", mod)
    monkeypatch.setattr(u, "_stream", lambda stream: 0)          # the Python path's stream
    return s


def on_gpu(*shape, dtype=torch.bfloat16, memory=True):
    """A contiguous tensor of host memory that says it is on a GPU (or one without memory)."""
    n = dtype.itemsize
    for x in shape:
        n *= x
    mem = torch.zeros(max(n, 16) + 16, dtype=torch.uint8)
    ptr = -(-mem.data_ptr() // 16) * 16 if memory else 0
    n = n if memory else 0
    dev = torch.device("cuda:0")
    storage = torch._C._construct_storage_from_data_pointer(ptr, dev, n)
    stride = [1]
    for x in reversed(shape[1:]):
        stride.insert(0, stride[0] * x)
    t = torch._C._construct_CUDA_Tensor_From_Storage_And_Metadata(
        dict(dtype=dtype, size=tuple(shape), stride=tuple(stride), storage_offset=0, device=dev, nbytes=n, data_ptr=ptr), storage)
    t.memory = mem
    return t


def cache(cls=u.Cache):
    shape = (B, H, (S + R) * T, 128)
    return cls(B, H, GH, GW, S, R, k_cache=on_gpu(*shape), v_cache=on_gpu(*shape))


def step_args():
    q, k, v = (on_gpu(B, N, H, 128) for _ in range(3))
    cos, sin = (on_gpu(N, 64, dtype=torch.float32) for _ in range(2))
    return q, k, v, cos, sin


def call(name, c):
    """One call of an entry point with every output given, and that output."""
    q, k, v, cos, sin = step_args()
    out = on_gpu(B, N, H, 128)
    if name == "append":
        return lambda: c.unstep_kv_append(0, C, q, k, v, cos, sin, q_rot=out), out
    if name == "append_qknorm":
        w = on_gpu(H * 128)
        return lambda: c.unstep_kv_append_qknorm(0, C, q, k, v, cos, sin, w, w, q_rot=out), out
    if name == "window_attn":
        return lambda: c.unstep_window_attn(0, C, W, q, out=out), out
    if name == "step":
        return lambda: c.unstep_step(0, C, W, q, k, v, cos, sin, q_rot=k, out=out), out
    if name == "linear":
        x, y = on_gpu(4, 16), on_gpu(4, 8)
        return lambda: u.unstep_linear(x, on_gpu(8, 16), on_gpu(8), out=y), y
    x = on_gpu(64)
    f = u.unstep_renoise if name == "renoise" else u.unstep_emit
    return lambda: f(x, on_gpu(64), 0.5, out=x), x


NAMES = ["append", "append_qknorm", "window_attn", "step", "linear", "renoise", "emit"]


@pytest.mark.parametrize("name", NAMES)
def test_library_error_is_raised_from_one_call(stub, monkeypatch, name):
    c = cache()
    monkeypatch.setattr(u, "lib", stub)
    f, out = call(name, c)
    assert f() is out and stub.calls.value == 1
    for code in (u.E_HIP, u.E_SHAPE):
        stub.calls.value, stub.fail_next.value = 0, code
        with pytest.raises(u.UnstepError, match="the stub's error") as e:
            f()
        assert e.value.code == code and stub.calls.value == 1
        assert f() is out and stub.calls.value == 2          # the error does not stay


@pytest.mark.parametrize("name", ["append", "append_qknorm", "step", "lse"])
def test_storage_without_memory_goes_to_the_library_as_null(stub, name):
    """Tables or a log-sum-exp whose storage has no memory (the typed data pointer of such a tensor
    throws): the library gets a null pointer, as from the Python path, and says what it says of one."""
    c = cache()
    q, k, v, cos, sin = step_args()
    w, out = on_gpu(H * 128), on_gpu(B, N, H, 128)
    bare = lambda *shape: on_gpu(*shape, dtype=torch.float32, memory=False)
    if name == "append":
        r = c.unstep_kv_append(0, C, q, k, v, bare(N, 64), sin, q_rot=out)
    elif name == "append_qknorm":
        r = c.unstep_kv_append_qknorm(0, C, q, k, v, cos, bare(N, 64), w, w, q_rot=out)
    elif name == "step":
        r = c.unstep_step(0, C, W, q, k, v, bare(N, 64), sin, q_rot=k, out=out, use_split=False)
    else:
        r = c.unstep_window_attn(0, C, W, q, out=out, lse=bare(B, H, N), use_split=False)
    assert r is out and stub.calls.value == 1
    assert stub.optional.value is None


@pytest.mark.parametrize("name", NAMES[:4])
def test_a_finalised_cache_is_refused(stub, name):
    """After __del__ the handle is gone: the library is asked with a null handle, not the freed one."""
    c = cache()
    f, out = call(name, c)
    assert f() is out and stub.handle.value is not None
    c.__del__()
    stub.calls.value = 0
    with pytest.raises(u.UnstepError) as e:              # the Python path, the library itself
        f()
    assert e.value.code == u.E_NULL and stub.calls.value == 0


@pytest.mark.parametrize("name", ["window_attn", "step"])
@pytest.mark.parametrize("method,how", [(m, h) for m in ("workspace", "workspace_bytes", "_step_workspace")
                                        for h in ("subclass", "class", "instance")] + [("_chunk_out", "subclass")])
def test_replaced_methods_are_asked(stub, monkeypatch, name, how, method):
    """A subclass or a program that replaces a scratch method (or a subclass that makes its own outputs)
    is asked on every call, as through the Python path."""
    scratch, asked = on_gpu(4096, dtype=torch.uint8), []
    own = getattr(u.Cache, method)

    def mine(self, *a):
        asked.append(method)
        return 1024 if method == "workspace_bytes" else own(self, *a) if method == "_chunk_out" else scratch

    cls = type("Own", (u.Cache,), {method: mine}) if how == "subclass" else u.Cache
    c = cache(cls)
    c._ws = on_gpu(2048, dtype=torch.uint8)
    stub.workspace.value = 1024
    if how == "class":
        monkeypatch.setattr(u.Cache, method, mine)
    elif how == "instance":
        monkeypatch.setattr(c, method, mine.__get__(c), raising=False)
    monkeypatch.setattr(u, "lib", stub)
    f, out = call(name, c)
    for n in (1, 2):
        assert f() is out and stub.calls.value == n
        if method == "_step_workspace" and name == "window_attn":
            assert asked == []
        else:
            assert len(asked) >= n
    assert stub.scratch.value == (scratch if method in ("workspace", "_step_workspace") and asked else c._ws).data_ptr()


@pytest.mark.parametrize("name", ["window_attn", "step"])
def test_own_scratch_methods_stay_native(stub, monkeypatch, name):
    c = cache(type("Plain", (u.Cache,), {}))             # a subclass that replaces nothing
    c._ws, stub.workspace.value = on_gpu(2048, dtype=torch.uint8), 1024
    monkeypatch.setattr(u, "lib", types.SimpleNamespace(unstep_cache_destroy=u.lib.unstep_cache_destroy))  # no Python path
    f, out = call(name, c)
    assert f() is out and stub.calls.value == 1 and stub.scratch.value == c._ws.data_ptr()
