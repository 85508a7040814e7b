"""The native marshalling of launch arguments: what it leaves to ctypes, what it raises, and that it does what the ctypes line does."""
import ctypes
import os
import re
import subprocess
import sys

import pytest
import torch

from paper_2409_16626_amd import hif8

P = 0x1000  # never dereferenced: n == 0, or the call is refused


def test_every_function_has_the_arguments_of_the_library():
    for name in [n for n in dir(hif8._native) if n.startswith("hif8_")]:
        args, _ = hif8._SIGS[name]
        f = getattr(hif8._native, name)
        assert f(*[object()] * len(args)) is NotImplemented and f(*[0] * (len(args) + 1)) is NotImplemented and f() is NotImplemented
        assert args[-1] is ctypes.c_void_p  # the stream
    src = open(hif8.__file__).read()
    assert len(re.findall(r"_native\.hif8_\w+\(", src)) >= 30


def test_usual_arguments_and_errors():
    f = hif8._native.hif8_encode_f32
    assert f(P, P, 0, 1.0, 0, 0) is None and f(None, None, 0, 1, 0, 0) is None  # nothing to do
    for bad, status in (((P, P, 16, 0.0, 0, 0), -3), ((None, P, 16, 1.0, 0, 0), -1), ((P, P, 16, 1.0, 5, 0), -2)):
        with pytest.raises(hif8.Hif8Error) as e:
            f(*bad)
        assert e.value.status == status
    with pytest.raises(hif8.Hif8Error):
        hif8.hif8_encode_f32(P, P, 16, scale=0.0, stream=0)


def test_truth_values_stream_objects_and_a_default_device():
    """pow2=True, a torch.cuda.Stream and torch.set_default_device are ordinary arguments: none of them goes through both ways."""
    f = hif8._native.hif8_encode_f32

    class Stream:
        cuda_stream = 0

    class Other:
        cuda_stream = "s"

    assert f(P, P, False, 1.0, True, 0) is None and f(P, P, 0, 1.0, 0, Stream()) is None
    assert f(P, P, 0, 1.0, 0, Other()) is NotImplemented and f(P, P, 0, 1.0, 0, Stream) is None and f(P, P, 0, 1.0, 0, True) is NotImplemented
    with pytest.raises(hif8.Hif8Error) as e:
        f(None, P, True, 1.0, 0, Stream())
    assert e.value.status == -1
    with torch.device("cpu"):
        assert f(P, P, 0, 1.0, 0, 0) is None
    torch.set_default_device("cpu")
    try:
        assert f(P, P, 0, 1.0, 0, 0) is None
    finally:
        torch.set_default_device(None)
    with pytest.raises(AttributeError):
        hif8.hif8_encode_f32(P, P, 0, stream="s")


class Sub(torch.Tensor):
    pass


def test_what_is_left_to_ctypes():
    f, q = hif8._native.hif8_encode_f32, hif8._native.hif8_quantize_tensor_f32
    cpu = torch.zeros(16)
    for args in ((cpu, P, 0, 1.0, 0, 0), (cpu.as_subclass(Sub), P, 0, 1.0, 0, 0), (P, P, -1, 1.0, 0, 0), (P, P, 1 << 64, 1.0, 0, 0), (P, P, 0.0, 1.0, 0, 0), (True, P, 0, 1.0, 0, 0),
                 (P, P, None, 1.0, 0, 0), (P, P, 0, None, 0, 0), (P, P, 0, 1.0, -1, 0), (P, P, 0, 1.0, 1 << 32, 0), (P, P, 0, 1.0, 0, None), (P, P, 0, 1.0, 0, "s"),
                 (1 << 70, P, 0, 1.0, 0, 0), ("p", P, 0, 1.0, 0, 0), (P, P, 0, 10 ** 400, 0, 0)):
        assert f(*args) is NotImplemented, args
    assert q(P, P, P, 0, 1.0, 1, 0, P, P, P, None, 0) is NotImplemented  # no tensor to take the bytes from
    with pytest.raises(ValueError):
        hif8.hif8_encode_f32(cpu, P, 0, stream=0)
    with pytest.raises(ctypes.ArgumentError):
        hif8.hif8_encode_f32(P, P, "n", stream=0)

    class Mode(torch.overrides.TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    with Mode():
        assert f(P, P, 0, 1.0, 0, 0) is NotImplemented
        with torch.device("cpu"):
            assert f(P, P, 0, 1.0, 0, 0) is NotImplemented
    with torch.device("cpu"), Mode():
        assert f(P, P, 0, 1.0, 0, 0) is NotImplemented
    assert f(P, P, 0, 1.0, 0, 0) is None
    assert not any(hasattr(hif8._native, n) for n in ("hif8_init", "hif8_calibrate_layer_f32", "hif8_multi_cast_f32"))


ROOT = os.path.dirname(os.path.dirname(os.path.abspath(hif8.__file__)))
IMPORT = """
import os, sys, warnings
from paper_2409_16626_amd import build
%s
with warnings.catch_warnings(record=True) as seen:
    warnings.simplefilter("always")
    from paper_2409_16626_amd import hif8
assert [w.category for w in seen if "native" in str(w.message)] == [RuntimeWarning], [str(w.message) for w in seen]
hif8.hif8_encode_f32(0x1000, 0x1000, 0, 1.0, stream=0)
for bad, status in ((dict(scale=0.0), -3), (dict(rounding_mode=5), -2)):
    try:
        hif8.hif8_encode_f32(0x1000, 0x1000, 16, stream=0, **bad)
    except hif8.Hif8Error as e:
        assert e.status == status
    else:
        assert False
print("went through ctypes")
"""


# nothing built and no compiler; nowhere to put it; built for another torch, and no compiler; a module that does not load; a library without
# one of its functions
@pytest.mark.parametrize("what", ["no_compiler", "read_only", "other_torch", "broken", "other_library"])
def test_package_without_native_marshalling(tmp_path, what):
    """The library is all that the package needs: without the extension module it warns, and its calls go through ctypes."""
    there = str(tmp_path / "_native_call.so")
    setup = {
        "no_compiler": "os.environ['PATH'] = '/nonexistent'; build.native_path = lambda: %r" % there,
        "read_only": "build.native_path = lambda: '/nonexistent/_native_call.so'",
        "other_torch": "os.environ['PATH'] = '/nonexistent'; import torch; torch.__version__ = '0.0.0'",
        "broken": "build.native_path = lambda: %r; open(%r, 'w').write('no module')" % (there, there),
        "other_library": """
import ctypes, importlib.util
class Loader:  # hands the module another library's handle
    def __init__(self, spec): self.real = spec.loader
    def create_module(self, spec): return self.real.create_module(spec)
    def exec_module(self, module):
        self.real.exec_module(module)
        set_up = module.set_up
        module.set_up = lambda handle, *rest: set_up(ctypes.CDLL('libc.so.6')._handle, *rest)
from_file = importlib.util.spec_from_file_location
def spec_of(name, path):
    spec = from_file(name, path)
    spec.loader = Loader(spec)
    return spec
importlib.util.spec_from_file_location = spec_of
""",
    }[what]
    r = subprocess.run([sys.executable, "-c", IMPORT % setup], cwd=ROOT, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=300)
    assert r.returncode == 0 and "went through ctypes" in r.stdout, r.stdout


def test_native_module_is_of_this_torch_python_and_header(monkeypatch, tmp_path):
    from paper_2409_16626_amd import build
    path = build.native_path()
    assert os.path.exists(path) and hif8._native.__file__ == path
    monkeypatch.setattr(torch, "__version__", "0.0.0")
    assert build.native_path() != path
    monkeypatch.undo()
    header = tmp_path / "hif8.h"
    header.write_text(open(build.NATIVE_INPUTS[1]).read() + "\n")
    monkeypatch.setattr(build, "NATIVE_INPUTS", [build.NATIVE_INPUTS[0], str(header)])
    assert build.native_path() != path


@pytest.mark.gpu
def test_same_as_ctypes_on_any_stream():
    hif8.hif8_init()
    x = torch.randn(3, 1000, device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    got = []
    side = torch.cuda.Stream()
    for case in range(5):
        codes, am, sc = torch.zeros(3000, dtype=torch.uint8, device="cuda"), torch.zeros(1, device="cuda"), torch.zeros(2, device="cuda")
        ws = torch.empty(hif8.hif8_quantize_workspace_bytes(), dtype=torch.uint8, device="cuda")
        torch.cuda.synchronize()
        if case == 0:  # torch's current stream
            assert hif8._native.hif8_quantize_tensor_f32(x, None, codes, 3000, 32768.0, 1, 0, am, sc, ws, None, None) is None
        elif case == 1:  # ctypes
            hif8._check(hif8.lib.hif8_quantize_tensor_f32(x.data_ptr(), None, codes.data_ptr(), 3000, 32768.0, 1, 0, am.data_ptr(), sc.data_ptr(), ws.data_ptr(), ws.numel(), None))
        elif case == 2:
            with torch.cuda.stream(side):
                hif8.hif8_quantize_tensor_f32(x, None, codes, 3000, am, sc, ws, 32768.0, True)
        elif case == 3:
            hif8.hif8_quantize_tensor_f32(x.view(-1), None, codes, 3000, am, sc, ws, 32768, 1, stream=side)
        else:
            hif8.hif8_quantize_tensor_f32(x.data_ptr(), None, codes.data_ptr(), 3000, am, sc, ws.data_ptr(), 32768.0, 1, stream=side.cuda_stream, workspace_bytes=ws.numel())
        torch.cuda.synchronize()
        got.append(torch.cat([codes.float(), am, sc]))
    assert all(torch.equal(g, got[0]) for g in got) and got[0][3000] == x.abs().max()
    with pytest.raises(ValueError):
        hif8.hif8_encode_f32(x.t(), torch.empty(3000, dtype=torch.uint8, device="cuda"), 3000)
    with pytest.raises(hif8.Hif8Error):  # a workspace of no bytes
        hif8.hif8_quantize_tensor_f32(x, None, torch.empty(3000, dtype=torch.uint8, device="cuda"), 3000, got[0][:1].clone(), got[0][:2].clone(), torch.empty(0, dtype=torch.uint8, device="cuda"))
