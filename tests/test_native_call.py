"""DsfqLinear's calls in native code (csrc/call.cpp): the outputs of the Python path, its errors, and nothing taken that the Python path would not."""
import importlib
import importlib.machinery
import importlib.util
import os
import shutil
import subprocess
import sys
import threading

import pytest
import torch

import paper_2509_21302_amd as q
from paper_2509_21302_amd import binding as B
from paper_2509_21302_amd import build


def test_the_module_is_built_and_knows_its_entry_points():
    assert B._call is not None
    q.load_library()
    with pytest.raises(ValueError):
        B._call.bind(len(B.LINEAR_KINDS), 0)
    with pytest.raises(TypeError):
        B._call.linear(0)


def test_the_library_is_built_where_the_module_cannot_be(monkeypatch, tmp_path, capsys):
    """No host compiler: libqvggt.so is linked all the same, and a module of an older source does not stay behind."""
    monkeypatch.setattr(build, "LIB", str(tmp_path / "libqvggt.so"))
    monkeypatch.setattr(build, "CALL", str(tmp_path / "_call.so"))
    monkeypatch.setattr(build, "BUILD", str(tmp_path))
    monkeypatch.setattr(build, "_compile", lambda src, save_temps: src)
    monkeypatch.setenv("CXX", str(tmp_path / "no-compiler"))
    (tmp_path / "_call.so").write_text("old")
    run = subprocess.run

    def link(cmd, **kw):
        if cmd[0] != build.HIPCC:
            return run(cmd, **kw)
        (tmp_path / "libqvggt.so.tmp").write_text("linked")
    monkeypatch.setattr(build.subprocess, "run", link)
    build.build()
    assert (tmp_path / "libqvggt.so").read_text() == "linked" and not os.path.exists(tmp_path / "_call.so")
    assert "_call.so was not built" in capsys.readouterr().err


@pytest.mark.parametrize("built_for,used", [(torch.__version__, True), ("1.0.0", False), (None, False)])
def test_a_module_of_another_torch_is_not_used(monkeypatch, tmp_path, built_for, used):
    shutil.copy(B.__file__, tmp_path / "binding.py")
    (tmp_path / "__init__.py").write_text("")
    (tmp_path / "_call.py").write_text("" if built_for is None else f"torch_version = {built_for!r}")
    name = f"another_build_{used}_{built_for is None}"
    spec = importlib.util.spec_from_file_location(name, tmp_path / "__init__.py", submodule_search_locations=[str(tmp_path)])
    monkeypatch.setitem(sys.modules, name, importlib.util.module_from_spec(spec))
    binding = importlib.import_module(name + ".binding")
    assert (binding._call is not None) == used
    assert build.CALL.endswith(importlib.machinery.EXTENSION_SUFFIXES[0]) and B._call.__file__ == build.CALL


@pytest.mark.parametrize("X", [torch.zeros(2, 128), torch.zeros(2, 128, dtype=torch.float16), torch.zeros(128), torch.zeros(2, 256)[:, ::2], None, 3])
def test_what_is_not_an_ordinary_device_tensor_is_left_to_the_python_path(X):
    w = torch.zeros(128)
    for kind in range(len(B.LINEAR_KINDS)):
        assert B.native_linear(kind, X, None, w, None, w, w, None, None, w, 16, 4) is None


def _layer(bits, act_bits, pre_gelu, K):
    g = torch.Generator(device="cuda:0").manual_seed(K + bits)
    W, X = torch.randn(144, K, device="cuda:0", generator=g) * 0.02, torch.randn(70, K, device="cuda:0", generator=g)
    bias = torch.randn(144, device="cuda:0", generator=g).to(torch.bfloat16)
    signs = (torch.randint(0, 2, (K,), device="cuda:0", generator=g, dtype=torch.int8) * 2 - 1).contiguous()
    return q.DsfqLinear(W.to(torch.bfloat16), bias, signs, X.to(torch.bfloat16), bits=bits, act_bits=act_bits, pre_gelu=pre_gelu), X


CASES = [(4, 4, False, 1024, torch.bfloat16), (4, 4, False, 256, torch.float32), (4, 4, True, 1024, torch.bfloat16), (8, 8, False, 1024, torch.bfloat16),
         (4, 8, False, 1024, torch.float32), (6, 6, False, 768, torch.bfloat16)]


@pytest.mark.gpu
@pytest.mark.parametrize("bits,act_bits,pre_gelu,K,dtype", CASES)
def test_the_same_output_as_the_python_path(monkeypatch, bits, act_bits, pre_gelu, K, dtype):
    layer, X = _layer(bits, act_bits, pre_gelu, K)
    X = X.to(dtype)
    taken = []
    native = B.native_linear
    monkeypatch.setattr(B, "native_linear", lambda *a: taken.append(native(*a)) or taken[-1])
    got = layer(X)
    out = torch.full((73, 144), 7.0, dtype=torch.bfloat16, device="cuda:0")
    assert layer(X, out[:70]).data_ptr() == out.data_ptr() and (out[70:] == 7.0).all().item()
    assert taken[0] is got and taken[1] is not None
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        on_side = layer(X)
    side.synchronize()
    monkeypatch.setattr(B, "native_linear", lambda *a: None)
    want = layer(X)
    assert got.shape == want.shape and got.dtype == torch.bfloat16 and got.device == want.device
    for y in (got, out[:70], on_side):
        assert torch.equal(y.view(torch.int16), want.view(torch.int16))


@pytest.mark.gpu
def test_errors_and_threads():
    layer, X = _layer(4, 4, False, 1024)
    X = X.to(torch.bfloat16)
    with pytest.raises(ValueError, match="contiguous"):
        layer(torch.cat([X, X], 1)[:, ::2])
    with pytest.raises(ValueError, match="device tensors"):
        layer(X.cpu())
    with pytest.raises(ValueError, match="unsupported dtype"):
        layer(X.half())
    with pytest.raises(q.QvggtError, match="QVGGT_ERR_ALIGN"):
        layer(torch.cat([X, X]).flatten()[1:1 + 1024].view(1, 1024))
    with pytest.raises(q.QvggtError, match="QVGGT_ERR_SHAPE"):
        layer(X, torch.empty(70, 17, dtype=torch.bfloat16, device="cuda:0"))
    assert layer(X[:0]).shape == (0, 144)
    want = layer(X)
    layers = [_layer(4, 4, False, 1024)[0] for _ in range(4)]         # a layer's workspace is one call's at a time
    bad = []

    def work(l):
        for _ in range(50):
            if not torch.equal(l(X), want):
                bad.append(l)
    threads = [threading.Thread(target=work, args=(l,)) for l in layers]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad


@pytest.mark.gpu
def test_an_error_of_the_allocation_is_raised_as_it_is():
    """What a dispatch mode raises where it sees the output's allocation, and the allocator's own error, keep their types."""
    from torch.utils._python_dispatch import TorchDispatchMode

    class Refused(Exception):
        pass

    class NoAllocation(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            if "empty" in func.__name__:
                raise Refused(func.__name__)
            return func(*args, **(kwargs or {}))
    layer, X = _layer(4, 4, False, 1024)
    X = X.to(torch.bfloat16)
    want = layer(X)
    with NoAllocation(), pytest.raises(Refused):
        layer(X)
    layer.N = 1 << 42
    with pytest.raises(torch.OutOfMemoryError):
        layer(X)
    layer.N = 144
    assert torch.equal(layer(X), want)


@pytest.mark.gpu
@pytest.mark.parametrize("which", ["float16", "one dimension", "three dimensions", "not contiguous", "subclass", "conjugate", "host bias", "strided bias", "host workspace",
                                   "strided output", "output of one dimension", "meta"])
def test_what_is_not_an_ordinary_tensor_on_the_device_is_left_to_the_python_path(which):
    """Each differs in one thing from arguments that are taken."""
    class Other(torch.Tensor):
        pass
    dev = "cuda:0"
    layer, X = _layer(4, 4, False, 1024)
    args = dict(X=X.to(torch.bfloat16), bias=layer.bias, out=torch.zeros(70, 144, dtype=torch.bfloat16, device=dev), ws=layer._workspace(70, X.device))

    def call():
        return B.native_linear(B.E2M3, args["X"], layer.signs, layer.inv_smooth, None, layer.Wf, layer.w_scale, args["bias"], args["out"], args["ws"], 144, 4)
    want = call()
    assert want is args["out"]
    want = want.clone()
    name, value = {"float16": ("X", X.half()), "one dimension": ("X", args["X"].flatten()), "three dimensions": ("X", args["X"][None]),
                   "not contiguous": ("X", torch.cat([args["X"]] * 2, 1)[:, ::2]), "subclass": ("X", args["X"].as_subclass(Other)),
                   "conjugate": ("X", torch.zeros(70, 1024, dtype=torch.complex64, device=dev).conj()), "host bias": ("bias", layer.bias.cpu()),
                   "strided bias": ("bias", torch.cat([layer.bias] * 2)[::2]), "host workspace": ("ws", args["ws"].cpu()),
                   "strided output": ("out", torch.zeros(144, 70, dtype=torch.bfloat16, device=dev).t()),
                   "output of one dimension": ("out", torch.zeros(70 * 144, dtype=torch.bfloat16, device=dev)),
                   "meta": ("X", args["X"].to("meta"))}[which]
    kept, args[name] = args[name], value
    assert call() is None
    args[name] = kept
    assert torch.equal(call().view(torch.int16), want.view(torch.int16))
