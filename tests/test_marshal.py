"""The binding's argument marshalling, native and through ctypes: what reaches the C function, and what is
refused.  The function called is a recorder with the signature of the real one."""
import ctypes as C
import os
import sysconfig

import numpy as np
import pytest
import torch

import paper_2509_08309_amd as H
from paper_2509_08309_amd import binding


@pytest.fixture(scope="module")
def lib():
    return binding.load(build_if_missing=True)


@pytest.fixture(params=["native", "ctypes"])
def recorder(request):
    """recorder(lib, name): (callable through the marshalling, list of the argument tuples that arrived)"""
    def make(lib, name):
        from paper_2509_08309_amd import _marshal
        argtypes = getattr(lib, name).argtypes
        types = [C.c_void_p if hasattr(t, "contents") else t for t in argtypes]
        got = []
        fn = C.CFUNCTYPE(C.c_int, *types)(lambda *a: got.append(a) or 5)
        address = C.cast(fn, C.c_void_p).value
        if request.param == "native":
            call = _marshal.bind(name, address)
        else:
            real = C.CFUNCTYPE(C.c_int, *argtypes)(address)
            real.argtypes = argtypes
            call = binding._by_ctypes(real)
        return (lambda *a, _keep=fn: call(*a)), got
    return make


def test_arguments_arrive_as_they_are(lib, recorder):
    call, got = recorder(lib, "hetis_attn_decode_ws")
    s = H.make_shape(4, 8, 8, 64, 16)
    t = torch.zeros(8, dtype=torch.float16)[3:]
    n = np.zeros(4, dtype=np.int32)
    big = (1 << 63) + 4096
    assert call(s, t, None, big, n, 4096, n[1:], np.int64(7), np.float32(0.125), t, 1 << 40, 1 << 35, None) == 5
    assert got == [(C.addressof(s), t.data_ptr(), None, big, n.ctypes.data, 4096, n.ctypes.data + 4, 7, 0.125,
                    t.data_ptr(), 1 << 40, 1 << 35, None)]
    call, got = recorder(lib, "hetis_kv_copy_tiles")
    a, b = H.make_pool(8, 64, 10), H.make_pool(4, 64, 1 << 33)
    assert call(a, 16, 32, b, 48, 64, 80, 96, 3, 112, 128, -2, 7) == 5
    assert call(None, 16, 32, None, 48, 64, 80, 96, 3, 112, 128, (1 << 32) + 1, 7) == 5
    assert got == [(C.addressof(a), 16, 32, C.addressof(b), 48, 64, 80, 96, 3, 112, 128, -2, 7),
                   (None, 16, 32, None, 48, 64, 80, 96, 3, 112, 128, 1, 7)]


def test_every_call_has_the_signature_that_ctypes_knows(lib, recorder):
    for name in vars(lib.call):
        call, got = recorder(lib, name)
        args, want = [], []
        for i, t in enumerate(getattr(lib, name).argtypes):
            struct = hasattr(t, "contents") and t._type_
            v = struct() if struct else 0.5 * i if t is C.c_float else 1000 + i
            args.append(v)
            want.append(C.addressof(v) if struct else v)
        assert call(*args) == 5 and got == [tuple(want)], name
        with pytest.raises(TypeError):
            call(*args[:-1])
        with pytest.raises(TypeError):
            call(*args, 0)


def test_what_is_no_argument_is_refused(lib, recorder):
    call, got = recorder(lib, "hetis_kv_append")
    ok = [H.make_shape(4, 8, 8, 64, 16)] + [16] * 5 + [4, 10, 16, 16, None]
    assert call(*ok) == 5
    for i, bad, err in ((0, None, TypeError), (0, H.make_pool(8, 64, 10), (TypeError, C.ArgumentError)), (1, "x", AttributeError),
                        (1, 1.5, AttributeError), (6, None, TypeError), (6, "x", ValueError)):
        args = list(ok)
        args[i] = bad
        with pytest.raises(err):
            call(*args)
    assert len(got) == 1
    from paper_2509_08309_amd import _marshal
    assert _marshal.bind("hetis_attn_version", 16) is None


def test_the_library_alone_is_enough(lib, monkeypatch):
    """Without an extension for this interpreter (another one's has another name) the library loads as it is,
    and its calls go through ctypes."""
    from paper_2509_08309_amd import build
    suffix = sysconfig.get_config_var("EXT_SUFFIX")
    assert "-" in suffix and binding.MARSHAL_PATH == build.MARSHAL and build.MARSHAL.endswith("_marshal" + suffix)
    monkeypatch.setattr(binding, "MARSHAL_PATH", os.path.join(binding.HERE, "_marshal.of-another-interpreter.so"))
    monkeypatch.setattr(binding, "_lib", None)
    alone = binding.load()
    s = H.make_shape(0, 8, 8, 64, 16)                       # refused before anything is launched
    args = (s, 16, 16, 16, 16, 16, 16, 4, 0.125, 16, 256, 256, None)
    assert alone.call.hetis_attn_decode_ws(*args) == lib.call.hetis_attn_decode_ws(*args) == binding.HETIS_ERR_BAD_SHAPE


def test_a_build_without_headers_is_one(monkeypatch):
    """No Python headers or no C++ compiler: nothing is current for want of the extension."""
    from paper_2509_08309_amd import build
    monkeypatch.setattr(build, "MARSHAL", os.path.join(build.HERE, "_marshal.of-another-interpreter.so"))
    monkeypatch.setattr(build, "sources", lambda: [])
    assert build.marshal_compiler() and not build.is_current()
    monkeypatch.setattr(build.sysconfig, "get_paths", lambda: {"include": "/nowhere"})
    assert build.marshal_compiler() is None and build.is_current()
