"""The compiled binding: what it refuses, in which order, and which numbers and pointers reach the library (objects that
answer like device tensors, whose calls end in the library's own argument checks)."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2506_19225_amd import vxl


class Like:
    """Answers like a contiguous device tensor."""
    is_cuda = True

    def __init__(self, shape, ptr=0x1000, contiguous=True):
        self.shape, self.ptr, self.contiguous = shape, ptr, contiguous

    def is_contiguous(self):
        return self.contiguous

    def data_ptr(self):
        return self.ptr

    def numel(self):
        return int(np.prod(self.shape))


DESC = vxl.make_desc(28, 4, 128, "bf16")
Q, KV, LEN = Like((2, 3, 28, 128)), Like((2, 4, 640, 128)), Like((2,))


@pytest.fixture(autouse=True)
def streams(monkeypatch):
    asked = []
    monkeypatch.setattr(torch.cuda, "is_initialized", lambda: True)
    monkeypatch.setattr(vxl, "_current_device", lambda: 0)
    monkeypatch.setattr(vxl, "_raw_stream", lambda dev: asked.append(dev) or 0)
    return asked


def decode(desc=DESC, q=Q, k=KV, v=KV, n=LEN, out=Q, lse=None, ws=None, stream=None):
    return vxl.bilevel_decode(desc, q, k, v, n, out, lse, ws, stream)


def status(*args, **kw):
    with pytest.raises(vxl.VxlError) as e:
        decode(*args, **kw)
    return e.value.status


@pytest.mark.parametrize("bad", [torch.zeros(2, 3, 28, 128), Like((2, 3, 28, 128), contiguous=False)])
def test_refuses_what_is_no_contiguous_device_tensor(bad, streams):
    for kw in (dict(q=bad), dict(k=bad), dict(v=bad), dict(n=bad), dict(out=bad), dict(lse=bad), dict(ws=bad)):
        with pytest.raises(AssertionError, match="contiguous CUDA tensors"):
            decode(**kw)
    assert not streams                                     # (a stream is asked for when all else is found good)


def test_refuses_other_objects(streams):
    for kw, error in ((dict(q=np.zeros((2, 3, 28, 128))), AttributeError), (dict(q=None), AttributeError),
                      (dict(desc=C.c_int(3)), TypeError), (dict(desc="text"), TypeError),
                      (dict(q=Like((2,))), IndexError), (dict(k=Like((2, 4))), IndexError), (dict(stream=5), AttributeError)):
        with pytest.raises(error):
            decode(**kw)
    with pytest.raises(TypeError, match="arguments expected"):
        vxl.native().bilevel_decode(DESC)


def test_what_reaches_the_library(streams):
    """A null output or length, a misaligned pointer, sizes of 0 and scratch memory too small for the sizes given
    are told apart by the library, which launches nothing for any of them."""
    assert status() == vxl.VXL_ERR_WORKSPACE and streams == [0]
    assert status(out=None) == status(n=None) == vxl.VXL_ERR_INVALID_ARG
    for kw in (dict(q=Like(Q.shape, 0x1008)), dict(k=Like(KV.shape, 0x1008)), dict(v=Like(KV.shape, 0x1008)),
               dict(out=Like(Q.shape, 0x1008)), dict(q=Like((0, 3, 28, 128))), dict(q=Like((2, 0, 28, 128))),
               dict(k=Like((2, 4, 0, 128)))):
        assert status(**kw) == vxl.VXL_ERR_INVALID_ARG
    need = vxl.workspace_bytes(vxl.OP_DECODE, None, DESC, 2, 3, 640)
    assert status(ws=Like((need - 1,))) == vxl.VXL_ERR_WORKSPACE
    assert status(ws=Like((need,), 0x1008)) == vxl.VXL_ERR_WORKSPACE
    assert status(desc=vxl.make_desc(28, 4, 96, "bf16")) == vxl.VXL_ERR_UNSUPPORTED


def test_a_null_layout_is_the_librarys_to_refuse():
    class Closed:
        handle = None
    x = Like((2, 4, 8, 128))
    for call in (lambda: vxl.chunk_prefill(Closed, DESC, x, x, x, x), lambda: vxl.chunk_score_topk(Closed, DESC, x, x, 1, x, x),
                 lambda: vxl.chunk_score_topk_mass(Closed, DESC, x, x, 1, x, x), lambda: vxl.pool_sparse_kv(Closed, DESC, x, x, x, x),
                 lambda: vxl.gather_bilevel_kv(Closed, DESC, x, x, x, x, x, x),
                 lambda: vxl.gather_bilevel_kv_pooled(Closed, DESC, x, x, x, x, x, x, x, x),
                 lambda: vxl.bilevel_decode_inplace(Closed, DESC, x, x, x, x, x, x, 8, x)):
        with pytest.raises(vxl.VxlError) as e:
            call()
        assert e.value.status == vxl.VXL_ERR_INVALID_ARG


# Every entry point with its arguments in order, tensors by the letter x (layouts are null ones: the library refuses those);
# the places of the scratch memory, whose number of elements it takes, and of the tensors that it takes sizes from.
X = Like((2, 4, 8, 128))
CALLS = [
    ("chunk_prefill", "layout desc x x x x x x", 7, ()), ("chunk_score_topk", "layout desc x x 1 x x x x 0 x", 10, (2,)),
    ("chunk_score_topk_mass", "layout desc x x 1 x x x x", 8, (2,)), ("gather_bilevel_kv", "layout desc x x x x x x x", None, (5,)),
    ("pool_sparse_kv", "layout desc x x x x", None, ()), ("gather_bilevel_kv_pooled", "layout desc x x x x x x x x x", None, (7,)),
    ("bilevel_decode", "desc x x x x x x x", 7, (1, 2)), ("bilevel_decode_inplace", "layout desc x x x x x x 8 x x x x", 12, (2,))]


class Closed:
    handle = None


@pytest.mark.parametrize("name,form", [c[:2] for c in CALLS])
def test_no_other_object_passes_for_an_address(name, form, streams):
    """A number, a truth value, bytes, a descriptor or a ctypes pointer where a tensor belongs, and anything but a descriptor
    where one belongs, are refused before the library sees them."""
    call, kinds = getattr(vxl, name), form.split()
    args = [Closed if x == "layout" else DESC if x == "desc" else X if x == "x" else int(x) for x in kinds]
    for i, kind in enumerate(kinds):
        wrong = {"x": (640, 0, True, False, b"\1\0", DESC, C.c_void_p(0x1000), C.byref(DESC), 1.5, "text"),
                 "desc": (None, 0x1000, True, b"\1\0", X, torch.zeros(4), C.c_void_p(0x1000), C.c_int(3), "text")}
        for bad in wrong.get(kind, ()):
            with pytest.raises(AttributeError if kind == "x" else TypeError):
                call(*args[:i], bad, *args[i + 1:])
    for bad in (1.5, b"ab", "text", X, DESC) if "layout" in kinds else ():
        with pytest.raises(TypeError):
            call(type("Other", (), {"handle": bad}), *args[1:])
    assert not streams
    if "layout" in kinds:                                    # (these arguments as they are reach the library)
        with pytest.raises(vxl.VxlError):
            call(*args)
        assert streams == [0]


@pytest.mark.parametrize("name,form,workspace,sized", CALLS)
def test_sizes_come_from_these_tensors(name, form, workspace, sized):
    class Asked(Like):
        def __init__(self):
            super().__init__((2, 4, 8, 128), 0x1008)       # (misaligned: the calls without a layout end here)
            self.asked = set()

        def __getattribute__(self, what):
            if what in ("shape", "numel"):
                self.asked.add(what)
            return object.__getattribute__(self, what)

    args = [Closed if x == "layout" else DESC if x == "desc" else Asked() if x == "x" else int(x) for x in form.split()]
    for x in args:
        if isinstance(x, Asked):
            x.asked.clear()
    with pytest.raises(vxl.VxlError) as e:
        getattr(vxl, name)(*args)
    assert e.value.status == vxl.VXL_ERR_INVALID_ARG
    asked = {i: x.asked for i, x in enumerate(args) if isinstance(x, Asked)}
    assert {i for i, a in asked.items() if "numel" in a} == ({workspace} if workspace else set())
    assert {i for i, a in asked.items() if "shape" in a} - {workspace} == set(sized)


def test_numbers_are_numbers():
    n = vxl.native()
    for bad in (None, 1.5, X, b"\1\0", DESC):
        for at in (4, 6):                                    # top_k, kbar_ready
            args = [None, DESC, X, X, 1, X, 0, X, X, X, X, None]
            args[at] = bad
            with pytest.raises(TypeError, match="a number expected"):
                n.chunk_score_topk(*args)


def test_calls_end_in_the_library_that_was_loaded(streams):
    """The binding calls the functions it was given, those of lib(), and none that the dynamic linker finds by the name of
    the library: another copy of it in the process stays apart."""
    n, got = vxl.native(), []
    form = C.CFUNCTYPE(C.c_int, *[C.c_void_p] * 2, *[C.c_int32] * 2, *[C.c_void_p] * 2, C.c_int32, *[C.c_void_p] * 4,
                       C.c_size_t, C.c_void_p)
    other = form(lambda *a: got.append(a) or vxl.VXL_ERR_UNSUPPORTED)
    own = [C.cast(getattr(vxl.lib(), "vxl_" + x), C.c_void_p).value for x in vxl._PATH]
    given = list(own)
    given[vxl._PATH.index("bilevel_decode")] = C.cast(other, C.c_void_p).value
    try:
        n.setup(vxl.AttnDesc, C.c_void_p, vxl._stream, *given)
        assert status(lse=Like((2, 3, 28), 0x2000), ws=Like((77,), 0x3000)) == vxl.VXL_ERR_UNSUPPORTED
    finally:
        n.setup(vxl.AttnDesc, C.c_void_p, vxl._stream, *own)
    assert got == [(C.addressof(DESC), 0x1000, 2, 3, 0x1000, 0x1000, 640, 0x1000, 0x1000, 0x2000, 0x3000, 77, None)]
    assert status() == vxl.VXL_ERR_WORKSPACE
    for bad in (own[:-1], own[:-1] + [0], own[:-1] + [None]):
        with pytest.raises(TypeError):
            n.setup(vxl.AttnDesc, C.c_void_p, vxl._stream, *bad)


def test_the_library_is_built_where_the_binding_cannot_be(monkeypatch, tmp_path):
    """By the compiler that builds the library; where that fails (no Python headers), the C library is there all the same, and
    the build says what is missing."""
    from paper_2506_19225_amd import build
    ran = []

    def run(cmd, **kw):
        ran.append(cmd)
        bad = any("vxl_torch" in x for x in cmd)
        return type("Done", (), {"returncode": int(bad), "stderr": "Python.h: No such file" if bad else "", "stdout": ""})

    monkeypatch.setattr(build, "OBJ", str(tmp_path))
    monkeypatch.setattr(build, "_compile", lambda src: src)
    monkeypatch.setattr(build.subprocess, "run", run)
    with pytest.raises(RuntimeError, match="(?s)vxl_torch.cpp.*Python.h"):
        build.build_lib()
    assert any(cmd[cmd.index("-o") + 1] == build.LIB for cmd in ran)
    assert {cmd[0] for cmd in ran} == {build._hipcc()}


def test_a_binding_of_another_torch_or_python_says_so(monkeypatch, tmp_path):
    from paper_2506_19225_amd import build
    import sysconfig
    assert vxl.BINDING_PATH == build.BINDING and vxl.BINDING_PATH.endswith(sysconfig.get_config_var("EXT_SUFFIX"))
    vxl.native()
    monkeypatch.setattr(vxl, "_native", None)
    with monkeypatch.context() as m:
        m.setattr(torch, "__version__", "0.0.1+other")
        with pytest.raises(RuntimeError, match="built for torch .*0.0.1.other.*build"):
            vxl.native()
    broken = tmp_path / "broken.so"
    broken.write_text("no library")
    for path in (broken, tmp_path / "missing.so"):
        monkeypatch.setattr(vxl, "BINDING_PATH", str(path))
        with pytest.raises(RuntimeError, match="paper_2506_19225_amd.build"):
            vxl.native()


def test_two_modules_in_a_process_stay_apart(streams):
    """Each with its own types, library and stream function, in either order of their first calls."""
    import importlib.util
    spec = importlib.util.spec_from_file_location("vxl_again", vxl.__file__)
    again = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(again)
    again._stream = lambda stream: 0
    desc = again.make_desc(28, 4, 128, "bf16")
    for _ in range(2):
        assert status() == vxl.VXL_ERR_WORKSPACE
        with pytest.raises(again.VxlError) as e:
            again.bilevel_decode(desc, Q, KV, KV, LEN, Q)
        assert e.value.status == vxl.VXL_ERR_WORKSPACE
    assert len(streams) == 2
    with pytest.raises(TypeError, match="a descriptor expected"):
        again.bilevel_decode(DESC, Q, KV, KV, LEN, Q)
