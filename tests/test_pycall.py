"""The native marshalling hands every argument to the right place.

A stand-in library that exports the entry points of moe.h and records what it
is called with takes the place of libmoe.so behind the binding: every wrapper is
called by keyword with a value of its own for each name, and each C parameter
must arrive with the value of its name in moe.h's prototypes.  Nothing is
launched, so this runs without a GPU."""
import ctypes
import inspect
import os
import re
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")

from paper_2607_26444_amd import build, moe  # noqa: E402

NAMES = ("moe_layout", "moe_layout_fixed", "moe_dispatch", "moe_combine", "moe_layout_dedup",
         "moe_dispatch_dedup", "moe_expand", "moe_combine_local", "moe_combine_dedup")


def prototypes():
    """C parameters (type, name) of each entry point, from the header."""
    text = re.sub(r"/\*.*?\*/", "", open(os.path.join(build.INCLUDE, "moe.h")).read(), flags=re.S)
    out = {}
    for name in NAMES:
        args = re.search(rf"\bint {name}\(([^)]*)\);", text).group(1)
        out[name] = [re.match(r"(.*?)(\w+)$", " ".join(a.split())).groups()
                     for a in args.split(",")]
    return out


PROTO = prototypes()


class Buf:
    """Stands in for a device tensor; its address is never followed."""
    is_cuda = True

    def __init__(self, addr, shape=None):
        self.addr, self.shape = addr, shape

    def data_ptr(self):
        return self.addr

    def numel(self):
        return self.addr // 16 + 3

    def element_size(self):
        return 4


class Stream:
    cuda_stream = 0x7F00DEADB000


# a value of its own for every integer name; T past 32 bits
INTEGERS = dict(dtype=1, H=7176, E=257, R=63, capacity=4099, scale_pitch=260)
T, K = (1 << 33) + 5, 31


def arguments(name):
    """{parameter of the wrapper: value}, tensors at distinct addresses."""
    args = {}
    for i, p in enumerate(inspect.signature(getattr(moe, name)).parameters):
        if p in INTEGERS:
            args[p] = INTEGERS[p]
        elif p == "stream":
            args[p] = Stream()
        else:
            args[p] = Buf(0x7F0000000000 + 0x1000 * (i + 1), (T, K) if p == "topk_idx" else None)
    return args


def expected(name, args):
    """What each C parameter must be, by its name in the header."""
    out = []
    for ctype, p in PROTO[name]:
        if p == "T":
            out.append(T)
        elif p == "k":
            out.append(K)
        elif p == "workspace_bytes":
            w = args["workspace"]
            out.append(w.numel() * w.element_size())
        elif p == "stream":
            out.append(args[p].cuda_stream)
        else:
            v = args[p]
            assert ("*" in ctype) == (v is None or isinstance(v, Buf)), (name, p)
            out.append(0 if v is None else v.addr if isinstance(v, Buf) else v)
    return out


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    """The recording library, bound behind the wrappers for this module."""
    d = tmp_path_factory.mktemp("stub")
    src, so = os.path.join(d, "stub.cpp"), os.path.join(d, "libstub.so")
    with open(src, "w") as f:
        f.write('#include "moe.h"\nextern "C" { unsigned long long rec[32]; int n_rec, code; }\n')
        for name, params in PROTO.items():
            f.write(f'extern "C" int {name}({", ".join(t + p for t, p in params)}) {{\n  n_rec = 0;\n')
            f.write("".join(f"  rec[n_rec++] = (unsigned long long){p};\n" for _, p in params))
            f.write("  return code;\n}\n")
    subprocess.run(["g++", "-shared", "-fPIC", "-I", build.INCLUDE, src, "-o", so], check=True)
    lib = ctypes.CDLL(so)
    calls = moe._calls()
    seen = []

    def get_stream(device):
        seen.append(device)
        return Stream.cuda_stream + 0x40
    calls.init(so, ctypes.ArgumentError, ctypes.c_int, lambda: 3, get_stream)

    class Stub:
        code = ctypes.c_int.in_dll(lib, "code")
        streams = seen

        @staticmethod
        def recorded():
            n = ctypes.c_int.in_dll(lib, "n_rec").value
            return list((ctypes.c_ulonglong * 32).in_dll(lib, "rec"))[:n]

    yield Stub
    calls.init(moe.LIB_PATH, ctypes.ArgumentError, ctypes.c_int, torch._C._cuda_getDevice,
               torch._C._cuda_getCurrentRawStream)


@pytest.mark.parametrize("name", NAMES)
def test_every_argument_arrives(stub, name):
    args = arguments(name)
    getattr(moe, name)(**args)
    assert stub.recorded() == expected(name, args)


@pytest.mark.parametrize("name", NAMES)
def test_none_is_null_for_every_pointer(stub, name):
    for p, v in arguments(name).items():
        if not isinstance(v, Buf) or p in ("topk_idx", "workspace"):
            continue   # these two have a size, and so are not optional
        args = arguments(name)
        args[p] = None
        getattr(moe, name)(**args)
        assert stub.recorded() == expected(name, args), p


@pytest.mark.parametrize("name", NAMES)
def test_no_stream_is_the_current_one(stub, name):
    args = arguments(name)
    del args["stream"]
    stub.streams.clear()
    getattr(moe, name)(**args)
    at = [p for _, p in PROTO[name]].index("stream")
    assert stub.recorded()[at] == Stream.cuda_stream + 0x40 and stub.streams == [3]


@pytest.mark.parametrize("name", NAMES)
def test_return_code_becomes_the_error(stub, name):
    stub.code.value = moe.MOE_EALIGN
    try:
        with pytest.raises(moe.MoeError, match=name) as e:
            getattr(moe, name)(**arguments(name))
    finally:
        stub.code.value = 0
    assert e.value.code == moe.MOE_EALIGN


def test_scale_pitch_defaults_to_packed(stub):
    for name in ("moe_dispatch", "moe_dispatch_dedup", "moe_expand"):
        args = arguments(name)
        del args["scale_pitch"]
        getattr(moe, name)(**args)
        assert stub.recorded() == expected(name, dict(args, scale_pitch=0)), name


def test_integers_as_ctypes_takes_them(stub):
    for given, got in ((ctypes.c_int(40), 40), (True, 1), (torch.tensor(9), 9), (-1, 2 ** 64 - 1),
                       (1 << 40, 0)):
        args = dict(arguments("moe_combine"), H=given)
        moe.moe_combine(**args)
        at = [p for _, p in PROTO["moe_combine"]].index("H")
        assert stub.recorded()[at] == got, given


def test_wrong_python_arguments(stub):
    def call(**change):
        moe.moe_combine(**dict(arguments("moe_combine"), **change))
    with pytest.raises(ctypes.ArgumentError):
        call(H=1.5)
    with pytest.raises(ctypes.ArgumentError):
        call(E=None)

    class Value:
        value = 5
    for other in (ctypes.c_long(3), ctypes.c_bool(True), Value()):   # not a c_int
        with pytest.raises(ctypes.ArgumentError):
            call(R=other)
    with pytest.raises(ValueError, match="device tensors"):
        call(y=torch.zeros(1))
    with pytest.raises(ValueError):
        call(topk_idx=Buf(64, (4,)))
    with pytest.raises(AttributeError):
        call(workspace=None)
    with pytest.raises(AttributeError):
        call(topk_idx=None)
    with pytest.raises(TypeError):
        moe._calls().combine(1, 2)


def test_other_interpreters_extension_is_not_taken(tmp_path):
    """The extension's name carries the interpreter's ABI tag: one built for
    another interpreter is not loaded, and the error says what to build."""
    assert os.path.exists(build.PYCALL) and ".cpython-" in os.path.basename(build.PYCALL)
    assert not os.path.exists(os.path.join(build.HERE, "_moecall.so"))
    pkg = tmp_path / "paper_2607_26444_amd"
    pkg.mkdir()
    for f in ("__init__.py", "moe.py", "libmoe.so"):
        os.symlink(os.path.join(build.HERE, f), pkg / f)
    os.symlink(build.PYCALL, pkg / "_moecall.cpython-399-x86_64-linux-gnu.so")
    run = subprocess.run([sys.executable, "-c", "from paper_2607_26444_amd import moe; moe._calls()"],
                         cwd=tmp_path, capture_output=True, text=True,
                         env=dict(os.environ, PYTHONPATH=str(tmp_path)))
    assert run.returncode != 0
    assert "RuntimeError: no _moecall for this interpreter" in run.stderr
