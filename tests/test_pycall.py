"""The native marshalling hands every argument to the right place: for calls
that the library refuses before any launch, it returns the code that the same
call through ctypes returns, whichever argument is the wrong one."""
import ctypes

import pytest

torch = pytest.importorskip("torch")

from paper_2607_26444_amd import moe  # noqa: E402


class Buf:
    """Stands in for a device tensor; its address is never followed."""
    is_cuda = True

    def __init__(self, addr=1 << 20, nbytes=1 << 30, shape=None):
        self.addr, self.nbytes, self.shape = addr, nbytes, shape

    def data_ptr(self):
        return self.addr

    def numel(self):
        return self.nbytes

    def element_size(self):
        return 1


class Stream:
    cuda_stream = 0


IDX = Buf(shape=(0, 2))     # T = 0: nothing is launched by the copy calls
E, R, H = 16, 4, 256
BAD = {"null": None, "odd": Buf((1 << 20) + 4), "small": Buf(nbytes=64), "float": 1.5,
       "big": 1 << 40, "minus": -1, "zero": 0, "three": 3,
       "T": Buf(shape=(5, 2)), "k": Buf(shape=(5, 99))}

# name, arguments in order (tensors b, integers, the index table, workspace w)
b, w, s = Buf(), Buf(), Stream()
CALLS = {
    "moe_layout": [IDX, E, R, b, b, b, b, b, b, w, b, s],
    "moe_layout_fixed": [IDX, E, R, 4, b, b, b, b, b, b, w, b, s],
    "moe_dispatch": [b, None, 0, H, E, R, IDX, b, b, b, None, b, w, b, s, 0],
    "moe_combine": [b, b, H, E, R, IDX, b, b, b, b, w, b, s],
    "moe_layout_dedup": [IDX, E, R, b, b, b, b, w, b, s],
    "moe_dispatch_dedup": [b, b, 1, H, E, R, IDX, b, b, b, b, b, w, b, s, 0],
    "moe_expand": [b, None, 0, H, E, R, IDX, b, b, b, b, b, b, None, b, w, b, s, 0],
    "moe_combine_local": [b, b, H, E, R, IDX, b, b, b, b, b, b, b, w, b, s],
    "moe_combine_dedup": [b, H, E, R, IDX, b, b, b, b, w, b, s],
}
# position of scale_pitch in the C call, which Python passes last
PITCH = {"moe_dispatch": 13, "moe_dispatch_dedup": 13, "moe_expand": 16}


def through_ctypes(name, args):
    """The C argument list by its documented order: pointers for tensors, T
    (and H where the call has one) and k around the table, the workspace's
    bytes after it."""
    ptr = moe._ptr
    args = list(args)
    pitch = args.pop() if name in PITCH else None
    stream, status, work = args.pop(), args.pop(), args.pop()
    idx = next(a for a in args if isinstance(a, Buf) and a.shape)
    T, k = idx.shape
    out, at = [], args.index(idx)
    head, tail = args[:at], args[at + 1:]
    if name.startswith("moe_layout"):
        out = [ptr(idx), T, k] + [a if isinstance(a, (int, float)) else ptr(a) for a in tail]
    else:
        h, e, r = head[-3:]
        out = [a if isinstance(a, (int, float)) else ptr(a) for a in head[:-3]]
        out += [T, h, k, e, r, ptr(idx)]
        out += [a if isinstance(a, (int, float)) else ptr(a) for a in tail]
    if pitch is not None:
        out.insert(PITCH[name], pitch)
    out += [ptr(work), work.nbytes if work else 0, ptr(status), stream.cuda_stream]
    return getattr(moe.lib(), name)(*out)


def native(name, args):
    return getattr(moe._calls(), name[4:])(*args)


CASES = [(n, i, k) for n, a in CALLS.items() for i in range(len(a)) for k in BAD
         if a[i] is not s and not (a[i] is w and k == "null")   # a workspace has a size
         and ((k in ("null", "odd", "small") and isinstance(a[i], Buf) and a[i] is not IDX)
              or (k in ("T", "k") and a[i] is IDX)
              or (k in ("big", "minus", "zero", "three") and isinstance(a[i], int)))]


@pytest.mark.parametrize("name,at,kind", CASES)
def test_same_code_as_ctypes(name, at, kind):
    args = list(CALLS[name])
    args[at] = BAD[kind]
    if kind == "T":     # tokens: refuse the batch by its experts, launch nothing
        args[args.index(BAD["T"]) + 1 if name.startswith("moe_layout")
             else args.index(BAD["T"]) - 1] = 5
    elif name.startswith("moe_layout"):   # T = 0 still launches: refuse it by R
        args[2] = 5
    want = through_ctypes(name, args)
    assert native(name, args) == want
    if kind in ("T", "k") or name.startswith("moe_layout"):
        assert want == moe.MOE_EINVAL


def test_wrong_python_arguments():
    with pytest.raises(ctypes.ArgumentError):
        moe.moe_combine(b, b, 1.5, E, R, IDX, b, b, b, b, w, b, s)
    with pytest.raises(ValueError, match="device tensors"):
        moe.moe_combine(torch.zeros(1), b, H, E, R, IDX, b, b, b, b, w, b, s)
    with pytest.raises(ValueError):
        moe.moe_layout(Buf(shape=(4,)), E, R, b, b, b, b, b, b, w, b, s)
    with pytest.raises(AttributeError):
        moe.moe_combine(b, b, H, E, R, IDX, b, b, b, b, None, b, s)
    assert native("moe_combine", [b, b, ctypes.c_int(H), E, R, IDX, b, b, b, b, w, b, s]) == 0
