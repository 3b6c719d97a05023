"""The native marshalling hands the library what ctypes hands it, and leaves everything out of the ordinary to ctypes."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2502_12574_amd import binding as hb

NAMES = ("hi_prefill_group", "hi_decode_group", "hi_decode_group_ragged", "hi_qkv_rope", "hi_out_proj")


class _Stream:
    cuda_stream = 0x7F0000001230


@pytest.fixture
def seen(monkeypatch):
    """The five functions replaced by ones that note their arguments, behind ctypes and behind the native module."""
    L, calls, keep = hb.lib(), [], []

    class Fake:
        pass

    fake = Fake()
    for name in NAMES:
        real = getattr(L, name)
        ragged = name.endswith("ragged")

        def note(*a, _name=name, _ragged=ragged):
            a = list(a)
            if _ragged:
                a[7] = [a[7][j] for j in range(a[3])]
            calls.append((_name, a))
            return -5
        f = C.CFUNCTYPE(C.c_int32, *real.argtypes)(note)
        keep.append(f)
        setattr(fake, name, f)
    monkeypatch.setattr(hb, "_lib", fake)
    monkeypatch.setattr(hb, "_native", None)
    hb._load_native()
    yield calls
    monkeypatch.undo()
    hb._native = None
    hb._load_native()               # bound to the library again


class _Noting:
    """The native module, with what its functions returned."""

    def __init__(self, module):
        self.module, self.returned = module, []

    def __getattr__(self, name):
        def call(*args):
            self.returned.append(getattr(self.module, name)(*args))
            return self.returned[-1]
        return call


def _both(seen, monkeypatch, call, ordinary):
    """what the call hands over natively (or by itself, if it is out of the ordinary), and through ctypes"""
    noting = _Noting(hb._native)
    monkeypatch.setattr(hb, "_native", noting)
    assert call() == -5
    assert noting.returned == ([-5] if ordinary else [None])         # None: left to ctypes, nothing called
    native = seen.pop()
    monkeypatch.setattr(hb, "_native", hb._CtypesOnly)
    assert call() == -5
    through_ctypes = seen.pop()
    assert not seen
    return native, through_ctypes


T = torch.zeros(64, dtype=torch.bfloat16)
CTX = C.c_void_p(0x123456789ABC)


ORDINARY = [
    lambda: hb.hi_prefill_group(CTX, 1, 2, 3, T, T[8:], None, 1 << 33, 77, 0x7F00_0000_1000, 4, 5, 6, 7 << 32, check=False),
    lambda: hb.hi_prefill_group(CTX, 0, 0, 8, T, T, T, 0, 1, T, check=False),
    lambda: hb.hi_decode_group(CTX, 1, 2, 3, T, T[8:], T, 1 << 33, T, -1, 0, 1, 0, check=False),
    lambda: hb.hi_decode_group(None, -1, True, 3, 0, T, T, -7, T, check=False),
    lambda: hb.hi_decode_group_ragged(CTX, 0, 0, 3, T, T, T, [0, 5, 1 << 34], T, check=False),
    lambda: hb.hi_qkv_rope(_Stream(), T, T, 4096, 32, 8, 1, 1 << 20, 5e5, 0, T, T, T, T, q_scale=hb.HI_Q_PRESCALE, check=False),
    lambda: hb.hi_qkv_rope(0, T, T, 4096, 32, 8, 1, 3, 0.0, 1, T, T, T, None, check=False),
    lambda: hb.hi_out_proj(None, T, T, 32, 4096, 1, 0, T, check=False),
]
# other number types, a tuple of lengths, an int for the base, more than 32 bits
OUT_OF_THE_ORDINARY = [
    lambda: hb.hi_decode_group(CTX, np.int64(1), 2, 3, T, T, T, np.int32(9), T, check=False),
    lambda: hb.hi_decode_group(CTX, (1 << 32) + 1, 2, 3, T, T, T, 9, T, check=False),
    lambda: hb.hi_decode_group_ragged(CTX, 0, 0, 2, T, T, T, (4, np.int64(6)), T, check=False),
    lambda: hb.hi_qkv_rope(_Stream(), T, T, 4096, 32, 8, 1, 3, 10000, 0, T, T, T, T, check=False),
]


@pytest.mark.parametrize("call,ordinary", [(c, True) for c in ORDINARY] + [(c, False) for c in OUT_OF_THE_ORDINARY])
def test_same_arguments_as_through_ctypes(seen, monkeypatch, call, ordinary):
    native, through_ctypes = _both(seen, monkeypatch, call, ordinary)
    assert native == through_ctypes


@pytest.mark.parametrize("call,error", [
    (lambda: hb.hi_decode_group(CTX, 0, 0, 1, object(), T, T, 1, T), AttributeError),
    (lambda: hb.hi_out_proj(object(), T, T, 32, 4096, 1, 0, T), AttributeError),
    (lambda: hb.hi_decode_group(CTX, 0, 1.5, 1, T, T, T, 1, T), C.ArgumentError),
    (lambda: hb.hi_decode_group_ragged(CTX, 0, 0, 1, T, T, T, [1, 2], T), IndexError),
    (lambda: hb.hi_out_proj(None, T, T, 32, 4096, 1, 0, T), hb.HiError),
])
def test_same_errors(seen, monkeypatch, call, error):
    monkeypatch.setattr(hb, "status_string", lambda st: "status")
    monkeypatch.setattr(hb, "last_error", lambda: "")
    with pytest.raises(error):
        call()


def test_without_the_extension(seen, monkeypatch):
    """Not built for this interpreter, the native marshalling is done without: the same calls, through ctypes."""
    import sys

    import paper_2502_12574_amd as package
    from paper_2502_12574_amd import build
    monkeypatch.setitem(sys.modules, package.__name__ + "._pycall", None)
    monkeypatch.delattr(package, "_pycall", raising=False)
    monkeypatch.setattr(hb, "_native", None)
    for call, name in ((lambda: hb.hi_prefill_group(CTX, 0, 0, 8, T, T, T, 0, 1, T, check=False), NAMES[0]),
                       (lambda: hb.hi_decode_group(CTX, 0, 0, 1, T, T, T, 5, T, check=False), NAMES[1]),
                       (lambda: hb.hi_decode_group_ragged(CTX, 0, 0, 2, T, T, T, [4, 6], T, check=False), NAMES[2]),
                       (lambda: hb.hi_qkv_rope(None, T, T, 4096, 32, 8, 1, 3, 1e4, 0, T, T, T, T, check=False), NAMES[3]),
                       (lambda: hb.hi_out_proj(None, T, T, 32, 4096, 1, 0, T, check=False), NAMES[4])):
        assert call() == -5 and seen.pop()[0] == name
    # and the library is built without a host compiler
    monkeypatch.setattr(build, "PYCALL", "/nonexistent/_pycall.so")
    monkeypatch.setattr(build.shutil, "which", lambda name: None)
    assert build.build_pycall() is None
