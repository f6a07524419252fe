"""CPU: the segmented product refuses on the host what would reach past its
output or break its 16-byte loads, before anything is launched.  Called through
the library's C++ symbol with a structure laid out as in internal.h."""

import ctypes as C

import pytest

from paper_2607_00981_amd import binding

INVALID = 1  # hipErrorInvalidValue


class Idx4(C.Structure):
    _fields_ = [("n", C.c_int * 3), ("s", C.c_longlong * 4)]


class SegGemm(C.Structure):
    _fields_ = [(x, C.c_int) for x in ("M", "N", "K", "kb", "n1", "n2", "nitems")] + [
        ("vec", C.c_bool), ("swap", C.c_bool), ("items", C.c_void_p), ("C", C.c_void_p), ("cm", Idx4), ("cn", Idx4),
        ("accumulate", C.c_int), ("c_last", C.c_longlong), ("c_len", C.c_longlong)]


def _call(**kw):
    """C(m, n) at m 12 + n of three items of 96 doubles (M = 8, N = 12, K = 6), with changes."""
    f = C.CDLL(binding.LIB_PATH)["_ZN3cct8seg_gemmERKNS_7SegGemmEP12ihipStream_t"]
    f.restype = C.c_int
    f.argtypes = [C.POINTER(SegGemm), C.c_void_p]
    one = (C.c_int * 3)(1, 1, 1)
    g = SegGemm(M=8, N=12, K=6, kb=5, n1=1, n2=1, nitems=3, vec=True, swap=False, items=4096, C=4096,
                cm=Idx4(one, (C.c_longlong * 4)(12, 0, 0, 0)), cn=Idx4(one, (C.c_longlong * 4)(1, 0, 0, 0)),
                accumulate=1, c_last=192, c_len=288)
    for k, x in kw.items():
        setattr(g, k, x)
    return f(C.byref(g), None)


@pytest.mark.parametrize("change", [
    {"c_len": 287}, {"c_last": 193}, {"c_last": -1}, {"M": 9}, {"N": 14}, {"K": 7}, {"N": 11, "c_len": 1 << 30},
    {"kb": 0}, {"kb": 7}, {"n2": 0}, {"items": None},
    {"cm": Idx4((C.c_int * 3)(1, 1, 0), (C.c_longlong * 4)(12, 0, 0, 0))},
    {"cn": Idx4((C.c_int * 3)(1, 1, 1), (C.c_longlong * 4)(-1, 0, 0, 0))},
])
def test_seg_gemm_refuses(change):
    assert _call(**change) == INVALID


def test_nothing_to_do_is_no_error():
    assert _call(nitems=0) == 0
