"""GPU: K-contiguous products whose K is less than one K tile, each operand in an
allocation of its own that it fills to the end: load units past K are masked,
and what they load has to lie inside the operand as well.  Called through the
library's C++ symbols with structures laid out as in internal.h; against numpy.
FP64: 4 K x 2^-53 of the largest product.  FP32 and split BF16: the operands are
numbers of few bits, so that their products and sums are exact."""

import ctypes as C

import numpy as np
import pytest

from paper_2607_00981_amd import binding

pytestmark = pytest.mark.gpu
L = C.c_longlong


class Idx2(C.Structure):
    _fields_ = [("inner", C.c_int), ("s_hi", L), ("s_lo", L)]


class NtArgs(C.Structure):
    _fields_ = [(x, C.c_int) for x in ("M", "N", "K", "batch")] + [
        ("A", C.c_void_p), ("lda", L), ("a_batch", L), ("B", C.c_void_p), ("ldb", L), ("b_batch", L),
        ("C", C.c_void_p), ("cm", Idx2), ("cn", Idx2), ("c_batch", L), ("alpha", C.c_double), ("beta", C.c_double),
        ("a_len", L), ("b_len", L), ("c_len", L), ("variant", C.c_int), ("b_kn", C.c_int), ("b_map", C.c_int),
        ("bnm", Idx2)]


class NtLpArgs(C.Structure):
    _fields_ = [(x, C.c_int) for x in ("M", "N", "K", "batch")] + [
        ("A", C.c_void_p), ("lda", L), ("a_batch", L), ("a_plane", L), ("B", C.c_void_p), ("ldb", L), ("b_batch", L),
        ("b_plane", L), ("C", C.c_void_p), ("cm", Idx2), ("cn", Idx2), ("c_batch", L), ("alpha", C.c_double),
        ("beta", C.c_double), ("a_len", L), ("b_len", L), ("c_len", L), ("variant", C.c_int), ("C32", C.c_void_p),
        ("il", C.c_int)]


class Device:
    """Buffers of exactly the arrays' sizes, freed together."""

    def __init__(self):
        binding.load()
        with open("/proc/self/maps") as f:
            path = sorted({line.split()[-1] for line in f if "libamdhip64" in line})[0]
        self.hip, self.held = C.CDLL(path), []
        self.hip.hipMalloc.argtypes = [C.POINTER(C.c_void_p), C.c_size_t]
        self.hip.hipMemcpy.argtypes = [C.c_void_p, C.c_void_p, C.c_size_t, C.c_int]
        self.hip.hipFree.argtypes = [C.c_void_p]

    def put(self, x):
        p = C.c_void_p()
        assert self.hip.hipMalloc(C.byref(p), x.nbytes) == 0
        self.held.append(p)
        assert self.hip.hipMemcpy(p, x.ctypes.data, x.nbytes, 1) == 0
        return p.value

    def get(self, p, like):
        out = np.empty_like(like)
        assert self.hip.hipMemcpy(out.ctypes.data, p, out.nbytes, 2) == 0
        return out

    def __enter__(self):
        return self

    def __exit__(self, *exc):
        for p in self.held:
            self.hip.hipFree(p)


def _stride(s):
    return Idx2(0, 0, s)


def _symbol(name, args):
    f = C.CDLL(binding.LIB_PATH)[name]
    f.argtypes = [C.POINTER(args), C.c_int, C.c_void_p]
    return f


# operands of whole pages (4096 bytes), of less and of more
@pytest.mark.parametrize("m,n,k,batch", [(256, 128, 2, 1), (128, 128, 4, 2), (64, 64, 8, 1), (36, 36, 6, 3),
                                         (100, 10, 10, 1), (144, 12, 12, 4), (40, 196, 14, 2), (33, 62, 18, 1)])
@pytest.mark.parametrize("layout", ["nk", "kn", "mapped"])
def test_fp64(m, n, k, batch, layout):
    rng = np.random.default_rng(m + n + k)
    a, b = rng.normal(size=(batch, m, k)), rng.normal(size=(batch, n, k))
    want = np.matmul(a, b.transpose(0, 2, 1))
    if layout == "nk":
        stored = b
    elif layout == "kn":
        stored = np.ascontiguousarray(b.transpose(0, 2, 1))
    else:  # [n / 2][k][2]: row k of B holds pairs of columns, 2 K apart
        stored = np.ascontiguousarray(b.reshape(batch, n // 2, 2, k).transpose(0, 1, 3, 2))
    gemm = _symbol("_ZN3cct7gemm_ntERKNS_6NtArgsENS_4PrecEP12ihipStream_t", NtArgs)
    with Device() as dev:
        pa, pb, c = dev.put(a), dev.put(stored), np.zeros((batch, m, n))
        for variant in (0, 1, 2, 3, 4, 5, 6, 7):
            print(f"[short products] {m} x {n} x {k}, batch {batch}, {layout}, variant {variant}", flush=True)
            pc = dev.put(c)
            g = NtArgs(M=m, N=n, K=k, batch=batch, A=pa, lda=k, a_batch=m * k, B=pb,
                       ldb={"nk": k, "kn": n, "mapped": 2}[layout], b_batch=n * k, C=pc, cm=_stride(n), cn=_stride(1),
                       c_batch=m * n, alpha=1.0, beta=0.0, a_len=a.size, b_len=b.size, c_len=c.size, variant=variant,
                       b_kn=layout != "nk", b_map=layout == "mapped", bnm=Idx2(2, 2 * k, 1))
            assert gemm(C.byref(g), 0, None) == 0
            got = dev.get(pc, c)
            assert np.abs(got - want).max() <= 4 * k * 2.0 ** -53 * float(np.abs(a).max() * np.abs(b).max())


@pytest.mark.parametrize("prec,m,n,k", [(1, 256, 64, 4), (1, 128, 36, 8), (1, 33, 40, 28), (2, 256, 64, 8),
                                        (2, 64, 128, 16), (2, 35, 41, 24)])
def test_low_precision(prec, m, n, k):
    rng = np.random.default_rng(m + n + k)
    a, b = (rng.integers(-8, 9, size=(x, k)).astype(np.float64) for x in (m, n))
    want = a @ b.T

    def planes(x):  # split BF16: the numbers are exact in the high plane
        hi = (x.astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
        return np.stack([hi, np.zeros_like(hi)])

    gemm = _symbol("_ZN3cct10gemm_nt_lpERKNS_8NtLpArgsENS_4PrecEP12ihipStream_t", NtLpArgs)
    with Device() as dev:
        pa, pb = (dev.put(x.astype(np.float32) if prec == 1 else planes(x)) for x in (a, b))
        c = np.zeros((m, n))
        for variant in (0, 1, 2, 3, 4):
            print(f"[short products] {m} x {n} x {k}, precision {prec}, variant {variant}", flush=True)
            pc = dev.put(c)
            g = NtLpArgs(M=m, N=n, K=k, batch=1, A=pa, lda=k, a_plane=m * k, B=pb, ldb=k, b_plane=n * k, C=pc,
                         cm=_stride(n), cn=_stride(1), alpha=1.0, beta=0.0, a_len=m * k, b_len=n * k, c_len=m * n,
                         variant=variant)
            assert gemm(C.byref(g), prec, None) == 0
            assert np.array_equal(dev.get(pc, c), want)
