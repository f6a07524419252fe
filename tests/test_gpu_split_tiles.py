"""GPU: the generally strided product where its tile depends on the split of K:
shapes on both sides of the rule (32 x 32 and 64 x 64 tiles, with and without
scratch for the split), ragged tiles and K ranges, batches.  Called through the
library's C++ symbol with a structure laid out as in internal.h; against a
float64 matmul, error at most K x 2^-53 x 4 times the largest |A| |B| product."""

import ctypes as C

import pytest
import torch

from paper_2607_00981_amd import binding

pytestmark = pytest.mark.gpu
L = C.c_longlong


class Idx2(C.Structure):
    _fields_ = [("inner", C.c_int), ("s_hi", L), ("s_lo", L)]


class GemmArgs(C.Structure):
    _fields_ = [(x, C.c_int) for x in ("M", "N", "K", "batch")] + [
        ("A", C.c_void_p), ("am", Idx2), ("ak", Idx2), ("a_batch", L), ("B", C.c_void_p), ("bk", Idx2), ("bn", Idx2),
        ("b_batch", L), ("C", C.c_void_p), ("cm", Idx2), ("cn", Idx2), ("c_batch", L), ("alpha", C.c_double),
        ("beta", C.c_double), ("a_len", L), ("b_len", L), ("c_len", L), ("split_ws", C.c_void_p), ("split_cap", L)]


def _stride(s):
    return Idx2(0, 0, s)


@pytest.mark.parametrize("m,n,k,batch,split", [
    (61, 61, 4097, 1, True), (100, 100, 4096, 1, True), (100, 100, 16385, 1, True), (128, 96, 8192, 1, True),
    (180, 180, 4100, 1, True), (240, 240, 1024, 1, True), (400, 400, 512, 1, True), (33, 20, 700, 5, True),
    (70, 70, 2000, 3, True), (180, 180, 4100, 1, False), (15, 17, 127, 2, True),
])
def test_strided_product(m, n, k, batch, split):
    print(f"[split tiles] {m} x {n} x {k}, batch {batch}, split {split}", flush=True)
    binding.load()
    gemm = C.CDLL(binding.LIB_PATH)["_ZN3cct4gemmERKNS_8GemmArgsENS_4PrecEP12ihipStream_t"]
    gemm.argtypes = [C.POINTER(GemmArgs), C.c_int, C.c_void_p]
    gen = torch.Generator(device="cuda").manual_seed(m + n + k)
    a = torch.randn((batch, m, k), device="cuda", dtype=torch.float64, generator=gen)
    b = torch.randn((batch, k, n), device="cuda", dtype=torch.float64, generator=gen)
    c = torch.randn((batch, m, n), device="cuda", dtype=torch.float64, generator=gen)
    want = -0.5 * torch.stack([x @ y for x, y in zip(a, b)]) + c
    ws = torch.empty(64 * batch * m * n, device="cuda", dtype=torch.float64)
    g = GemmArgs(M=m, N=n, K=k, batch=batch, A=a.data_ptr(), am=_stride(k), ak=_stride(1), a_batch=m * k,
                 B=b.data_ptr(), bk=_stride(n), bn=_stride(1), b_batch=k * n, C=c.data_ptr(), cm=_stride(n),
                 cn=_stride(1), c_batch=m * n, alpha=-0.5, beta=1.0, a_len=a.numel(), b_len=b.numel(),
                 c_len=c.numel(), split_ws=ws.data_ptr() if split else None, split_cap=ws.numel())
    torch.cuda.synchronize()
    assert gemm(C.byref(g), 0, torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    assert float((c - want).abs().max()) <= 4 * k * 2.0 ** -53 * float(a.abs().max() * b.abs().max())
