"""The weight-gradient launches refuse problems their kernels do not take before
any HIP call (host only): widths and strides that are not multiples of 8, no
tokens, operands of 2 GiB and more, gradients that are not dense, invalid counts."""
import ctypes as C

import pytest

import paper_2202_11836_amd as P

INVALID_VALUE = 1  # hipErrorInvalidValue


class GemmArgs(C.Structure):  # (the fields these checks read, and room for the others)
    _fields_ = ([(n, C.c_void_p) for n in ("A", "B", "C", "C2", "bias", "aux", "aux2", "dsum")]
                + [(n, C.c_int) for n in ("dsum_S", "M", "N", "K")]
                + [(n, C.c_int64) for n in ("lda", "ldb", "ldc", "ldaux")] + [("rest", C.c_char * 512)])


def problem(M, N, K, lda, ldb, ldc):
    return dict(M=M, N=N, K=K, lda=lda, ldb=ldb, ldc=ldc)


GOOD = problem(64, 192, 100, 64, 192, 192)


@pytest.mark.parametrize("p", [
    dict(GOOD, M=60, lda=64), dict(GOOD, N=188, ldc=188), dict(GOOD, lda=68), dict(GOOD, ldb=196),
    dict(GOOD, ldc=200), dict(GOOD, K=0), dict(GOOD, M=-64), dict(GOOD, K=1 << 24),
    dict(GOOD, K=1 << 24, lda=8)])
def test_refused(p):
    lib = P.load_library()
    args = GemmArgs(**p)
    out = (C.c_void_p * 4)()
    tail = (C.c_char * 4096)()
    for tile in (2, 3, 5):
        assert lib._Z14gemm_mid_wgradPK8GemmArgsPKPfiiRK8TailJobsP12ihipStream_t(
            C.byref(args), out, 1, tile, tail, None) == INVALID_VALUE
    if p["ldc"] == p["N"]:
        assert lib._Z21gemm_bf16_wgrad_groupPK8GemmArgsiP12ihipStream_t(
            C.byref(args), 1, None) == INVALID_VALUE


def test_refused_counts():
    lib = P.load_library()
    tail, out = (C.c_char * 4096)(), (C.c_void_p * 8)()
    args = (GemmArgs * 8)(*[GemmArgs(**GOOD)] * 8)
    call = lib._Z14gemm_mid_wgradPK8GemmArgsPKPfiiRK8TailJobsP12ihipStream_t
    assert all(call(args, out, n, 3, tail, None) == INVALID_VALUE for n in (-1, 0, 5))
    assert call(None, out, 1, 3, tail, None) == INVALID_VALUE
    assert call(args, None, 1, 3, tail, None) == INVALID_VALUE
