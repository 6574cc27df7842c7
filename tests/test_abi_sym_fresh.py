"""o2m_sym_fresh reports the argument errors of the call its op names, before
any GPU work (no compute call is made)."""
import ctypes

import pytest

import paper_2609_05419_amd as o2m

P = ctypes.c_void_p(0x1000)


def call(op=b"h", uplo=b"L", n=4, k=4, A=P, lda=4, B=P, ldb=4, C=P, ldc=4, N=16, rule=0):
    return o2m._L.o2m_sym_fresh(op, uplo, n, k, A, lda, B, ldb, C, ldc, N, rule, None)


@pytest.mark.parametrize("op", [b"h", b"s", b"x", b"y"])
def test_errors(op):
    two = op in (b"x", b"y")
    assert call(op, uplo=b"Q") == -1
    assert call(op, n=-1) == -2
    assert call(op, k=-1) == -3
    assert call(op, A=None) == -4
    assert call(op, lda=3) == -5
    assert call(op, C=None) == (-8 if two else -6)
    assert call(op, ldc=3) == (-9 if two else -7)
    assert call(op, N=0) == call(op, N=23) == -20
    assert call(op, k=149131) == -21
    assert call(op, rule=2) == -26
    assert call(op, n=0) == 0
    if two:
        assert call(op, B=None) == -6 and call(op, ldb=3) == -7


@pytest.mark.parametrize("op", [b"z", b"c", b"g", b"r", b"?"])
def test_other_ops_are_refused(op):
    assert call(op) == -1
