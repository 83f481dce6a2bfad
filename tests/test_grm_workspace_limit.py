"""The int8 path of the relationship matrix keeps a second operand; panels that
would not fit the card with it keep the fp64 kernel's workspace, the sample-major
operand and little more."""
import ctypes

import pytest

from paper_1410_4803_amd import _native as N

GIB = 1 << 30


def _bytes(n, V):
    g = N.Genotypes(0x1000, n, V, 0, None)
    b = ctypes.c_size_t(0)
    rc = N.load().pg_grm_workspace_bytes(ctypes.byref(g), 0, 0, 0, ctypes.byref(b))
    assert rc == 0
    return b.value


def _operand(n, V):
    return -(-n // 128) * 128 * (-(-V // 256) * 16) * 4


@pytest.mark.parametrize("n,V", [(100000, 3000000), (130000, 800000), (1000000, 150000),
                                 (40000, 4000000)])
def test_large_panels_take_one_operand(n, V):
    assert _operand(n, V) <= _bytes(n, V) < 1.02 * _operand(n, V) + 40 * V


@pytest.mark.parametrize("n,V", [(10000, 71307), (50000, 2000000)])
def test_others_take_two(n, V):
    assert _bytes(n, V) > 2 * _operand(n, V)
