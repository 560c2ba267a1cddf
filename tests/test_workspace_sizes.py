"""Workspace queries: a size may depend on what its entry point documents and on nothing else, and less work never
needs more, so that a program can keep one workspace for calls that differ in the rest."""
import ctypes

import pytest

U32 = ctypes.c_uint32


def _trace(S, n, t_end):
    some = 256                                                    # (a query looks at no memory)
    return S._Trace(n, t_end, some, some, some)


def _orders_need(S, n, first, P):
    need = ctypes.c_size_t(0)
    tr = _trace(S, n, 2 * n)
    assert S.lib.stalloc_make_orders(ctypes.byref(tr), first, P, 1000, None, None, None, ctypes.byref(need), None) == 0
    return need.value


@pytest.mark.parametrize("n", [1, 96, 2048, 2049, 6144, 199748, 6_291_457, 7_000_000])
def test_windows_of_orders_share_a_workspace(n):
    import paper_2507_16274_amd as S
    last = 0
    for P in (1, 2, 3, 4, 64, 4096):
        sizes = {_orders_need(S, n, first, P) for first in (0, 1, 2, 3, 4, 5, 256, 0xffffffff - P)}
        assert len(sizes) == 1, (P, sizes)
        assert sizes.pop() >= last
        last = _orders_need(S, n, 0, P)
