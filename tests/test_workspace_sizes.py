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


@pytest.mark.gpu
@pytest.mark.parametrize("n", [96, 1023, 1024, 2048, 3071, 3072, 6144, 19840, 32768])
def test_plans_of_one_length_share_a_workspace(n):
    """(the query asks for the device's LDS) Fewer rows never need more; whatever t_end, as long as a list of all placed
    blocks fits LDS (from 9096 requests on tables by allocation time are part of the workspace)."""
    import torch
    import paper_2507_16274_amd as S
    torch.cuda.init()

    def need(t_end, P, offsets, sized):
        size = ctypes.c_size_t(0)
        tr = _trace(S, n, t_end)
        args = (ctypes.byref(tr), 256, P, 256 if offsets else None, 256, 256, 256, 256)
        if sized:
            assert S.lib.stalloc_plan_sized(*args, 1 << 20, 1 << 16, None, ctypes.byref(size), None) == 0
        else:
            assert S.lib.stalloc_plan(*args, None, ctypes.byref(size), None) == 0
        return size.value

    times = (1, n // 2 + 1, 2 * n, 4 * n + 4096, 4 * n + 4097, 1 << 20)
    for offsets in (True, False):
        for sized in (True, False):
            by_rows = [[need(t_end, P, offsets, sized) for t_end in times] for P in (1, 64, 512, 513, 4096)]
            for fewer, more in zip(by_rows, by_rows[1:]):
                assert all(a <= b for a, b in zip(fewer, more)), by_rows
            if n <= S.lib.stalloc_plan_lds_capacity():
                assert all(len(set(sizes)) == 1 for sizes in by_rows), by_rows


@pytest.mark.gpu
@pytest.mark.parametrize("n", [7300, 7404, 8200, 9095])
def test_no_tables_by_allocation_time_up_to_their_length(n):
    """Calls of up to 9095 requests carry none of the long-list kernel's tables, also where no list fits LDS: one workspace
    does for every t_end."""
    import torch
    import paper_2507_16274_amd as S
    torch.cuda.init()
    for P in (1, 512, 4096):
        sizes = set()
        for t_end in (1, 2 * n, 4 * n + 4096, 4 * n + 4097, 1 << 20):
            need = ctypes.c_size_t(0)
            assert S.lib.stalloc_plan(ctypes.byref(_trace(S, n, t_end)), 256, P, 256, 256, 256, 256, 256, None,
                                      ctypes.byref(need), None) == 0
            sizes.add(need.value)
        assert len(sizes) == 1, (P, sizes)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [10_500, 49_920])
def test_lists_in_the_workspace_are_as_many_as_workgroups_run(n):
    """One workgroup per CU places plans with its list in the workspace, two lists of 24-byte entries each."""
    import torch
    import paper_2507_16274_amd as S
    cus = torch.cuda.get_device_properties(0).multi_processor_count

    def need(P):
        size = ctypes.c_size_t(0)
        assert S.lib.stalloc_plan_sized(ctypes.byref(_trace(S, n, 2 * n)), 256, P, 256, 256, None, 256, 256, 1 << 20, 1, None,
                                        ctypes.byref(size), None) == 0
        return size.value

    assert need(cus) - need(1) >= (cus - 1) * 2 * 24 * n
    assert need(4096) - need(cus) <= 4 * 4096 + 256                   # a mark per plan


@pytest.mark.gpu
@pytest.mark.parametrize("n", [4300, 5000, 5600, 8200, 9095])
def test_lists_in_the_workspace_lie_where_the_index_of_the_bitmap_kernels_may(n):
    """A trace is placed by the one or the other, so a call needs room for the larger of the two."""
    import torch
    import paper_2507_16274_amd as S
    torch.cuda.init()

    def need(P, largest_size):
        size = ctypes.c_size_t(0)
        assert S.lib.stalloc_plan_sized(ctypes.byref(_trace(S, n, 2 * n)), 256, P, 256, 256, None, 256, 256, largest_size, 1, None,
                                        ctypes.byref(size), None) == 0
        return size.value

    index, lists = need(1, 8), need(4096, 1 << 20)                  # with sizes for the bitmap kernels, and without
    assert need(4096, 8) <= max(index, lists) + 4 * 4096 + 24 * n + (1 << 15)        # (marks, and words per request and timestamp)


@pytest.mark.gpu
def test_very_many_windows_need_no_room_for_intervals():
    """What a window adds to the workspace of the dynamic reusable space is its place in the sorted sequence (twice), and for every part of
    the plan (one, with this many windows) what is covered and found there."""
    import torch
    import paper_2507_16274_amd as S
    torch.cuda.init()

    def need(k):
        size = ctypes.c_size_t(0)
        assert S.lib.stalloc_reusable_space(ctypes.byref(_trace(S, 6144, 12288)), 256, 256, k, 0, None, 256, 256, 256, None,
                                            ctypes.byref(size), None) == 0
        return size.value

    windows = 1 << 24
    assert need(2 * windows) - need(windows) <= windows * (2 * 16 + 8 + 8 + 8 + 4 + 4) + 4096
    assert need(4096) - need(1) <= (128 << 20) + 4096 * 256 * 20 + (1 << 20)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [96, 512, 513])
def test_short_calls_carry_no_index(n):
    """Up to 4096 plans of up to 512 requests are placed in registers: no index of requests with overlapping lifetimes is part of those
    calls; it is from 4097 plans on, so that the size jumps there and never falls."""
    import torch
    import paper_2507_16274_amd as S
    torch.cuda.init()

    def need(P):
        size = ctypes.c_size_t(0)
        assert S.lib.stalloc_plan(ctypes.byref(_trace(S, n, 2 * n)), 256, P, 256, 256, 256, 256, 256, None, ctypes.byref(size), None) == 0
        return size.value

    index = n * n                                                 # (256 entries of two bytes for each request at least)
    assert need(1) <= need(64) <= need(4096) <= need(4097)
    assert (need(4097) - need(4096) >= index) == (n <= 512)
