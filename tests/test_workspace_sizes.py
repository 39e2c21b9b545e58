"""Workspaces that callers sized once stay large enough: the sizes the solves
report are pinned, and so are the smallest ones the adjoint takes."""
import ctypes

import pytest

from paper_1502_07303_amd import fmm


def shapes(n):
    return [(1 + (7 * i) % 33, 1 + (11 * i) % 29, 1 + (5 * i) % 41) for i in range(n)]


@pytest.mark.parametrize("n,edge,dtype,want", [(1, 8, 0, 14848), (2, 4, 0, 22016), (7, 8, 1, 732672), (10, 16, 0, 1948672),
                                               (64, 8, 0, 8546304), (300, 8, 1, 54650112)])
def test_batch_workspace(n, edge, dtype, want):
    lib = fmm.load_library()
    buf = ctypes.create_string_buffer(64)
    arr = (fmm.FmmProblem * n)()
    for q, s in zip(arr, shapes(n)):
        q.n0, q.n1, q.n2 = s
        q.h = 1.0
        q.F = q.T_out = ctypes.addressof(buf)
    o = fmm.make_opts(tile_edge=edge)
    assert lib.fmm_batch_workspace_bytes(n, arr, dtype, ctypes.byref(o)) == want


@pytest.mark.parametrize("n,want", [(1, 2048), (2, 18688), (7, 604928), (64, 9490176), (300, 49014272)])
def test_smallest_adjoint_workspace(n, want):
    lib = fmm.load_library()
    arr = (fmm.FmmAdjointProblem * n)()
    for q, s in zip(arr, shapes(n)):
        q.n0, q.n1, q.n2 = s
        q.h = 1.0
    assert lib.fmm_adjoint_workspace_bytes_min(n, arr) == want
    assert lib.fmm_adjoint_workspace_bytes(n, arr) >= want
    assert lib.fmm_adjoint_workspace_bytes_min(0, arr) == lib.fmm_adjoint_workspace_bytes(0, arr) == 0
    arr[n - 1].n1 = 0
    assert lib.fmm_adjoint_workspace_bytes_min(n, arr) == lib.fmm_adjoint_workspace_bytes(n, arr) == 0
