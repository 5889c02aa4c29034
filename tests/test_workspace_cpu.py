"""CPU checks of the workspace sizes: what runs on the library's own scratch."""
import ctypes as C
import os

import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2303_16492_amd", "libtrsgd.so")

pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="library not built")


def _run_size(I, R, prec, m, m_H=0, law="U", scaled=True):
    from paper_2303_16492_amd import _lib as L, api
    dt = torch.float64 if prec == "f64" else torch.float32
    p = L.tr_problem()
    p.desc = api.make_desc(I, R, dt, torch.float16 if prec == "f16" else dt)
    c = L.tr_config()
    c.m, c.m_H, c.scaled = m, m_H, int(scaled)
    c.law = {"U": L.TR_LAW_UNIFORM, "L": L.TR_LAW_LEVERAGE, "E": L.TR_LAW_EUCLID, "O": L.TR_LAW_OPTIMAL}[law]
    c.prec = {"f64": L.TR_PREC_F64, "f32": L.TR_PREC_F32, "bf16": L.TR_PREC_BF16, "f16": L.TR_PREC_F16}[prec]
    return L.lib().tr_run_workspace_size(C.byref(p), C.byref(c))


# Workspaces of 10 to 16.7 MB with one block of sample groups per CU (two in
# FP64, of 32 rows) and the law's workspace behind the step's: tr_run_noalloc has
# taken these, so they keep fitting its scratch whatever more groups would gain.
@pytest.mark.parametrize("I,R,prec,m,m_H,law", [
    ([864, 864, 864], [14, 14, 14], "f32", 1272, 0, "U"), ([941, 95, 90], [15, 9, 12], "f32", 3722, 0, "U"),
    ([75, 27, 36], [12, 12, 12], "f32", 12532, 0, "E"), ([819, 5, 4], [12, 12, 12], "f32", 3128, 0, "U"),
    ([77, 77, 77, 77, 77], [14, 3, 10, 14, 16], "f32", 6048, 9, "L"), ([1183, 1183], [9, 9], "f64", 1526, 3, "O"),
    ([468, 468], [4, 10], "f64", 28550, 0, "L"), ([126, 155, 1118], [10, 15, 1], "f64", 1085, 0, "L"),
    ([3, 488, 1214], [6, 16, 4], "f64", 5809, 0, "E"), ([3857, 1141], [14, 9], "f32", 774, 0, "L"),
    ([11, 3, 2, 2, 3, 4, 5, 6], [8, 12, 10, 16, 1, 7, 8, 5], "f32", 17386, 119, "U"),
    ([104, 104, 104, 104], [12, 6, 1, 6], "f32", 29074, 0, "E")])
def test_runs_that_fitted_the_library_scratch_still_do(I, R, prec, m, m_H, law):
    from paper_2303_16492_amd import _lib as L
    assert 0 < _run_size(I, R, prec, m, m_H, law) <= L.TR_NOALLOC_SCRATCH_BYTES


def test_larger_runs_keep_a_size_above_the_scratch():
    from paper_2303_16492_amd import _lib as L
    assert _run_size([400, 400, 400], [16, 16, 16], "f32", 60000) > L.TR_NOALLOC_SCRATCH_BYTES


def test_an_entry_workspace_serves_smaller_batches():
    """The workspace of a batch of B entries is enough for every smaller batch: no
    size falls as B grows, across the batch sizes where the split over workgroups
    changes."""
    from paper_2303_16492_amd import _lib as L, api
    sizes = sorted({max(1, e) for b in (64, 2048, 8192) for w in (1, 2, 4, 8, 16) for e in (b * w - 1, b * w, b * w + 1)}
                   | {1 << k for k in range(19)} | {3 << k for k in range(17)})
    for I, R in [([1, 1], [16, 12]), ([2, 145], [16, 6]), ([2049, 5, 6], [4, 8, 4]), ([40, 30, 5], [7, 9, 3]),
                 ([14456, 826, 580, 9, 2], [3, 2, 2, 7, 8]), ([16, 16, 16, 16], [11] * 4), ([6] * 8, [5] * 8),
                 ([32] * 5, [8] * 5)]:
        d = api.make_desc(I, R, torch.float32)
        c = L.tr_completion_config()
        last = last_c = 0
        for B in sizes:
            size = L.lib().tr_entry_workspace_size(C.byref(d), B)
            c.B = B
            size_c = L.lib().tr_completion_workspace_size(C.byref(d), C.byref(c))
            assert size >= last and size_c >= last_c, (I, R, B)
            assert size > 0 and size_c > 0
            last, last_c = size, size_c
