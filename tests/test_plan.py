"""Planning (host only) of feeders whose segments nearly all conflict."""
import ctypes
import time

import numpy as np
import pytest


def star(m):
    """m leaves at the slack, a segment each: one common head."""
    return [-1] + [0] * m


def path(m):
    """A path of m nodes, a segment each: every region holds the ones below."""
    return [-1] + list(range(m))


@pytest.mark.parametrize("parent", [star(20000), path(6000)], ids=["star", "path"])
def test_plan_of_many_conflicting_segments(parent):
    """The conflicts are ordered without listing every pair of them (200 and 18
    million here, several seconds and up to 1 GB when they were listed): well
    below a second of processor time.  The path's tops, found by climbing, take
    the most of it, 18 million steps."""
    import paper_2510_19608_amd as okr
    B = okr.binding
    n = len(parent)
    a = dict(parent=np.array(parent, np.int32), phase=np.full(n, 7, np.uint8),
             eligible=np.r_[0, np.ones(n - 1)].astype(np.uint8), segment=np.arange(-1, n - 1, dtype=np.int32))
    T = B.Topology(n, *(a[k].ctypes.data for k in ("parent", "phase", "eligible", "segment")))
    h = okr.okr_create(None)
    try:
        mg, ws, sz = B.make_margins({}), ctypes.c_size_t(), B.Sizes()
        t0 = time.process_time()
        rc = okr.lib().okr_plan(h, ctypes.byref(T), ctypes.byref(mg), 2, ctypes.byref(ws), ctypes.byref(sz))
        took = time.process_time() - t0
        assert rc == okr.OKR.OK and sz.n_segments == n - 1
        print(f"planned {n} nodes in {took:.3f} s")
        assert took < 1.0
    finally:
        okr.okr_destroy(h)
