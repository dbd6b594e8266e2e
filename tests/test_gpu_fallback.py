"""The per-XCD barrier's counter-tree fallback on the GPU: a kernel of the test's own runs it
with fewer groups than XCDs or with arrival blocks too small for the members, so that some
registration does not fit and every round takes the tree."""

import ctypes
import os

import numpy as np
import pytest

import oracle
from conftest import ROOT, announce

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def run(ctx):
    path = os.path.join(ROOT, "tests", "device", "libsp_device_tests.so")
    if not os.path.exists(path):
        import __graft_entry__
        __graft_entry__._builder().build_device_tests()
    lib = ctypes.CDLL(path)

    def call(nwg, lanes, rounds, seed, coherent, groups, xblock):
        out = np.zeros(nwg, np.uint32)
        info = np.zeros(2, np.uint32)
        announce("barrier fallback", f"nwg={nwg} lanes={lanes} rounds={rounds}",
                 f"coherent={coherent} groups={groups} xblock={xblock}")
        rc = lib.sp_test_barrier_fallback(*(ctypes.c_uint32(v) for v in
                                            (nwg, lanes, rounds, seed, coherent, groups, xblock)),
                                          out.ctypes.data_as(ctypes.c_void_p),
                                          info.ctypes.data_as(ctypes.c_void_p))
        assert rc == 0 and info[1] == 0, (rc, info)
        return out, int(info[0])
    return call


@pytest.mark.parametrize("coherent", [0, 1])
@pytest.mark.parametrize("nwg,lanes", [(9, 64), (64, 256), (300, 192), (1024, 64), (1024, 256)])
def test_registrations_that_do_not_fit_take_the_tree(ctx, run, nwg, lanes, coherent):
    xcds = ctx.info["xcd_count"]
    want = oracle.barrier_closed(17, nwg, 300)
    chk, over = run(nwg, lanes, 300, 17, coherent, xcds, 1)  # one member per block
    assert over >= nwg - xcds and (chk == want).all()
    if xcds > 1:  # the upper half of the XCD ids shares groups with the lower
        chk, over = run(nwg, lanes, 300, 17, coherent, xcds // 2, nwg)
        assert over > 0 and (chk == want).all()


@pytest.mark.parametrize("coherent", [0, 1])
def test_the_same_kernel_without_overflow(ctx, run, coherent):
    chk, over = run(300, 192, 300, 17, coherent, ctx.info["xcd_count"], 300)
    assert over == 0 and (chk == oracle.barrier_closed(17, 300, 300)).all()
