"""How many workgroups of 1-16 wavefronts a CU is sure to hold at once.  The expected counts
were measured on an MI355X: grids of workgroups that note their start, spin for a fixed time
and end, without waiting for each other; the largest count per CU at which no workgroup of 20
grids started after another one's end.  Rows: wave slots per SIMD (512 VGPRs / the kernel's).
"""
import ctypes

import pytest

import oracle
from conftest import announce

# VGPRs, wave slots per SIMD, workgroups per CU at 1, 2, ... wavefronts per workgroup
MEASURED = [
    (56, 8, [32, 16, 10, 8, 5, 4, 4, 4, 3, 2, 2, 2, 2, 2, 2, 2]),
    (72, 7, [28, 14, 9, 7, 4, 3, 3, 3, 2, 2, 2, 2, 1, 1, 1, 1]),
    (80, 6, [24, 12, 7, 6, 3, 3, 3, 3, 2, 2, 2, 2, 1, 1, 1, 1]),
    (96, 5, [20, 10, 6, 5, 3, 2, 2, 2, 1, 1, 1, 1, 1, 1, 1, 1]),
    (128, 4, [16, 8, 5, 4, 2, 2, 2, 2, 1, 1, 1, 1, 1, 1, 1, 1]),
    (168, 3, [12, 6, 3, 3, 1, 1, 1, 1, 1, 1, 1, 1]),
    (256, 2, [8, 4, 2, 2, 1, 1, 1, 1]),
]


@pytest.mark.parametrize("vgprs,slots,counts", MEASURED)
def test_workgroups_per_cu_are_the_measured_ones(vgprs, slots, counts):
    from paper_1110_4623_amd import _native as N
    for waves, want in enumerate(counts, 1):
        o = N.Occupancy(runtime_per_cu=4 * slots // waves, vgprs=vgprs, lds_bytes=2048,
                        lanes=64 * waves)
        assert N.lib.sp_resident_per_cu(ctypes.byref(o)) == want, waves


@pytest.mark.gpu
@pytest.mark.parametrize("waves,per_cu", [(3, 10), (5, 5), (6, 4), (7, 4), (10, 2)])
def test_barrier_runs_at_the_count_and_is_refused_above_it(ctx, waves, per_cu):
    import paper_1110_4623_amd as sp
    lanes, most = 64 * waves, per_cu * ctx.info["cu_count"]
    announce("barrier at the residency limit", f"nwg={most} lanes={lanes} rounds=50")
    b = sp.Barrier(ctx, "default", most)
    try:
        chk, st = b.run_hash(lanes, 50, 9)
        assert st["resident_per_cu"] == per_cu
        assert (chk == oracle.barrier_closed(9, most, 50)).all()
    finally:
        b.close()
    b = sp.Barrier(ctx, "default", most + 1)
    try:
        with pytest.raises(sp.SpNotResident):
            b.run_hash(lanes, 1, 9)
    finally:
        b.close()
