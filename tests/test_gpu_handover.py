"""Hand-overs between workgroups at the sizes where their paths can go wrong: slot indices
that wrap and do not divide evenly, queues that run empty, one and several wavefronts per
workgroup.  Results are whole numbers and equal the oracle's."""

import pytest

import oracle
from conftest import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("coherent", [0, 1])
@pytest.mark.parametrize("K,nwg,lanes,total", [
    (8, 64, 64, 40_000),     # one unit per XCD, every queue past its 4096 slots
    (13, 301, 192, 60_000),  # queues of one and of two units, more tickets than slots
    (257, 2048, 64, 70_000),  # 33 units in one queue: 4092 of its 4096 slots in use
    (300, 40, 128, 3_000),   # more units than workgroups: nobody waits
])
def test_xcd_chain_slots(ctx, K, nwg, lanes, total, coherent):
    """The per-XCD chains' grants through the XCD's L2: every pair is admitted once, at
    most K are inside, and the guarded words lose no update."""
    import paper_1110_4623_amd as sp
    announce("xcd chain", K, nwg, lanes, total, coherent)
    s = sp.Semaphore(ctx, "xcd_chain", K, coherent_cs=coherent)
    try:
        r = s.run(nwg, lanes, total, 200, 5, track=True, data=True)
    finally:
        s.close()
    assert (r["chk"] == oracle.sem_closed(5, nwg, total)).all()
    assert 1 <= r["maxocc"] <= K and r["occ"] == 0
    assert r["state"][1:] == (total, total, total)
    assert int(r["data"].astype("u8").sum()) == total
