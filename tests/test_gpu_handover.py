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


@pytest.mark.parametrize("passes", [1, 2, 255])
@pytest.mark.parametrize("nwg,lanes,L,W", [
    (2048, 64, 1, 1),      # one wavefront, one word
    (2048, 256, 3, 257),   # stores of four wavefronts over nine lines
    (512, 1024, 2, 1000),  # sixteen wavefronts, two workgroups per CU
    (777, 192, 1, 33),     # CUs with three and with four contenders
])
def test_cu_cohort_handover(ctx, nwg, lanes, L, W, passes):
    """A hand-over within a CU waits for no store; the one that leaves the CU waits for
    every holder before it.  Each word's count is exact however often the lock moves."""
    import paper_1110_4623_amd as sp
    announce("cu cohort", nwg, lanes, L, W, passes)
    m = sp.Mutex(ctx, "cu_cohort", L, W, cohort_passes=passes, verify=1)
    try:
        words, st, _ = m.run(nwg, lanes, 12_345, 50, 3)
    finally:
        m.close()
    assert st["device_error"] == 0
    assert (words == oracle.mutex_closed(3, nwg, 12_345, L, W)).all()


@pytest.mark.parametrize("passes", [1, 3, 255])
@pytest.mark.parametrize("pad", [4, 128])
def test_xcd_cohort_handover(ctx, pad, passes):
    """Grants through the XCD's L2, also where words of several XCDs share a line."""
    import paper_1110_4623_amd as sp
    announce("cohort", pad, passes)
    m = sp.Mutex(ctx, "cohort", 5, 70, cohort_passes=passes, pad_bytes=pad, verify=1)
    try:
        words, st, _ = m.run(600, 128, 20_001, 100, 3)
    finally:
        m.close()
    assert st["device_error"] == 0
    assert (words == oracle.mutex_closed(3, 600, 20_001, 5, 70)).all()


@pytest.mark.parametrize("coherent", [0, 1])
@pytest.mark.parametrize("nwg,L", [
    (24, 4), (23, 3), (25, 5), (96, 6), (95, 6),   # around the spin / XCD-cohort lines
    (639, 1), (640, 1), (1280, 1), (1279, 1),      # around the XCD-cohort / CU-cohort lines
])
def test_default_mutex_lines(ctx, nwg, L, coherent):
    """A default mutex on both sides of each line, the first run of every mutex recorded
    into a graph (so nothing is allocated for it) and replayed with runs in between."""
    import paper_1110_4623_amd as sp
    announce("default mutex", nwg, L, coherent)
    want = oracle.mutex_closed(9, nwg, 3000, L, 9)
    m = sp.Mutex(ctx, "default", L, 9, coherent_cs=coherent)
    g = sp.Graph(ctx)
    try:
        with g:
            m.launch(nwg, 64, 3000, 100, 9)
        for _ in range(2):
            g.launch(2)
            assert (m.words() == want).all()
            words, _, _ = m.run(nwg, 64, 3000, 100, 9)
            assert (words == want).all()
    finally:
        g.close()
        m.close()


@pytest.mark.parametrize("coherent", [0, 1])
@pytest.mark.parametrize("nwg,lanes", [
    (9, 64),        # XCDs with one member and with two
    (504, 64), (512, 64), (520, 256),   # 63, 64 and 65 members: around a group of arrivals
    (1032, 128),    # two groups and one member, two wavefronts
    (2048, 64),     # four groups, one wavefront to scan them
])
def test_xcd_barrier_arrivals(ctx, nwg, lanes, coherent):
    """The arrival bytes wrap every 256 rounds; a scan compares 64 members at a time."""
    import paper_1110_4623_amd as sp
    announce("xcd barrier", nwg, lanes, coherent)
    b = sp.Barrier(ctx, "xcd", nwg, coherent_cs=coherent)
    try:
        chk, _ = b.run_hash(lanes, 700, 17)
        assert b.info()["xcd_path"]
    finally:
        b.close()
    assert (chk == oracle.barrier_closed(17, nwg, 700)).all()


@pytest.mark.parametrize("offset", [0, 1, 2, 3])
@pytest.mark.parametrize("K", [1, 2, 3, 5, 301])
def test_resets_reach_their_range_and_no_more(ctx, K, offset):
    """A run resets its arrays with 16-byte stores between their aligned ends: an output of
    K words at any word offset is reset whole, and its neighbours keep their values."""
    import ctypes

    import paper_1110_4623_amd as sp
    from paper_1110_4623_amd import _native as N
    if ctx.torch is None:
        pytest.skip("needs torch's device tensors")
    announce("resets", K, offset)
    s = sp.Semaphore(ctx, "sleep", K)
    out = ctx.torch.full((K + 16,), 77, dtype=ctx.torch.int32, device="cuda")
    chk, state, st = ctx.zeros(64), ctx.zeros(8), N.Stats()
    try:
        for total in (1000, 500):  # the second run finds the first one's words
            rc = N.lib.sp_sem_run(s.h, 64, 64, total, 0, 5, 0, ctx.ptr(chk), ctx.ptr(state),
                                  ctypes.c_void_p(out.data_ptr() + 4 * (4 + offset)),
                                  ctypes.byref(st), ctx.stream())
            assert rc == 0 and st.device_error == 0 and st.kernel_ms > 0
            got = out.cpu().numpy()
            assert got[4 + offset:4 + offset + K].sum() == total
            assert (got[:4 + offset] == 77).all() and (got[4 + offset + K:] == 77).all()
    finally:
        s.close()


@pytest.mark.parametrize("nwg,producers", [(2, 1), (257, 1), (300, 299), (1024, 512)])
def test_ring_totals_over_all_workgroups(ctx, nwg, producers):
    """The totals of more and of fewer workgroups than the adding kernel has lanes."""
    import numpy as np

    import paper_1110_4623_amd as sp
    announce("ring totals", nwg, producers)
    r = sp.bounded_buffer(ctx, "array", nwg, producers, 32, 3001, 7, values=True)
    assert r["taken"] == r["put"] == 3001 and r["left"] == 0 and 1 <= r["max_count"] <= 32
    assert r["sum"] == int(r["values"].astype(np.uint64).sum())
    assert r["xor"] == int(np.bitwise_xor.reduce(r["values"]))


@pytest.mark.parametrize("T,stride", [(1, 4), (255, 4), (1000, 64), (1 << 20, 4),
                                      ((1 << 20) + 1, 8), ((2 << 20) + 77, 12)])
def test_finals_of_strided_words(ctx, T, stride):
    """Final words read through the staging: none, one and several times its size, on a
    fresh and on a caller's buffer."""
    import numpy as np

    import paper_1110_4623_amd as sp
    import sp_inputs
    announce("strided finals", T, stride)
    perm = sp_inputs.permutation(T, 3)
    buf = ctx.zeros(T * stride // 4 + 5)
    for b in (None, buf):
        finals, _, _ = sp.bench_atomic(ctx, "add", 16, 64, T, stride, "per_lane", 3, 3, perm, b)
        pos = (np.arange(16 * 64)[:, None] + np.arange(3)[None, :]) % T
        want = np.bincount(perm[pos].ravel(), minlength=T).astype(np.uint32)
        assert finals.dtype == np.uint32 and (finals == want).all()


@pytest.mark.parametrize("reps", [1, 3])
@pytest.mark.parametrize("n16,nwg", [
    (1, 0), (63, 1), (64, 1), (65, 2), (2047, 1), (2049, 1), (16 * 2048 + 5, 3),
    (8192 * 64 - 1, 0), (8192 * 64 + 1, 0), (1_000_003, 777), (5 << 20, 0),
])
def test_stream_sums_at_piece_edges(ctx, n16, nwg, reps):
    """Pieces of whole wavefront loads, empty last pieces, loads left over from a step of
    eight, more workgroups than sum slots; the sum is exact."""
    import numpy as np

    import paper_1110_4623_amd as sp
    announce("stream", n16, nwg, reps)
    words = np.random.default_rng(n16).integers(0, 1 << 32, 4 * n16, dtype=np.uint64)
    words = words.astype(np.uint32)
    buf = ctx.upload(words)
    s, st = sp.stream_read(ctx, buf, 16 * n16, reps=reps, nwg=nwg)
    assert s == reps * int(words.sum(dtype=np.uint64)) and st["device_error"] == 0


def test_stream_sum_in_a_graph(ctx):
    """A recorded read adds to its own output: replays beside eager reads of the same
    context keep both sums."""
    import ctypes

    import numpy as np

    import paper_1110_4623_amd as sp
    from paper_1110_4623_amd import _native as N
    announce("stream in a graph")
    a, b = (ctx.upload(np.full(1 << 20, v, np.uint32)) for v in (3, 5))
    out, st = ctx.zeros(1, "u64"), N.Stats()
    g = sp.Graph(ctx)
    with g:
        assert N.lib.sp_bench_stream(ctx.h, ctx.ptr(a), 4 << 20, 0, 2, ctx.ptr(out),
                                     ctypes.byref(st), ctx.stream()) == 0
    for _ in range(3):
        g.launch()
        assert sp.stream_read(ctx, b, 4 << 20)[0] == 5 << 20
        assert int(ctx.read(out, "u64", 1)[0]) == 2 * 3 << 20
    g.close()


@pytest.mark.parametrize("coherent", [0, 1])
@pytest.mark.parametrize("kind", ["sleep", "array", "chain", "xcd_chain", "cohort"])
@pytest.mark.parametrize("K,nwg,lanes", [(2, 2, 64), (2, 64, 256), (3, 3, 128), (4, 257, 64),
                                         (64, 65, 192)])
def test_pool_slots_returned_behind_the_post(ctx, kind, K, nwg, lanes, coherent):
    """A holder admitted before its predecessor's slot is back: every update of the pool's
    words is kept, with as many holders as slots and with one more."""
    import paper_1110_4623_amd as sp
    if kind == "xcd_chain" and K < ctx.info["xcd_count"]:
        pytest.skip("a unit per XCD at least")
    announce("pool", kind, K, nwg, lanes, coherent)
    s = sp.Semaphore(ctx, kind, K, coherent_cs=coherent)
    try:
        r = s.run(nwg, lanes, 5000, 0, 11, track=True, data=True)
    finally:
        s.close()
    assert (r["chk"] == oracle.sem_closed(11, nwg, 5000)).all()
    assert 1 <= r["maxocc"] <= K and int(r["data"].astype("u8").sum()) == 5000


@pytest.mark.parametrize("coherent", [0, 1])
@pytest.mark.parametrize("kind", ["central", "tree", "flag", "xcd"])
@pytest.mark.parametrize("nwg,lanes", [(1, 64), (2, 128), (7, 64), (8, 64), (9, 192), (255, 64),
                                       (256, 128), (257, 1024 // 4), (511, 320), (2047, 256)])
def test_exchange_layout(ctx, nwg, lanes, kind, coherent):
    """Workgroup counts around whole blocks of the exchange's layout, rounds past the count
    (the reader comes round to its first slot), one round and none."""
    import paper_1110_4623_amd as sp
    announce("exchange layout", kind, nwg, lanes, coherent)
    b = sp.Barrier(ctx, kind, nwg, coherent_cs=coherent)
    try:
        for rounds in (1, 2, min(2 * nwg + 3, 300), 0):
            chk, st = b.run_hash(lanes, rounds, 13)
            assert st["device_error"] == 0
            assert (chk == oracle.barrier_closed(13, nwg, rounds)).all()
    finally:
        b.close()


@pytest.mark.parametrize("mode", ["persistent", "launch"])
def test_chain_lengths_around_an_iteration(ctx, mode):
    """Hash chains of every length from none to four iterations of the unrolled loop."""
    import numpy as np

    import paper_1110_4623_amd as sp
    import sp_inputs
    announce("chain lengths", mode)
    reqs = dict(sp_inputs.request_table(66, 1e5, 9))
    reqs["L"] = np.arange(66, dtype=np.asarray(reqs["L"]).dtype)
    if mode == "persistent":
        out, _, r = sp.serve(ctx, reqs, nwg=32, seed=9)
    else:
        out, _, r = sp.serve_launch_per_request(ctx, reqs, seed=9)
    assert r["completed"] == 66
    assert (out == oracle.chain_batch(9, reqs["L"])).all()
