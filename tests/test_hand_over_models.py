"""The hand-overs as the device runs them, on all interleavings: the CU-cohort lock's grant
ahead of its section's stores with the completion count behind it, and the bounded buffer's
signal by a store of a counter loaded under the mutex.  Each planted mistake is caught."""

import pytest

from oracle.modelcheck import CondHeldSignalModel, CuCohortEarlyGrantModel, explore

# (xcd, cu) per agent: hand-overs within a CU, between CUs of an XCD and (CU4) between XCDs
CU3 = ((0, 0), (0, 0), (0, 1))
CU4 = ((0, 0), (0, 0), (0, 1), (1, 2))


@pytest.mark.parametrize("pl,ops,B", [(CU3, 2, 2), (CU3, 2, 3), (CU4, 1, 2), (CU4, 1, 3),
                                      (((0, 0), (0, 0)), 3, 3)])
def test_cu_cohort_early_grant_correct(pl, ops, B):
    """Mutual exclusion, no stale read of either guarded word though a store may land in the
    L2 long after the grant, every acquisition completes, every level ends released."""
    r = explore(CuCohortEarlyGrantModel(pl, ops, B))
    assert r.ok, r.violation


@pytest.mark.parametrize("pl,ops,B", [(CU3, 2, 2), (CU3, 2, 3), (CU4, 1, 2)])
@pytest.mark.parametrize("mutant", ["no_count_wait", "count_before_store", "no_acquire",
                                    "group_by_xcd"])
def test_cu_cohort_early_grant_mutants_read_stale(mutant, pl, ops, B):
    """Without the wait for the earlier holders' count, with a count ahead of one's own
    store, without the acquire or with groups that span CUs a holder misses an update."""
    r = explore(CuCohortEarlyGrantModel(pl, ops, B, mutant))
    assert not r.ok and "stale" in r.violation


@pytest.mark.parametrize("pl,ops,B", [(CU3, 2, 2), (CU3, 2, 3), (CU4, 1, 2)])
def test_cu_cohort_record_behind_the_grant_fails(pl, ops, B):
    assert not explore(CuCohortEarlyGrantModel(pl, ops, B, "record_after_grant")).ok


def test_cu_cohort_early_grant_without_waiter_deadlocks():
    assert explore(CuCohortEarlyGrantModel(CU3, 1, 3, "no_waiter_check")).deadlock


@pytest.mark.parametrize("P,Cn,items,C", [(1, 1, 3, 1), (1, 2, 2, 1), (2, 1, 2, 1),
                                          (2, 2, 1, 1), (1, 2, 3, 2), (2, 2, 2, 1)])
def test_signal_held_correct(P, Cn, items, C):
    r = explore(CondHeldSignalModel(P, Cn, items, C))
    assert r.ok, r.violation


@pytest.mark.parametrize("mutant,P,Cn,items", [("store_unlocked", 2, 2, 2),
                                               ("peek_unlocked", 1, 1, 3),
                                               ("peek_unlocked", 2, 1, 2)])
def test_signal_without_the_mutex_loses_a_wakeup(mutant, P, Cn, items):
    assert explore(CondHeldSignalModel(P, Cn, items, 1, mutant=mutant)).deadlock
