"""The launch autotuner's choice (CPU: the timings are made up)."""
import pytest

from paper_2302_13590_amd import autotune as A


@pytest.mark.parametrize("quick", [False, True])
def test_the_library_s_own_launch_is_a_candidate(quick):
    """No schedule and no block asked for, with and without ordering: what only that launch reaches
    (four lanes per particle, the block chosen by size) can be recorded."""
    cands = A.candidates(quick)
    for sort in (1, 2):
        assert dict(schedule=0, sort=sort) in cands
    assert len({tuple(sorted(c.items())) for c in cands}) == len(cands)


def test_the_fastest_is_taken():
    cands = A.candidates()
    best, table = A.tune(lambda c: 1.0 if c == dict(schedule=0, sort=1) else 2.0, cands, reps=1)
    assert best == dict(schedule=0, sort=1) and len(table) == len(cands)


def test_an_entry_s_schedule_names_the_kernel():
    own = dict(schedule=0, sort=1)
    assert A.recorded(own, 1) == own
    assert A.recorded(own, 2) == dict(schedule=2, sort=1)
    for c in A.candidates():
        if c["schedule"]:
            assert A.recorded(c, c["schedule"]) == c
