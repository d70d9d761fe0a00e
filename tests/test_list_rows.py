"""The list kernel's rows run out: the host model shows that the workloads of
list_rows_cases do that, over and over, from events and from TIDE's moves, and what the packed leaves leave free at every pool size; the GPU
runs them against the oracle."""
import pytest

from list_rows_cases import lru_replay, thinned_leaves
from parity import compare_counters, oracle_counters, oracle_log, same_log
from test_list_entry import lib  # noqa: F401  (a fixture)

# slots, SRAM residents, seed, rounds, one in how many stays, lengths
CASES = [(300, 120, 4, 11, 28, (5, 15)), (600, 200, 0, 11, 28, (5, 15)), (600, 300, 2, 10, 28, (10, 11)),
         (1500, 700, 3, 8, 24, (10, 11)), (4096, 1500, 4, 5, 24, (10, 11))]


def test_packed_leaves_leave_rows_free(lib):  # noqa: F811
    """After a pack both lists together use at most their full leaves and two
    partly filled ones; the rows beyond are the insertions until the next."""
    for n in range(1, 4097):
        slots = (n + 63) // 64 * 64
        rows = lib.rows(slots)
        used = slots // 64 + 1          # two lists: one partly filled leaf more
        assert rows - used >= 2 and rows <= 192, n
        if slots >= 3072:
            assert rows == 152 and rows - used >= 87
        else:
            assert rows == 3 * (slots // 64) + 8


@pytest.mark.parametrize("case", CASES)
def test_the_workloads_run_out_of_rows(lib, case):  # noqa: F811
    w = thinned_leaves(*case)
    n_rows = lib.rows((case[0] + 63) // 64 * 64)
    for row, least in ((0, 2), (1, 2)):
        r = lru_replay(w.traces[0], oracle_log(w, row, log_cap=1 << 18), n_rows)
        assert sum(r.packs.values()) >= least and r.most == n_rows, (row, r.packs)


def test_packs_come_from_every_insertion(lib):  # noqa: F811
    """Over the cases, an event's own insertion and both of a TIDE move find no
    row free."""
    seen = {"event": 0, "promoted": 0, "demoted": 0}
    for case in CASES:
        w = thinned_leaves(*case)
        r = lru_replay(w.traces[0], oracle_log(w, 1, log_cap=1 << 18), lib.rows((case[0] + 63) // 64 * 64))
        for k in seen:
            seen[k] += r.packs[k]
    assert all(seen.values()), seen


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES)
def test_lists_that_are_packed(case):
    from paper_2609_09643_amd.unison import Simulator
    w = thinned_leaves(*case)
    want = oracle_counters(w)
    s = Simulator(w, log_cap=1 << 17, variant=14)
    s.run(flags=2)
    compare_counters(s.counters(), want, label="rows %s" % (case,))
    for i in range(w.n_sims):
        assert same_log(s.log(i), oracle_log(w, i, log_cap=1 << 17)), "sim %d log" % i
    s.run(max_events=w.traces[0].n_events * 2 // 3)
    s.run(flags=1)
    compare_counters(s.counters(), want, label="rows %s split" % (case,))
