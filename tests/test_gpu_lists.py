"""The sorted-list kernel (variant 14 for batches without online tables) where
its shapes change: leaves that split and empty, windows cut anywhere, ties that
run over several leaves, timers that fire in numbers.  Every result against the
oracle."""
import numpy as np
import pytest

from paper_2609_09643_amd import synth
from parity import compare_counters, oracle_counters, oracle_log, same_log
from test_gpu_lane import Sim, workload
from tracekit import trace_from_events

pytestmark = pytest.mark.gpu

LISTS = 14


def offline(w):
    w.params = w.params[w.params["hazard_online"] == 0].copy()
    return w


@pytest.mark.parametrize("step", [1, 63, 64, 65, 200])
def test_windows_cut_anywhere(step):
    w = offline(workload(n_sessions=24 if step == 1 else 90, n_slots=12 if step == 1 else 40))
    s = Sim(w, log_cap=1 << 14, variant=LISTS)
    for e in range(0, w.traces[0].n_events, step):
        s.run(flags=(1 if e else 0) | 2, max_events=step)
    compare_counters(s.counters(), oracle_counters(w), label="step %d" % step)
    for i in range(w.n_sims):
        assert same_log(s.log(i), oracle_log(w, i)), "step %d sim %d log" % (step, i)


@pytest.mark.parametrize("n_slots", [1, 2, 33, 63, 64, 65, 129, 512, 513, 1000])
def test_resident_counts_around_leaf_sizes(n_slots):
    w = offline(workload(n_sessions=max(40, 3 * n_slots // 2), n_slots=n_slots, seed=n_slots))
    s = Sim(w, variant=LISTS)
    s.run()
    want = oracle_counters(w)
    compare_counters(s.counters(), want, label="slots %d" % n_slots)
    s.run(max_events=w.traces[0].n_events // 2)
    s.run(flags=1)
    compare_counters(s.counters(), want, label="slots %d split" % n_slots)


@pytest.mark.parametrize("sram,hbm", [(40, 4000), (2000, 2000), (4000, 40)])
def test_large_pools_with_ties(sram, hbm):
    """Pools of hundreds of residents in either tier: equal keys over several
    leaves (turn-0 sessions share a SPEAR key).  (Rows that run out and are
    packed: test_list_rows.py.)"""
    w = offline(workload(n_sessions=700, n_slots=600, seed=sram))
    w.params["cap_sram_B"] = sram * 40 * synth.MIB
    w.params["cap_hbm_B"] = hbm * 40 * synth.MIB
    w.params["ttl_ns"] = 20 * synth.NS
    s = Sim(w, log_cap=1 << 15, variant=LISTS)
    s.run(flags=2)
    compare_counters(s.counters(), oracle_counters(w), label="sram %d" % sram)
    for i in range(0, w.n_sims, 3):
        assert same_log(s.log(i), oracle_log(w, i, log_cap=1 << 15)), "sim %d log" % i


@pytest.mark.parametrize("n_slots", [256, 257, 600])
@pytest.mark.parametrize("online", [0, 1])
def test_chosen_kernel_on_both_sides_of_the_line(n_slots, online):
    """The kernel chosen by resident count, with and without a row whose
    hazard table grows online."""
    w = workload(n_sessions=700, n_slots=n_slots, seed=5 + n_slots)
    if not online:
        w = offline(w)
    s = Sim(w)
    s.run(max_events=500)
    s.run(flags=1)
    compare_counters(s.counters(), oracle_counters(w), label="auto %d online %d" % (n_slots, online))


@pytest.mark.parametrize("tide", [0, 1])
def test_the_largest_session_expires_from_the_last_slot(tide):
    """Session 2^20 - 1 in slot 4,095 of a full pool of 4,096: its entry is the
    word 0xFFFFFFFF.  Its timer fires alone, and beside others in either tier."""
    top, n = (1 << 20) - 1, 4095

    def workload_with(last):
        ev = [(10 + i, i, synth.KIND_ARRIVE, 0, 20) for i in range(n)]
        ev.append((10_000, last, synth.KIND_ARRIVE, 0, 5))      # the last free slot
        ev.append((10_001, last, synth.KIND_GAP_START, 0, 0))
        ev += [(10_002 + i, s, synth.KIND_GAP_START, 0, 0) for i, s in enumerate((7, 3, 4000))]
        ev.append((10_100, 9, synth.KIND_GAP_START, 0, 0))
        ev.append((10_101, 7, synth.KIND_ARRIVE, 1, 21))       # 7 is gone or resident, by the row
        ev.append((30_000, last, synth.KIND_ARRIVE, 1, 6))
        ev.append((30_001, last, synth.KIND_DONE, 1, 0))
        ev.append((60_000, 3, synth.KIND_ARRIVE, 1, 20))
        tr = trace_from_events(ev, last + 1)
        rows = []
        for cap_s in (0, 10, 1 << 40):   # all in HBM; only the last session in SRAM; all in SRAM
            for ttl in (0, 98, 100, 1000):
                p = synth.default_params(1)
                p["policy"], p["tide"], p["ttl_ns"] = synth.POLICY_TIMEOUT, tide, ttl
                p["cap_sram_B"], p["cap_hbm_B"], p["n_slots"] = cap_s, 1 << 40, 4096
                rows.append(p[0])
        return synth.Workload("top", [tr], [tr.turns], np.array(rows, dtype=synth.SIM_PARAMS_DTYPE))

    s = Sim(workload_with(top), log_cap=1 << 13)
    s.run(flags=2)
    got = s.counters()
    # The oracle runs the same trace with the last session as number 4,095 (its
    # scans of 2^20 entries would take minutes): ids keep their order, so only
    # that id differs in the records.
    small = workload_with(n)
    want = oracle_counters(small)
    assert all(c["expire"] >= 5 and c["error"] == 0 for c in want)
    got["digest"] = got["victim_digest"] = 0
    compare_counters(got, [dict(c, digest=0, victim_digest=0) for c in want], label="top")
    for i in range(small.n_sims):
        log = oracle_log(small, i).copy()
        log["a"][log["a"] == n] = top
        assert same_log(s.log(i), log), "sim %d log" % i
