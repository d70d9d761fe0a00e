"""Launches of a few events: a table left by any kernel is resumed by any other,
and the kernels chosen by a launch's length give one simulation's decisions
whatever the lengths of its launches.  Every result against the oracle."""
import numpy as np
import pytest

from paper_2609_09643_amd import synth
from parity import compare_counters, oracle_counters, oracle_log, same_log
from test_gpu_lane import Sim, dual_workload, workload

pytestmark = pytest.mark.gpu


def offline(w):
    w.params = w.params[w.params["hazard_online"] == 0].copy()
    return w


def replay(w, lengths, variants=None, log_cap=1 << 14, override=0xFF):
    """The workload in launches of the given lengths, over and over, each on the
    next of `variants` (None: chosen)."""
    from paper_2609_09643_amd.unison import lib
    s = Sim(w, log_cap=log_cap)
    n = max(t.n_events for t in w.traces)
    e = k = 0
    while e < n:
        if variants:
            assert lib().unison_debug_force_variant(s.ctx, variants[k % len(variants)]) == 0
        s.run(policy=override, flags=(1 if e else 0) | 2, max_events=lengths[k % len(lengths)])
        e += lengths[k % len(lengths)]
        k += 1
    return s


def check(s, w, want, label):
    compare_counters(s.counters(), want, label=label)
    for i in range(w.n_sims):
        assert same_log(s.log(i), oracle_log(w, i)), "%s sim %d log" % (label, i)


@pytest.mark.parametrize("n_sessions,n_slots,variants",
                         [(16, 12, (5, 13)), (16, 16, (13, 0, 14, 5)), (60, 40, (7, 13, 15)),
                          (200, 150, (8, 13, 14)), (300, 200, (12, 13, 10, 15)), (420, 300, (12, 14, 13)),
                          (700, 600, (14, 10, 15, 12, 14, 15))])
def test_tables_pass_between_kernels(n_sessions, n_slots, variants):
    w = workload(n_sessions=n_sessions, n_slots=n_slots, seed=n_sessions)
    want = oracle_counters(w)
    for lengths in ((7, 64, 1, 130), (33,)):
        check(replay(w, lengths, variants), w, want, "%d %s" % (n_sessions, lengths))
    w = offline(w)   # variant 14 as lists
    check(replay(w, (50, 3), variants), w, oracle_counters(w), "offline %d" % n_sessions)


@pytest.mark.parametrize("n_sessions,n_slots", [(3, 3), (16, 12), (17, 17), (60, 40), (200, 150), (256, 64),
                                                (300, 200), (420, 300), (700, 600)])
@pytest.mark.parametrize("online", [0, 1])
def test_chosen_kernels_over_launch_lengths(n_sessions, n_slots, online):
    w = workload(n_sessions=n_sessions, n_slots=n_slots, seed=n_sessions + 1)
    if not online:
        w = offline(w)
    want = oracle_counters(w)
    for lengths in ((1, 2, 3, 5, 9, 11, 20, 60, 80), (4,), (100, 1)):
        check(replay(w, lengths), w, want, "%d %s" % (n_sessions, lengths))


@pytest.mark.parametrize("n_sessions,n_slots", [(20, 12), (300, 200), (500, 400)])
def test_chosen_kernels_of_the_dual_design(n_sessions, n_slots):
    w = dual_workload(n_slots, n_sessions)
    check(replay(w, (1, 2, 4, 70, 19, 21), log_cap=1 << 13), w, oracle_counters(w), "dual")


def test_a_policy_for_all_rows_in_short_launches():
    """The register tables' lane-group map is the parameter rows'; a launch
    under one policy for all rows stays on the lane kernel."""
    w = offline(workload(n_sessions=16, n_slots=12, seed=3))
    s = replay(w, (2, 1, 40), override=synth.POLICY_LRU)
    w.params["policy"] = synth.POLICY_LRU
    check(s, w, oracle_counters(w), "override")


@pytest.mark.parametrize("n_slots", [60, 200, 2000])
def test_short_launches_of_tables_beyond_lds(n_slots):
    """5,000 sessions: the streamed table for short launches, and the wide-table
    kernel, whose LDS slots many simulations resume from."""
    w = offline(workload(n_sessions=5000, n_slots=n_slots, seed=n_slots, mean=1))
    w.params = w.params[[0, 2, 5, 7]].copy()
    w.params["ttl_ns"] = 60 * synth.NS
    n = 2500
    want = oracle_counters(w, max_events=n)
    s = Sim(w)
    for k, (m, variant) in enumerate(((1500, -1), (3, -1), (20, -1), (70, -1), (307, 15), (100, 14 if n_slots > 512 else 13),
                                      (500, -1))):
        from paper_2609_09643_amd.unison import lib
        assert lib().unison_debug_force_variant(s.ctx, variant) == 0
        s.run(flags=1 if k else 0, max_events=m)
    compare_counters(s.counters(), want, label="wide %d" % n_slots)


def test_short_launches_by_batch_size():
    """16-session tables: 1,024 simulations over 5 events a launch (register
    tables below 6) and 8 (the lane kernel) against one launch."""
    w = synth.c3_sweep()
    few = synth.Workload("few", w.traces, w.lut_pops, w.params[::16][:1024].copy(), w.flat_luts)
    one = Sim(few)
    one.run()
    want = one.counters().view(np.uint64)
    for step in (5, 8):
        s = Sim(few)
        for e in range(0, max(t.n_events for t in w.traces), step):
            s.run(flags=1 if e else 0, max_events=step)
        assert np.array_equal(s.counters().view(np.uint64), want), step


@pytest.mark.parametrize("n_sessions,n_slots", [(16, 12), (60, 40), (200, 150), (300, 200), (420, 300)])
def test_short_and_long_launches_under_capture(n_sessions, n_slots):
    """A fresh short launch, a long one and the rest recorded into one graph:
    no launch waits for the stream, and every replay gives the eager result."""
    import torch
    w = workload(n_sessions=n_sessions, n_slots=n_slots, seed=n_sessions + 2)
    want = oracle_counters(w)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        s = Sim(w)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=side):
            s.run(max_events=2)
            s.run(flags=1, max_events=100)
            s.run(flags=1, max_events=1)
            s.run(flags=1)
        for k in range(3):
            g.replay()
            compare_counters(s.counters(), want, label="replay %d" % k)
            s.run(max_events=5)      # the eager path's own use of the same tables
            torch.cuda.synchronize()
