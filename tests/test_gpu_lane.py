"""The lane kernel (residents sorted across one wavefront's lanes, events
prepared 64 to a window) where its shapes change: windows cut at and around 64
events, resident counts around each register width, a resident evicted in a
later launch without an event of its own, session ids up to 2^20 - 1.  Every
result against the oracle, decision by decision."""
import numpy as np
import pytest

import oracle
from paper_2609_09643_amd import synth
from parity import compare_counters, oracle_counters, oracle_log, same_log

pytestmark = pytest.mark.gpu

LANE = 13


def Sim(*a, **k):
    from paper_2609_09643_amd.unison import Simulator
    return Simulator(*a, **k)


def workload(n_sessions=90, n_slots=64, seed=11, sids=None, mean=5):
    """Every policy and score form, with and without TIDE and online tables,
    on one trace whose pool keeps evicting."""
    rng = np.random.Generator(np.random.PCG64(seed))
    turns = synth.geometric_turns(rng, n_sessions, mean)
    kvb = np.array([64, 128, 160], dtype=np.uint32)[rng.permutation(n_sessions) % 3] * synth.KIB
    tr = synth.build_trace(rng, turns, synth.poisson_arrivals(rng, n_sessions, 20.0),
                           synth.gaps_mixture, kvb)
    if sids is not None:
        tr.sid = np.asarray(sids, np.uint32)[tr.sid]
        wide = np.zeros(int(max(sids)) + 1, np.uint32)
        wide[np.asarray(sids)] = kvb
        tr.kvb = wide
        n_turns = np.zeros(wide.shape[0], np.uint32)
        n_turns[np.asarray(sids)] = turns
        tr.turns = n_turns
    rows = []
    for pol, mode, tide, online in ((0, 0, 1, 0), (0, 0, 0, 0), (0, 1, 1, 0), (0, 0, 1, 1), (0, 1, 1, 1),
                                    (1, 0, 0, 0), (1, 0, 1, 0), (2, 0, 0, 0), (2, 0, 1, 0),
                                    (3, 0, 1, 0), (4, 0, 1, 0)):
        p = synth.default_params(1)
        p["policy"], p["score_mode"], p["tide"], p["hazard_online"] = pol, mode, tide, online
        p["cap_sram_B"] = n_slots * 40 * synth.MIB
        p["cap_hbm_B"] = n_slots * 120 * synth.MIB
        p["ttl_ns"] = 3 * synth.NS
        p["n_slots"] = n_slots
        rows.append(p[0])
    return synth.Workload("lane", [tr], [turns], np.array(rows, dtype=synth.SIM_PARAMS_DTYPE))


@pytest.mark.parametrize("step", [1, 63, 64, 65, 200])
def test_windows_cut_anywhere(step):
    w = workload(n_sessions=24 if step == 1 else 90, n_slots=12 if step == 1 else 40)
    s = Sim(w, log_cap=1 << 14, variant=LANE)
    n = w.traces[0].n_events
    for e in range(0, n, step):
        s.run(flags=(1 if e else 0) | 2, max_events=step)
    compare_counters(s.counters(), oracle_counters(w), label="step %d" % step)
    for i in range(w.n_sims):
        assert same_log(s.log(i), oracle_log(w, i)), "step %d sim %d log" % (step, i)


@pytest.mark.parametrize("n_slots", [1, 2, 63, 64, 65, 128, 129, 256, 257, 512])
def test_resident_counts_around_each_width(n_slots):
    w = workload(n_sessions=max(40, 3 * n_slots // 2), n_slots=n_slots, seed=n_slots)
    s = Sim(w, variant=LANE)
    s.run()
    want = oracle_counters(w)
    compare_counters(s.counters(), want, label="slots %d" % n_slots)
    s.run(max_events=w.traces[0].n_events // 2)
    s.run(flags=1)
    compare_counters(s.counters(), want, label="slots %d split" % n_slots)


def dual_workload(n_slots, n_sessions):
    w = workload(n_sessions=n_sessions, n_slots=n_slots, seed=n_slots + 1)
    rows = []
    for r in w.params:
        if r["hazard_online"]:
            continue
        for sync in (synth.DUAL_NONE, synth.DUAL_EVERY, synth.DUAL_EIGHT, synth.DUAL_GAP):
            q = r.copy()
            q["dual_sync"] = sync
            rows.append(q)
    w.params = np.array(rows, dtype=synth.SIM_PARAMS_DTYPE)
    return w


@pytest.mark.parametrize("n_slots,step", [(12, 1), (40, 64), (40, 77), (100, 90), (200, 1000)])
def test_dual_copies_across_launches(n_slots, step):
    """The dual design's copies through launches cut anywhere, every second
    one on the streamed-table kernel, which reads and refreshes the copies in
    the workspace."""
    from paper_2609_09643_amd.unison import lib
    w = dual_workload(n_slots, 20 if step == 1 else 60 if n_slots < 100 else 300)
    n = w.traces[0].n_events
    for swap in (False, True):
        s = Sim(w, log_cap=1 << 13)
        for i, e in enumerate(range(0, n, step)):
            if swap:
                assert lib().unison_debug_force_variant(s.ctx, 11 if i % 2 else -1) == 0
            s.run(flags=(1 if e else 0) | 2, max_events=step)
        compare_counters(s.counters(), oracle_counters(w), label="dual %d/%d swap %d" % (n_slots, step, swap))
        for i in range(0, w.n_sims, 5):
            assert same_log(s.log(i), oracle_log(w, i)), "dual sim %d log" % i


def test_dual_rows_with_online_tables():
    w = dual_workload(40, 60)
    w.params["hazard_online"] = np.arange(w.n_sims) % 3 == 0
    s = Sim(w)
    s.run()
    compare_counters(s.counters(), oracle_counters(w), label="dual online")


def test_session_ids_up_to_the_largest():
    top = (1 << 20) - 1
    sids = [top - 3 * k for k in range(60)] + list(range(0, 900, 30))
    w = workload(n_sessions=len(sids), n_slots=30, sids=sids)
    w.params = w.params[:3]
    s = Sim(w, variant=LANE)
    s.run(max_events=150)
    s.run(flags=1)
    compare_counters(s.counters(), oracle_counters(w), label="large ids")


def test_small_tables_choose_by_batch_size():
    """Batches of 16-session tables on both sides of the 4,096-simulation
    line: the same counters from the lane kernel and the register tables."""
    w = synth.c3_sweep()
    rows = w.params[::4][:4096].copy()
    few = synth.Workload("few", w.traces, w.lut_pops, rows, w.flat_luts)
    many = synth.Workload("many", w.traces, w.lut_pops, np.concatenate([rows, rows[:1]]), w.flat_luts)
    a, b = Sim(few), Sim(many)
    a.run()
    b.run()
    ca, cb = a.counters(), b.counters()
    assert np.array_equal(ca.view(np.uint64), cb[:4096].view(np.uint64))


@pytest.mark.parametrize("mean", [1, 2])
@pytest.mark.parametrize("n_slots", [2, 64, 65, 128, 200, 257, 512])
def test_online_tables_that_change_at_every_turn(n_slots, mean):
    """Sessions of one or two turns under online tables: a completion every few
    events, each changing every resident's key and the order of a full pool."""
    w = workload(n_sessions=n_slots + 20, n_slots=n_slots, seed=n_slots + mean, mean=mean)
    rows = [r for r in w.params if r["hazard_online"]]
    for r in list(rows):
        for cap in (0, 3, n_slots // 2):
            q = r.copy()
            q["online_sessions"] = cap
            rows.append(q)
    w.params = np.array(rows, dtype=synth.SIM_PARAMS_DTYPE)
    w.params["cap_sram_B"] = n_slots * 100 * synth.MIB
    w.params["cap_hbm_B"] = n_slots * 1000 * synth.MIB
    want = oracle_counters(w)
    for variant in (LANE, None):   # 257 to 384 residents of few turns have a rule of their own
        s = Sim(w, log_cap=1 << 13, variant=variant)
        s.run(flags=2, max_events=w.traces[0].n_events // 3)
        s.run(flags=3)
        compare_counters(s.counters(), want, label="online %d mean %d" % (n_slots, mean))
        for i in range(w.n_sims):
            assert same_log(s.log(i), oracle_log(w, i)), "sim %d log" % i
