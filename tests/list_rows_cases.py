"""Workloads that run the list kernel out of free rows, and a host model of its
leaf directories (csrc/lane.hip ListSim) that counts how often that happens."""
import bisect

import numpy as np

from paper_2609_09643_amd import synth
from tracekit import trace_from_events

LEAF = 64


class Rows:
    """The rows of both lists."""

    def __init__(self, n):
        self.free = n
        self.packs = {"event": 0, "promoted": 0, "demoted": 0}
        self.most = 0
        self.total = n


class Leaves:
    """One list: leaves in order, each a sorted list of (key order, session)."""

    def __init__(self, rows):
        self.rows = rows
        self.leaves = []

    def take(self):
        assert self.rows.free > 0
        self.rows.free -= 1
        self.rows.most = max(self.rows.most, self.rows.total - self.rows.free)

    def find(self, e):
        return max(0, bisect.bisect_right([lf[0] for lf in self.leaves], e) - 1)

    def insert(self, e, other, why):
        if self.rows.free == 0:
            self.pack()
            other.pack()
            self.rows.packs[why] += 1
        if not self.leaves:
            self.take()
            self.leaves.append([e])
            return
        p = self.find(e)
        if len(self.leaves[p]) == LEAF:
            self.take()
            self.leaves.insert(p + 1, self.leaves[p][LEAF // 2:])
            del self.leaves[p][LEAF // 2:]
            p = self.find(e)
        bisect.insort(self.leaves[p], e)

    def remove(self, e):
        p = self.find(e)
        self.leaves[p].remove(e)
        if not self.leaves[p]:
            del self.leaves[p]
            self.rows.free += 1

    def pack(self):
        flat = [e for lf in self.leaves for e in lf]
        was = len(self.leaves)
        self.leaves = [flat[i:i + LEAF] for i in range(0, len(flat), LEAF)]
        self.rows.free += was - len(self.leaves)


def lru_replay(trace, log, n_rows):
    """The lists over an LRU simulation's decision log: keys are event times, the
    oldest first, ties to the smaller id."""
    rows = Rows(n_rows)
    lists = {1: Leaves(rows), 2: Leaves(rows)}     # SRAM, HBM
    at = {}        # resident -> (tier, entry or None while it is served)
    by_ev = {}
    for r in log:
        by_ev.setdefault(int(r["ev"]), []).append((int(r["op"]), int(r["a"]), int(r["b"])))

    def put(s, tier, e, why):
        lists[tier].insert(e, lists[3 - tier], why)
        at[s] = (tier, e)

    def drop(s):
        tier, e = at.pop(s)
        if e is not None:
            lists[tier].remove(e)
        return e

    for k in range(trace.n_events):
        s, kind, t = int(trace.sid[k]), int(trace.info[k]) >> 24, int(trace.t_ns[k])
        if kind == synth.KIND_ARRIVE:
            if s in at:
                drop(s)
        elif s in at:
            put(s, at[s][0], (t, s), "event")
        for op, a, b in by_ev.get(k, ()):
            if op in (1, 2):
                drop(a)
            elif op == 7:
                at[a] = (b, None)
            elif op == 4:
                put(a, 1, drop(a), "promoted")
            elif op == 5:
                p, d = drop(a), drop(b)
                put(b, 2, d, "demoted")
                put(a, 1, p, "promoted")
    return rows


def thinned_leaves(n_slots, sram, seed, rounds, keep, lengths=(10, 11), spare=40):
    """A pool of n_slots that fills in order (leaves of 32 by appending), then
    rounds in which all but one in `keep` of the latest sessions run another turn,
    which leaves an entry or two in their leaves and appends the rest; at last
    some sessions end and new ones arrive."""
    rng = np.random.Generator(np.random.PCG64(seed))
    t, ev, turn = 1000, [], {}
    order = list(range(n_slots))

    def run(s, length):
        nonlocal t
        k = turn.get(s, -1) + 1
        turn[s] = k
        ev.append((t, s, synth.KIND_ARRIVE, k, length))
        ev.append((t + 400, s, synth.KIND_GAP_START, k, 0))
        t += int(rng.integers(500, 3000)) * 1000
    size = rng.integers(*lengths, n_slots)   # a prefix never shrinks
    for s in order:
        run(s, int(size[s]))
    old, recent = [], order
    for _ in range(rounds):
        stay = rng.random(len(recent)) < 1 / keep
        old += [s for s, k in zip(recent, stay) if k]
        recent = [s for s, k in zip(recent, stay) if not k]
        for s in recent:
            run(s, int(size[s]))
    order = old + recent
    for s in range(n_slots, n_slots + spare):
        run(s, int(rng.integers(1, 30)))
        done = order.pop(0)
        k = turn[done] + 1
        ev.append((t, done, synth.KIND_ARRIVE, k, int(size[done]) + 2))
        ev.append((t + 1, done, synth.KIND_DONE, k, 0))
        t += 2000
    tr = trace_from_events_fast(ev, n_slots + spare)
    rows = []
    for pol, mode, td in ((synth.POLICY_LRU, 0, 0), (synth.POLICY_LRU, 0, 1), (synth.POLICY_TIMEOUT, 0, 1),
                          (synth.POLICY_BELADY, 0, 1), (synth.POLICY_SPEAR, 0, 1), (synth.POLICY_SPEAR, 1, 1)):
        p = synth.default_params(1)
        p["policy"], p["score_mode"], p["tide"] = pol, mode, td
        p["cap_sram_B"], p["cap_hbm_B"], p["n_slots"] = sram * 10, 1 << 40, n_slots
        p["dma_B_per_us"] = 1
        p["ttl_ns"] = int(t * 0.6)
        rows.append(p[0])
    return synth.Workload("rows", [tr], [tr.turns], np.array(rows, dtype=synth.SIM_PARAMS_DTYPE))


def trace_from_events_fast(ev, n_sessions):
    """trace_from_events with the next arrivals found in one pass."""
    tr = trace_from_events([(a, b, synth.KIND_DONE if c == synth.KIND_GAP_START else c, d, e)
                            for a, b, c, d, e in ev], n_sessions)
    tr.info = np.array([(c << 24) | d for _, _, c, d, _ in ev], np.uint32)
    nxt = {}
    for i in range(len(ev) - 1, -1, -1):
        a, b, c, _, _ = ev[i]
        if c == synth.KIND_GAP_START:
            tr.next_ns[i] = nxt.get(b, synth.U64_MAX)
        elif c == synth.KIND_ARRIVE:
            nxt[b] = a
    return tr
