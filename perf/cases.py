"""The work that users of this framework have it do, as measurable cases.

A case is a plain dict; `prepare` builds what a program holds before the call
(traces, hazard tables and parameter rows in a Simulator, or the score inputs
of a ranking study on the GPU), `run` makes one pass through the public entry
points.  Five kinds cover the framework:

  sweep   many independent simulations of short traces (policy, capacity and
          hazard-table sweeps); the counters stay on the GPU
  trace   one paper-scale trace under the residency policies side by side;
          the counters are read back, as a study script does
  study   the batches the paper's studies launch: fixed-point formats, online
          hazard tables, components, session slots, dual register files
  live    tens of thousands of concurrently live sessions
  rank    the ranking-fidelity pass: hazard fit, gap EMAs, both scores and
          Kendall tau-b per fixed-point format (n_per = 0: scores of a pool only)

Every output is defined bit by bit (integer counters and digests of every
decision, fp32 scores with a fixed order of roundings, integer scores, pair
counts), so the tolerance is "exact" throughout.
"""
import numpy as np
import torch

from paper_2609_09643_amd import synth
from paper_2609_09643_amd import unison as U

POLICY_MIXES = {
    # SPEAR+TIDE beside the offline bound
    "pair": ((synth.POLICY_SPEAR, 0), (synth.POLICY_BELADY, 0)),
    # the four residency policies
    "four": ((synth.POLICY_SPEAR, 0), (synth.POLICY_LRU, 0), (synth.POLICY_TIMEOUT, 0),
             (synth.POLICY_BELADY, 0)),
    # every policy and both score forms
    "all": ((synth.POLICY_SPEAR, 0), (synth.POLICY_SPEAR, 1), (synth.POLICY_LRU, 0),
            (synth.POLICY_TIMEOUT, 0), (synth.POLICY_BELADY, 0), (synth.POLICY_ETA, 0)),
}
STUDIES = ("formats", "online", "components", "slots", "dual")
PENALTY_US = 5e8


def listed():
    return [
        # the smallest call: the 16-session trace under SPEAR+TIDE and Belady,
        # as an interactive what-if or a smoke test runs it
        {"name": "tiny_pair", "kind": "sweep", "sims": 2, "sessions": 16, "turns": 12, "traces": 1,
         "mix": "pair"},
        # the headline sweep: 4,096 capacity x hazard points under each of four policies
        {"name": "capacity_sweep", "kind": "sweep", "sims": 16384, "sessions": 16, "turns": 12,
         "traces": 8, "mix": "four"},
        # an ordinary sweep of odd sizes: every policy, both score forms, mixed in one batch
        {"name": "mixed_sweep_53", "kind": "sweep", "sims": 1511, "sessions": 53, "turns": 17,
         "traces": 5, "mix": "all"},
        # a sweep over traces of a few hundred sessions, the size of the paper's smaller traces
        {"name": "mixed_sweep_203", "kind": "sweep", "sims": 999, "sessions": 203, "turns": 9,
         "traces": 3, "mix": "all"},
        # the paper-scale trace, four policies side by side: one long chain of decisions each
        {"name": "paper_trace", "kind": "trace", "sessions": 1415, "turns": 33596, "slots": 64,
         "scale": 8, "mix": "four"},
        # the fixed-point format study: 27 formats with the exact divider and with a
        # 16-bit reciprocal table, and the fp32 reference, on 6 traces x 3 envelopes
        {"name": "format_study", "kind": "study", "study": "formats", "recip": 16, "turns": 33596},
        # online hazard tables rebuilt from the first n completions
        {"name": "online_study", "kind": "study", "study": "online", "recip": 0, "turns": 33596},
        # the unified register file against the dual copies
        {"name": "dual_study", "kind": "study", "study": "dual", "recip": 0, "turns": 33596},
        # 65,536 live sessions in tables too large for LDS
        {"name": "live_set", "kind": "live", "sims": 16, "traces": 2, "sessions": 65536,
         "turns": 150000, "slots": 4096},
        # ranking fidelity of large snapshots: C5's two formats and a nanosecond-resolution
        # one whose scores pass 32 bits
        {"name": "rank_4096", "kind": "rank", "snapshots": 10000, "n_per": 4096, "pool": 65536,
         "formats": "16/32/1000/0,12/32/1000/0,12/64/1/0"},
        # the format study's ranking gate: 7,265 snapshots of 64 sessions
        {"name": "rank_64", "kind": "rank", "snapshots": 7265, "n_per": 64, "pool": 65536,
         "formats": "8/32/1/0,8/32/1000/0,8/32/1000000/0,10/24/1000/12,10/32/1000/16,"
                    "12/24/1/20,12/32/1000/0,12/32/1000000/24,12/64/1/0"},
        # the scores of a very large session pool, in bulk
        {"name": "pool_scores", "kind": "rank", "snapshots": 0, "n_per": 0, "pool": 8000003,
         "formats": "12/32/1000/0,12/32/1000/16"},
    ]


def _log_int(rng, lo, hi):
    """An integer spread evenly over the logarithm of [lo, hi]."""
    return int(min(hi, max(lo, round(lo * (hi / lo) ** rng.random()))))


def _formats(rng, n):
    return ",".join("%d/%d/%d/%d" % (rng.choice((8, 10, 12, 16)), rng.choice((24, 32, 64)),
                                     rng.choice((1, 1000, 1000000)), rng.choice((0, 0, 12, 16, 20, 24)))
                    for _ in range(n))


def draw(rng):
    kind = rng.choice(("sweep", "sweep", "sweep", "trace", "study", "live", "rank", "rank", "rank"))
    if kind == "sweep":
        sessions = _log_int(rng, 3, 256)
        # bounded by the events of all simulations together
        turns = _log_int(rng, 2, 24)
        most = max(2, min(16384, 30_000_000 // (sessions * turns * 2)))
        return {"kind": kind, "sims": _log_int(rng, 2, most), "sessions": sessions, "turns": turns,
                "traces": rng.randint(1, 8), "mix": rng.choice(("pair", "four", "all"))}
    if kind == "trace":
        # 64 slots at a paper-like pool, or a pool and slot count several times as large
        scale = rng.choice((1, 3, 8, 16))
        sessions = _log_int(rng, 260, 3000)
        return {"kind": kind, "sessions": sessions, "turns": sessions * rng.randint(4, 12),
                "slots": _log_int(rng, 16, 512), "scale": scale, "mix": rng.choice(("four", "all"))}
    if kind == "study":
        study = rng.choice(STUDIES)
        return {"kind": kind, "study": study, "recip": rng.choice((0, 12, 16, 20, 24)),
                "turns": rng.randint(6000, 20000)}
    if kind == "live":
        sessions = _log_int(rng, 5000, 65536)
        return {"kind": kind, "sims": rng.randint(1, 24), "traces": rng.randint(1, 2),
                "sessions": sessions, "turns": int(sessions * rng.uniform(1.2, 2.2)),
                "slots": _log_int(rng, 500, 8192)}
    if rng.random() < 0.25:
        return {"kind": kind, "snapshots": 0, "n_per": 0, "pool": _log_int(rng, 1000, 6_000_000),
                "formats": _formats(rng, 2)}
    n_per = _log_int(rng, 2, 4096)
    most = max(4, min(10000, 30_000_000 // n_per))
    return {"kind": kind, "snapshots": _log_int(rng, 4, most), "n_per": n_per,
            "pool": _log_int(rng, max(5000, n_per), 65536), "formats": _formats(rng, rng.randint(1, 3))}


# ------------------------------------------------------------------ workloads

def _pcg(seed):
    return np.random.Generator(np.random.PCG64(seed))


def _sweep(case, seed):
    """Short traces of about `turns` turns a session; the rows run over the
    mix's policies, then traces, then capacities, hazard tables and penalties."""
    rng = _pcg(seed)
    n, ntr = case["sessions"], case["traces"]
    uniform = case["mix"] != "all"
    traces = []
    for _ in range(ntr):
        turns = np.full(n, case["turns"]) if uniform else synth.geometric_turns(rng, n, case["turns"])
        kvb = np.full(n, 128 * synth.KIB) if uniform else \
            np.array([64, 128, 160], dtype=np.uint32)[rng.permutation(n) % 3] * synth.KIB
        gaps = synth.gaps_single if uniform else synth.gaps_mixture
        traces.append(synth.build_trace(rng, turns, synth.poisson_arrivals(rng, n, 5.0), gaps, kvb))
    pops = [tr.turns for tr in traces] + [synth.hazard_population(seed + 1128, 128),
                                          synth.hazard_population(seed + 1496, 496)]
    mix = POLICY_MIXES[case["mix"]]
    sims = case["sims"]
    p = synth.default_params(sims)
    i = np.arange(sims)
    # contiguous blocks per policy (four: as a sweep script lays them out), or interleaved
    pol_i = i * len(mix) // sims if uniform else i % len(mix)
    pol = np.array([m[0] for m in mix])[pol_i]
    p["policy"] = pol
    p["score_mode"] = np.array([m[1] for m in mix])[pol_i]
    p["tide"] = np.isin(pol, (synth.POLICY_SPEAR, synth.POLICY_BELADY))
    within = i - np.ceil(pol_i * sims / len(mix)).astype(np.int64) if uniform else i // len(mix)
    per_trace = max(1, -(-sims // (len(mix) * ntr)))
    p["trace"] = np.minimum(within // per_trace, ntr - 1) if uniform else within % ntr
    cell = within % per_trace if uniform else within // ntr
    scale = max(1, n // 16)
    p["cap_sram_B"] = np.array(synth.C3_SRAM_MIB)[(cell // 64) % 8] * scale * synth.MIB
    p["cap_hbm_B"] = np.array(synth.C3_HBM_GIB)[(cell // 8) % 8] * scale * synth.GIB
    v = cell % 8
    p["lut"] = np.where(v // 2 < 2, p["trace"], ntr + (v // 2) - 2)
    pen = np.array(synth.C3_PENALTY)[v % 2]
    p["penalty_us"] = pen.astype(np.float32)
    p["p_z"] = pen.astype(np.uint64)
    p["ttl_ns"] = np.where(pol == synth.POLICY_TIMEOUT, np.array(synth.C3_TTL_S)[v], 30) * synth.NS
    return synth.Workload("sweep", traces, pops, p)


def _trace(case, seed):
    rng = _pcg(seed)
    n = case["sessions"]
    turns = synth.geometric_turns(rng, n, case["turns"] / n, total=case["turns"])
    kvb = np.array([64, 128, 160], dtype=np.uint32)[rng.permutation(n) % 3] * synth.KIB
    tr = synth.build_trace(rng, turns, synth.poisson_arrivals(rng, n, 5.0), synth.gaps_mixture, kvb)
    mix = POLICY_MIXES[case["mix"]]
    p = synth.default_params(len(mix))
    for q, (pol, mode) in enumerate(mix):
        synth.set_policy(p[q:q + 1], pol)
        p["score_mode"][q] = mode
    p["cap_sram_B"] = case["scale"] * 10_000 * 128 * synth.KIB
    p["cap_hbm_B"] = case["scale"] * 50_000 * 128 * synth.KIB
    p["n_slots"] = case["slots"]
    return synth.Workload("trace", [tr], [tr.turns], p)


def _study(case, seed):
    """The study batches on six stand-in traces of 128 to 496 sessions."""
    rng = _pcg(seed)
    share = case["turns"] / synth.FIDELITY_TURNS
    n_all = sum(synth.FIDELITY_SESSIONS)
    turns = synth.fix_total(rng, synth.lognormal_turns(rng, n_all, median=max(2.0, 16.5 * share)),
                            max(case["turns"], n_all))
    traces, at = [], 0
    for n in synth.FIDELITY_SESSIONS:
        kvb = np.array([64, 128, 160], dtype=np.uint32)[rng.permutation(n) % 3] * synth.KIB
        traces.append(synth.build_trace(rng, turns[at:at + n], synth.poisson_arrivals(rng, n, 0.2),
                                        synth.gaps_mixture, kvb))
        at += n
    study = case["study"]
    if study == "formats":
        fmts = synth.format_grid_dividers((0, case["recip"]) if case["recip"] else (0,))
        return synth.format_sweep(traces=traces, formats=fmts)[0]
    if study == "online":
        return synth.attainment_workload(traces)[0]
    if study == "components":
        return synth.component_ablation(traces)[0]
    if study == "slots":
        return synth.slot_sweep(traces)[0]
    return synth.dual_ablation(traces)[0]


def _live(case, seed):
    """All sessions arrive within a minute of `sessions` / 65,536 and stay
    live; SPEAR+TIDE over hazard tables and penalties."""
    n, ntr = case["sessions"], case["traces"]
    traces = []
    for t in range(ntr):
        rng = _pcg(seed * 1000 + t)
        turns = synth.geometric_turns(rng, n, case["turns"] / n, total=case["turns"])
        first = np.sort(rng.uniform(0.0, 60.0 * n / 65536, n))
        traces.append(synth.build_trace(rng, turns, first, synth.gaps_mixture,
                                        np.full(n, 160 * synth.KIB)))
    pops = [tr.turns for tr in traces] + [synth.hazard_population(seed + 2128, 128),
                                          synth.hazard_population(seed + 2496, 496)]
    p = synth.default_params(case["sims"])
    synth.set_policy(p, synth.POLICY_SPEAR)
    i = np.arange(case["sims"])
    p["trace"] = i % ntr
    v = (i // ntr) % 8
    p["lut"] = np.where(v // 2 < 2, p["trace"], ntr + v // 2 - 2)
    pen = np.array(synth.C3_PENALTY)[v % 2]
    p["penalty_us"] = pen.astype(np.float32)
    p["p_z"] = pen.astype(np.uint64)
    p["cap_sram_B"] = 512 * synth.MIB
    p["cap_hbm_B"] = 288 * synth.GIB
    p["n_slots"] = case["slots"]
    return synth.Workload("live", traces, pops, p)


WORKLOADS = {"sweep": _sweep, "trace": _trace, "study": _study, "live": _live}


def _parse(formats):
    return [tuple(int(v) for v in f.split("/")) for f in formats.split(",")]


def _rank_inputs(case, seed):
    """A session pool on the host: turn index, completion flag, the latest gaps."""
    rng = _pcg(seed)
    n, hist = case["pool"], 8
    turn = np.minimum(rng.geometric(1 / 23.7, n) - 1, 60).astype(np.uint8)
    done = (rng.random(n) < 0.02).astype(np.uint8)
    n_hist = np.minimum(turn, hist).astype(np.uint8)
    if n > 262_144:   # a large pool repeats drawn gaps at other places, plus whole microseconds
        base = np.rint(synth.gaps_mixture(rng, 262_144) * synth.NS).astype(np.uint64)
        gaps = base[rng.integers(0, base.size, n * hist)].reshape(n, hist)
        gaps += (rng.integers(0, 1000, n, dtype=np.uint64) * np.uint64(1000))[:, None]
    else:
        gaps = np.rint(synth.gaps_mixture(rng, n * hist) * synth.NS).astype(np.uint64).reshape(n, hist)
    gaps[np.arange(hist)[None, :] >= n_hist[:, None]] = 0
    pop = synth.lognormal_turns(_pcg(seed + 1000), 128)
    return gaps, n_hist, turn, done, pop


def _to_gpu(a):
    a = a.view({np.dtype(np.uint64): np.int64, np.dtype(np.uint32): np.int32}.get(a.dtype, a.dtype))
    return torch.from_numpy(a).to("cuda")


def prepare(case, seed):
    if case["kind"] != "rank":
        sim = U.Simulator(WORKLOADS[case["kind"]](case, seed))
        if case["kind"] in ("sweep", "live"):
            return {"sim": sim, "dev": torch.as_tensor(_Counters(sim), device="cuda")}
        return {"sim": sim}
    gaps, n_hist, turn, done, pop = (_to_gpu(a) for a in _rank_inputs(case, seed))
    st = {"formats": _parse(case["formats"]), "gaps": gaps, "n_hist": n_hist, "turn": turn,
          "done": done, "pop": pop, "idx": None}
    if case["snapshots"]:
        # each snapshot holds n_per distinct sessions of the pool
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        parts, at = [], 0
        while at < case["snapshots"]:
            k = min(128, case["snapshots"] - at)
            r = torch.rand(k, case["pool"], device="cuda", generator=g)
            parts.append(r.argsort(dim=1)[:, :case["n_per"]].to(torch.int32))
            at += k
        st["idx"] = torch.cat(parts).contiguous()
    return st


class _Counters:
    """The counters of a simulator's batch where they lie on the GPU: a row of
    25 64-bit words per simulation, the last two of them doubles."""

    def __init__(self, sim):
        self.__cuda_array_interface__ = {"shape": (sim.n_sims, U.COUNTERS_DTYPE.itemsize // 8),
                                         "typestr": "<i8", "version": 2,
                                         "data": (sim.counters_device(), False)}


def run(state):
    if "sim" in state:
        sim = state["sim"]
        sim.run()
        if "dev" in state:
            c = state["dev"]
            return {"counts": c[:, :23], "sums": c[:, 23:].view(torch.float64)}
        c = sim.counters()
        words = c.view(np.uint64).reshape(sim.n_sims, -1)
        return {"counts": words[:, :23].view(np.int64), "sums": words[:, 23:].view(np.float64)}
    d, n = U.hazard_counts(state["pop"])
    first = state["formats"][0]
    g, gq = U.ema_replay(state["gaps"], state["n_hist"], first[1], first[2])
    x = U.score_fp32(state["turn"], g, state["done"], d, n, PENALTY_US)
    out = {"g": g, "x": x}
    for k, (bh, bg, tau, recip) in enumerate(state["formats"]):
        if k and (bg, tau) != state["formats"][k - 1][1:3]:
            gq = U.ema_replay(state["gaps"], state["n_hist"], bg, tau)[1]
        y = U.score_fixed(state["turn"], gq, state["done"], d, n, bh,
                          int(round(PENALTY_US * 1000 / tau)), recip)
        out["y%d" % k] = y
        if state["idx"] is not None:
            out["counts%d" % k], out["top1_%d" % k] = U.kendall(x, y, state["idx"])
    return out


# ------------------------------------------------------------------- measures

def _shape(case):
    """(simulated events of one run, events of the traces, sessions, simulations)."""
    kind = case["kind"]
    if kind == "sweep":
        ev = 2 * case["sessions"] * case["turns"]
        return ev * case["sims"], ev * case["traces"], case["sessions"] * case["traces"], case["sims"]
    if kind == "trace":
        ev, sims = 2 * case["turns"], len(POLICY_MIXES[case["mix"]])
        return ev * sims, ev, case["sessions"], sims
    if kind == "live":
        ev = 2 * case["turns"]
        return ev * case["sims"], ev * case["traces"], case["sessions"] * case["traces"], case["sims"]
    sims = {"formats": 18 * (1 + 27 * (2 if case["recip"] else 1)), "online": 128,
            "components": 216, "slots": 42, "dual": 24}[case["study"]]
    ev = 2 * case["turns"]
    return ev * sims // 6, ev, sum(synth.FIDELITY_SESSIONS), sims


def work(case):
    if case["kind"] != "rank":
        events, trace_events, sessions, sims = _shape(case)
        # each trace's 36-byte events and sessions, the parameter rows and the
        # counters once; per simulated event its EMA and its score
        return {"bytes": 36 * trace_events + 4 * sessions + (144 + 200) * sims, "flops": 10 * events}
    pool, nf = case["pool"], len(_parse(case["formats"]))
    n, m = case["snapshots"], case["n_per"]
    # gap histories, turn and done once, g and x written, an integer score per
    # format; per snapshot and format the pairs' order: m log2 m comparisons of
    # both rankings
    return {"bytes": pool * (8 * 8 + 3 + 8 + 8 * nf) + 4 * n * m + nf * n * 41,
            "flops": pool * (8 * 8 + 10) + nf * n * m * max(1.0, np.log2(max(m, 2))) * 2}


def tolerance(case):
    return "exact"


def exact(case, seed):
    """The gap EMA and the SPEAR score of the pool in 64 bits; integer outputs
    are exact by definition, and a simulation's sums follow from its decisions."""
    if case["kind"] != "rank":
        return None
    gaps, n_hist, turn, done, pop = _rank_inputs(case, seed)
    us = np.minimum(gaps // np.uint64(1000), np.uint64(0xFFFFFFFF)).astype(np.float64)
    g = np.zeros(case["pool"])
    for k in range(us.shape[1]):
        g = np.where(k < n_hist, (3.0 * us[:, k] + 7.0 * g) / 10.0, g)
    t = np.arange(51)
    d = (pop[None, :] == t[:, None] + 1).sum(axis=1)
    n = (pop[None, :] > t[:, None]).sum(axis=1)
    h = np.where(n > 0, d / np.maximum(n, 1), 0.0)
    sigma = np.maximum(0.01, 1.0 - h)[np.minimum(turn, 50)]
    x = np.where(done > 0, np.inf, g / sigma + (1.0 - sigma) * PENALTY_US)
    return {"g": g, "x": x}
