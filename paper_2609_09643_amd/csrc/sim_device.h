// sim_device.h -- what the simulation kernels share (gfx950): cross-lane
// moves and wavefront reductions, the policies' keys, event records, the
// per-simulation state and counters, and the hazard table in LDS.
#pragma once

#include "unison_device.h"

#pragma clang fp contract(off)

namespace unison {

// ------------------------------------------------------- cross-lane moves

// Every pattern used here reads a lane of the same row, so no lane needs a
// fallback value (mov_dpp leaves the destination's old value unspecified).
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}

// Partner value for butterfly step M.  Before step M every aligned block of
// M lanes holds one value; the partner lane lies in the sibling block.
template <int M>
__device__ __forceinline__ uint32_t xchg(uint32_t v) {
  if constexpr (M == 1) return dpp<0xB1>(v);   // quad_perm [1,0,3,2]
  else if constexpr (M == 2) return dpp<0x4E>(v);  // quad_perm [2,3,0,1]
  else if constexpr (M == 4) return dpp<0x141>(v);  // row_half_mirror
  else if constexpr (M == 8) return dpp<0x140>(v);  // row_mirror
  else if constexpr (M == 16) return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, 0x401F);  // xor 16
  else return (uint32_t)__shfl_xor((int)v, 32);
}

struct Cand {
  uint64_t key;
  uint32_t sid;
};

__device__ __forceinline__ bool max_better(uint64_t ka, uint32_t sa, uint64_t kb, uint32_t sb) {
  return ka > kb || (ka == kb && sa < sb);
}
__device__ __forceinline__ bool min_better(uint64_t ka, uint32_t sa, uint64_t kb, uint32_t sb) {
  return ka < kb || (ka == kb && sa < sb);
}
__device__ __forceinline__ Cand cand_none_max() { return Cand{0ull, kNone}; }
__device__ __forceinline__ Cand cand_none_min() { return Cand{~0ull, kNone}; }

// Max (MAX) or min of a 32-bit value over each aligned group of W lanes;
// every lane of the group ends with it.
template <int W, int M, bool MAX>
__device__ __forceinline__ uint32_t group_ext32(uint32_t v) {
  if constexpr (M < W) {
    const uint32_t o = xchg<M>(v);
    return group_ext32<W, M * 2, MAX>(MAX ? (o > v ? o : v) : (o < v ? o : v));
  } else {
    return v;
  }
}

// Max (MAX) or min of a packed 64-bit value over each aligned group of W
// lanes, as two 32-bit words, most significant first: the group's best high
// word, then the best low word among the lanes that hold it (the others enter
// the empty value).  Each word's step is one max or min with a lane permute,
// which the compiler folds into one DPP instruction, where a 64-bit step
// needs two permutes, a compare and two selects.
template <int W, bool MAX>
__device__ __forceinline__ uint64_t reduce_words(uint64_t c) {
  const uint32_t hi = (uint32_t)(c >> 32);
  const uint32_t h = group_ext32<W, 1, MAX>(hi);
  const uint32_t lo = hi == h ? (uint32_t)c : (MAX ? 0u : ~0u);
  return ((uint64_t)h << 32) | group_ext32<W, 1, MAX>(lo);
}

template <int W, int M>
__device__ __forceinline__ uint32_t reduce_min32(uint32_t c) {
  if constexpr (M < W) {
    const uint32_t o = xchg<M>(c);
    return reduce_min32<W, M * 2>(o < c ? o : c);
  } else {
    return c;
  }
}

// Every lane of an aligned group of W lanes ends with the winner (ties to
// the smaller session id): the key's two words, most significant first, then
// the smallest id among the lanes still tied, each over the lanes that hold
// the best word so far (the others enter the empty value).
template <int W, bool MAX>
__device__ __forceinline__ Cand reduce_group(Cand c) {
  const uint32_t empty = MAX ? 0u : ~0u;
  const uint32_t khi = (uint32_t)(c.key >> 32), klo = (uint32_t)c.key;
  const uint32_t h = group_ext32<W, 1, MAX>(khi);
  const bool tied = khi == h;
  const uint32_t l = group_ext32<W, 1, MAX>(tied ? klo : empty);
  const uint32_t s = group_ext32<W, 1, false>(tied && klo == l ? c.sid : ~0u);
  return Cand{((uint64_t)h << 32) | l, s};
}

// Whole-wavefront max (MAX) or min of a 32-bit value, uniform: a DPP
// butterfly inside each row of 16 lanes, then the four row results compared
// in scalar registers (no cross-row permute through the LDS crossbar).
template <bool MAX>
__device__ __forceinline__ uint32_t ext32(uint32_t a, uint32_t b) {
  return MAX ? (a > b ? a : b) : (a < b ? a : b);
}
template <bool MAX>
__device__ __forceinline__ uint32_t wave_ext32(uint32_t v) {
  v = ext32<MAX>(v, xchg<1>(v));
  v = ext32<MAX>(v, xchg<2>(v));
  v = ext32<MAX>(v, xchg<4>(v));
  v = ext32<MAX>(v, xchg<8>(v));
  const uint32_t r0 = (uint32_t)__builtin_amdgcn_readlane((int)v, 0);
  const uint32_t r1 = (uint32_t)__builtin_amdgcn_readlane((int)v, 16);
  const uint32_t r2 = (uint32_t)__builtin_amdgcn_readlane((int)v, 32);
  const uint32_t r3 = (uint32_t)__builtin_amdgcn_readlane((int)v, 48);
  return ext32<MAX>(ext32<MAX>(r0, r1), ext32<MAX>(r2, r3));
}
// One phase of a lexicographic wavefront reduction over N words per lane:
// the best word M among the active ones; with NARROW, a word stays active
// only where it equals M, so the next phase breaks the ties.
template <bool MAX, bool NARROW, int N>
__device__ __forceinline__ uint32_t lex_phase(const uint32_t (&w)[N], bool (&act)[N]) {
  uint32_t v = MAX ? 0u : ~0u;
#pragma unroll
  for (int k = 0; k < N; ++k) v = act[k] ? ext32<MAX>(v, w[k]) : v;
  const uint32_t m = wave_ext32<MAX>(v);
  if constexpr (NARROW) {
#pragma unroll
    for (int k = 0; k < N; ++k) act[k] = act[k] && w[k] == m;
  }
  return m;
}

// Sum mod 2^64 over the wavefront; every lane ends with it.
__device__ __forceinline__ uint64_t wave_sum64_step(uint64_t v, uint32_t lo, uint32_t hi) {
  return v + (((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ uint64_t wave_sum64(uint64_t v) {
  v = wave_sum64_step(v, xchg<1>((uint32_t)v), xchg<1>((uint32_t)(v >> 32)));
  v = wave_sum64_step(v, xchg<2>((uint32_t)v), xchg<2>((uint32_t)(v >> 32)));
  v = wave_sum64_step(v, xchg<4>((uint32_t)v), xchg<4>((uint32_t)(v >> 32)));
  v = wave_sum64_step(v, xchg<8>((uint32_t)v), xchg<8>((uint32_t)(v >> 32)));
  v = wave_sum64_step(v, xchg<16>((uint32_t)v), xchg<16>((uint32_t)(v >> 32)));
  v = wave_sum64_step(v, xchg<32>((uint32_t)v), xchg<32>((uint32_t)(v >> 32)));
  return v;
}

// Pins a value to a vector register.  A workgroup-per-simulation kernel keeps
// its long-lived per-simulation state (pool usage, counters) there: held in
// scalar registers it would exceed them and spill on every event.
__device__ __forceinline__ uint32_t in_vgpr(uint32_t v) {
  asm volatile("" : "+v"(v));
  return v;
}
__device__ __forceinline__ uint64_t in_vgpr(uint64_t v) {
  return ((uint64_t)in_vgpr((uint32_t)(v >> 32)) << 32) | in_vgpr((uint32_t)v);
}
__device__ __forceinline__ double in_vgpr(double v) {
  return __longlong_as_double((long long)in_vgpr((uint64_t)__double_as_longlong(v)));
}

__device__ __forceinline__ uint32_t uni32(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}
__device__ __forceinline__ uint64_t uni64(uint64_t v) {
  return ((uint64_t)uni32((uint32_t)(v >> 32)) << 32) | uni32((uint32_t)v);
}
// A condition every lane of the wavefront evaluates alike (UNI), as a scalar
// branch condition: values pinned to vector registers would otherwise make
// the compiler treat the branch as divergent (exec masking, merges of every
// live value at the join).
template <bool UNI>
__device__ __forceinline__ bool uc(bool c) {
  if constexpr (UNI) return __builtin_amdgcn_ballot_w64(c) != 0ull;
  else return c;
}

// ------------------------------------------------------------ keys

template <uint32_t POL, uint32_t SMODE>
struct Pol {
  static constexpr bool spear = POL == kSpear;
  static constexpr bool fixed = spear && SMODE == 1;
  static constexpr bool belady = POL == kBelady;
  static constexpr bool eta = POL == kEta;
  // the key is the session's next arrival: true (Belady) or predicted (ETA)
  static constexpr bool nextkey = belady || eta;
  static constexpr bool timeout = POL == kTimeout;
  static constexpr bool recency = POL == kLru || POL == kTimeout;
  static constexpr bool has_inf = spear || nextkey;
  static constexpr uint64_t inf_key = (spear && !fixed) ? 0x7F800000ull : ~0ull;
};

// The simulation's hazard table lives in LDS: its counts d(t), n(t) of
// eq. (hazard) and both derived forms, h as fp32 and h_q (eq. (hq)).  An
// online table (online_cap > 0) grows by one session at each of the first
// online_cap completions.
struct KeyCtx {
  float* hf;            // LDS [52]
  uint32_t* hq;         // LDS [52]
  uint32_t* hd;         // LDS [52]
  uint32_t* hn;         // LDS [52]
  float P;
  uint32_t lambda;
  uint64_t p_z;
  bool pack44;          // times fit 44 bits and ids 20 bits: recency / Belady keys pack
  uint32_t online_cap;  // completions an online table still may count; 0: fixed table
  const uint64_t* eta;  // the trace's ETA table: expected wait per tool class, ns (global)
  uint32_t recip_bits;  // eq. (t1) by a reciprocal of this many fraction bits; 0: exact
};

// Adds a completed session of Tn turns to the counts (n(t) += 1 for t < Tn,
// d(Tn - 1) += 1) and rebuilds the entries it changed; t is split over
// `width` cooperating lanes starting at `lane`.
__device__ __forceinline__ void hazard_add_counts(const KeyCtx& K, uint32_t Tn, uint32_t lane,
                                                  uint32_t width) {
  for (uint32_t t = lane; t < kLut; t += width) {
    const uint32_t dn = t < Tn ? 1u : 0u;
    const uint32_t dd = t + 1u == Tn ? 1u : 0u;
    if (dn | dd) {
      const uint32_t d = K.hd[t] + dd;
      const uint32_t n = K.hn[t] + dn;
      K.hd[t] = d;
      K.hn[t] = n;
      K.hf[t] = hazard_f32(d, n);
      K.hq[t] = hazard_q(d, n, K.lambda);
    }
  }
}

// The hazard entry eq. (hazard) / eq. (hq) of a session at turn index t
// (clamped to 50): fp32 bits of h for the fp32 score, h_q for the integer one.
template <uint32_t POL, uint32_t SMODE>
__device__ __forceinline__ uint32_t hazard_of(const KeyCtx& K, uint32_t meta) {
  using PT = Pol<POL, SMODE>;
  if constexpr (PT::spear) {
    uint32_t t = meta_turn(meta);
    t = t < 50u ? t : 50u;
    return PT::fixed ? K.hq[t] : __float_as_uint(K.hf[t]);
  } else {
    return 0u;
  }
}

// "Larger key = evict first".  SPEAR: the score (eq. (esp) or eq. (scoreq))
// from the entry's hazard value hz (hazard_of); completed sessions take
// S_max.  LRU / timeout: older last event first.  Belady: later next arrival
// first.
template <uint32_t POL, uint32_t SMODE>
__device__ __forceinline__ uint64_t key_of(const KeyCtx& K, uint32_t meta, uint32_t hz, float g,
                                           uint64_t gq, uint64_t last, uint64_t next) {
  using PT = Pol<POL, SMODE>;
  if constexpr (PT::spear) {
    const bool done = meta_phase(meta) == kDoneP;
    if constexpr (PT::fixed) {
      const uint64_t s = spear_fixed(hz, gq, K.lambda, K.p_z, K.recip_bits);
      return done ? ~0ull : s;
    } else {
      const float s = spear_f32(__uint_as_float(hz), g, K.P);
      return done ? 0x7F800000ull : (uint64_t)__float_as_uint(s);
    }
  } else if constexpr (PT::nextkey) {
    return next;
  } else {
    return ~0ull - last;
  }
}

// A session's timer has fired (now - last > ttl) exactly when last lies below
// this threshold: last never exceeds now, and nothing fires while now <= ttl.
__device__ __forceinline__ uint64_t idle_threshold(uint64_t now, uint64_t ttl) {
  return now > ttl ? now - ttl : 0ull;
}

struct Entry {
  uint32_t meta;
  float g;
  uint64_t gq;
  uint32_t len;
  uint32_t kvb;
  uint64_t last;
  uint64_t next;
};

struct TraceView {
  const uint64_t* t;
  const uint32_t* sid;
  const uint32_t* info;
  const uint32_t* len;
  const uint64_t* next;
  const uint32_t* tool;  // or null: every gap is tool class 0
  uint64_t n_ev;
  uint32_t n_sess;
};

struct Ev {
  uint64_t t;
  uint32_t sid, info, len, tool;
  uint64_t next;
};

// The event record; the next arrival only where the key reads it (Belady),
// the tool class only where it predicts one (ETA).
template <bool NEXT, bool TOOL>
__device__ __forceinline__ Ev load_ev(const TraceView& tr, uint64_t e) {
  Ev v;
  v.t = tr.t[e];
  v.sid = tr.sid[e];
  v.info = tr.info[e];
  v.len = tr.len[e];
  v.next = NEXT ? tr.next[e] : ~0ull;
  v.tool = (TOOL && tr.tool) ? tr.tool[e] : 0u;
  return v;
}

// ------------------------------------------------------------- state and counters

struct Scalars {
  uint64_t used_s, used_h, dma_free_at, prev_t, log_len;
  uint32_t n_res, n_table, hi;
  uint64_t hit_s_bytes, hit_h_bytes, miss_tok, prev_s_bytes, prev_h_bytes;
};

// Counters as kept during a run: event-bounded counts in 32 bits.
struct Cnt {
  uint32_t requests, hit_sram, hit_hbm, miss, bypass, evict, expire, promote, swap, tide_passes,
      events, prefetch_hits, vict_diff, prom_diff;
  uint64_t dma_bytes, tokens_total, tokens_computed, extra_prefill, score_evals, resident_evals,
      digest, victim_digest, error;
  double amat, ttft;
};

__device__ __forceinline__ Cnt cnt_from(const unison_counters& c) {
  Cnt k;
  k.requests = (uint32_t)c.requests;
  k.hit_sram = (uint32_t)c.hit_sram;
  k.hit_hbm = (uint32_t)c.hit_hbm;
  k.miss = (uint32_t)c.miss;
  k.bypass = (uint32_t)c.bypass;
  k.evict = (uint32_t)c.evict;
  k.expire = (uint32_t)c.expire;
  k.promote = (uint32_t)c.promote;
  k.swap = (uint32_t)c.swap;
  k.tide_passes = (uint32_t)c.tide_passes;
  k.events = (uint32_t)c.events;
  k.prefetch_hits = (uint32_t)c.prefetch_hits;
  k.vict_diff = (uint32_t)c.vict_diff;
  k.prom_diff = (uint32_t)c.prom_diff;
  k.dma_bytes = c.dma_bytes;
  k.tokens_total = c.tokens_total;
  k.tokens_computed = c.tokens_computed;
  k.extra_prefill = c.extra_prefill_tok;
  k.score_evals = c.score_evals;
  k.resident_evals = c.resident_evals;
  k.digest = c.digest;
  k.victim_digest = c.victim_digest;
  k.error = c.error;
  k.amat = c.amat_sum_ns;
  k.ttft = c.ttft_sum_ns;
  return k;
}

__device__ __forceinline__ unison_counters cnt_to(const Cnt& k) {
  unison_counters c;
  c.requests = k.requests;
  c.hit_sram = k.hit_sram;
  c.hit_hbm = k.hit_hbm;
  c.miss = k.miss;
  c.bypass = k.bypass;
  c.evict = k.evict;
  c.expire = k.expire;
  c.promote = k.promote;
  c.swap = k.swap;
  c.dma_bytes = k.dma_bytes;
  c.tide_passes = k.tide_passes;
  c.tokens_total = k.tokens_total;
  c.tokens_computed = k.tokens_computed;
  c.extra_prefill_tok = k.extra_prefill;
  c.score_evals = k.score_evals;
  c.resident_evals = k.resident_evals;
  c.digest = k.digest;
  c.victim_digest = k.victim_digest;
  c.events = k.events;
  c.error = k.error;
  c.prefetch_hits = k.prefetch_hits;
  c.vict_diff = k.vict_diff;
  c.prom_diff = k.prom_diff;
  c.amat_sum_ns = k.amat;
  c.ttft_sum_ns = k.ttft;
  return c;
}

__device__ __forceinline__ void pin_vgpr(Scalars& S) {
  S.used_s = in_vgpr(S.used_s);
  S.used_h = in_vgpr(S.used_h);
  S.dma_free_at = in_vgpr(S.dma_free_at);
  S.prev_t = in_vgpr(S.prev_t);
  S.log_len = in_vgpr(S.log_len);
  S.n_res = in_vgpr(S.n_res);
  S.n_table = in_vgpr(S.n_table);
  S.hi = in_vgpr(S.hi);
  S.hit_s_bytes = in_vgpr(S.hit_s_bytes);
  S.hit_h_bytes = in_vgpr(S.hit_h_bytes);
  S.miss_tok = in_vgpr(S.miss_tok);
  S.prev_s_bytes = in_vgpr(S.prev_s_bytes);
  S.prev_h_bytes = in_vgpr(S.prev_h_bytes);
}

__device__ __forceinline__ void pin_vgpr(unison_sim_params& p) {
  p.tide = in_vgpr(p.tide);
  p.cap_sram_B = in_vgpr(p.cap_sram_B);
  p.cap_hbm_B = in_vgpr(p.cap_hbm_B);
  p.n_slots = in_vgpr(p.n_slots);
  p.dma_B_per_us = in_vgpr(p.dma_B_per_us);
  p.ttl_ns = in_vgpr(p.ttl_ns);
  p.b_g = in_vgpr(p.b_g);
  p.tau_ns = in_vgpr(p.tau_ns);
}

__device__ __forceinline__ void pin_vgpr(Cnt& k) {
  k.requests = in_vgpr(k.requests);
  k.hit_sram = in_vgpr(k.hit_sram);
  k.hit_hbm = in_vgpr(k.hit_hbm);
  k.miss = in_vgpr(k.miss);
  k.bypass = in_vgpr(k.bypass);
  k.evict = in_vgpr(k.evict);
  k.expire = in_vgpr(k.expire);
  k.promote = in_vgpr(k.promote);
  k.swap = in_vgpr(k.swap);
  k.tide_passes = in_vgpr(k.tide_passes);
  k.events = in_vgpr(k.events);
  k.prefetch_hits = in_vgpr(k.prefetch_hits);
  k.vict_diff = in_vgpr(k.vict_diff);
  k.prom_diff = in_vgpr(k.prom_diff);
  k.dma_bytes = in_vgpr(k.dma_bytes);
  k.tokens_total = in_vgpr(k.tokens_total);
  k.tokens_computed = in_vgpr(k.tokens_computed);
  k.extra_prefill = in_vgpr(k.extra_prefill);
  k.score_evals = in_vgpr(k.score_evals);
  k.resident_evals = in_vgpr(k.resident_evals);
  k.digest = in_vgpr(k.digest);
  k.victim_digest = in_vgpr(k.victim_digest);
  k.error = in_vgpr(k.error);
  k.amat = in_vgpr(k.amat);
  k.ttft = in_vgpr(k.ttft);
}

struct LogSink {
  bool on;             // logging requested (a launch-wide, uniform flag)
  unison_record* rec;  // this simulation's records
  uint32_t cap;
  bool lead;           // the one lane that stores records
  bool victims;        // also record each event's scan result
};

// The simulation's hazard table into LDS: the counts of its fixed table, or
// of its online table so far (none on a fresh run), and h in both forms.
__device__ __forceinline__ void load_hazard(const SimArgs& a, const unison_sim_params& P,
                                            uint32_t sim, const KeyCtx& K, uint32_t lane,
                                            uint32_t width) {
  const bool online = P.hazard_online != 0;
  const bool fresh = online && !(a.flags & UNISON_RUN_CONTINUE);
  const uint32_t* kd = online ? a.hcount + (size_t)sim * 2 * kLut : a.lut_d + (size_t)P.lut * kLut;
  const uint32_t* kn = online ? kd + kLut : a.lut_n + (size_t)P.lut * kLut;
  for (uint32_t t = lane; t < kLut; t += width) {
    const uint32_t d = fresh ? 0u : kd[t];
    const uint32_t n = fresh ? 0u : kn[t];
    K.hd[t] = d;
    K.hn[t] = n;
    K.hf[t] = hazard_f32(d, n);
    K.hq[t] = hazard_q(d, n, K.lambda);
  }
}

// An online table's counts at the end of the launch, for a later CONTINUE
// and for unison_read_hazard (a fixed table never changes: nothing to store).
__device__ __forceinline__ void store_hazard(const SimArgs& a, const unison_sim_params& P,
                                             uint32_t sim, const KeyCtx& K, uint32_t lane,
                                             uint32_t width) {
  if (!P.hazard_online) return;
  uint32_t* out = a.hcount + (size_t)sim * 2 * kLut;
  for (uint32_t t = lane; t < kLut; t += width) {
    out[t] = K.hd[t];
    out[kLut + t] = K.hn[t];
  }
}

__device__ __forceinline__ void load_scalars(const SimState& st, Scalars& S) {
  S.used_s = st.used_s;
  S.used_h = st.used_h;
  S.dma_free_at = st.dma_free_at;
  S.prev_t = st.prev_t;
  S.log_len = st.log_len;
  S.n_res = st.n_res;
  S.n_table = st.n_table;
  S.hi = st.hi;
  S.hit_s_bytes = st.hit_s_bytes;
  S.hit_h_bytes = st.hit_h_bytes;
  S.miss_tok = st.miss_tok;
  S.prev_s_bytes = st.prev_s_bytes;
  S.prev_h_bytes = st.prev_h_bytes;
}

__device__ __forceinline__ void store_scalars(SimState& st, const Scalars& S, uint64_t next_event) {
  st.next_event = next_event;
  st.used_s = S.used_s;
  st.used_h = S.used_h;
  st.dma_free_at = S.dma_free_at;
  st.prev_t = S.prev_t;
  st.log_len = S.log_len;
  st.n_res = S.n_res;
  st.n_table = S.n_table;
  st.hi = S.hi;
  st.hit_s_bytes = S.hit_s_bytes;
  st.hit_h_bytes = S.hit_h_bytes;
  st.miss_tok = S.miss_tok;
  st.prev_s_bytes = S.prev_s_bytes;
  st.prev_h_bytes = S.prev_h_bytes;
}

// eq. (hr-amat) sums from the exact integer totals, rounded once: the same
// quantities the per-request f64 sums approximate.
__device__ __forceinline__ void finish_costs(const Scalars& S, const unison_sim_params& P, Cnt& C) {
  const double a = (double)S.hit_s_bytes * P.t_s_ns_per_B;
  const double b = (double)S.hit_h_bytes * P.t_h_ns_per_B;
  const double c = (double)S.miss_tok * P.t_p_ns_per_tok;
  C.amat = (a + b) + c;
  const double d = (double)S.prev_s_bytes * P.t_s_ns_per_B;
  const double f = (double)S.prev_h_bytes * P.t_h_ns_per_B;
  const double h = (double)C.tokens_computed * P.t_p_ns_per_tok;
  C.ttft = (d + f) + h;
}

__device__ __forceinline__ uint32_t sim_policy(const SimArgs& a, const unison_sim_params& P) {
  return a.policy_override == UNISON_POLICY_PARAMS ? P.policy : a.policy_override;
}

}  // namespace unison
