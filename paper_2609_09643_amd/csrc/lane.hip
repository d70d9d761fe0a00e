// lane.hip -- one wavefront per simulation with the residents sorted across
// its lanes (gfx950).
//
// What bounds a single simulation is the chain of dependent instructions of
// one event after the other, at about 8 cycles each for a lone wavefront.  So
// everything about an event that does not depend on the pool leaves that
// chain: a window of 64 events is prepared with one event per lane (the gap
// EMAs of eq. (ema) and eq. (ema-int) along each session's events, the keys,
// the KV sizes, the TIDE budgets of eq. (budget)), from table entries gathered
// one window ahead, and what an event only reports (hits, tokens, bytes, its
// scan victim) is noted in its lane and summed 64 events at a time.
//
// The chain that is left works on residents that are kept in victim order:
// position i of the order sits in lane i % 64 of register i / 64, as (key,
// session, slot, tier).  The scan victim of an event is position 0, TIDE's
// candidates are the last HBM and the first SRAM position, and one comparison
// per register finds where a key belongs; entries move over by one lane with
// a whole-wavefront DPP shift.  A session being served is no candidate
// (Alg. 1), so it only holds its slot (id, KV bytes, flags).
//
// Every branch of the chain is uniform and every loop in it has one exit (a
// divergent branch, or a loop left from two places, makes the compiler
// linearise the control flow around it, with copies of all live state at every
// join); decision records are queued in LDS and hashed 64 at a time outside it.
//
// Measured (67,192 events, 1,415 sessions, 64 slots): 0.48 us per event under
// SPEAR+TIDE and 0.33 under LRU, about 1,080 and 735 cycles in the chain and 60
// in the window's preparation, against 1.28 for residents in unsorted register
// slots with three wavefront reductions per event and the table in LDS.
// Above 256 residents the order moves to sorted lists in LDS (ListSim).
// 128 VGPRs keep four wavefronts on a SIMD: with 200 (sums and window
// constants in registers) 4,096 simulations of 16 sessions took 225 us, now 167.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "list_entry.h"
#include "sim_device.h"

#pragma clang fp contract(off)

// Writes one lane of a register (v_writelane_b32): clang has the instruction as
// an LLVM intrinsic only.
extern "C" __device__ __attribute__((const)) int unison_writelane(int v, int lane, int old) __asm(
    "llvm.amdgcn.writelane.i32");

namespace unison {

namespace {

__device__ __forceinline__ uint32_t rl(uint32_t v, uint32_t l) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)l);
}
__device__ __forceinline__ uint64_t rl(uint64_t v, uint32_t l) {
  return ((uint64_t)rl((uint32_t)(v >> 32), l) << 32) | rl((uint32_t)v, l);
}
__device__ __forceinline__ uint32_t wl(uint32_t old, uint32_t l, uint32_t v) {
  return (uint32_t)unison_writelane((int)v, (int)l, (int)old);
}
__device__ __forceinline__ uint64_t wl(uint64_t old, uint32_t l, uint64_t v) {
  return ((uint64_t)wl((uint32_t)(old >> 32), l, (uint32_t)(v >> 32)) << 32) |
         wl((uint32_t)old, l, (uint32_t)v);
}
// Lane i takes lane i + 1's value (lane 63: 0), or lane i - 1's (lane 0: 0).
__device__ __forceinline__ uint32_t from_above(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x130, 0xF, 0xF, true);
}
__device__ __forceinline__ uint32_t from_below(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x138, 0xF, 0xF, true);
}
__device__ __forceinline__ uint64_t from_above(uint64_t v) {
  return ((uint64_t)from_above((uint32_t)(v >> 32)) << 32) | from_above((uint32_t)v);
}
__device__ __forceinline__ uint64_t from_below(uint64_t v) {
  return ((uint64_t)from_below((uint32_t)(v >> 32)) << 32) | from_below((uint32_t)v);
}
// Lane i takes lane i ^ M's value, for the M that a sorting network asks for.
template <int M>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v) {
  if constexpr (M == 1) return dpp<0xB1>(v);         // quad_perm [1,0,3,2]
  else if constexpr (M == 2) return dpp<0x4E>(v);    // quad_perm [2,3,0,1]
  else if constexpr (M == 3) return dpp<0x1B>(v);    // quad_perm [3,2,1,0]
  else if constexpr (M == 4) return dpp<0x1B>(dpp<0x141>(v));
  else if constexpr (M == 7) return dpp<0x141>(v);   // row_half_mirror
  else if constexpr (M == 8) return dpp<0x141>(dpp<0x140>(v));
  else if constexpr (M == 15) return dpp<0x140>(v);  // row_mirror
  else if constexpr (M < 32) return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, (M << 10) | 0x1F);
  else return (uint32_t)__shfl_xor((int)v, M);
}
template <int M>
__device__ __forceinline__ uint64_t lane_xor(uint64_t v) {
  return ((uint64_t)lane_xor<M>((uint32_t)(v >> 32)) << 32) | lane_xor<M>((uint32_t)v);
}
// Lane l's value, l per lane.
__device__ __forceinline__ uint32_t from_lane(uint32_t v, uint32_t l) { return (uint32_t)__shfl((int)v, (int)l); }
__device__ __forceinline__ uint64_t from_lane(uint64_t v, uint32_t l) {
  return ((uint64_t)from_lane((uint32_t)(v >> 32), l) << 32) | from_lane((uint32_t)v, l);
}
__device__ __forceinline__ uint64_t ballot(bool c) { return __builtin_amdgcn_ballot_w64(c); }
__device__ __forceinline__ uint32_t pop64(uint64_t m) { return (uint32_t)__builtin_popcountll(m); }

// Orders the wavefront's own memory accesses before and after this point.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 1 when a <= b, else 0, for uniform values in scalar registers (gfx950 has no
// scalar 64-bit order comparison; the compiler would go through vector
// registers).
__device__ __forceinline__ uint32_t le64(uint64_t a, uint64_t b) {
  uint32_t r;
  asm("s_sub_u32 %0, %3, %1\n\ts_subb_u32 %0, %4, %2\n\ts_cselect_b32 %0, 0, 1"
      : "=&s"(r)
      : "s"((uint32_t)a), "s"((uint32_t)(a >> 32)), "s"((uint32_t)b), "s"((uint32_t)(b >> 32))
      : "scc");
  return r;
}
// The same wherever the values are: the list pool's bytes may sit in vector
// registers, which the scalar form's operands cannot.
__device__ __forceinline__ uint32_t le_u64(uint64_t a, uint64_t b) { return a <= b ? 1u : 0u; }
// The lowest set bit's index, kNone for none.
__device__ __forceinline__ uint32_t first_set(uint64_t m) {
  uint32_t r;
  asm("s_ff1_i32_b64 %0, %1" : "=s"(r) : "s"(m));
  return r;
}
// The highest set bit's index, kNone for none.
__device__ __forceinline__ uint32_t last_set(uint64_t m) {
  uint32_t r;
  asm("s_flbit_i32_b64 %0, %1" : "=s"(r) : "s"(m));
  return r == kNone ? kNone : 63u - r;
}

// n / b for a divisor known in advance: inv = floor((2^64 - 1) / b), one high
// product and at most two corrections (the estimate falls short by at most 2).
__device__ __forceinline__ uint64_t div_by(uint64_t n, uint64_t b, uint64_t inv) {
  uint64_t q = __umul64hi(n, inv);
  uint64_t r = n - q * b;
  if (r >= b) { ++q; r -= b; }
  if (r >= b) ++q;
  return q;
}

// What only a window's preparation uses of the launch's constants, one word per
// lane of a register: held in scalar registers, they would make the chain spill
// at every event; a window reads them back with one instruction a word.
struct Consts {
  uint32_t v;
  __device__ __forceinline__ void put(uint32_t i, uint32_t x) { v = wl(v, i, x); }
  __device__ __forceinline__ void put(uint32_t i, uint64_t x) {
    put(i, (uint32_t)x);
    put(i + 1, (uint32_t)(x >> 32));
  }
  template <class T>
  __device__ __forceinline__ void put(uint32_t i, const T* p) { put(i, (uint64_t)p); }
  __device__ __forceinline__ uint32_t u32(uint32_t i) const { return rl(v, i); }
  __device__ __forceinline__ uint64_t u64(uint32_t i) const {
    return ((uint64_t)rl(v, i + 1) << 32) | rl(v, i);
  }
  template <class T>
  __device__ __forceinline__ T* ptr(uint32_t i) const {
    typedef __attribute__((address_space(1))) T G;
    return (T*)(G*)u64(i);
  }
  // The words may not be kept in scalar registers from one window to the next.
  __device__ __forceinline__ void fresh() { asm volatile("" : "+v"(v)); }
};
enum : uint32_t {
  kCMg = 0, kCGq = 2, kCLast = 4, kCNext = 6, kCLen = 8, kCKvb = 10, kCEvT = 12, kCEvNext = 14,
  kCEvSid = 16, kCEvInfo = 18, kCEvLen = 20, kCEvTool = 22, kCEta = 24, kCLog = 26, kCDma = 28,
  kCDmaInv = 30, kCTau = 32, kCTtl = 34, kCPz = 36, kCEnd = 38, kCLambda = 40, kCRecip, kCP, kCBg,
  kCLogCap, kCIdBits, kCHasTool, kCDual, kCView = 48, kCStride = 50, kCSync = 52, kCReq = 54
};

// Queued records: the chain stops for a flush once kQueueFlush are waiting,
// and one event adds at most its scan victim, a record per resident that
// expires or is evicted, its own placement and two per resident that TIDE
// promotes or swaps (a session TIDE moved up stays up for the pass).
constexpr uint32_t kQueueFlush = 64;
constexpr uint32_t queue_entries(uint32_t residents) { return kQueueFlush + 2u + 4u * residents; }

// hazard_add_counts over one wavefront without a divergent branch: lanes from
// 51 on rewrite the tables' unused 52nd entry.
__device__ __forceinline__ void add_completion(const KeyCtx& K, uint32_t Tn, uint32_t lane) {
  const uint32_t t = lane < kLut ? lane : kLut;
  const uint32_t d = t < kLut ? K.hd[t] + (t + 1u == Tn ? 1u : 0u) : 0u;
  const uint32_t n = t < kLut ? K.hn[t] + (t < Tn ? 1u : 0u) : 0u;
  K.hd[t] = d;
  K.hn[t] = n;
  K.hf[t] = hazard_f32(d, n);
  K.hq[t] = hazard_q(d, n, K.lambda);
  wave_sync();
}

// One window's events as loaded, an event per lane.
struct EvRegs {
  uint64_t t, next;
  uint32_t sid, info, len, tool;
};
// The table entries of a window's sessions.
struct TabRegs {
  uint64_t mg, gq, last;
  uint32_t len, kvb;
};
// The dual design's copies of them, the index of the session's latest event
// and the live table's next arrival.
struct CopyRegs {
  uint64_t gq, last, next, seen, live_next;
  float g;
  uint32_t turn;
  bool done;
};

// An event's word in the chain: its session (below 2^20) and flags.
constexpr uint32_t kWNewBit = 25;
constexpr uint32_t kWArrive = 1u << 24, kWNew = 1u << kWNewBit, kWOnset = 1u << 26, kWBig = 1u << 27;
static_assert(UNISON_MAX_SESSIONS <= (1u << 20), "session ids take 20 bits");

// Values spread over a wavefront: index i sits in lane i % 64 of register i / 64.
template <int SPL>
struct Spread {
  template <class T>
  __device__ __forceinline__ static T get(const T (&a)[SPL], uint32_t i) {
    T v = rl(a[0], i & 63u);
#pragma unroll
    for (int j = 1; j < SPL; ++j) {
      const T o = rl(a[j], i & 63u);
      v = (i >> 6) == (uint32_t)j ? o : v;
    }
    return v;
  }
  template <class T>
  __device__ __forceinline__ static void set(T (&a)[SPL], uint32_t i, T v) {
#pragma unroll
    for (int j = 0; j < SPL; ++j) {
      const T n = wl(a[j], i & 63u, v);
      a[j] = SPL == 1 || (i >> 6) == (uint32_t)j ? n : a[j];
    }
  }
  // Register j's lane l as an index, or `other` for no lane.
  __device__ __forceinline__ static uint32_t at(uint32_t l, int j, uint32_t other) {
    if constexpr (SPL == 1) return l;
    else return l == kNone ? other : (uint32_t)j * 64u + l;
  }
};

// An order entry: session << 11 | slot << 2 | completed << 1 | in SRAM.
constexpr uint32_t kSidShift = 11, kDoneB = 2u, kSram = 1u;
static_assert(kTierSram == 1 && kTierHbm == 2, "a tier's low bit is the SRAM flag");

// Evictable residents in victim order (larger key first, ties to the smaller
// id): the key, and the entry complemented, so that an empty position is 0 in
// both and sorts last.
template <int SPL, class KT>
struct Order : Spread<SPL> {
  using Spread<SPL>::get;
  using Spread<SPL>::set;
  using Spread<SPL>::at;
  uint32_t lane;
  KT skey[SPL];
  uint32_t snot[SPL];

  __device__ __forceinline__ void init(uint32_t l) {
    lane = l;
#pragma unroll
    for (int j = 0; j < SPL; ++j) {
      skey[j] = 0;
      snot[j] = 0;
    }
  }
  // The position of a resident that is in the order.
  __device__ __forceinline__ uint32_t pos_of(uint32_t sid) const {
    const uint32_t top = (uint32_t)((int)~(sid << kSidShift) >> kSidShift);
    uint32_t p = kNone;
#pragma unroll
    for (int j = SPL - 1; j >= 0; --j)
      p = at(first_set(ballot((uint32_t)((int)snot[j] >> kSidShift) == top)), j, p);
    return p;
  }
  // The entry at position p (kNone: empty).
  __device__ __forceinline__ uint32_t entry(uint32_t p) const { return ~get(snot, p); }
  __device__ __forceinline__ uint32_t front() const { return ~rl(snot[0], 0u); }
  __device__ __forceinline__ static uint32_t slot_in(uint32_t x) { return (x >> 2) & 511u; }
  template <bool FRONT, class T>
  __device__ __forceinline__ void close_gap(T (&a)[SPL], uint32_t pos) const {
#pragma unroll
    for (int j = 0; j < SPL; ++j) {
      T t = from_above(a[j]);
      if constexpr (SPL > 1) {
        if (j + 1 < SPL) t = wl(t, 63u, rl(a[j + 1 < SPL ? j + 1 : j], 0u));
      }
      a[j] = !FRONT && (uint32_t)j * 64u + lane < pos ? a[j] : t;
    }
  }
  __device__ __forceinline__ void remove_at(uint32_t pos) {
    close_gap<false>(skey, pos);
    close_gap<false>(snot, pos);
  }
  __device__ __forceinline__ void pop_front() {
    close_gap<true>(skey, 0u);
    close_gap<true>(snot, 0u);
  }
  template <class T>
  __device__ __forceinline__ static void open_gap(T (&a)[SPL], const bool (&before)[SPL]) {
#pragma unroll
    for (int j = SPL - 1; j >= 0; --j) {
      T t = from_below(a[j]);
      if constexpr (SPL > 1) {
        if (j > 0) t = wl(t, 0u, rl(a[j > 0 ? j - 1 : 0], 63u));
      }
      a[j] = before[j] ? a[j] : t;
    }
  }
  __device__ __forceinline__ void insert(KT key, uint32_t entry_word) {
    const uint32_t n = ~entry_word;
    bool before[SPL];
    uint32_t pos = 0;
#pragma unroll
    for (int j = 0; j < SPL; ++j) {
      before[j] = (skey[j] > key) | ((skey[j] == key) & (snot[j] > n));
      pos += pop64(ballot(before[j]));
    }
    open_gap(skey, before);
    open_gap(snot, before);
    set(skey, pos, key);
    set(snot, pos, n);
  }
  // TIDE's candidates: the smallest key in HBM, ties to the smaller id
  // (eq. (promote)), and the largest key in SRAM (eq. (demote)).  kNone: none.
  __device__ __forceinline__ uint64_t hbm(int j) const { return ballot((snot[j] & 1u) != 0u); }
  __device__ __forceinline__ uint32_t last_hbm() const {
    uint64_t m[SPL];
    uint32_t p = kNone;
#pragma unroll
    for (int j = 0; j < SPL; ++j) {
      m[j] = hbm(j);
      p = at(last_set(m[j]), j, p);
    }
    if (p == kNone) return kNone;
    const KT k = get(skey, p);
#pragma unroll
    for (int j = SPL - 1; j >= 0; --j) p = at(first_set(ballot(skey[j] == k) & m[j]), j, p);
    return p;
  }
  __device__ __forceinline__ uint32_t first_sram() const {
    uint32_t p = kNone;
#pragma unroll
    for (int j = SPL - 1; j >= 0; --j)
      p = at(first_set(ballot(snot[j] != 0u) & ~hbm(j)), j, p);
    return p;
  }
  // Whether every position precedes the next (empty positions last).
  __device__ __forceinline__ bool sorted() const {
    uint64_t bad = 0;
#pragma unroll
    for (int j = 0; j < SPL; ++j) {
      KT k = from_above(skey[j]);
      uint32_t n = from_above(snot[j]);
      if (j + 1 < SPL) {
        k = wl(k, 63u, rl(skey[j + 1 < SPL ? j + 1 : j], 0u));
        n = wl(n, 63u, rl(snot[j + 1 < SPL ? j + 1 : j], 0u));
      }
      bad |= ballot((k > skey[j]) | ((k == skey[j]) & (n > snot[j])));
    }
    return bad == 0ull;
  }
  // A bitonic sorting network over the 64 SPL positions, every comparator's
  // larger value to the lower position: K = 2, 4, ... halves that are each in
  // order, merged by one step against the mirrored position (i ^ (K - 1)) and then
  // steps at distance K / 4, K / 8, ... 1.
  template <int M>
  __device__ __forceinline__ void lane_step(uint32_t l) {
    constexpr uint32_t kTop = M & 32 ? 32u : M & 16 ? 16u : M & 8 ? 8u : M & 4 ? 4u : M & 2 ? 2u : 1u;
    const bool low = (l & kTop) == 0u;
#pragma unroll
    for (int j = 0; j < SPL; ++j) {
      const KT k = lane_xor<M>(skey[j]);
      const uint32_t n = lane_xor<M>(snot[j]);
      const bool more = (skey[j] > k) | ((skey[j] == k) & (snot[j] > n));
      skey[j] = more == low ? skey[j] : k;
      snot[j] = more == low ? snot[j] : n;
    }
  }
  // Registers j and j ^ X, lane against lane or against the mirrored lane.
  template <int X, bool MIRROR>
  __device__ __forceinline__ void reg_step() {
#pragma unroll
    for (int j = 0; j < SPL; ++j) {
      const int i = (j ^ X) < SPL ? j ^ X : j;
      if (j < i) {
        const KT ka = MIRROR ? lane_xor<63>(skey[j]) : skey[j], kb = MIRROR ? lane_xor<63>(skey[i]) : skey[i];
        const uint32_t na = MIRROR ? lane_xor<63>(snot[j]) : snot[j], nb = MIRROR ? lane_xor<63>(snot[i]) : snot[i];
        const bool up = (kb > skey[j]) | ((kb == skey[j]) & (nb > snot[j]));
        const bool down = MIRROR ? (skey[i] > ka) | ((skey[i] == ka) & (snot[i] > na)) : up;
        skey[j] = up ? kb : skey[j];
        snot[j] = up ? nb : snot[j];
        skey[i] = down ? ka : skey[i];
        snot[i] = down ? na : snot[i];
      }
    }
  }
  template <int S>
  __device__ __forceinline__ void steps(uint32_t l) {
    if constexpr (S >= 64) reg_step<S / 64, false>();
    else lane_step<S>(l);
    if constexpr (S > 1) steps<S / 2>(l);
  }
  template <int K>
  __device__ __forceinline__ void merges(uint32_t l) {
    if constexpr (K > 2) merges<K / 2>(l);
    if constexpr (K > 64) reg_step<K / 64 - 1, true>();
    else lane_step<K - 1>(l);
    if constexpr (K > 2) steps<K / 4>(l);
  }
  // (The lane's number anew: the steps' lane masks, known throughout the launch,
  // would take scalar registers from the chain.)
  __device__ __forceinline__ void sort() { merges<64 * SPL>(in_vgpr(lane)); }
  // The session of an order entry; kNone for the empty one.
  __device__ __forceinline__ static uint32_t sid_of(uint32_t x) {
    return (uint32_t)((int)x >> kSidShift);
  }
};

// DUAL: the dual register-file design, eq. (rf), eq. (stale): both engines
// decide from copies of the key fields that are refreshed together, so one
// order by the copies' keys serves both; the live order beside it tells which
// decisions the unified file would have taken differently.
template <int SPL, uint32_t POL, uint32_t SMODE, bool DUAL>
struct LaneSim : Spread<SPL> {
  using Spread<SPL>::get;
  using Spread<SPL>::set;
  using Spread<SPL>::at;
  using PT = Pol<POL, SMODE>;
  // fp32 scores are 32-bit keys; integer scores and times take 64 bits
  using KT = typename std::conditional<PT::spear && !PT::fixed, uint32_t, uint64_t>::type;
  static constexpr bool kList = false;
  static constexpr int kRegs = SPL;
  static constexpr uint32_t kSlots = 64u * SPL;
  using O = Order<SPL, KT>;
  static constexpr uint32_t kPref = 2u;         // slot flags: kSram and this
  static constexpr bool kGapEma = PT::spear || PT::belady;  // others read it for TIDE only

  uint32_t lane;
  Order<SPL, KT> live;
  Order<SPL, KT> copy;   // DUAL only
  // slots: every resident, also while it is served
  uint32_t ssid[SPL], sfl[SPL];
  uint64_t ssz[SPL];
  // online tables: what a resident's key is recomputed from
  uint32_t sturn[SPL];
  uint64_t sema[SPL];

  __device__ __forceinline__ void init() {
    live.init(lane);
    copy.init(lane);
#pragma unroll
    for (int j = 0; j < SPL; ++j) {
      ssid[j] = kNone;
      sfl[j] = 0;
      ssz[j] = 0;
      sturn[j] = 0;
      sema[j] = 0;
    }
  }
  // The order the engines decide by.
  __device__ __forceinline__ Order<SPL, KT>& order() {
    if constexpr (DUAL) return copy;
    else return live;
  }
  __device__ __forceinline__ void insert(KT key, KT copy_key, uint32_t x) {
    live.insert(key, x);
    if constexpr (DUAL) copy.insert(copy_key, x);
  }
  __device__ __forceinline__ void remove(uint32_t sid) {
    live.remove_at(live.pos_of(sid));
    if constexpr (DUAL) copy.remove_at(copy.pos_of(sid));
  }
  // The front of the deciding order, session sid, leaves.
  __device__ __forceinline__ void pop_front(uint32_t sid) {
    order().pop_front();
    if constexpr (DUAL) live.remove_at(live.pos_of(sid));
  }
  // The entry at position p of the deciding order changes from x to y.
  __device__ __forceinline__ void change(uint32_t p, uint32_t x, uint32_t y) {
    set(order().snot, p, ~y);
    if constexpr (DUAL) set(live.snot, live.pos_of(x >> kSidShift), ~y);
  }
  // The copies are refreshed.
  __device__ __forceinline__ void sync() {
#pragma unroll
    for (int j = 0; j < SPL; ++j) {
      copy.skey[j] = live.skey[j];
      copy.snot[j] = live.snot[j];
    }
  }
  // The slot of resident sid, or kNone.
  __device__ __forceinline__ uint32_t slot_of(uint32_t sid) const {
    uint32_t s = kNone;
#pragma unroll
    for (int j = SPL - 1; j >= 0; --j) s = at(first_set(ballot(ssid[j] == sid)), j, s);
    return s;
  }
  // The slot a new resident takes (residents never exceed 64 SPL).
  __device__ __forceinline__ uint32_t free_slot() const {
    uint32_t s = 0;
#pragma unroll
    for (int j = SPL - 1; j >= 0; --j) s = at(first_set(ballot(ssid[j] == kNone)), j, s);
    return s;
  }

  // A key in the form the order compares.
  __device__ __forceinline__ static KT key_from(const KeyCtx& K, bool done, uint32_t turn, float g,
                                                uint64_t gq, uint64_t t, uint64_t next) {
    const uint32_t m = make_meta(done ? kDoneP : kGap, kTierNone, turn);
    return (KT)key_of<POL, SMODE>(K, m, hazard_of<POL, SMODE>(K, m), g, gq, t, next);
  }
  // After a change of the hazard table: every ordered resident's key, and the order
  // where it changed.  One by one into their ranks, 512 residents took about 85 us
  // and 256 about 40, more than the rest of 20 events: 256 sessions of one turn, all
  // completing, 10.9 ms against 2.1 in register tables.
  __device__ __forceinline__ void rescore(const KeyCtx& K) {
    if constexpr (PT::spear) {
      KT fresh[SPL];
#pragma unroll
      for (int j = 0; j < SPL; ++j)
        fresh[j] = key_from(K, false, sturn[j], __uint_as_float((uint32_t)sema[j]), sema[j], 0ull, 0ull);
      // the keys from slot order to the present order
#pragma unroll
      for (int j = 0; j < SPL; ++j) {
        const uint32_t x = ~live.snot[j], s = live.slot_in(x);
        KT v = from_lane(fresh[0], s & 63u);
#pragma unroll
        for (int i = 1; i < SPL; ++i) {
          const KT o = from_lane(fresh[i], s & 63u);
          v = (s >> 6) == (uint32_t)i ? o : v;
        }
        live.skey[j] = live.snot[j] == 0u ? (KT)0 : (x & kDoneB) ? (KT)PT::inf_key : v;
      }
      if (__builtin_expect(!live.sorted(), 0)) live.sort();
    }
  }
};

// Pools of more residents than registers hold in order: two sorted lists, one
// per tier, of leaves of up to 64 entries in LDS, an entry per lane.  A list's
// directory -- its leaves in order, each with its first entry, its row and its
// count -- sits in registers as an Order, so finding an entry's leaf is a
// comparison per register, and an insertion or removal reads and writes one row.
// The first entry of a list is in its directory: the scan victim is the better
// of two fronts, TIDE's demotion candidate the SRAM list's.  A full leaf splits
// in halves; when no row is free both lists are packed into full leaves.
// A session's residency (slot, tier) lies in the workspace and, for the events
// of the current window, in their lanes; a resident's KV bytes in its LDS slot.
// Bound by the same chain as the register orders, with an LDS round trip or two
// per change (about 0.8 us per event).  65,536 live sessions (16 simulations of
// 300,000 events, about 1,100 resident of 4,096 slots): 613 ms with unsorted LDS
// slots and three wavefront reductions per event, 243 here; the paper-scale trace
// at 512 and 1,400 slots 112 ms (register orders) and 166 (table in LDS) before,
// 67 at both here.
constexpr int kDirRegs = 3;
constexpr uint32_t kListQueue = 256;  // queued records; a pass over the pool flushes in between
constexpr uint32_t kStIn = 4u, kStSlot = 3u;  // a residency word: kSram, kPref, kStIn, slot << 3
static_assert(list_rows(kListResidents) <= 64u * kDirRegs, "a directory holds every row");

template <class KT>
struct Dir : Order<kDirRegs, KT> {
  using B = Order<kDirRegs, KT>;
  using B::lane;
  using B::skey;
  using B::snot;
  uint32_t leaf[kDirRegs];  // row << 7 | count
  uint32_t n;               // leaves

  __device__ __forceinline__ void reset(uint32_t l) {
    this->init(l);
#pragma unroll
    for (int j = 0; j < kDirRegs; ++j) leaf[j] = 0;
    n = 0;
  }
  // The leaf an entry belongs to: the last one whose first entry does not
  // follow it, else the first.
  __device__ __forceinline__ uint32_t find(KT key, uint32_t e) const {
    uint32_t c = 0;
#pragma unroll
    for (int j = 0; j < kDirRegs; ++j)
      c += pop64(ballot(((skey[j] > key) | ((skey[j] == key) & (snot[j] >= e))) &
                        ((uint32_t)j * 64u + lane < n)));
    return c ? c - 1u : 0u;
  }
  // Leaves whose first key is larger than `key`.
  __device__ __forceinline__ uint32_t above(KT key) const {
    uint32_t c = 0;
#pragma unroll
    for (int j = 0; j < kDirRegs; ++j)
      c += pop64(ballot((skey[j] > key) & ((uint32_t)j * 64u + lane < n)));
    return c;
  }
  __device__ __forceinline__ void put(uint32_t p, KT key, uint32_t e, uint32_t lf) {
    B::set(skey, p, key);
    B::set(snot, p, e);
    B::set(leaf, p, lf);
  }
  __device__ __forceinline__ void open(uint32_t p, KT key, uint32_t e, uint32_t lf) {
    bool before[kDirRegs];
#pragma unroll
    for (int j = 0; j < kDirRegs; ++j) before[j] = (uint32_t)j * 64u + lane < p;
    B::open_gap(skey, before);
    B::open_gap(snot, before);
    B::open_gap(leaf, before);
    put(p, key, e, lf);
    ++n;
  }
  __device__ __forceinline__ void close(uint32_t p) {
    this->template close_gap<false>(skey, p);
    this->template close_gap<false>(snot, p);
    this->template close_gap<false>(leaf, p);
    --n;
  }
};

template <uint32_t POL, uint32_t SMODE>
struct ListSim {
  using PT = Pol<POL, SMODE>;
  using KT = typename std::conditional<PT::spear && !PT::fixed, uint32_t, uint64_t>::type;
  using D = Dir<KT>;
  static constexpr bool kList = true;
  static constexpr uint32_t kSlots = kListResidents;
  static constexpr uint32_t kPref = 2u;
  static constexpr bool kGapEma = PT::spear || PT::belady;

  uint32_t lane;
  D hbm, sram;
  KT* lkey;         // LDS [rows][64]
  uint32_t* lent;   // LDS [rows][64]: session << 12 | slot, complemented
  uint64_t* ssz;    // LDS [slots]: KV bytes
  uint32_t* where;  // workspace [sessions]: residency words
  uint32_t rows_free;          // per lane: bit b for row b * 64 + lane
  uint64_t used, done, pref;   // per lane: bit b for slot b * 64 + lane

  // LDS: the slots, the rows' keys, the rows' entries.
  __device__ __forceinline__ void init(uint32_t l, uint64_t* lds, uint32_t slots, uint32_t rows, uint32_t* w) {
    lane = l;
    ssz = lds;
    lkey = reinterpret_cast<KT*>(lds + slots);
    lent = reinterpret_cast<uint32_t*>(lkey + rows * 64u);
    where = w;
    hbm.reset(l);
    sram.reset(l);
    rows_free = 0;
    for (uint32_t b = 0; b < (uint32_t)kDirRegs; ++b) rows_free |= b * 64u + l < rows ? 1u << b : 0u;
    used = slots < kListResidents ? ~0ull << (slots >> 6) : 0ull;  // slots is a multiple of 64
    done = pref = 0;
  }
  __device__ __forceinline__ static KT key_from(const KeyCtx& K, bool fin, uint32_t turn, float g,
                                                uint64_t gq, uint64_t t, uint64_t next) {
    const uint32_t m = make_meta(fin ? kDoneP : kGap, kTierNone, turn);
    return (KT)key_of<POL, SMODE>(K, m, hazard_of<POL, SMODE>(K, m), g, gq, t, next);
  }
  __device__ __forceinline__ static uint32_t entry_of(uint32_t sid, uint32_t slot) {
    return ~list_word(sid, slot);
  }
  __device__ __forceinline__ static uint32_t sid_in(uint32_t e) { return list_sid(~e); }
  __device__ __forceinline__ static uint32_t slot_in(uint32_t e) { return list_slot(~e); }
  __device__ __forceinline__ uint64_t mine(uint32_t slot) const {
    return lane == (slot & 63u) ? 1ull << (slot >> 6) : 0ull;
  }
  __device__ __forceinline__ static uint32_t bit(uint64_t m, uint32_t slot) {
    return (uint32_t)(rl(m, slot & 63u) >> (slot >> 6)) & 1u;
  }
  // A free slot (residents never exceed the slots).
  __device__ __forceinline__ uint32_t take_slot() {
    const uint32_t l = first_set(ballot(used != ~0ull));
    const uint32_t s = (uint32_t)__builtin_ctzll(~rl(used, l)) * 64u + l;
    used |= mine(s);
    done &= ~mine(s);
    pref &= ~mine(s);
    return s;
  }
  __device__ __forceinline__ void free_slot(uint32_t s) { used &= ~mine(s); }
  // (The index in a vector register keeps the readfirstlane: of an address known
  // to be uniform it is dropped, and the value stays out of the scalar registers.)
  __device__ __forceinline__ uint64_t size(uint32_t slot) const { return uni64(ssz[in_vgpr(slot)]); }

  __device__ __forceinline__ uint32_t take_row() {
    const uint32_t l = first_set(ballot(rows_free != 0u));
    const uint32_t b = (uint32_t)__builtin_ctz(rl(rows_free, l));
    rows_free &= lane == l ? ~(1u << b) : ~0u;
    return b * 64u + l;
  }
  __device__ __forceinline__ void give_row(uint32_t r) {
    rows_free |= lane == (r & 63u) ? 1u << (r >> 6) : 0u;
  }
  // Every leaf full but the last.  Rows are refilled in order: a row is written
  // once the rows before it and itself have been read.
  __device__ __forceinline__ void pack(D& d) {
    KT bk = 0;
    uint32_t be = 0, nb = 0, out = 0;
    const uint32_t was = d.n;
    for (uint32_t p = 0; p < was; ++p) {
      const uint32_t lf = D::get(d.leaf, p), c = lf & 127u, i = (lf >> 7) * 64u + lane;
      const KT k = lkey[i];
      const uint32_t e = lent[i];
      const int from = (int)((lane - nb) & 63u);
      const KT rk = (KT)__shfl((unsigned long long)k, from);
      const uint32_t re = __shfl(e, from);
      bk = lane < nb ? bk : rk;
      be = lane < nb ? be : re;
      nb += c;
      if (nb >= 64u) {
        const uint32_t row = D::get(d.leaf, out) >> 7;
        lkey[row * 64u + lane] = bk;
        lent[row * 64u + lane] = be;
        d.put(out, rl(bk, 0u), rl(be, 0u), row << 7 | 64u);
        ++out;
        bk = rk;
        be = re;
        nb -= 64u;
      }
    }
    if (nb) {
      const uint32_t row = D::get(d.leaf, out) >> 7;
      lkey[row * 64u + lane] = bk;
      lent[row * 64u + lane] = be;
      d.put(out, rl(bk, 0u), rl(be, 0u), row << 7 | nb);
      ++out;
    }
    for (uint32_t p = out; p < was; ++p) give_row(D::get(d.leaf, p) >> 7);
    d.n = out;
  }
  __device__ __forceinline__ void split(D& d, uint32_t p) {
    const uint32_t row = D::get(d.leaf, p) >> 7, up = take_row();
    const KT k = lkey[row * 64u + lane];
    const uint32_t e = lent[row * 64u + lane];
    const int from = (int)((lane + 32u) & 63u);
    const KT uk = (KT)__shfl((unsigned long long)k, from);
    const uint32_t ue = __shfl(e, from);
    lkey[up * 64u + lane] = uk;
    lent[up * 64u + lane] = ue;
    D::set(d.leaf, p, row << 7 | 32u);
    d.open(p + 1u, rl(k, 32u), rl(e, 32u), up << 7 | 32u);
  }
  __device__ __forceinline__ void insert(D& d, KT key, uint32_t e) {
    if (ballot(rows_free != 0u) == 0ull) {
      pack(hbm);
      pack(sram);
    }
    if (d.n == 0u) {
      const uint32_t row = take_row();
      lkey[row * 64u + lane] = key;
      lent[row * 64u + lane] = e;
      d.open(0u, key, e, row << 7 | 1u);
    } else {
      uint32_t p = d.find(key, e);
      uint32_t lf = D::get(d.leaf, p);
      if ((lf & 127u) == 64u) {
        split(d, p);
        p = d.find(key, e);
        lf = D::get(d.leaf, p);
      }
      const uint32_t i = (lf >> 7) * 64u + lane;
      const KT k = lkey[i];
      const uint32_t x = lent[i];
      const bool before = (lane < (lf & 127u)) & ((k > key) | ((k == key) & (x > e)));
      const uint32_t q = pop64(ballot(before));
      const KT kb = from_below(k);
      const uint32_t xb = from_below(x);
      lkey[i] = before ? k : lane == q ? key : kb;
      lent[i] = before ? x : lane == q ? e : xb;
      D::set(d.leaf, p, lf + 1u);
      if (q == 0u) {
        D::set(d.skey, p, key);
        D::set(d.snot, p, e);
      }
    }
  }
  // Entry q of leaf p leaves.
  __device__ __forceinline__ void remove_at(D& d, uint32_t p, uint32_t q, uint32_t lf, KT k, uint32_t x) {
    if ((lf & 127u) == 1u) {
      give_row(lf >> 7);
      d.close(p);
    } else {
      const KT ka = from_above(k);
      const uint32_t xa = from_above(x), i = (lf >> 7) * 64u + lane;
      k = lane < q ? k : ka;
      x = lane < q ? x : xa;
      lkey[i] = k;
      lent[i] = x;
      D::set(d.leaf, p, lf - 1u);
      if (q == 0u) {
        D::set(d.skey, p, rl(k, 0u));
        D::set(d.snot, p, rl(x, 0u));
      }
    }
  }
  __device__ __forceinline__ void remove_at(D& d, uint32_t p, uint32_t q) {
    const uint32_t lf = D::get(d.leaf, p), i = (lf >> 7) * 64u + lane;
    remove_at(d, p, q, lf, lkey[i], lent[i]);
  }
  __device__ __forceinline__ void remove(D& d, KT key, uint32_t e) {
    if (d.n) {
      const uint32_t p = d.find(key, e), lf = D::get(d.leaf, p), i = (lf >> 7) * 64u + lane;
      const KT k = lkey[i];
      const uint32_t x = lent[i];
      const uint32_t q = first_set(ballot((lane < (lf & 127u)) & (x == e)));
      if (q != kNone) remove_at(d, p, q, lf, k, x);
    }
  }
  // An entry whose key is not at hand, near the front.
  __device__ __forceinline__ void remove_walking(D& d, uint32_t e) {
    bool more = d.n != 0u;
    for (uint32_t p = 0; more; ++p) {
      const uint32_t lf = D::get(d.leaf, p), i = (lf >> 7) * 64u + lane;
      const KT k = lkey[i];
      const uint32_t x = lent[i];
      const uint32_t q = first_set(ballot((lane < (lf & 127u)) & (x == e)));
      more = q == kNone && p + 1u < d.n;
      if (q != kNone) remove_at(d, p, q, lf, k, x);
    }
  }
  // The smallest key, ties to the smaller id (d not empty): its leaf and position.
  struct At {
    uint32_t p, q, e;
    KT key;
  };
  __device__ __forceinline__ At back(const D& d) const {
    At r;
    r.p = d.n - 1u;
    uint32_t lf = D::get(d.leaf, r.p), i = (lf >> 7) * 64u + lane;
    KT k = lkey[i];
    uint32_t x = lent[i];
    r.key = rl(k, (lf & 127u) - 1u);
    r.q = first_set(ballot((lane < (lf & 127u)) & (k == r.key)));
    r.e = rl(x, r.q);
    if (r.q == 0u && r.p) {
      // the tie may begin in an earlier leaf: inside the last one that begins
      // with a larger key, or with the leaf after that
      const uint32_t c = d.above(r.key);
      r.p = c;
      r.e = D::get(d.snot, c);
      if (c) {
        lf = D::get(d.leaf, c - 1u);
        i = (lf >> 7) * 64u + lane;
        k = lkey[i];
        x = lent[i];
        const uint32_t q = first_set(ballot((lane < (lf & 127u)) & (k == r.key)));
        if (q != kNone) {
          r.p = c - 1u;
          r.q = q;
          r.e = rl(x, q);
        }
      }
    }
    return r;
  }
  // The scan victim is the better of the two fronts (none: empty()).
  // (Uniform conditions that outlive a branch are words: as truth values the
  // compiler keeps lane masks of them and selects in vector registers.)
  __device__ __forceinline__ uint32_t empty() const { return (hbm.n | sram.n) == 0u ? 1u : 0u; }
  __device__ __forceinline__ uint32_t front_in_sram() const {
    const KT hk = rl(hbm.skey[0], 0u), sk = rl(sram.skey[0], 0u);
    const uint32_t he = rl(hbm.snot[0], 0u), se = rl(sram.snot[0], 0u);
    const uint32_t ge = hk <= sk ? 1u : 0u;
    uint32_t first = hk == sk ? (se > he ? 1u : 0u) : ge;
    first = hbm.n == 0u ? 1u : first;
    return sram.n == 0u ? 0u : first;
  }
  __device__ __forceinline__ uint32_t front(uint32_t in_sram) const {
    return in_sram ? rl(sram.snot[0], 0u) : rl(hbm.snot[0], 0u);
  }
  // The smallest id with a key above th, as its entry's complement: in the first n
  // leaves, d.above(th) of them (0: kNone, which may also be an entry).
  __device__ __forceinline__ uint32_t fired(const D& d, KT th, uint32_t n) const {
    uint32_t best = kNone;
    for (uint32_t p = 0; p < n; ++p) {
      const uint32_t lf = D::get(d.leaf, p), i = (lf >> 7) * 64u + lane;
      const uint32_t x = ~lent[i];
      const uint32_t v = ((lane < (lf & 127u)) & (lkey[i] > th)) ? x : kNone;
      const uint32_t m = uni32(wave_ext32<false>(v));
      best = m < best ? m : best;
    }
    return best;
  }
};

// The wavefront's 64-bit sums, 64 words each in LDS.
enum : uint32_t { kSTok, kSComp, kSExtra, kSMiss, kSHitS, kSPrevS, kSHitH, kSPrevH, kSEvals, kSResEvals,
                  kSDigest, kSVictim, kSums };

// The pool's scalars, and what a launch adds to a simulation's counters.
struct Pool {
  uint64_t used_s, used_h, dma_free, log_len, requests, last_sync;
  uint32_t n_res, n_table;
};
struct Totals {
  uint64_t hit_s, hit_h, miss_tok, prev_s, prev_h, dma_bytes, tok, comp, extra, evals, res_evals,
      digest, victim_digest;
  uint32_t hi, req, n_hs, n_hh, n_pf, n_byp, n_evict, n_exp, n_pro, n_swap, passes, vict_diff,
      prom_diff;
};

// Events [e_io, end) of one simulation.
template <uint32_t POL, uint32_t SMODE, bool DUAL, class LS>
__device__ __forceinline__ void lane_events(const SimArgs& a, const unison_sim_params& P,
                                            const KeyCtx& K, const TraceView& tr, size_t tb,
                                            const uint32_t* kvb_of, uint64_t* view, uint2* queue, uint64_t* sums,
                                            LS& T,
                                            Pool& pool, Totals& W, const LogSink& L, uint64_t& e_io,
                                            uint64_t end) {
  using PT = Pol<POL, SMODE>;
  using KT = typename LS::KT;
  constexpr uint64_t kGolden = 0x9e3779b97f4a7c15ull;
  const uint32_t lane = T.lane;
  const uint64_t below = (1ull << lane) - 1ull;
  Consts c{0u};
  c.put(kCMg, a.t_mg + tb);
  c.put(kCGq, a.t_gq + tb);
  c.put(kCLast, a.t_last + tb);
  c.put(kCNext, a.t_next + tb);
  c.put(kCLen, a.t_len + tb);
  c.put(kCKvb, kvb_of);
  c.put(kCEvT, tr.t);
  c.put(kCEvNext, tr.next);
  c.put(kCEvSid, tr.sid);
  c.put(kCEvInfo, tr.info);
  c.put(kCEvLen, tr.len);
  c.put(kCEvTool, tr.tool);
  c.put(kCEta, K.eta);
  c.put(kCLog, L.rec);
  c.put(kCDma, uni64(P.dma_B_per_us));
  // the DMA busy time divides by the bandwidth: one reciprocal per launch
  c.put(kCDmaInv, uni64(~0ull / P.dma_B_per_us));
  c.put(kCTau, uni64(P.tau_ns));
  c.put(kCTtl, uni64(P.ttl_ns));
  c.put(kCPz, uni64(K.p_z));
  c.put(kCEnd, end);
  c.put(kCLambda, uni32(K.lambda));
  c.put(kCRecip, uni32(K.recip_bits));
  c.put(kCP, uni32(__float_as_uint(K.P)));
  c.put(kCBg, uni32(P.b_g));
  c.put(kCLogCap, L.cap);
  c.put(kCIdBits, tr.n_sess > 1u ? 32u - (uint32_t)__builtin_clz(tr.n_sess - 1u) : 0u);
  c.put(kCHasTool, PT::eta && tr.tool != nullptr ? 1u : 0u);
  if constexpr (DUAL) {
    c.put(kCDual, uni32(P.dual_sync));
    c.put(kCView, view);
    c.put(kCStride, (uint64_t)a.max_sessions);
    c.put(kCSync, (uint64_t)0);           // 1 + the index of the latest refresh
    c.put(kCReq, pool.requests);    // requests so far
  }
  const auto key_ctx = [&]() {
    KeyCtx v = K;
    v.lambda = c.u32(kCLambda);
    v.p_z = c.u64(kCPz);
    v.recip_bits = c.u32(kCRecip);
    v.P = __uint_as_float(c.u32(kCP));
    return v;
  };
  const bool tide = uni32(P.tide) != 0;
  const uint32_t online = DUAL ? 0u : K.online_cap;
  const uint32_t log_on = L.on ? 1u : 0u, log_victims = L.victims ? 1u : 0u;
  const bool ema = LS::kGapEma || tide;
  const uint64_t cap_s = uni64(P.cap_sram_B), cap_h = uni64(P.cap_hbm_B);
  const uint64_t slots = uni64(P.n_slots);
  const uint32_t n_slots = slots < LS::kSlots ? (uint32_t)slots : LS::kSlots;  // residents fit the slots

  uint64_t used_s = pool.used_s, used_h = pool.used_h, dma_free = pool.dma_free;
  uint32_t n_res = uni32(pool.n_res), n_table = uni32(pool.n_table);

  uint64_t log_len = in_vgpr(pool.log_len);
  uint64_t dma_bytes = 0;
  uint32_t passes = 0, hi = 0, vict_diff = 0, prom_diff = 0;
  // per lane, summed over the wavefront at the end; the 64-bit sums in LDS
#pragma unroll
  for (uint32_t i = 0; i < kSums; ++i) sums[i * 64u + lane] = 0ull;
  const auto add = [&](uint32_t i, uint64_t v) { sums[i * 64u + lane] += v; };
  uint32_t n_req = 0, n_hs = 0, n_hh = 0, n_pf = 0, n_evict = 0, n_exp = 0, n_byp = 0, n_pro = 0,
           n_swap = 0;
  uint32_t q_n = 0;  // queued decision records

  const auto load_events = [&](uint64_t b) {
    const uint64_t last = c.u64(kCEnd) - 1;
    const uint64_t i = b + lane < last ? b + lane : last;
    EvRegs v;
    v.t = c.ptr<uint64_t>(kCEvT)[i];
    v.sid = c.ptr<uint32_t>(kCEvSid)[i];
    v.info = c.ptr<uint32_t>(kCEvInfo)[i];
    v.len = c.ptr<uint32_t>(kCEvLen)[i];
    v.next = PT::belady ? c.ptr<uint64_t>(kCEvNext)[i] : ~0ull;
    v.tool = PT::eta && c.u32(kCHasTool) ? c.ptr<uint32_t>(kCEvTool)[i] : 0u;
    return v;
  };
  const auto gather = [&](uint32_t sid) {
    TabRegs v;
    v.mg = c.ptr<uint64_t>(kCMg)[sid];
    v.gq = PT::fixed ? c.ptr<uint64_t>(kCGq)[sid] : 0ull;
    v.last = c.ptr<uint64_t>(kCLast)[sid];
    v.len = c.ptr<uint32_t>(kCLen)[sid];
    v.kvb = c.ptr<uint32_t>(kCKvb)[sid];
    return v;
  };

  const auto gather_copy = [&](uint32_t sid) {
    CopyRegs v{};
    if constexpr (DUAL) {
      const uint64_t* v0 = c.ptr<uint64_t>(kCView);
      const uint64_t st = c.u64(kCStride);
      const uint64_t x = v0[sid];
      v.g = __uint_as_float((uint32_t)(x >> 32));
      v.turn = meta_turn((uint32_t)x);
      v.done = meta_phase((uint32_t)x) == kDoneP;
      v.gq = PT::fixed ? v0[st + sid] : 0ull;
      v.last = v0[2 * st + sid];
      v.next = PT::nextkey ? v0[3 * st + sid] : ~0ull;
      v.seen = v0[4 * st + sid];
      v.live_next = PT::nextkey ? c.ptr<uint64_t>(kCNext)[sid] : ~0ull;
    }
    return v;
  };

  uint64_t base = e_io;
  EvRegs cur = load_events(base);
  TabRegs tab = gather(cur.sid);
  CopyRegs cp = gather_copy(cur.sid);
  EvRegs nxt = load_events(base + 64);

  while (base < end) {
    c.fresh();
    const uint32_t cnt = end - base < 64 ? (uint32_t)(end - base) : 64u;
    const uint64_t all = cnt < 64u ? (1ull << cnt) - 1ull : ~0ull;
    const bool valid = lane < cnt;
    const uint64_t now = cur.t;
    const uint32_t sid = cur.sid, kind = cur.info >> 24, turn_ev = cur.info & 0xFFFFFFu;
    const uint32_t ln = cur.len;

    // ---- the window, an event per lane ----
    // the lanes of each lane's own session: those that agree in every id bit
    const uint32_t n_bits = c.u32(kCIdBits);
    uint32_t same_lo = (uint32_t)all, same_hi = (uint32_t)(all >> 32);
    for (uint32_t b = 0; b < n_bits; ++b) {
      const uint32_t mine = 0u - ((sid >> b) & 1u);
      const uint64_t set = ballot(mine != 0u);
      same_lo &= ~((uint32_t)set ^ mine);
      same_hi &= ~((uint32_t)(set >> 32) ^ mine);
    }
    const uint64_t same = ((uint64_t)same_hi << 32) | same_lo;
    const uint64_t earlier = same & below;
    const bool newest = valid && (same & ~below & ~(1ull << lane)) == 0ull;
    const int prev = valid && earlier ? 63 - __builtin_clzll(earlier) : -1;
    // the register file's entry before the event, then after it
    float g_in = __uint_as_float((uint32_t)(tab.mg >> 32));
    uint64_t gq_in = tab.gq, last_in = tab.last;
    uint32_t len_in = tab.len, turn_in = meta_turn((uint32_t)tab.mg);
    const bool arrive = kind == kArrive;
    const bool fresh = arrive && turn_ev == 0u;
    float g = 0.0f;
    uint64_t gq = 0;
    uint32_t len_out = 0, turn = 0;
    uint64_t ready = ballot(prev < 0);
    for (;;) {
      const uint64_t gap = now - last_in;  // eq. (gap)
      const bool upd = arrive && !fresh;
      if (ema) g = upd ? ema_f32(g_in, gap) : g_in;
      else g = g_in;
      if constexpr (PT::fixed) gq = upd ? ema_int(gq_in, gap, c.u32(kCBg), c.u64(kCTau)) : gq_in;
      if (fresh) {
        g = 0.0f;
        gq = 0;
      }
      len_out = arrive ? ln : len_in;
      turn = arrive ? turn_ev : turn_in;
      if (ready == ~0ull) break;
      const int p = prev < 0 ? (int)lane : prev;
      const float pg = __shfl(g, p);
      const uint64_t pq = PT::fixed ? __shfl((unsigned long long)gq, p) : 0ull;
      const uint64_t pt = __shfl((unsigned long long)now, p);
      const uint32_t pl = __shfl(len_out, p), pn = __shfl(turn, p);
      const bool take = prev >= 0 && ((ready >> p) & 1ull);
      g_in = take ? pg : g_in;
      gq_in = take ? pq : gq_in;
      last_in = take ? pt : last_in;
      len_in = take ? pl : len_in;
      turn_in = take ? pn : turn_in;
      ready |= ballot(take);
    }
    const uint32_t len_prev = fresh ? 0u : len_in;
    uint64_t next = kind == kGapStart ? cur.next : ~0ull;
    if constexpr (PT::eta) {
      // the predicted return: gap onset + the expected wait of the gap's tool class
      if (kind == kGapStart) next = sat_add(now, c.ptr<uint64_t>(kCEta)[cur.tool < kEtaClasses ? cur.tool : 0u]);
    }
    KT key = LS::key_from(key_ctx(), kind == kDone, turn, g, gq, now, next);
    // The copies' entry before the event.  It is the live entry after the
    // session's previous event if a refresh fell at or after that event, else
    // what the copies held before it.
    KT copy_key = 0;
    uint64_t m_sync = 0;
    uint64_t next_out = next;  // the live entry's next arrival after the event
    if constexpr (DUAL) {
      const uint32_t mode = c.u32(kCDual);
      const uint64_t m_arr = ballot(valid && arrive);
      const uint32_t nth = (uint32_t)c.u64(kCReq) + pop64(m_arr & (below | (1ull << lane)));
      m_sync = ballot(valid && (mode == UNISON_DUAL_EVERY   ? kind != kDone
                                : mode == UNISON_DUAL_EIGHT ? arrive && nth % 8u == 0u
                                                            : kind == kGapStart));
      const uint64_t sync_before = m_sync & below;
      // event indices + 1; 0: no refresh yet
      const uint64_t last_sync = c.u64(kCSync);
      const CopyRegs v = cp;
      float vg = v.g;
      uint64_t vq = v.gq, vlast = v.last, vnext = v.next;
      uint32_t vturn = v.turn;
      bool vdone = v.done;
      if (arrive) next_out = v.live_next;  // an arrival keeps the one before it
      uint64_t go = ballot(prev < 0);
      const bool late = prev < 0 ? sync_before != 0ull || last_sync > v.seen
                                 : (sync_before >> (prev < 0 ? 0 : prev)) != 0ull;
      if (prev < 0 && late) {
        vg = __uint_as_float((uint32_t)(tab.mg >> 32));
        vq = tab.gq;
        vlast = tab.last;
        vnext = v.live_next;
        vturn = meta_turn((uint32_t)tab.mg);
        vdone = false;  // a completed session has no later event
      }
      while (go != ~0ull) {
        const int p = prev < 0 ? (int)lane : prev;
        const bool take = prev >= 0 && ((go >> p) & 1ull) && !((go >> lane) & 1ull);
        // after the previous event ...
        const float ag = __shfl(g, p);
        const uint64_t aq = PT::fixed ? __shfl((unsigned long long)gq, p) : 0ull;
        const uint64_t al = __shfl((unsigned long long)now, p), an = __shfl((unsigned long long)next_out, p);
        const uint32_t at = __shfl(turn, p);
        // ... and what the copies held before it
        const float bg = __shfl(vg, p);
        const uint64_t bq = PT::fixed ? __shfl((unsigned long long)vq, p) : 0ull;
        const uint64_t bl = __shfl((unsigned long long)vlast, p), bn = __shfl((unsigned long long)vnext, p);
        const uint32_t bt = __shfl(vturn, p);
        const bool bd = __shfl((int)vdone, p) != 0;
        if (take) {
          vg = late ? ag : bg;
          vq = late ? aq : bq;
          vlast = late ? al : bl;
          vnext = late ? an : bn;
          vturn = late ? at : bt;
          vdone = late ? false : bd;
          if (arrive) next_out = an;
        }
        go |= ballot(take);
      }
      copy_key = LS::key_from(key_ctx(), vdone, vturn, vg, vq, vlast, vnext);
      if (newest) {
        c.ptr<uint64_t>(kCView)[sid] = (uint64_t)make_meta(vdone ? kDoneP : kGap, kTierNone, vturn) |
                                       ((uint64_t)__float_as_uint(vg) << 32);
        uint64_t* const v1 = c.ptr<uint64_t>(kCView) + c.u64(kCStride);
        v1[sid] = vq;
        v1[c.u64(kCStride) + sid] = vlast;
        v1[2 * c.u64(kCStride) + sid] = vnext;
        // the event's index, where the second copy will be
        v1[3 * c.u64(kCStride) + sid] = base + lane;
      }
      if (m_sync) c.put(kCSync, (uint64_t)(base + 64u - (uint32_t)__builtin_clzll(m_sync)));
      c.put(kCReq, (uint64_t)(c.u64(kCReq) + pop64(m_arr)));
    }
    // a list finds an arriving session's entry by the key of its last gap onset
    // and its size by the length before the event
    KT key_in = 0;
    uint64_t size_in = 0;
    uint32_t st = 0;
    if constexpr (LS::kList) {
      st = T.where[sid];
      const KT pk = (KT)__shfl((unsigned long long)key, prev < 0 ? (int)lane : prev);
      key_in = LS::key_from(key_ctx(), false, meta_turn((uint32_t)tab.mg),
                            __uint_as_float((uint32_t)(tab.mg >> 32)), tab.gq, tab.last,
                            PT::nextkey ? c.ptr<uint64_t>(kCNext)[sid] : ~0ull);
      key_in = prev < 0 ? key_in : pk;
      size_in = (uint64_t)len_in * tab.kvb;
    }
    const uint64_t size = (uint64_t)ln * tab.kvb;
    uint64_t budget = 0;
    if (tide) {
      // eq. (budget) / eq. (budgetq): Delta is the session's gap EMA in us
      uint64_t delta_us;
      if constexpr (PT::fixed) {
        const uint64_t tau = c.u64(kCTau);
        if (gq < (1ull << 32) && tau < (1ull << 32)) {
          delta_us = (gq * tau) / 1000u;
        } else {
          const unsigned __int128 d = ((unsigned __int128)gq * tau) / 1000u;
          delta_us = d > (unsigned __int128)~0ull ? ~0ull : (uint64_t)d;
        }
      } else {
        delta_us = (uint64_t)g;
      }
      budget = sat_mul(delta_us, c.u64(kCDma));
    }
    // each session's newest entry back to the table (tiers follow at the end)
    if (newest) {
      const uint32_t ph = arrive ? kServing : kind == kGapStart ? kGap : kDoneP;
      c.ptr<uint64_t>(kCMg)[sid] = (uint64_t)make_meta(ph, kTierNone, turn) | ((uint64_t)__float_as_uint(g) << 32);
      if constexpr (PT::fixed) c.ptr<uint64_t>(kCGq)[sid] = gq;
      c.ptr<uint32_t>(kCLen)[sid] = len_out;
      c.ptr<uint64_t>(kCLast)[sid] = now;
      if constexpr (PT::nextkey) {
        if (DUAL || !arrive) c.ptr<uint64_t>(kCNext)[sid] = next_out;
      }
    }
    wave_sync();
    const uint32_t kvb = tab.kvb;
    // the next window's entries and the events after it, in flight meanwhile
    cur = nxt;
    tab = gather(cur.sid);
    cp = gather_copy(cur.sid);
    nxt = load_events(base + 128);

    // the event's word: its session, and what the chain asks about it
    const bool onset_l = kind == kGapStart;
    const uint32_t word = sid | (arrive ? kWArrive : 0u) | (fresh ? kWNew : 0u) |
                          (onset_l ? kWOnset : 0u) | (size > cap_s && size > cap_h ? kWBig : 0u);
    uint64_t m_free = tide ? ballot(valid && onset_l && now >= dma_free) : 0ull;
    uint64_t thr = 0;
    if constexpr (PT::timeout) thr = ~idle_threshold(now, c.u64(kCTtl));  // a timer fired: key > thr
    hi = valid && fresh && sid + 1u > hi ? sid + 1u : hi;
    uint32_t o_code = 0, o_vic = 0;  // the event's outcome and scan victim, noted in its lane
    uint32_t w_evals = 0, w_res = 0;

    // Decision records queue in LDS as (event in window | op << 6 | b << 12, a)
    // and are hashed, counted and logged 64 at a time outside the chain.
    const auto emit = [&](uint32_t k, uint32_t op, uint32_t x, uint32_t y) {
      queue[q_n] = make_uint2(k | (op << 6) | (y << 12), x);
      ++q_n;
    };
    // (Without a divergent branch, so that it may stand inside the chain's loops:
    // lanes past the end read, hash and store the last record again.)
    const auto flush = [&]() {
      wave_sync();
      for (uint32_t q0 = 0; q0 < q_n; q0 += 64u) {
        const uint32_t m = q_n - q0 < 64u ? q_n - q0 : 64u;
        const bool in = lane < m;
        const uint2 r = queue[q0 + (in ? lane : m - 1u)];
        const uint32_t op = in ? (r.x >> 6) & 7u : 0u;
        const uint32_t ev = (uint32_t)base + (r.x & 63u);
        const auto second = [](uint32_t x) {
          const uint32_t o = (x >> 6) & 7u;
          return o == kOpPlace || o == kOpSwap ? x >> 12 : kNone;
        };
        // placements and bypasses are hashed from the window, an event per lane
        const uint64_t hash = rec_hash(ev, op, r.y, second(r.x));
        const uint64_t mask = 0ull - (uint64_t)(in & (op != kOpVictim) & (op != kOpPlace) & (op != kOpBypass));
        add(kSDigest, hash & mask);
        n_evict += op == kOpEvict ? 1u : 0u;
        n_exp += op == kOpExpire ? 1u : 0u;
        n_pro += op == kOpPromote ? 1u : 0u;
        n_swap += op == kOpSwap ? 1u : 0u;
        if (log_on) {
          const uint64_t at = uni64(log_len), cap = c.u32(kCLogCap);
          if (at < cap) {
            const uint64_t fit = cap - at < m ? cap - at : m;
            const uint32_t i = lane < (uint32_t)fit ? lane : (uint32_t)fit - 1u;
            const uint2 w = queue[q0 + i];
            c.ptr<unison_record>(kCLog)[at + i] =
                unison_record{(uint32_t)base + (w.x & 63u), (w.x >> 6) & 7u, w.y, second(w.x)};
          }
          log_len += m;
        }
      }
      wave_sync();
      q_n = 0;
    };
    if constexpr (LS::kList) {
    const auto set_state = [&](uint32_t v, uint32_t w) {
      st = sid == v ? w : st;
      T.where[v] = w;
    };
    const auto leave = [&](uint32_t x, uint32_t in_sram) {
      const uint32_t slot = LS::slot_in(x);
      const uint64_t sz = T.size(slot), m = 0ull - (uint64_t)in_sram;
      used_s -= sz & m;
      used_h -= sz & ~m;
      --n_res;
      n_table -= LS::bit(T.done, slot);  // a completed session leaves the table
      T.free_slot(slot);
      set_state(LS::sid_in(x), 0u);
    };
    // ---- the chain, one event after the other (every branch is uniform) ----
    for (uint32_t k = 0; k < cnt; ++k) {
      const uint32_t wd = rl(word, k);
      const uint32_t s = wd & (kWArrive - 1u);
      if (q_n >= kQueueFlush) flush();
      if constexpr (PT::timeout) {
        // TTL timers that fired since the previous event, smallest id first
        const KT th = rl(thr, k);
        uint32_t in_h = T.hbm.above(th), in_s = T.sram.above(th);
        while (in_h + in_s != 0u) {
          const uint32_t ch = T.fired(T.hbm, th, in_h), cs = T.fired(T.sram, th, in_s);
          const uint32_t in_sram = fired_in_sram(in_h, in_s, ch, cs);
          const uint32_t c = in_sram ? cs : ch;
          emit(k, kOpExpire, c >> kListSlotBits, 0u);
          leave(~c, in_sram);
          if (in_sram) T.remove_walking(T.sram, ~c);
          else T.remove_walking(T.hbm, ~c);
          if (q_n >= kListQueue - 4u) flush();
          in_h = T.hbm.above(th);
          in_s = T.sram.above(th);
        }
      }
      const uint32_t at = rl(st, k);  // the session's residency
      if (wd & kWArrive) {
        n_table += (wd >> kWNewBit) & 1u;
        w_evals += n_table;
        w_res += n_res;
        uint32_t code = 0;
        if (at & kStIn) {
          const uint64_t sz = rl(size_in, k);
          const uint32_t slot = at >> kStSlot;
          used_s -= at & kSram ? sz : 0ull;
          used_h -= at & kSram ? 0ull : sz;
          code = at & kSram ? at & 3u : 4u;
          --n_res;
          T.free_slot(slot);
          if (at & kSram) T.remove(T.sram, rl(key_in, k), LS::entry_of(s, slot));
          else T.remove(T.hbm, rl(key_in, k), LS::entry_of(s, slot));
        }
        uint32_t none = T.empty(), in_sram = T.front_in_sram();
        uint32_t x = T.front(in_sram);
        const uint32_t v0 = none ? kNone : LS::sid_in(x);
        o_vic = wl(o_vic, k, v0);
        if (log_victims) emit(k, kOpVictim, v0, 0u);
        // Alg. 1 capacity branch: evict the argmax victim until the session fits
        uint32_t place = 0;  // the tier, 0: bypassed
        const uint64_t sz = rl(size, k);
        const uint32_t want_h = code >> 2;
        if (!(wd & kWBig)) {
          for (;;) {
            const uint32_t room = (n_res - n_slots) >> 31;  // n_res < n_slots
            const uint32_t fit_s = room & le_u64(used_s + sz, cap_s);
            const uint32_t fit_h = room & le_u64(used_h + sz, cap_h);
            // SRAM first, for an HBM resident's request HBM first
            place = fit_s + 2u * (fit_h & ((fit_s ^ 1u) | want_h));
            place = place == 3u ? kTierHbm : place;
            if (place | none) break;
            emit(k, kOpEvict, LS::sid_in(x), 0u);
            leave(x, in_sram);
            if (in_sram) T.remove_at(T.sram, 0u, 0u);
            else T.remove_at(T.hbm, 0u, 0u);
            none = T.empty();
            in_sram = T.front_in_sram();
            x = T.front(in_sram);
            if (q_n >= kListQueue - 4u) flush();
          }
        }
        o_code = wl(o_code, k, code | (place << 4));
        if (log_on) emit(k, place ? kOpPlace : kOpBypass, s, place);
        if (place) {
          used_s += place & 1u ? sz : 0ull;
          used_h += place & 1u ? 0ull : sz;
          ++n_res;
          const uint32_t f = T.take_slot();
          T.ssz[f] = sz;
          set_state(s, kStIn | (f << kStSlot) | (place & 1u));
        } else if (at & kStIn) {
          set_state(s, 0u);
        }
      } else {
        const bool onset = (wd & kWOnset) != 0u;
        if (at & kStIn) {
          const uint32_t slot = at >> kStSlot;
          if (!onset) T.done |= T.mine(slot);
          if (at & kSram) T.insert(T.sram, rl(key, k), LS::entry_of(s, slot));
          else T.insert(T.hbm, rl(key, k), LS::entry_of(s, slot));
        }
        w_evals += n_table;
        w_res += n_res;
        const uint32_t v0 = T.empty() ? kNone : LS::sid_in(T.front(T.front_in_sram()));
        o_vic = wl(o_vic, k, v0);
        if (log_victims) emit(k, kOpVictim, v0, 0u);
        n_table -= !onset && !(at & kStIn) ? 1u : 0u;
        if ((m_free >> k) & 1ull) {
          uint64_t left = rl(budget, k), moved = 0;
          ++passes;
          bool more = T.hbm.n != 0u;
          while (more) {
            more = false;
            const auto b = T.back(T.hbm);
            const uint32_t ps = LS::slot_in(b.e);
            const uint64_t sp = T.size(ps);
            // past the budget or the SRAM, neither a promotion nor a swap is legal
            uint32_t may = le_u64(sp, left) & le_u64(sp, cap_s);
            if constexpr (PT::has_inf) may &= b.key != (KT)PT::inf_key ? 1u : 0u;
            if (may) {
              uint64_t sd = 0;
              more = le_u64(used_s + sp, cap_s) != 0u;
              const bool swap = !more && T.sram.n != 0u;
              const KT dk = rl(T.sram.skey[0], 0u);
              const uint32_t de = rl(T.sram.snot[0], 0u);
              if (swap) {
                sd = T.size(LS::slot_in(de));
                more = ((b.key < dk ? 1u : 0u) & le_u64(sd, left - sp) &
                        le_u64(used_s - sd + sp, cap_s) & le_u64(used_h - sp + sd, cap_h)) != 0u;
              }
              if (more) {
                used_s = used_s - sd + sp;
                used_h = used_h - sp + sd;
                T.remove_at(T.hbm, b.p, b.q);
                if (swap) {
                  const uint32_t ds = LS::slot_in(de);
                  T.remove_at(T.sram, 0u, 0u);
                  T.insert(T.hbm, dk, de);
                  set_state(LS::sid_in(de), kStIn | (ds << kStSlot) | (LS::bit(T.pref, ds) ? LS::kPref : 0u));
                }
                T.insert(T.sram, b.key, b.e);
                T.pref |= T.mine(ps);
                set_state(LS::sid_in(b.e), kStIn | (ps << kStSlot) | kSram | LS::kPref);
                left -= sp + sd;
                moved += sp + sd;
                emit(k, swap ? kOpSwap : kOpPromote, LS::sid_in(b.e), swap ? LS::sid_in(de) : 0u);
                if (q_n >= kListQueue - 4u) flush();
              }
            }
            more = more && T.hbm.n != 0u;
          }
          if (moved) {
            // DMA busy for ceil(moved * 1000 / B) ns
            const uint64_t b = c.u64(kCDma);
            const uint64_t busy = moved < (1ull << 53) && b < (1ull << 53)
                                      ? div_by(moved * 1000u + b - 1u, b, c.u64(kCDmaInv))
                                      : dma_ns(moved, b);
            dma_free = sat_add(rl(now, k), busy);
            m_free = ballot(valid && onset_l && now >= dma_free);
            dma_bytes += moved;
          }
        }
      }
    }
    flush();
    } else {
    constexpr int SPL = LS::kRegs;
    using O = typename LS::O;
    // A resident leaves the pool: its bytes, its slot.
    const auto leave = [&](uint32_t x) {
      const uint32_t slot = O::slot_in(x);
      const uint64_t sz = LS::get(T.ssz, slot);
      used_s -= x & kSram ? sz : 0ull;
      used_h -= x & kSram ? 0ull : sz;
      --n_res;
      n_table -= (x >> 1) & 1u;  // a completed session leaves the table
      LS::set(T.ssid, slot, kNone);
    };

    // ---- the chain, one event after the other (every branch is uniform) ----
    for (uint32_t k = 0; k < cnt;) {
      uint32_t stop = cnt;
      for (; k < stop; ++k) {
        const uint32_t wd = rl(word, k);
        const uint32_t s = wd & (kWArrive - 1u);
        if constexpr (PT::timeout) {
          // TTL timers that fired since the previous event, smallest id first
          const uint64_t th = rl(thr, k);
          while (LS::get(T.live.skey, 0) > th) {
            uint32_t c = kNone;
#pragma unroll
            for (int j = 0; j < SPL; ++j) c = T.live.skey[j] > th && ~T.live.snot[j] < c ? ~T.live.snot[j] : c;
            c = uni32(wave_ext32<false>(c));
            emit(k, kOpExpire, c >> kSidShift, 0u);
            leave(c);
            T.remove(c >> kSidShift);
            stop = q_n >= kQueueFlush ? k + 1u : stop;
          }
        }
        const uint32_t slot = T.slot_of(s);
        if (wd & kWArrive) {
          n_table += (wd >> kWNewBit) & 1u;
          w_evals += n_table;
          w_res += n_res;
          uint32_t code = 0;
          if (slot != kNone) {
            const uint32_t fl = LS::get(T.sfl, slot);
            const uint64_t sz = LS::get(T.ssz, slot);
            used_s -= fl & kSram ? sz : 0ull;
            used_h -= fl & kSram ? 0ull : sz;
            code = fl & kSram ? fl & 3u : 4u;
            --n_res;
            LS::set(T.ssid, slot, kNone);
            T.remove(s);
          }
          uint32_t x = T.order().front();
          o_vic = wl(o_vic, k, O::sid_of(x));
          if (log_victims) emit(k, kOpVictim, O::sid_of(x), 0u);
          // Alg. 1 capacity branch: evict the argmax victim until the session fits
          uint32_t place = 0;  // the tier, 0: bypassed
          const uint64_t sz = rl(size, k);
          const uint32_t want_h = code >> 2;
          if (!(wd & kWBig)) {
            for (;;) {
              const uint32_t room = (n_res - n_slots) >> 31;  // n_res < n_slots
              const uint32_t fit_s = room & le64(used_s + sz, cap_s);
              const uint32_t fit_h = room & le64(used_h + sz, cap_h);
              // SRAM first, for an HBM resident's request HBM first
              place = fit_s + 2u * (fit_h & ((fit_s ^ 1u) | want_h));
              place = place == 3u ? kTierHbm : place;
              if ((place != 0u) | (x == kNone)) break;
              emit(k, kOpEvict, x >> kSidShift, 0u);
              leave(x);
              // eq. (stale): would the live file agree?
              if constexpr (DUAL) vict_diff += T.live.front() >> kSidShift != x >> kSidShift ? 1u : 0u;
              T.pop_front(x >> kSidShift);
              x = T.order().front();
              stop = q_n >= kQueueFlush ? k + 1u : stop;
            }
          }
          o_code = wl(o_code, k, code | (place << 4));
          if (log_on) {
            emit(k, place ? kOpPlace : kOpBypass, s, place);
            stop = q_n >= kQueueFlush ? k + 1u : stop;
          }
          if (place) {
            used_s += place & 1u ? sz : 0ull;
            used_h += place & 1u ? 0ull : sz;
            ++n_res;
            const uint32_t f = T.free_slot();
            LS::set(T.ssid, f, s);
            LS::set(T.ssz, f, sz);
            LS::set(T.sfl, f, place & 1u);
          }
        } else {
          const bool onset = (wd & kWOnset) != 0u;
          if (slot != kNone) {
            const uint32_t fl = LS::get(T.sfl, slot);
            if (online) {
              LS::set(T.sturn, slot, rl(turn, k));
              LS::set(T.sema, slot, PT::fixed ? rl(gq, k) : (uint64_t)rl(__float_as_uint(g), k));
            }
            T.insert(rl(key, k), DUAL ? rl(copy_key, k) : (KT)0, (s << kSidShift) | (slot << 2) | (onset ? 0u : kDoneB) |
                                     (fl & kSram));
          }
          // an online hazard table counts the completed session before the scan
          // (the branch weights, here and at the sort, keep that code out of the way of
          // the other rows' chain: without them it costs 1.2 % of the paper-scale trace)
          if (!onset && __builtin_expect(online != 0u, 0) && uni32(K.hn[0]) < K.online_cap) {
            add_completion(K, rl(turn, k) + 1u, lane);
            T.rescore(key_ctx());
            key = LS::key_from(key_ctx(), kind == kDone, turn, g, gq, now, next);
          }
          w_evals += n_table;
          w_res += n_res;
          const uint32_t v0 = O::sid_of(T.order().front());
          o_vic = wl(o_vic, k, v0);
          if (log_victims) {
            emit(k, kOpVictim, v0, 0u);
            stop = q_n >= kQueueFlush ? k + 1u : stop;
          }
          n_table -= !onset && slot == kNone ? 1u : 0u;
          if ((m_free >> k) & 1ull) {
            uint64_t left = rl(budget, k), moved = 0;
            ++passes;
            bool more = true;
            while (more) {
              more = false;
              const uint32_t p = T.order().last_hbm();
              if (p != kNone) {
                const KT pk = LS::get(T.order().skey, p);
                const uint32_t px = T.order().entry(p);
                const uint32_t ps = O::slot_in(px);
                const uint64_t sp = LS::get(T.ssz, ps);
                // past the budget or the SRAM, neither a promotion nor a swap is legal
                uint32_t may = le64(sp, left) & le64(sp, cap_s);
                if constexpr (PT::has_inf) may &= pk != (KT)PT::inf_key ? 1u : 0u;
                if (may) {
                  uint32_t d = kNone, dx = 0, ds = 0;
                  uint64_t sd = 0;
                  more = le64(used_s + sp, cap_s) != 0u;
                  if (!more) {
                    d = T.order().first_sram();
                    if (d != kNone) {
                      dx = T.order().entry(d);
                      ds = O::slot_in(dx);
                      sd = LS::get(T.ssz, ds);
                      more = ((pk < LS::get(T.order().skey, d) ? 1u : 0u) & le64(sd, left - sp) &
                              le64(used_s - sd + sp, cap_s) & le64(used_h - sp + sd, cap_h)) != 0u;
                    }
                  }
                  if (more) {
                    if constexpr (DUAL) {
                      const uint32_t lp = T.live.last_hbm();
                      prom_diff += T.live.entry(lp) >> kSidShift != px >> kSidShift ? 1u : 0u;
                    }
                    used_s = used_s - sd + sp;
                    used_h = used_h - sp + sd;
                    T.change(p, px, px | kSram);
                    LS::set(T.sfl, ps, LS::get(T.sfl, ps) | kSram | LS::kPref);
                    if (d != kNone) {
                      T.change(d, dx, dx & ~kSram);
                      LS::set(T.sfl, ds, LS::get(T.sfl, ds) & ~kSram);
                    }
                    left -= sp + sd;
                    moved += sp + sd;
                    emit(k, d == kNone ? kOpPromote : kOpSwap, px >> kSidShift,
                         d == kNone ? 0u : dx >> kSidShift);
                    stop = q_n >= kQueueFlush ? k + 1u : stop;
                  }
                }
              }
            }
            if (moved) {
              // DMA busy for ceil(moved * 1000 / B) ns
              const uint64_t b = c.u64(kCDma);
              const uint64_t busy = moved < (1ull << 53) && b < (1ull << 53)
                                        ? div_by(moved * 1000u + b - 1u, b, c.u64(kCDmaInv))
                                        : dma_ns(moved, b);
              dma_free = sat_add(rl(now, k), busy);
              m_free = ballot(valid && onset_l && now >= dma_free);
              dma_bytes += moved;
            }
          }
        }
        if constexpr (DUAL) {
          if ((m_sync >> k) & 1ull) T.sync();
        }
      }
      flush();
    }
    }

    // ---- the window's accounting, an event per lane: eq. (hr-amat), eq. (prered) ----
    add(kSEvals, lane == 0 ? w_evals : 0u);
    add(kSResEvals, lane == 0 ? w_res : 0u);
    const bool h_s = valid && (o_code & 1u), h_h = valid && (o_code & 4u);
    n_hs += h_s ? 1u : 0u;
    n_hh += h_h ? 1u : 0u;
    n_pf += h_s && (o_code & LS::kPref) ? 1u : 0u;
    if (valid && arrive) {
      const uint32_t tier = o_code >> 4;  // where the session was placed
      add(kSDigest, rec_hash((uint32_t)(base + lane), tier ? kOpPlace : kOpBypass, sid,
                             tier ? tier : kNone));
      n_byp += tier ? 0u : 1u;
      ++n_req;
      const uint64_t old = (uint64_t)len_prev * kvb;
      const bool h = h_s || h_h;
      add(kSTok, ln);
      add(kSComp, h ? ln - len_prev : ln);
      if (h) {
        add(h_s ? kSHitS : kSHitH, size);
        add(h_s ? kSPrevS : kSPrevH, old);
      } else {
        add(kSExtra, len_prev);
        add(kSMiss, ln);
      }
    }
    // odd weight per event: a different victim at any one event changes the sum
    if (valid) add(kSVictim, ((uint64_t)o_vic + 1u) * ((2ull * (base + lane) + 1ull) * kGolden));
    base += cnt;
  }

  e_io = base;
  pool = Pool{used_s, used_h, dma_free, log_len, 0ull, DUAL ? c.u64(kCSync) : 0ull, n_res, n_table};
  const auto sum = [&](uint32_t i) { return wave_sum64(sums[i * 64u + lane]); };
  const auto sum32 = [](uint32_t v) { return (uint32_t)wave_sum64(v); };
  W.hi = wave_ext32<true>(hi);
  W.hit_s = sum(kSHitS);
  W.hit_h = sum(kSHitH);
  W.miss_tok = sum(kSMiss);
  W.prev_s = sum(kSPrevS);
  W.prev_h = sum(kSPrevH);
  W.req = sum32(n_req);
  W.n_hs = sum32(n_hs);
  W.n_hh = sum32(n_hh);
  W.n_pf = sum32(n_pf);
  W.n_byp = sum32(n_byp);
  W.n_evict = sum32(n_evict);
  W.n_exp = sum32(n_exp);
  W.n_pro = sum32(n_pro);
  W.n_swap = sum32(n_swap);
  W.passes = passes;
  W.vict_diff = vict_diff;
  W.prom_diff = prom_diff;
  W.dma_bytes = dma_bytes;
  W.tok = sum(kSTok);
  W.comp = sum(kSComp);
  W.extra = sum(kSExtra);
  W.evals = sum(kSEvals);
  W.res_evals = sum(kSResEvals);
  W.digest = sum(kSDigest);
  W.victim_digest = sum(kSVictim);
}

// lds, cap: a list pool's LDS and its slots.
template <uint32_t POL, uint32_t SMODE, bool DUAL, class LS>
__device__ __forceinline__ void lane_run(const SimArgs& a, uint32_t sim, const KeyCtx& K0,
                                         uint2* queue, uint64_t* sums, uint64_t* lds, uint32_t cap) {
  using KT = typename LS::KT;
  using PT = Pol<POL, SMODE>;
  // each instance computes its own addresses: shared ones would be hoisted
  // above the switch over policies and stay live in every instance
  asm volatile("" : "+s"(sim));
  const unison_sim_params& P = a.params[sim];
  const uint32_t lane = threadIdx.x;
  const uint64_t eb = a.ev_off[P.trace], ee = a.ev_off[P.trace + 1];
  const uint64_t sb = a.sess_off[P.trace];
  const uint32_t n_sess = (uint32_t)(a.sess_off[P.trace + 1] - sb);
  const TraceView tr{a.ev_t + eb, a.ev_sid + eb, a.ev_info + eb, a.ev_len + eb, a.ev_next + eb,
                     a.ev_tool ? a.ev_tool + eb : nullptr, ee - eb, n_sess};
  const size_t tb = (size_t)sim * a.max_sessions;
  const bool cont = (a.flags & UNISON_RUN_CONTINUE) != 0;
  KeyCtx K = K0;
  K.P = P.penalty_us;
  K.lambda = (1u << P.b_h) - 1u;
  K.p_z = P.p_z;
  K.pack44 = false;  // keys compare as they are
  K.online_cap = uni32(P.hazard_online ? P.online_sessions : 0u);
  K.eta = a.eta + (size_t)P.trace * kEtaClasses;
  K.recip_bits = P.recip_bits;

  uint64_t e = 0;
  bool ok = true;
  LS T;
  if constexpr (LS::kList) {
    T.init(lane, lds, cap, list_rows(cap), a.t_slot + tb);
    for (uint32_t i = lane; i < n_sess; i += 64) T.where[i] = 0u;
  } else {
    T.lane = lane;
    T.init();
  }
  if (cont) {
    e = uni64(a.state[sim].next_event);
    ok = uni64(a.counters[sim].error) == 0ull;
  } else {
    for (uint32_t i = lane; i < n_sess; i += 64) {
      a.t_mg[tb + i] = 0;
      a.t_gq[tb + i] = 0;
      a.t_len[tb + i] = 0;
      a.t_last[tb + i] = 0;
      a.t_next[tb + i] = ~0ull;
    }
  }
  __syncthreads();
  // residents never exceed min(N_sess, sessions): the launcher picks a kernel that holds them
  const uint64_t max_res = P.n_slots < n_sess ? P.n_slots : n_sess;
  const bool dual_ok = DUAL ? a.views && !P.hazard_online : !P.dual_sync;
  bool fits = dual_ok && max_res <= (LS::kList ? cap : LS::kSlots);
  uint64_t* const view = DUAL ? a.views + (size_t)sim * 8 * a.max_sessions : nullptr;
  ok = ok && fits;

  // a resumed table's residents take slots, in session order
  if (cont && ok) {
    uint32_t n = 0;
    for (uint32_t b = 0; b < n_sess && ok; b += 64) {
      const uint32_t i = b + lane;
      const bool in = i < n_sess;
      const uint64_t x = in ? a.t_mg[tb + i] : 0ull;
      const uint32_t m = (uint32_t)x;
      const uint64_t q = in ? a.t_gq[tb + i] : 0ull;
      const uint64_t last = in ? a.t_last[tb + i] : 0ull, next = in ? a.t_next[tb + i] : ~0ull;
      const uint64_t sz = in ? (uint64_t)a.t_len[tb + i] * a.sess_kvb[sb + i] : 0ull;
      const float g = __uint_as_float((uint32_t)(x >> 32));
      const bool done = meta_phase(m) == kDoneP;
      const KT key = LS::key_from(K, done, meta_turn(m), g, q, last, next);
      KT copy_key = 0;
      if constexpr (DUAL) {
        const size_t st = a.max_sessions;
        const uint64_t vx = in ? view[i] : 0ull;
        copy_key = LS::key_from(K, meta_phase((uint32_t)vx) == kDoneP, meta_turn((uint32_t)vx),
                                __uint_as_float((uint32_t)(vx >> 32)), in ? view[st + i] : 0ull,
                                in ? view[2 * st + i] : 0ull, in ? view[3 * st + i] : ~0ull);
      }
      // while the launch runs only the slots know the tiers: a resident that
      // leaves without an event of its own must not keep one in the table
      if (in && meta_tier(m) != kTierNone)
        *reinterpret_cast<uint32_t*>(a.t_mg + tb + i) = with_tier(m, kTierNone) & ~kPrefetched;
      for (uint64_t bits = ballot(in && meta_tier(m) != kTierNone); bits; bits &= bits - 1u) {
        if (n >= (LS::kList ? cap : LS::kSlots)) {
          ok = fits = false;
          break;
        }
        const uint32_t l = (uint32_t)__builtin_ctzll(bits);
        const uint32_t mm = rl(m, l), s = b + l;
        const uint32_t fl = (meta_tier(mm) == kTierSram ? kSram : 0u) |
                            ((mm & kPrefetched) ? LS::kPref : 0u);
        if constexpr (LS::kList) {
          const uint32_t f = T.take_slot(), e = LS::entry_of(s, f);
          T.ssz[f] = rl(sz, l);
          T.where[s] = kStIn | (f << kStSlot) | fl;
          if (fl & LS::kPref) T.pref |= T.mine(f);
          if (meta_phase(mm) == kDoneP) T.done |= T.mine(f);
          if (meta_phase(mm) != kServing) {
            if (fl & kSram) T.insert(T.sram, rl(key, l), e);
            else T.insert(T.hbm, rl(key, l), e);
          }
        } else {
        LS::set(T.ssid, n, s);
        LS::set(T.sfl, n, fl);
        LS::set(T.ssz, n, rl(sz, l));
        LS::set(T.sturn, n, meta_turn(mm));
        LS::set(T.sema, n, PT::fixed ? rl(q, l) : (uint64_t)rl((uint32_t)(x >> 32), l));
        if (meta_phase(mm) != kServing)
          T.insert(rl(key, l), DUAL ? rl(copy_key, l) : (KT)0, (s << kSidShift) | (n << 2) |
                                   (meta_phase(mm) == kDoneP ? kDoneB : 0u) | (fl & kSram));
        }
        ++n;
      }
    }
  }
  const bool log_on = (a.flags & UNISON_RUN_LOG) && a.log_cap;
  const LogSink L{log_on, log_on ? a.log + (size_t)sim * a.log_cap : nullptr, a.log_cap, lane == 0,
                  log_on && (a.flags & UNISON_RUN_LOG_VICTIM) != 0};
  const uint64_t e0 = e;
  if constexpr (DUAL) {
    // While the launch runs, the first copy holds each session's entry as the
    // copies did before its latest event, and the second copy's first field
    // that event's index: none since this launch began (a resumed launch's
    // copies are as the last one left them).
    if (ok) {
      const size_t st = a.max_sessions;
      for (uint32_t i = lane; i < n_sess; i += 64) {
        if (!cont) {
          view[i] = 0;
          view[st + i] = 0;
          view[2 * st + i] = 0;
          view[3 * st + i] = ~0ull;
        }
        view[4 * st + i] = e0;
      }
      __syncthreads();
    }
  }
  uint64_t bad = 0;
  Totals W{};
  Pool pool{};
  if (cont) {
    const SimState& st = a.state[sim];
    pool = Pool{uni64(st.used_s), uni64(st.used_h), uni64(st.dma_free_at), uni64(st.log_len),
                uni64(a.counters[sim].requests), 0ull, uni32(st.n_res), uni32(st.n_table)};
  }
  if (ok) {
    const uint64_t bad_at = a.first_bad[P.trace];
    uint64_t end = (e >= tr.n_ev || tr.n_ev - e < a.max_events) ? tr.n_ev : e + a.max_events;
    if (bad_at < end) {
      end = bad_at;
      bad = bad_at + 1;
    }
    if (e < end)
      lane_events<POL, SMODE, DUAL>(a, P, K, tr, tb, a.sess_kvb + sb, view, queue, sums, T, pool, W, L, e, end);
    __syncthreads();
    if constexpr (DUAL) {
      // both copies as the latest refresh left them
      const size_t st = a.max_sessions;
      for (uint32_t i = lane; i < n_sess; i += 64) {
        const bool late = pool.last_sync > view[4 * st + i];
        const uint64_t x = late ? a.t_mg[tb + i] : view[i];
        const uint64_t q = late ? a.t_gq[tb + i] : view[st + i];
        const uint64_t l = late ? a.t_last[tb + i] : view[2 * st + i];
        const uint64_t n = late ? a.t_next[tb + i] : view[3 * st + i];
        view[i] = view[4 * st + i] = x;
        view[st + i] = view[5 * st + i] = q;
        view[2 * st + i] = view[6 * st + i] = l;
        view[3 * st + i] = view[7 * st + i] = n;
      }
    }
    // the residents' tiers into the table
    __syncthreads();
    if constexpr (LS::kList) {
      for (uint32_t i = lane; i < n_sess; i += 64) {
        const uint32_t st = T.where[i];
        if (st & kStIn) {
          uint32_t* w = reinterpret_cast<uint32_t*>(a.t_mg + tb + i);
          *w = with_tier(*w, (st & kSram) ? kTierSram : kTierHbm) | ((st & LS::kPref) ? kPrefetched : 0u);
        }
      }
    } else {
#pragma unroll
    for (int j = 0; j < LS::kRegs; ++j)
      if (T.ssid[j] != kNone) {
        uint32_t* w = reinterpret_cast<uint32_t*>(a.t_mg + tb + T.ssid[j]);
        *w = with_tier(*w, (T.sfl[j] & kSram) ? kTierSram : kTierHbm) |
             ((T.sfl[j] & LS::kPref) ? kPrefetched : 0u);
      }
    }
  }
  store_hazard(a, P, sim, K, lane, 64);
  if (lane == 0) {
    Scalars S{};
    Cnt C = cnt_from(unison_counters{});
    if (cont) {
      load_scalars(a.state[sim], S);
      C = cnt_from(a.counters[sim]);
    }
    if (!fits) C.error = ~0ull;
    if (bad) C.error = bad;
    S.used_s = pool.used_s;
    S.used_h = pool.used_h;
    S.dma_free_at = pool.dma_free;
    S.log_len = pool.log_len;
    S.n_res = pool.n_res;
    S.n_table = pool.n_table;
    if (S.hi > n_sess) S.hi = n_sess;
    S.hi = W.hi > S.hi ? W.hi : S.hi;
    S.hit_s_bytes += W.hit_s;
    S.hit_h_bytes += W.hit_h;
    S.miss_tok += W.miss_tok;
    S.prev_s_bytes += W.prev_s;
    S.prev_h_bytes += W.prev_h;
    C.requests += W.req;
    C.hit_sram += W.n_hs;
    C.hit_hbm += W.n_hh;
    C.miss += W.req - W.n_hs - W.n_hh;
    C.prefetch_hits += W.n_pf;
    C.bypass += W.n_byp;
    C.evict += W.n_evict;
    C.expire += W.n_exp;
    C.promote += W.n_pro;
    C.swap += W.n_swap;
    C.tide_passes += W.passes;
    C.vict_diff += W.vict_diff;
    C.prom_diff += W.prom_diff;
    C.dma_bytes += W.dma_bytes;
    C.tokens_total += W.tok;
    C.tokens_computed += W.comp;
    C.extra_prefill += W.extra;
    C.score_evals += W.evals;
    C.resident_evals += W.res_evals;
    C.digest += W.digest;
    C.victim_digest += W.victim_digest;
    C.events += (uint32_t)(e - e0);
    finish_costs(S, P, C);
    store_scalars(a.state[sim], S, e);
    a.counters[sim] = cnt_to(C);
  }
}

template <int SPL, uint32_t POL, uint32_t SMODE, bool DUAL>
__device__ __forceinline__ void lane_row(const SimArgs& a, uint32_t sim, const KeyCtx& K,
                                         uint2* queue, uint64_t* sums) {
  if constexpr (DUAL) {
    if (uni32(a.params[sim].dual_sync)) {
      lane_run<POL, SMODE, true, LaneSim<SPL, POL, SMODE, true>>(a, sim, K, queue, sums, nullptr, 0u);
      return;
    }
  }
  lane_run<POL, SMODE, false, LaneSim<SPL, POL, SMODE, false>>(a, sim, K, queue, sums, nullptr, 0u);
}

// DUAL: a batch with rows of the dual design (the others run as ever).
template <int SPL, bool DUAL>
__global__ __launch_bounds__(64, SPL == 1 && !DUAL ? 4 : SPL <= 2 ? 2 : 1)
void sim_lane_kernel(SimArgs a) {
  __shared__ float s_hf[52];
  __shared__ uint32_t s_hq[52];
  __shared__ uint32_t s_hd[52];
  __shared__ uint32_t s_hn[52];
  __shared__ uint2 s_queue[queue_entries(64u * SPL)];
  __shared__ uint64_t s_sums[kSums * 64u];
  const uint32_t sim = blockIdx.x;
  const unison_sim_params& P = a.params[sim];
  KeyCtx K{};
  K.hf = s_hf;
  K.hq = s_hq;
  K.hd = s_hd;
  K.hn = s_hn;
  K.lambda = (1u << P.b_h) - 1u;
  load_hazard(a, P, sim, K, threadIdx.x, 64);
  __syncthreads();
  switch (sim_policy(a, P)) {
    case kSpear:
      if (P.score_mode) lane_row<SPL, kSpear, 1, DUAL>(a, sim, K, s_queue, s_sums);
      else lane_row<SPL, kSpear, 0, DUAL>(a, sim, K, s_queue, s_sums);
      break;
    case kLru: lane_row<SPL, kLru, 0, DUAL>(a, sim, K, s_queue, s_sums); break;
    case kTimeout: lane_row<SPL, kTimeout, 0, DUAL>(a, sim, K, s_queue, s_sums); break;
    case kBelady: lane_row<SPL, kBelady, 0, DUAL>(a, sim, K, s_queue, s_sums); break;
    default: lane_row<SPL, kEta, 0, DUAL>(a, sim, K, s_queue, s_sums); break;
  }
}

// Residents in sorted lists (ListSim).  Rows with an online hazard table, whose
// keys all change with every completed session, are left to the wide-table kernel.
__global__ __launch_bounds__(64, 1) void sim_list_kernel(SimArgs a, uint32_t cap) {
  __shared__ float s_hf[52];
  __shared__ uint32_t s_hq[52];
  __shared__ uint32_t s_hd[52];
  __shared__ uint32_t s_hn[52];
  __shared__ uint2 s_queue[kListQueue];
  __shared__ uint64_t s_sums[kSums * 64u];
  extern __shared__ uint64_t s_pool[];
  const uint32_t sim = blockIdx.x;
  const unison_sim_params& P = a.params[sim];
  KeyCtx K{};
  K.hf = s_hf;
  K.hq = s_hq;
  K.hd = s_hd;
  K.hn = s_hn;
  K.lambda = (1u << P.b_h) - 1u;
  load_hazard(a, P, sim, K, threadIdx.x, 64);
  __syncthreads();
  const auto go = [&](auto pol, auto mode) {
    constexpr uint32_t POL = decltype(pol)::value, SMODE = decltype(mode)::value;
    lane_run<POL, SMODE, false, ListSim<POL, SMODE>>(a, sim, K, s_queue, s_sums, s_pool, cap);
  };
  using std::integral_constant;
  constexpr integral_constant<uint32_t, 0> zero{};
  switch (sim_policy(a, P)) {
    case kSpear:
      if (P.score_mode) go(integral_constant<uint32_t, kSpear>{}, integral_constant<uint32_t, 1>{});
      else go(integral_constant<uint32_t, kSpear>{}, zero);
      break;
    case kLru: go(integral_constant<uint32_t, kLru>{}, zero); break;
    case kTimeout: go(integral_constant<uint32_t, kTimeout>{}, zero); break;
    case kBelady: go(integral_constant<uint32_t, kBelady>{}, zero); break;
    default: go(integral_constant<uint32_t, kEta>{}, zero); break;
  }
}

template <bool DUAL>
hipError_t launch_width(const SimArgs& a, uint64_t max_res, hipStream_t stream) {
  const dim3 grid(a.n_sims), block(64);
  if (max_res <= 64) hipLaunchKernelGGL((sim_lane_kernel<1, DUAL>), grid, block, 0, stream, a);
  else if (max_res <= 128) hipLaunchKernelGGL((sim_lane_kernel<2, DUAL>), grid, block, 0, stream, a);
  else if (max_res <= 256) hipLaunchKernelGGL((sim_lane_kernel<4, DUAL>), grid, block, 0, stream, a);
  else if (max_res <= 512) hipLaunchKernelGGL((sim_lane_kernel<8, DUAL>), grid, block, 0, stream, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace

// max_res: the most residents any simulation can hold, at most 512.
hipError_t launch_lanes(const SimArgs& a, uint64_t max_res, hipStream_t stream) {
  return a.dual ? launch_width<true>(a, max_res, stream) : launch_width<false>(a, max_res, stream);
}

// max_res: the most residents any simulation can hold, at most kListResidents.
// No row has an online table or the dual design.
hipError_t launch_lists(const SimArgs& a, uint64_t max_res, hipStream_t stream) {
  if (max_res > kListResidents) return hipErrorInvalidValue;
  const uint32_t cap = (uint32_t)((max_res ? max_res : 1) + 63) / 64u * 64u;
  const size_t lds = (size_t)cap * 8u + (size_t)list_rows(cap) * 64u * 12u;
  hipLaunchKernelGGL(sim_list_kernel, dim3(a.n_sims), dim3(64), lds, stream, a, cap);
  return hipGetLastError();
}

}  // namespace unison
