// vsh_persistent.hip -- the batched form: persistent waves that keep every
// lane busy with a fresh event until the work runs out.
//
// The paper's parallel veto algorithm (Sec. 2) runs one step for all events
// in lockstep and leaves finished events idle until the last one reaches the
// cutoff (Fig. 3; Fig. 7 shows the long tail).  Here each lane of a resident
// wave owns one event slot.  After every `period` veto cycles the wave takes a
// ballot of its idle lanes; if at least `threshold` are idle (or all are), one
// lane claims that many event indices from a global work counter with a
// single atomic, and the idle lanes take consecutive indices in lane order
// (prefix count of the ballot below the lane).  A lane whose event finishes
// copies the final partons and summary to the event's own output position.
// A wave exits when the counter is exhausted and none of its lanes is busy.
//
// The work space is a list of segments (request, event range), so events of
// several requests share one launch (serving); observables and histograms are
// computed afterwards per request by k_obs over its output records.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cstring>
#include <type_traits>
#include <vector>

#include "vsh_internal.hpp"
#include "vsh_observables.hpp"
#include "vsh_persistent.hpp"
#include "vsh_shower.hpp"

namespace vsh {

__device__ __forceinline__ uint32_t find_segment(const Segment* segs, uint32_t n, uint64_t w) {
  uint32_t lo = 0, hi = n;  // segs[k].start ascending; find last k with start <= w
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) / 2;
    if (segs[mid].start <= w) lo = mid;
    else hi = mid;
  }
  return lo;
}

// Claim work for the idle lanes of this wave (see the file comment).  Returns
// true for a lane that took an event; sets req/ev and, once the counter is
// exhausted, drained.  Claims are whole multiples of kGranule events, so with
// kGranule = 16 every claim starts on a 16-event boundary and each 128-byte
// line of a record column (16 doubles of consecutive events) belongs to one
// wave: for events that evolve in place, where neighbouring events of
// one line would otherwise be written by waves on different XCDs.  A wave of
// fewer than 64 events (wave_lanes, see events_per_wave) takes them all in
// one claim: such launches hold every event at once, and their waves share
// lines, as those of the one- and two-byte columns always do (an XCD's L2
// writes back the bytes written there).
template <uint32_t kGranule>
__device__ __forceinline__ bool refill(const PersistArgs& A, bool busy, uint32_t wave_lanes, uint32_t lane,
                                      uint32_t& since, bool& drained, uint32_t& req, uint64_t& ev) {
  const uint64_t idle = __ballot(!busy) & (~0ull >> (64 - wave_lanes));
  const uint32_t n_idle = __popcll(idle);
  const uint32_t take = wave_lanes < 64 ? n_idle : n_idle / kGranule * kGranule;
  if (drained || take == 0 || (n_idle != wave_lanes && (since < A.period || n_idle < A.threshold)))
    return false;
  since = 0;
  const uint32_t leader = __ffsll((unsigned long long)idle) - 1;
  unsigned long long base = 0;
  if (lane == leader) base = atomicAdd(A.next, (unsigned long long)take);
  base = __shfl(base, leader);
  if (base + take >= A.total) drained = true;
  if (busy) return false;
  const uint32_t rank = __popcll(idle & ((1ull << lane) - 1));
  const uint64_t w = base + rank;
  if (rank >= take || w >= A.total) return false;  // lanes past wave_lanes have rank n_idle
  const uint32_t sg = find_segment(A.segs, A.n_segs, w);
  req = A.segs[sg].req;
  ev = A.segs[sg].lo + (w - A.segs[sg].start);
  return true;
}

// Start event ev of request R in working slot `slot`.  In place, the slots
// are R's own output records, where the matrix-element pass has already
// left the LO partons and their partner links.
template <bool kInPlace>
__device__ __forceinline__ void start_event(EvState& s, const PersistArgs& A, const ReqDev& R, uint64_t ev,
                                            uint64_t slot) {
  const double ecm = R.ecm ? R.ecm[ev] : R.ecm0;
  const double tcut = R.tcut ? R.tcut[ev] : R.tcut0;
  const Keyed key = make_keyed(R.seed, R.first + ev);
  if (kInPlace) lo_state(s, key, ecm, tcut, R.t_over, (int)R.out.cap);
  else start_from_record(s, R.out, ev, A.slots, slot, key, ecm, tcut, R.t_over, (int)R.out.cap);
}

// Record a finished event: its summary, and (unless in place) its partons
// copied from the working slot to the request's output.
template <bool kInPlace>
__device__ __forceinline__ void finish_event(const EvState& s, const PersistArgs& A, const ReqDev& R, uint64_t ev,
                                             uint64_t slot) {
  if (!kInPlace) {
    const Records& o = R.out;
    for (int a = 0; a < s.n; ++a) {
      const uint64_t from = (uint64_t)a * A.slots.stride + slot;
      const uint64_t to = (uint64_t)a * o.stride + ev;
      o.E[to] = A.slots.E[from];
      o.x[to] = A.slots.x[from];
      o.y[to] = A.slots.y[from];
      o.z[to] = A.slots.z[from];
      o.pid[to] = A.slots.pid[from];
      o.col[to] = A.slots.col[from];
      o.acol[to] = A.slots.acol[from];
    }
  }
  write_state(s, R.sum, ev);
}

template <bool kInPlace, bool kMassive = false>
__global__ void __launch_bounds__(256) k_shower_persistent(PersistArgs A) {
  const uint64_t L = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;  // this lane's working slot
  const uint32_t lane = __lane_id();
  const uint32_t wave_lanes = __popcll(__ballot(1));
  EvState s = {};
  s.status = kDone;
  bool busy = false;
  bool drained = false;
  uint32_t req = 0;
  uint64_t ev = 0;  // event index within its request
  uint64_t slot = L;
  uint32_t since = 0;
  while (true) {
    if (refill<(kInPlace ? 16u : 1u)>(A, busy, wave_lanes, lane, since, drained, req, ev)) {
      slot = kInPlace ? ev : L;
      start_event<kInPlace>(s, A, A.reqs[req], ev, slot);
      busy = true;
    }
    if (!__any(busy)) break;  // counter exhausted and nothing left in this wave
    if (busy) {
      if constexpr (kMassive) veto_cycle_massive(s, A.slots, slot, A.reqs[req].qm);
      else veto_cycle(s, A.slots, slot);
      if (s.status == kRunning && s.cycle >= A.reqs[req].cycle_limit) s.status = kCycleLimitHit;
      if (s.status != kRunning) {
        finish_event<kInPlace>(s, A, A.reqs[req], ev, slot);
        busy = false;
      }
    }
    ++since;
  }
}

// ---------------------------------------------------------------------------
// Flattened mapping.  Same refill as above, but each veto cycle's trials of a
// wave's 64 events are spread over its 64 lanes: the work items are the
// partons of all busy events, taken 64 per round; item (owner o, parton i)
// runs that parton's dipole ends.  A gluon item (two ends, three Philox
// blocks and two trials per end) costs about four quark items (one end, one
// block, one trial), so gluon and quark partons get rounds of their own: first
// the gluons of every event (event-major), padded to a whole round, then the
// quarks.  Each event keeps a bit mask of its gluon slots in LDS, so item r of
// an owner is its r-th set (or clear) bit.  Trials are ranked by their
// single-precision bounds (trial_bound): an item's lowest bound, with its
// (i, k, K) below it in one 64-bit key, goes into its owner's minimum in LDS by
// an atomic, what it displaces into the runner-up's.  Each owner then computes
// the exact scale of its winner and decides its own cycle; where the runner-up
// is not proven to lose, its lane compares all the cycle's trials exactly in
// the paper's loop order (the first of equal trials wins).  Against exact
// logarithms for every trial and a segmented maximum by shuffles, 10^6 events:
// plain LEP showers 3.04 -> 2.63 ms, t_C = 0.25 GeV^2 at 500 GeV 27.8 -> 20.6.
// ---------------------------------------------------------------------------
// Launch-wide constants of the kernels whose events all belong to one
// request: each event's key is make_keyed(seed, first + its record column)
// and the cycle limit is one, so neither is kept per event in LDS (kOne),
// and, for four waves per SIMD (kFour, records of at most 128 partons), the
// item list (whose free tail holds the stale partons) is shorter (its
// overflow takes the offsets' path): 8.1 KB + 1 or 2 KB of masks, sixteen
// blocks per CU (a list of 1124 entries, fourteen at 128 partons: 2% slower at
// 200 GeV).  With
// 256-parton records the layout leaves room for one more block per CU.
struct OneRequest {
  uint64_t seed, first;
  uint32_t climit;
};
constexpr uint32_t kOneAboveCap = 64;  // massive plain kernel: the per-event layout up to here
constexpr uint32_t kFourMaxCap = 128;  // massless: four-wave builds up to here (LDS-bound above)

template <bool kMassive_, bool kOne_, bool kFour_ = false, bool kRegW_ = false>
struct FlatShared {
  static constexpr bool kOne = kOne_, kFour = kFour_, kRegW = kRegW_;
  double lt[64], tcut[64], ltc[64], cfac[64];
  uint32_t slot[64];  // record columns (a launch covers fewer than 2^32)
  uint32_t key[4][kOne ? 1 : 64];
  uint32_t cycle[64];
  uint8_t rank[64];     // of the events that make trials: their first pair
  uint8_t ranked[64];   // and the events in order of rank
  uint32_t gstart[65], qstart[65];  // per-owner item offsets in the gluon and quark sections
  uint32_t sstart[65];              // per-owner offsets in the list of stale partons
  // the cycle's items, owner << 10 | parton: gluon items (a gluon twice,
  // once per dipole end, when rounds allow), then quark items, then the
  // stale partons in what the items leave free (two spare entries)
  alignas(4) uint16_t item[(kFour ? 768 : kRegW ? 1124 : 1408) + 4];
  // per (event, cycle) pair: its trials' lowest bound << 32 | packed (i, k, K),
  // and the lowest bound of the others
  uint64_t best[64];
  uint32_t second[64];
  // per pair: the lowest one's uniform and coefficients (unless kRedraw); later, of
  // cycles evaluated ahead, ln t, t, z (and, in best, the weight)
  double pair[3][64];
  uint32_t counts[64];  // the cycle's trials (low 16 bits) and active ends (high 16 bits) per owner
  uint32_t climit[kOne ? 1 : 64];  // each event's cycle limit
  double wsh[kRegW ? 1 : 64];  // each event's shower weight (weighted veto), unless held in a register
  double mc[kMassive_ ? 64 : 1], mb[kMassive_ ? 64 : 1];  // each event's charm and bottom masses
};

// per-owner gluon masks, then per-owner stale masks (partons whose cached end
// coefficients must be recomputed), ceil(cap / 64) words each, in dynamic LDS
extern __shared__ uint64_t flat_gmask[];

__device__ __forceinline__ uint32_t mask_words(uint32_t cap) { return (cap + 63) / 64; }


__device__ __forceinline__ uint32_t owner_of(const uint32_t* start, uint32_t j) {
  uint32_t lo = 0, hi = 64;  // last o with start[o] <= j (owners with no items have start[o] == start[o+1])
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) / 2;
    if (start[mid] <= j) lo = mid;
    else hi = mid;
  }
  return lo;
}

// position of the r-th (from 0) set bit of x; x has more than r set bits
__device__ __forceinline__ uint32_t select64(uint64_t x, uint32_t r) {
  uint32_t pos = 0;
#pragma unroll
  for (uint32_t w = 32; w >= 1; w >>= 1) {
    const uint32_t c = __popcll(x & ((1ull << w) - 1));
    if (r >= c) {
      r -= c;
      x >>= w;
      pos += w;
    }
  }
  return pos;
}

// slot of the r-th gluon (gluon = true) or r-th quark of an event's mask
__device__ __forceinline__ uint32_t select_slot(const uint64_t* m, uint32_t words, uint32_t r, bool gluon) {
  for (uint32_t w = 0; w < words; ++w) {
    const uint64_t x = gluon ? m[w] : ~m[w];
    const uint32_t c = __popcll(x);
    if (r < c) return 64 * w + select64(x, r);
    r -= c;
  }
  return 0;  // not reached for r below the owner's count
}

// The gluon mask of the event in column `slot`, from its partons' ids, and
// its stale mask with every parton set.
__device__ __forceinline__ void mask_init(uint64_t* m, uint64_t* st, uint32_t words, const Records& r,
                                          uint64_t slot, int n) {
  for (uint32_t w = 0; w < words; ++w) {
    m[w] = 0ull;
    const int lo = 64 * (int)w;
    st[w] = n >= lo + 64 ? ~0ull : (n > lo ? (1ull << (n - lo)) - 1ull : 0ull);
  }
  for (int a = 0; a < n; ++a)
    if (r.pid[(uint64_t)a * r.stride + slot] == kGluon) m[a >> 6] |= 1ull << (a & 63);
}

__device__ __forceinline__ void set_bit(uint64_t* m, int a) {
  if (a >= 0 && a != kNoPartner) m[a >> 6] |= 1ull << (a & 63);
}

// Trials of parton i of the event in column `slot`.  Each lane's event keeps,
// per parton, one cache entry of kCacheWords words at
// rec[((col * cap) + i) * kCacheWords]: its id and its spectators in
// ascending order (packed in word 0), then per end the trial coefficients
// (quark kernel or g -> g g, and g -> f fbar; 0 = no phase space; a quark
// end keeps the g -> f fbar form cfac T_R/2 (z+ - z-) too, from which the
// decision recovers the end's range and mass).  An entry
// changes only when an emission touches the parton or its partners, which
// marks it stale: then it is rebuilt from the records (the values a
// recomputation gives).  A fresh parton needs nothing but its entry.  Same
// trials, same order, same winner as parton_trials.
__device__ __forceinline__ uint64_t pack_meta(int pid, int k1, int k2) {
  return (uint64_t)(uint8_t)(int8_t)pid | ((uint64_t)(uint16_t)k1 << 8) | ((uint64_t)(uint16_t)k2 << 24);
}

// The entry of parton i of column o of a wave's cache (the wave's first column
// at ec.rec): the base is the same for all lanes and the offset fits 32 bits,
// so the address costs three instructions instead of a dozen.
template <int kW>
__device__ __forceinline__ uint64_t* entry_at(const EndCache& ec, uint32_t o, uint32_t i) {
  return (uint64_t*)((char*)ec.rec + (o * ec.cap + i) * (uint32_t)(8 * kW));
}
template <int kW>
__device__ __forceinline__ EndCache wave_cache(const EndCache& ec, uint64_t wave_col) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)wave_col),
                 hi = __builtin_amdgcn_readfirstlane((uint32_t)(wave_col >> 32));
  return EndCache{ec.rec ? ec.rec + (((uint64_t)hi << 32) | lo) * ec.cap * kW : ec.rec, ec.cap};
}

// Rebuild the cache entry of parton i of the event in column `slot` from the
// records (the stale rounds of a cycle).
__device__ __forceinline__ void entry_build(double cfac, double tcut, const Records& r, uint64_t slot, int i,
                                            const EndCache& ec, uint32_t col) {
  uint64_t* ent = entry_at<kCacheWords>(ec, col, (uint32_t)i);
  const uint64_t oi = (uint64_t)i * r.stride + slot;
  const int pid_i = r.pid[oi];
  int k1 = r.cpart[oi], k2 = r.apart[oi];
  if (k2 == k1) k2 = kNoPartner;
  if (k1 > k2) {
    const int t = k1;
    k1 = k2;
    k2 = t;
  }
  const P4 pi = r.load(i, slot);
  uint64_t w[kCacheWords];
  w[0] = pack_meta(pid_i, k1, k2);
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int k = e == 0 ? k1 : k2;
    double ia = 0.0, ib = 0.0;  // 0: no end, or no phase space above the cutoff
    if (k != kNoPartner) {
      double q2, zm, zp, L;
      if (!end_coeffs(cfac, tcut, pid_i, pi, r.load(k, slot), q2, zm, zp, L, ia, ib)) ia = ib = 0.0;
    }
    w[1 + 2 * e] = (uint64_t)__double_as_longlong(ia);
    w[2 + 2 * e] = (uint64_t)__double_as_longlong(ib);
  }
#pragma unroll
  for (int q = 0; q < kCacheWords; ++q) ent[q] = w[q];
}

// The same for an event with quark masses: per end the four class
// coefficients of massive_end_coeffs.
__device__ __forceinline__ void entry_build_massive(double cfac, double tcut, const Records& r, uint64_t slot, int i,
                                                    const EndCache& ec, uint32_t col, const QuarkMasses& qm) {
  uint64_t* ent = entry_at<kMCacheWords>(ec, col, (uint32_t)i);
  const uint64_t oi = (uint64_t)i * r.stride + slot;
  const int pid_i = r.pid[oi];
  int k1 = r.cpart[oi], k2 = r.apart[oi];
  if (k2 == k1) k2 = kNoPartner;
  if (k1 > k2) {
    const int t = k1;
    k1 = k2;
    k2 = t;
  }
  const P4 pi = r.load(i, slot);
  const TrialCtx c{Keyed{0u, 0u, 0u, 0u}, 0.0, tcut, 0.0, cfac, 0u};  // the ranges read t_C and cfac only
  uint64_t w[kMCacheWords];
  w[0] = pack_meta(pid_i, k1, k2);
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int k = e == 0 ? k1 : k2;
    double cc[4] = {0.0, 0.0, 0.0, 0.0};
    if (k != kNoPartner) massive_end_coeffs(c, pid_i, r.pid[(uint64_t)k * r.stride + slot], pi, r.load(k, slot), qm, cc);
#pragma unroll
    for (int q = 0; q < 4; ++q) w[1 + 4 * e + q] = (uint64_t)__double_as_longlong(cc[q]);
  }
#pragma unroll
  for (int q = 0; q < kMCacheWords; ++q) ent[q] = w[q];
}

// An item's end-cache entry, when loaded ahead of its round.
struct Ent5 {
  uint64_t w[kCacheWords];
};

// A parton's id, its spectators in ascending order and its ends' trial
// coefficients: (1/ca, 1/cb), or with quark masses the four of
// massive_end_coeffs; 0 for no phase space above the cutoff.
template <bool kMassive>
struct Ends {
  static constexpr int kC = kMassive ? 4 : 2;
  int pid, k[2];
  double c[2][kC];
};

// Those of ends e_lo .. e_hi of parton i: from its fresh cache entry
// (kCached; the stale rounds rebuilt it; already loaded if pre) or from the
// records.
template <bool kCached, bool kMassive>
__device__ __forceinline__ Ends<kMassive> load_ends(const TrialCtx& c, const Records& r, uint64_t slot, int i, int e_lo,
                                                    int e_hi, const EndCache& ec, uint32_t col, bool pre,
                                                    const Ent5& pw, const QuarkMasses& qm) {
  constexpr int kC = Ends<kMassive>::kC;
  Ends<kMassive> E;
  if constexpr (kCached) {
    constexpr int kW = kMassive ? kMCacheWords : kCacheWords;
    static_assert(kW == 1 + 2 * kC);
    const uint64_t* ent = entry_at<kW>(ec, col, (uint32_t)i);
    uint64_t w[kW];
#pragma unroll
    for (int q = 0; q < kW; ++q) {
      if constexpr (kMassive) w[q] = ent[q];
      else w[q] = pre ? pw.w[q] : ent[q];
    }
    E.pid = (int)(int8_t)(uint8_t)(w[0] & 0xFFu);
    E.k[0] = (int)((w[0] >> 8) & 0xFFFFu);
    E.k[1] = (int)((w[0] >> 24) & 0xFFFFu);
#pragma unroll
    for (int e = 0; e < 2; ++e)
#pragma unroll
      for (int q = 0; q < kC; ++q) E.c[e][q] = __longlong_as_double((long long)w[1 + kC * e + q]);
  } else {
    const uint64_t oi = (uint64_t)i * r.stride + slot;
    E.pid = r.pid[oi];
    int k1 = r.cpart[oi], k2 = r.apart[oi];
    if (k2 == k1) k2 = kNoPartner;
    E.k[0] = k1 < k2 ? k1 : k2;
    E.k[1] = k1 < k2 ? k2 : k1;
    const P4 pi = r.load(i, slot);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int k = E.k[e];
#pragma unroll
      for (int q = 0; q < kC; ++q) E.c[e][q] = 0.0;
      if (e < e_lo || e > e_hi || k == kNoPartner) continue;
      if constexpr (kMassive) {
        massive_end_coeffs(c, E.pid, r.pid[(uint64_t)k * r.stride + slot], pi, r.load(k, slot), qm, E.c[e]);
      } else {
        double q2, zm, zp, L;
        if (!end_coeffs(c.cfac, c.tcut, E.pid, pi, r.load(k, slot), q2, zm, zp, L, E.c[e][0], E.c[e][1]))
          E.c[e][0] = E.c[e][1] = 0.0;
      }
    }
  }
  return E;
}

// Trials of one item, ranked by their bounds: ends e_lo .. e_hi of parton i (a
// massless gluon's item takes one or both of its ends; a quark's both, the
// second empty as a quark has one colour partner).
template <bool kMassive>
__device__ __forceinline__ void item_bounds(const TrialCtx& c, int i, const Ends<kMassive>& E, int e_lo, int e_hi,
                                            LowTrial& low, uint32_t& trials, uint32_t& ends) {
  // the q-th end of the item is end e_lo + q: lanes of gluon items with
  // different ends and of quark items take their first end together
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int e = e_lo + q;
    const int k = e == 0 ? E.k[0] : E.k[1];
    if (e > e_hi || k == kNoPartner) continue;
    if constexpr (kMassive) {  // both ends, in order
      end_bounds_massive(c.key, c.cycle, i, k, E.pid, E.c[q], low, trials, ends);
    } else {
      const double ia = e == 0 ? E.c[0][0] : E.c[1][0], ib = e == 0 ? E.c[0][1] : E.c[1][1];
      if (ia == 0.0) continue;  // no phase space above the cutoff
      ends += 1;
      end_bounds(c.key, c.cycle, i, k, E.pid, ia, ib, low, trials);
    }
  }
}

// The winner of one cycle of the event in column `slot` (n partons) by the
// exact comparison in the paper's loop order (strict maximum above `best`):
// packed (i, k, K), its scale in `best` and its end's coefficients.  One lane,
// where the bounds did not prove the order.
template <bool kCached, bool kMassive>
__device__ __forceinline__ uint32_t exact_winner(const TrialCtx& c, const Records& r, uint64_t slot, int n,
                                                 const EndCache& ec, uint32_t col, const QuarkMasses& qm,
                                                 double& best, double& ca, double& cb) {
  uint32_t idx = kNoTrial, trials = 0, ends = 0;
#pragma unroll 1
  for (int i = 0; i < n; ++i) {
    const Ends<kMassive> E =
        load_ends<kCached, kMassive>(c, r, slot, i, 0, 1, ec, col, false, Ent5{}, qm);
#pragma unroll 1
    for (int e = 0; e < 2; ++e) {
      const int k = e ? E.k[1] : E.k[0];
      if (k == kNoPartner) continue;
      double cc[Ends<kMassive>::kC];
#pragma unroll
      for (int q = 0; q < Ends<kMassive>::kC; ++q) cc[q] = e ? E.c[1][q] : E.c[0][q];
      int K = -1;
      if constexpr (kMassive) K = end_draws_massive(c, i, k, E.pid, cc, best, trials, ends);
      else if (cc[0] != 0.0) K = end_draws(c, i, k, E.pid, cc[0], cc[1], best, trials);
      if (K >= 0) {
        idx = pack_trial(i, k, K);
        ca = cc[0];
        cb = cc[1];
      }
    }
  }
  return idx;
}

// Load the end-cache entry of the item at list position `at` into pw; false
// (nothing loaded) past the cycle's items or the list's end.
__device__ __forceinline__ bool prefetch_entry(const uint16_t* item, uint32_t at, uint32_t n_items, uint32_t n_list,
                                               const EndCache& ec, Ent5& pw) {
  if (at >= n_items || at >= n_list) return false;
  const uint32_t it = item[at];
  const uint64_t* ent = entry_at<kCacheWords>(ec, it >> 10, it & 1023u);
#pragma unroll
  for (int q = 0; q < kCacheWords; ++q) pw.w[q] = ent[q];
  return true;
}

// One veto cycle of every busy event of this wave whose last accepted
// emission has been built, the trials spread over the lanes; each owner lane
// then decides its own event's cycle.  An accepted emission stays pending
// (the event makes no trials meanwhile) until at least half of the busy
// events have one; then the wave builds them together (a quarter, three
// quarters and all of them measured slower on LEP, mixed and stress events).
// Deferring an emission changes nothing in the event: its random numbers are
// keyed by the event's own cycle.  The event of the calling lane sits in
// column `slot` of `slots`; its gluon mask at gm + lane * words.
constexpr uint32_t kEmitDiv = 2;

// kCached: the kernel has an end cache (ec); the cycle then starts with
// rounds that rebuild the entries of stale partons, so that every trial
// round reads fresh entries only.  Without it, each item computes its
// parton's coefficients itself.  kMassive: the events carry quark masses
// (qm, the calling lane's event's); no end cache, the owner recomputes its
// winner's range from the records.
// kAhead: the owner's trial constants (key, scales, cycle) are reloaded from
// LDS after the rounds, so their registers are free during them; for
// massless cached events each round then loads the end-cache entries of the
// next round's items while it reduces its winners.  The four-wave builds
// take it to fit 128 registers; at three waves the plain kernel takes it
// with quark masses only (for massless events it measured 1% slower there).
//
// kAheadCycles (cached events): a wave cycle may evaluate K = 2^m
// consecutive veto cycles of each event that makes trials.  A trial's scale
// is ln t + ln(R)/c, with c fixed until an emission changes the event, so
// between emissions the winner of a veto cycle (the lowest |ln R|/c) does
// not depend on the scale it starts from; only the decision does.  The
// rounds therefore draw the trials of cycles c .. c+K-1 together (item j of
// cycle k at position j K + k of its section, keyed by that cycle), each
// (event, cycle) pair keeps its lowest bound, then one lane per pair takes
// that trial's exact ln(R)/c, chains
// the scales in order (ln t of cycle k = that of cycle k-1 plus the pair's
// best, the same additions a cycle-by-cycle evaluation makes) and makes the
// pair's CheckCutoff, alpha_s and AcceptOrVeto with the pair's accept block.
// Each event then takes its pairs in order up to the first that ends the
// cycle sequence (cutoff, acceptance, cycle limit); later pairs are dropped
// and drawn again, keyed by the same cycles, after the emission.  K is the
// largest power of two with at most 64 pairs, at most kAheadMax cycles and
// at most kAheadRounds more rounds than one cycle's items take (2, 3, 5, 8 and
// 16 rounds at 500 GeV: 21.1, 20.5, 20.0, 19.8, 19.8 ms per 10^6 events; LEP
// within 1%).  With quark masses it took 250000 events from 1.71 to 1.36 ms.
constexpr uint32_t kAheadLgMax = 3;  // kAheadMax = 8
constexpr uint32_t kAheadRounds = 8;
enum : uint32_t { kPairVeto = 0, kPairAccept = 1, kPairDone = 2, kPairLimit = 3 };

__device__ __forceinline__ uint32_t list_pos(uint32_t v, uint32_t vg, uint32_t n_g, uint32_t lg) {
  return v < vg ? v >> lg : n_g + ((v - vg) >> lg);
}

template <bool kCached, bool kMassive = false, bool kAhead = false, bool kAheadCycles = false, bool kOne = false,
          class SH>
__device__ __forceinline__ void flat_cycle(SH& sh, const OneRequest& one, uint64_t* gm, uint32_t words, EvState& s, bool busy,
                                           bool& pend, Pending& pd, const Records& slots, uint64_t slot,
                                           const EndCache& cache, uint64_t wave_col, uint32_t lane,
                                           const QuarkMasses& qm = QuarkMasses{0.0, 0.0, 0.0, 0.0, 0.0}) {
  // kRedraw: the winner's uniform and coefficients are drawn and read again
  // when the cycle is decided; otherwise each round's lanes that hold a pair's
  // best write them to LDS.  The long showers of large records have enough
  // rounds per cycle for the first (500 GeV, 256 partons: 20.6 against 21.7 ms
  // per 10^6 events), the others do not (mixed energies: 7.4 against 7.2 ms
  // per 3 10^6).
  constexpr bool kRedraw = kCached && !kMassive && kOne && !SH::kFour;
  const EndCache ec = wave_cache<kMassive ? kMCacheWords : kCacheWords>(cache, wave_col);
  const bool trial = busy && !pend;
  // this lane's event's shower weight: in LDS, or (kRegW) in the event state
  auto wsh = [&]() -> double& {
    if constexpr (SH::kRegW) return s.wsh;
    else return sh.wsh[lane];
  };
  // the key and cycle limit of the event in column o of this wave
  // (kOne: the seed's words come from LDS at each use, so that the
  // compiler does not hold Philox's round keys in registers for the kernel)
  auto key_of = [&](uint32_t o) -> Keyed {
    if constexpr (kOne) {
      const uint64_t ev = one.first + sh.slot[o];
      return Keyed{(uint32_t)ev, (uint32_t)(ev >> 32), sh.key[2][0], sh.key[3][0]};
    } else {
      return Keyed{sh.key[0][o], sh.key[1][o], sh.key[2][o], sh.key[3][o]};
    }
  };
  auto climit_of = [&](uint32_t o) -> uint32_t {
    if constexpr (kOne) return one.climit;
    else return sh.climit[o];
  };
  uint64_t* mym = gm + (uint64_t)lane * words;
  uint64_t* sm = gm + (uint64_t)64 * words;  // stale masks
  uint64_t* mys = sm + (uint64_t)lane * words;
  // --- publish the events that make trials, the item ranges of both
  // sections and of the stale partons (counts in 21-bit fields: at most 64
  // events of 1024 partons)
  constexpr uint64_t kF = (1ull << 21) - 1;
  uint32_t ng = 0, ns = 0;
  if (trial)
    for (uint32_t w = 0; w < words; ++w) {
      const int lo = 64 * (int)w;
      const uint64_t live = s.n >= lo + 64 ? ~0ull : (s.n > lo ? (1ull << (s.n - lo)) - 1ull : 0ull);
      ng += __popcll(mym[w] & live);
      if (kCached) ns += __popcll(mys[w] & live);
    }
  const uint64_t mine = trial ? ((uint64_t)ng | ((uint64_t)((uint32_t)s.n - ng) << 21) | ((uint64_t)ns << 42)) : 0ull;
  const uint64_t incl = wave_inclusive_sum(mine);  // every lane of the wave takes part
  const uint64_t excl = incl - mine;
  const uint64_t tot = lane63(incl);
  const uint32_t n_g1 = (uint32_t)(tot & kF), n_q = (uint32_t)((tot >> 21) & kF), n_s = (uint32_t)(tot >> 42);
  // cycles evaluated ahead: K = 2^lg_ (1 without kAheadCycles); a trialing
  // event's rank is the number of trialing lanes below its own
  uint32_t lg_ = 0;
  const uint64_t tmask = kAheadCycles ? __ballot(trial) : 0ull;
  if (kAheadCycles) {
    const uint32_t n_tr = (uint32_t)__popcll(tmask), n1 = n_g1 + n_q, r1 = (n1 + 63) / 64;
    while (lg_ < kAheadLgMax && (n_tr << (lg_ + 1)) <= 64u && ((n1 << (lg_ + 1)) + 63) / 64 <= r1 + kAheadRounds)
      ++lg_;
  }
  const uint32_t lg = lg_, K = 1u << lg_;
  // (kPairs: the pairs' decision serves K = 1 too: one copy of its arithmetic,
  // and fewer registers; kRedraw's kernels keep the owners' own for K = 1, 2.5%
  // faster at 500 GeV)
  constexpr bool kPairs = kAheadCycles && !kRedraw;
  const bool ahead = kPairs || (kAheadCycles && lg_ > 0);
  // A massless gluon's two dipole ends become two items (half the longest
  // lane's work in a round) whenever that takes no more rounds than one item
  // per gluon; otherwise, and with quark masses, one item per gluon.
  const uint32_t kge = !kMassive && (K * (2 * n_g1 + n_q) + 63) / 64 == (K * (n_g1 + n_q) + 63) / 64 ? 2u : 1u;
  const uint32_t n_g = kge * n_g1;
  const uint32_t vg = K * n_g, vt = vg + K * n_q;  // positions of the rounds: gluon items, then quark items
  if (kAheadCycles && trial) {
    const uint32_t rk = __builtin_amdgcn_mbcnt_hi((uint32_t)(tmask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)tmask, 0u));
    sh.rank[lane] = (uint8_t)(rk << lg_);
    sh.ranked[rk] = (uint8_t)lane;
  }
  sh.gstart[lane] = kge * (uint32_t)(excl & kF);
  sh.qstart[lane] = (uint32_t)((excl >> 21) & kF);
  sh.sstart[lane] = (uint32_t)(excl >> 42);
  if (lane == 63) {
    sh.gstart[64] = n_g;
    sh.qstart[64] = n_q;
    sh.sstart[64] = n_s;
  }
  // list length; a spare entry past its end takes the writes beyond it, so
  // the listing loops need no branch.  The stale partons follow the items.
  constexpr uint32_t kItems = sizeof(sh.item) / sizeof(sh.item[0]) - 2;
  const uint32_t sbase = n_g + n_q < kItems ? n_g + n_q : kItems;
  if (n_g + n_q + n_s <= kItems && !__any(trial && s.n > 32)) {
    // all in the list, and each event's masks one word: half the instructions
    // of the general listing below, which are a tenth of an LEP shower's
    if (trial) {
      const uint32_t live = s.n >= 32 ? ~0u : (1u << s.n) - 1u, m = (uint32_t)mym[0], top = lane << 10;
      uint16_t* w = sh.item + n_g + (uint32_t)((excl >> 21) & kF);
      for (uint32_t x = ~m & live; x; x &= x - 1) *w++ = (uint16_t)(top | (uint32_t)__builtin_ctz(x));  // quarks
      if (kge == 2) {  // both of a gluon's ends at once
        uint32_t* w2 = (uint32_t*)sh.item + (uint32_t)(excl & kF);
        for (uint32_t x = m & live; x; x &= x - 1) *w2++ = (top | (uint32_t)__builtin_ctz(x)) * 0x10001u;
      } else {
        w = sh.item + (uint32_t)(excl & kF);
        for (uint32_t x = m & live; x; x &= x - 1) *w++ = (uint16_t)(top | (uint32_t)__builtin_ctz(x));
      }
      if (kCached) {
        w = sh.item + sbase + (uint32_t)(excl >> 42);
        for (uint32_t x = (uint32_t)mys[0] & live; x; x &= x - 1) *w++ = (uint16_t)(top | (uint32_t)__builtin_ctz(x));
      }
    }
  } else if (trial) {  // list this event's items (beyond the lists' lengths rounds search the offsets instead)
    uint32_t gpos = kge * (uint32_t)(excl & kF), qpos = n_g + (uint32_t)((excl >> 21) & kF),
             spos = (uint32_t)(excl >> 42);
    for (uint32_t w = 0; w < words; ++w) {
      const int lo = 64 * (int)w;
      const uint64_t live = s.n >= lo + 64 ? ~0ull : (s.n > lo ? (1ull << (s.n - lo)) - 1ull : 0ull);
      const uint32_t top = (lane << 10) | (uint32_t)lo;
      for (uint64_t x = mym[w] & live; x; x &= x - 1) {  // gluons, ascending
        const uint16_t item = (uint16_t)(top | (uint32_t)__builtin_ctzll(x));
        sh.item[gpos < kItems ? gpos : kItems] = item;
        sh.item[gpos + kge - 1 < kItems ? gpos + kge - 1 : kItems] = item;  // the second end's item
        gpos += kge;
      }
      for (uint64_t x = ~mym[w] & live; x; x &= x - 1) {  // quarks, ascending
        sh.item[qpos < kItems ? qpos : kItems] = (uint16_t)(top | (uint32_t)__builtin_ctzll(x));
        ++qpos;
      }
      if (kCached)
        for (uint64_t x = mys[w] & live; x; x &= x - 1) {  // stale partons
          sh.item[sbase + spos < kItems ? sbase + spos : kItems] = (uint16_t)(top | (uint32_t)__builtin_ctzll(x));
          ++spos;
        }
    }
  }
  sh.lt[lane] = s.lt;
  sh.tcut[lane] = s.tcut;
  sh.ltc[lane] = s.ltc;
  sh.cfac[lane] = s.cfac;
  sh.slot[lane] = (uint32_t)slot;
  if constexpr (!kOne) {
    sh.key[0][lane] = s.key.ev_lo;
    sh.key[1][lane] = s.key.ev_hi;
    sh.key[2][lane] = s.key.k0;
    sh.key[3][lane] = s.key.k1;
  } else if (lane == 0) {
    sh.key[2][0] = (uint32_t)one.seed;
    sh.key[3][0] = (uint32_t)(one.seed >> 32);
  }
  sh.cycle[lane] = s.cycle;
  sh.best[lane] = ~0ull;
  sh.second[lane] = kNoBound;
  sh.counts[lane] = 0;
  if (kMassive) {
    sh.mc[lane] = qm.c;
    sh.mb[lane] = qm.b;
  }
  __syncthreads();
  // --- rebuild the cache entries of the stale partons, 64 per round
  if (kCached && n_s > 0) {
    for (uint32_t r0 = 0; r0 < n_s; r0 += 64) {
      const uint32_t at = r0 + lane;
      if (at < n_s) {
        uint32_t o, i;
        if (sbase + at < kItems) {
          const uint32_t it = sh.item[sbase + at];
          o = it >> 10;
          i = it & 1023u;
        } else {
          o = owner_of(sh.sstart, at);
          i = select_slot(sm + (uint64_t)o * words, words, at - sh.sstart[o], true);
        }
        if constexpr (kMassive)
          entry_build_massive(sh.cfac[o], sh.tcut[o], slots, sh.slot[o], (int)i, ec, o,
                              QuarkMasses{0.0, 0.0, 0.0, sh.mc[o], sh.mb[o]});
        else
          entry_build(sh.cfac[o], sh.tcut[o], slots, sh.slot[o], (int)i, ec, o);
      }
    }
    __threadfence_block();  // the rebuilt entries are stored before any trial round reads them
    __syncthreads();
    if (trial)
      for (uint32_t w = 0; w < words; ++w) mys[w] = 0ull;
  }
  // --- trials, 64 items per round: the gluon items, then the quark items
  // (a round may hold the end of one and the start of the other: its quark
  // lanes finish early, in time the round takes for its gluons anyway); with
  // cycles evaluated ahead, item j of a section takes its positions j K ..
  // j K + K - 1, one per cycle, so each (event, cycle) run strides by K
  // the end-cache entry of the lane's item in the coming round is loaded
  // while the current round reduces its winners (an item past the list's
  // end loads its own)
  constexpr bool kPre = kAhead && kCached && !kMassive;
  Ent5 pw{{0ull, 0ull, 0ull, 0ull, 0ull}};
  bool pre = false;
  if (kPre) pre = prefetch_entry(sh.item, list_pos(lane, vg, n_g, lg), n_g + n_q, kItems, ec, pw);
  // (the rounds' code compiled twice: one cycle at a time it takes no cycle
  // index and no pair rank)
  auto rounds = [&](auto kA) {
    constexpr bool A = decltype(kA)::value;
    const uint32_t lg = A ? lg_ : 0u, K = 1u << lg;
    for (uint32_t r0 = 0; r0 < vt; r0 += 64) {
      const uint32_t at = r0 + lane;  // position in the rounds
      const bool gsec = at < vg;
      const uint32_t* st = gsec ? sh.gstart : sh.qstart;
      const uint32_t vbase = gsec ? 0u : vg;  // first position of the section
      const uint32_t j = (at - vbase) >> lg;  // item index within the section
      const uint32_t k = (at - vbase) & (K - 1u);  // cycle ahead
      const bool active = at < vt;
      LowTrial low;
      uint32_t i = 0, pr = 63;
      if (active) {
        uint32_t o;
        const uint32_t lp = (gsec ? 0u : n_g) + j;  // list position
        if (lp < kItems) {
          const uint32_t it = sh.item[lp];
          o = it >> 10;
          i = it & 1023u;
        } else {
          o = owner_of(st, j);
          i = select_slot(gm + (uint64_t)o * words, words, gsec ? (j - st[o]) / kge : j - st[o], gsec);
        }
        // a gluon item's ends: both, or (two items per gluon) the parity of
        // its place in the owner's run
        const int e_lo = gsec && kge == 2 ? (int)((j - st[o]) & 1u) : 0, e_hi = gsec && kge == 2 ? e_lo : 1;
        pr = A ? sh.rank[o] | k : o;
        const TrialCtx c{key_of(o), 0.0, sh.tcut[o], 0.0, sh.cfac[o], sh.cycle[o] + k};
        QuarkMasses om{0.0, 0.0, 0.0, 0.0, 0.0};
        if constexpr (kMassive) om = QuarkMasses{0.0, 0.0, 0.0, sh.mc[o], sh.mb[o]};
        const Ends<kMassive> E = load_ends<kCached, kMassive>(c, slots, sh.slot[o], (int)i, e_lo, e_hi, ec, o,
                                                              kPre && pre, pw, om);
        uint32_t nt = 0, ne = 0;
        item_bounds(c, (int)i, E, e_lo, e_hi, low, nt, ne);
        atomicAdd(&sh.counts[pr], nt | (ne << 16));  // at most 12 x 1024 trials and 2048 ends per cycle
      }
      // into the pair's lowest and second-lowest bounds: whichever of the
      // pair's running best and this item's is not the lower goes, with the
      // item's own second, into the runner-up
      const uint64_t key = ((uint64_t)low.m << 32) | ((i << 14) | low.k);
      if (low.m != kNoBound) {
        const uint32_t old = (uint32_t)(atomicMin((unsigned long long*)&sh.best[pr], key) >> 32);
        const uint32_t hi = old > low.m ? old : low.m;
        atomicMin(&sh.second[pr], hi < low.m2 ? hi : low.m2);
      }
      if (kPre) pre = prefetch_entry(sh.item, list_pos(r0 + 64 + lane, vg, n_g, lg), n_g + n_q, kItems, ec, pw);
      if constexpr (!kRedraw) {
        __syncthreads();  // one wave: the atomics above are done
        if (low.m != kNoBound && sh.best[pr] == key) {
          sh.pair[0][pr] = low.u;
          sh.pair[1][pr] = low.ca;
          if constexpr (!kMassive) sh.pair[2][pr] = low.cb;
        }
      }
    }
  };
  if (ahead) rounds(std::true_type{});
  else if constexpr (!kPairs) rounds(std::false_type{});
  __syncthreads();
  if (kAhead) {  // the event's trial constants, published to LDS above, come back from there
    s.key = key_of(lane);
    s.lt = sh.lt[lane];
    s.tcut = sh.tcut[lane];
    s.ltc = sh.ltc[lane];
    s.cfac = sh.cfac[lane];
    s.cycle = sh.cycle[lane];
  }
  // The exact winner of the pair in position pr (event o of n_o partons, cycle
  // `cyc`), its scale counted from lt0: packed (i, k, K) or kNoTrial.
  auto winner = [&](uint32_t pr, uint32_t o, int n_o, uint32_t cyc, double lt0, double& v, double& ca,
                    double& cb) -> uint32_t {
#pragma clang fp contract(off)  // as in end_draws
    const uint64_t key = sh.best[pr];
    uint32_t idx = (uint32_t)key;
    if (key == ~0ull) return kNoTrial;
    const TrialCtx c{key_of(o), lt0, sh.tcut[o], 0.0, sh.cfac[o], cyc};
    const int W = (int)(idx & 15u);
    double u;
    if constexpr (kRedraw) {
      const int i = (int)(idx >> 14), k = (int)((idx >> 4) & 1023u);
      const Ends<kMassive> E = load_ends<kCached, kMassive>(c, slots, sh.slot[o], i, 0, 1, ec, o, false,
                                                            Ent5{}, qm);
      const bool e1 = k == E.k[1];
      u = trial_uniform(c.key, cyc, i, k, W);
      ca = e1 ? E.c[1][0] : E.c[0][0];
      cb = e1 ? E.c[1][1] : E.c[0][1];
    } else {
      u = sh.pair[0][pr];
      ca = sh.pair[1][pr];
      if constexpr (!kMassive) cb = sh.pair[2][pr];
    }
    double d;
    if constexpr (kMassive) d = log_fast(u) / ca;
    else d = log_fast(u) * (W <= 10 ? ca : cb);
    v = lt0 + d;
    // (no runner-up: NaN; 1e-13 covers scales that round to equal doubles)
    constexpr double kLn2 = 0.69314718055994530942;
    if ((double)__uint_as_float(sh.second[pr]) * kLn2 <= 1e-13 - d) {
      QuarkMasses om{0.0, 0.0, 0.0, 0.0, 0.0};
      if constexpr (kMassive) om = QuarkMasses{0.0, 0.0, 0.0, sh.mc[o], sh.mb[o]};
      v = -INFINITY;
      idx = exact_winner<kCached, kMassive>(c, slots, sh.slot[o], n_o, ec, o, om, v, ca, cb);
    }
    return idx;
  };
  // --- each owner that made trials decides its cycle
  if (ahead) {
    // one lane per (event, cycle) pair: the pair's scale, cutoff and veto;
    // its outcome goes into `second`, above it the winner
    const uint32_t n_pairs = (uint32_t)__popcll(tmask) << lg;
    const uint32_t o = lane < n_pairs ? sh.ranked[lane >> lg] : lane;  // the pair's event
    const double asmax = __shfl(s.asmax, (int)o);  // its trial alpha_s
    const int n_o = __shfl(s.n, (int)o);
    const uint32_t rk = lane >> lg, k = lane & (K - 1u), cyc = sh.cycle[o] + k;
    uint32_t wi = kNoTrial;
    double v = 0.0, wia = 0.0, wib = 0.0;
    if (lane < n_pairs && cyc < climit_of(o)) wi = winner(lane, o, n_o, cyc, 0.0, v, wia, wib);
    sh.pair[0][lane] = v;
    __syncthreads();
    double l = sh.lt[o];
    if (lane < n_pairs)
      for (uint32_t q = 0; q <= k; ++q) l += sh.pair[0][(rk << lg) | q];  // the winners' scales, in cycle order
    __syncthreads();
    if (lane < n_pairs) {
      uint32_t f = kPairVeto;
      double t = 0.0, z = 0.0, wf = 1.0;
      if (cyc >= climit_of(o)) {
        f = kPairLimit;
      } else if (wi == kNoTrial || !(l > sh.ltc[o])) {
        f = kPairDone;  // no end with phase space above the cutoff, or below it
      } else {
        const U4 a = key_of(o).draw(cyc, kPurposeAccept, 0);
        double prob;
        t = exp(l);
        if constexpr (kMassive) {
          const MWinner W = massive_winner(
              TrialCtx{key_of(o), 0.0, sh.tcut[o], 0.0, sh.cfac[o], cyc}, slots, sh.slot[o], (int)(wi >> 14),
              (int)((wi >> 4) & 1023u), (int)(wi & 15u), QuarkMasses{0.0, 0.0, 0.0, sh.mc[o], sh.mb[o]});
          z = trial_z(W.w, unit(a.x, a.y));
          prob = massive_prob(W, l, t, z, asmax);
        } else {
          Winner w{0.0, 0.0, 0.0, 0.0, -1, 0, 0};
          w.K = (int)(wi & 15u);
          end_from_inverse(sh.cfac[o], sh.tcut[o], w.K, wia, wib, w);
          z = trial_z(w, unit(a.x, a.y));
          prob = massless_ratio(w.K, l, t, z, w.rq2, asmax);
        }
        if (prob >= 0.0 && accept_test(prob, a, wf)) f = kPairAccept;
      }
      sh.second[lane] = (wi << 6) | f;
      sh.pair[0][lane] = l;
      sh.pair[1][lane] = t;
      sh.pair[2][lane] = z;
      sh.best[lane] = (uint64_t)__double_as_longlong(wf);
    }
    __syncthreads();
    // each event takes its pairs in cycle order up to the first that ends
    // the sequence: the steps of a cycle-by-cycle decision
    if (trial) {
      for (uint32_t k = 0; k < K; ++k) {
        const uint32_t pr = sh.rank[lane] | k;
        const uint32_t f = sh.second[pr] & 63u;
        if (f == kPairLimit) {
          s.status = kCycleLimitHit;
          break;
        }
        s.trials += sh.counts[pr] & 0xFFFFu;
        s.ends += sh.counts[pr] >> 16;
        const uint32_t this_cycle = s.cycle++;
        if (f == kPairDone) {
          s.status = kDone;
          break;
        }
        s.lt = sh.pair[0][pr];
        wsh() *= __longlong_as_double((long long)sh.best[pr]);
        if (f == kPairAccept) {
          if (s.n == s.cap) {
            s.status = kOverflow;
          } else {
            const uint32_t wi = sh.second[pr] >> 6;
            pd = Pending{sh.pair[1][pr], sh.pair[2][pr], (int)(wi >> 14), (int)((wi >> 4) & 1023u),
                         (int)(wi & 15u), this_cycle};
            pend = true;
          }
          break;
        }
      }
    }
  } else if (!kPairs && trial) {
    s.trials += sh.counts[lane] & 0xFFFFu;
    s.ends += sh.counts[lane] >> 16;
    double best = s.ltc, wia = 0.0, wib = 0.0;
    uint32_t wi = winner(lane, lane, s.n, s.cycle, s.lt, best, wia, wib);
    if (wi != kNoTrial && !(best > s.ltc)) wi = kNoTrial;  // below the cutoff
    const U4 acc = accept_draw(s);
    if constexpr (kMassive) {
      MWinner W{Winner{0.0, 0.0, 0.0, 0.0, -1, 0, 0}, 0.0, 0.0, 0.0, 0.0, 1.0, false};
      if (wi != kNoTrial)
        W = massive_winner(trial_ctx(s), slots, slot, (int)(wi >> 14), (int)((wi >> 4) & 1023u), (int)(wi & 15u), qm);
      pend = veto_decide_massive(s, best, W, acc, pd, wsh());
    } else {
      Winner w{0.0, 0.0, 0.0, 0.0, -1, 0, 0};
      if (wi != kNoTrial) {
        w.i = (int)(wi >> 14);
        w.k = (int)((wi >> 4) & 1023u);
        w.K = (int)(wi & 15u);
        end_from_inverse(s.cfac, s.tcut, w.K, wia, wib, w);
      }
      pend = veto_decide_drawn(s, best, w, acc, pd, wsh());
    }
  }
  // --- pending emissions, built together; the new parton's type goes into the mask
  const uint32_t n_pend = __popcll(__ballot(pend));
  const uint32_t n_busy = __popcll(__ballot(busy));
  if (n_pend > 0 && kEmitDiv * n_pend >= n_busy && pend) {
    const int j = s.n;
    // i's and k's colour partners before the emission, loaded beside the
    // emission's own reads: j takes the place of one partner of each, so
    // with i, j and k they are the partners afterwards
    const uint64_t oi = (uint64_t)pd.i * slots.stride + slot, ok = (uint64_t)pd.k * slots.stride + slot;
    const int pci = slots.cpart[oi], pai = slots.apart[oi], pck = slots.cpart[ok], pak = slots.apart[ok];
    if constexpr (kMassive) emit_massive(s, slots, slot, pd, qm);
    else emit(s, slots, slot, pd);
    if (pd.K <= 10) mym[j >> 6] |= 1ull << (j & 63);               // gluon emitted
    else mym[pd.i >> 6] &= ~(1ull << (pd.i & 63));                 // g -> f fbar: i is now a quark
    // ends whose momenta or partners changed: those of i, j, k and of the
    // other colour partners of i and k (partner links are symmetric)
    set_bit(mys, pd.i);
    set_bit(mys, j);
    set_bit(mys, pd.k);
    set_bit(mys, pci);
    set_bit(mys, pai);
    set_bit(mys, pck);
    set_bit(mys, pak);
    pend = false;
  }
  if (busy && !pend && s.status == kRunning && s.cycle >= climit_of(lane)) s.status = kCycleLimitHit;
}

// The flattened kernels' shared state: plain; in place; in staging slots.
template <bool kMassive, bool kOne, bool kFour>
using PlainShared = FlatShared<kMassive, kOne, kFour, kOne && !kFour && !kMassive>;
template <bool kMassive, bool kOne, bool kFour>
using PersistShared = FlatShared<kMassive, kOne, kFour, kOne && !kFour>;

size_t flat_lds_bytes(uint32_t cap) { return (size_t)2 * 64 * ((cap + 63) / 64) * 8; }

// Blocks of a flattened kernel that a CU's LDS holds (allocated in units of
// 1280 bytes).
template <class SH>
static uint32_t lds_blocks(uint32_t cap) {
  constexpr size_t kLds = 160 * 1024, kUnit = 1280;
  return (uint32_t)(kLds / ((sizeof(SH) + flat_lds_bytes(cap) + kUnit - 1) / kUnit * kUnit));
}

// Waves that a launch of the flattened kernels spreads its events over: those
// that the device's compute units hold at once.  By registers sixteen blocks
// per CU in the four-wave builds, twelve in the others, eight in staging slots
// with quark masses; by LDS fewer in large records (the masks: twelve at 256
// partons, six at 1024).  Massless records above 128 partons take eleven: at 256
// partons twelve are 5% faster for 150000 events and 5% slower for 20000.  With
// quark masses, twelve against four per CU: calls of 5000 events 393 and 372 us,
// 20000 566 and 618, 60000 875 and 978.  By registers alone and by LDS too, plain
// showers at 500 GeV: 256 partons with masses (12 and 10) 20000 events 1.93 and
// 1.67 ms, 150000 6.9 and 5.7; 512 massless (11 and 9) 2800 0.75 and 0.70, 60000
// 2.7 and 2.2; 1024 (11 and 6) 20000 1.69 and 1.48.
enum class FlatKind { kPlain, kInPlace, kStaged };
static uint32_t flat_waves(uint32_t n_cu, uint32_t cap, bool massive, FlatKind kind) {
  const bool four = !massive && cap <= kFourMaxCap;
  uint32_t lds = 0, regs = massive ? 12u : 11u;
  if (kind == FlatKind::kStaged) {
    lds = massive ? lds_blocks<PersistShared<true, false, false>>(cap) : lds_blocks<PersistShared<false, false, false>>(cap);
    regs = massive ? 8u : 12u;
  } else if (four) {
    lds = lds_blocks<PlainShared<false, true, true>>(cap);
    regs = 16u;
  } else if (!massive) {
    lds = lds_blocks<PlainShared<false, true, false>>(cap);
  } else if (kind == FlatKind::kInPlace) {
    lds = lds_blocks<PersistShared<true, true, false>>(cap);
  } else {
    lds = cap > kOneAboveCap ? lds_blocks<PlainShared<true, true, false>>(cap)
                             : lds_blocks<PlainShared<true, false, false>>(cap);
  }
  return n_cu * std::min(regs, lds);
}

// Events that a wave holds at once.  A small launch is bound by the chain of
// wave cycles of its longest wave, and 64 events to a wave left most of the
// chip idle (100 events: two waves): a wave of few events runs shorter cycles
// and evaluates up to eight veto cycles ahead from the start, so the events
// are spread until every resident wave has some.  Plain LEP shower, 64 events
// per wave and this rule: 100 events 392 and 114 us, 5003 events 509 and 195,
// 20000 events 532 and 272, 140000 events 743 and 666; from 64 events per
// resident wave on (262144) both are the same.  Past the resident waves the
// spreading costs throughput (20000 events, 2 per wave: 375 us).
static uint32_t events_per_wave(uint64_t n, uint64_t waves) {
  return (uint32_t)std::min<uint64_t>(64, (n + waves - 1) / waves);
}

// Plain one-launch form with the flattened mapping: wave w owns per_wave
// consecutive events of the batch (already started by k_me) from start to
// cutoff, with no refill; finished lanes only stop contributing trial work.
// kFour (massless, at most 128 partons): four resident waves per SIMD (128
// registers, a few spilled; 8.1 KB of LDS and the masks), the trial constants
// reloaded from LDS after the rounds (kAhead); otherwise three waves, the
// massive instantiation reloading them too to fit without spilling.
template <bool kMassive, bool kOne, bool kFour = false>
__global__ void __launch_bounds__(64, kFour ? 4 : 3)
    k_shower_plain_flat(Records r, Summary sm, EventInputs in, uint32_t n, EndCache ec, uint32_t per_wave) {
  // above 128 partons: the weight in a register and the shorter list, for
  // twelve blocks per CU instead of eleven at 256 (500 GeV, 10^6 events: 18.9 ->
  // 18.1 ms)
  using SH = PlainShared<kMassive, kOne, kFour>;
  constexpr bool kRegW = SH::kRegW;
  __shared__ SH sh;
  const OneRequest one{in.seed, in.first, in.cycle_limit};
  const uint32_t lane = threadIdx.x;
  const uint32_t words = mask_words(r.cap);
  const uint64_t e = (uint64_t)blockIdx.x * per_wave + lane;
  EvState s = {};
  s.status = kDone;
  bool busy = lane < per_wave && e < n;
  bool pend = false;
  Pending pd{};
  if (busy) {
    init_state(s, r, e, make_keyed(in.seed, in.first + e), in.ecm_of(e), in.tcut_of(e), in.t_over,
               sm.i[kSiN * sm.stride + e], (int)r.cap);
    if constexpr (!kOne) sh.climit[lane] = in.cycle_limit;
    if constexpr (!kRegW) sh.wsh[lane] = 1.0;
    mask_init(flat_gmask + (uint64_t)lane * words, flat_gmask + (uint64_t)(64 + lane) * words, words, r, e, s.n);
  }
  while (__any(busy)) {
    flat_cycle<true, kMassive, kMassive || kFour, true, kOne>(sh, one, flat_gmask, words, s, busy, pend, pd, r, e, ec,
                                                          e - lane, lane, in.qm);
    if (busy && s.status != kRunning) {
      if constexpr (!kRegW) s.wsh = sh.wsh[lane];
      write_state(s, sm, e);
      busy = false;
    }
    __syncthreads();
  }
}

// cache: [event][cap] entries of kCacheWords words (column = event), or null
void launch_shower_plain_flat(const Records& r, const Summary& s, const EventInputs& in, uint32_t n,
                              uint64_t* cache, uint32_t n_cu, hipStream_t st) {
  if (!n) return;
  const EndCache ec{cache, r.cap};
  const uint32_t waves = flat_waves(n_cu, r.cap, in.massive != 0, FlatKind::kPlain);
  // the long showers of records above 128 partons take up to an eighth more
  // events one to a wave, the last starting as the first ones end (256 partons at
  // 500 GeV, two to a wave and one: 2700 events with masses 0.98 and 0.92 ms, 2900
  // massless 0.71 and 0.67; 4400 LEP events, 64 partons: 0.165 and 0.173)
  const uint32_t pw = r.cap > kFourMaxCap && n <= waves + waves / 8 ? 1 : events_per_wave(n, waves);
  const dim3 g((n + pw - 1) / pw), b(64);
  const size_t lds = flat_lds_bytes(r.cap);
  // Massless events: the single-request LDS layout; up to 128 partons per
  // record it leaves room for four blocks per SIMD, which the four-wave
  // build fills with 128 registers by reloading its trial constants from
  // LDS after the rounds (and loading the next round's cache entries
  // ahead); above that the masks make LDS the bound and the three-wave
  // build is faster.  With quark masses: the per-event layout up to 64
  // partons, single-request above.
  if (in.massive) {
    if (r.cap > kOneAboveCap) hipLaunchKernelGGL((k_shower_plain_flat<true, true>), g, b, lds, st, r, s, in, n, ec, pw);
    else hipLaunchKernelGGL((k_shower_plain_flat<true, false>), g, b, lds, st, r, s, in, n, ec, pw);
  } else {
    if (r.cap > kFourMaxCap) hipLaunchKernelGGL((k_shower_plain_flat<false, true>), g, b, lds, st, r, s, in, n, ec, pw);
    else hipLaunchKernelGGL((k_shower_plain_flat<false, true, true>), g, b, lds, st, r, s, in, n, ec, pw);
  }
}

// kCached: A.cache holds an end cache per lane (always when in place; the
// serving epochs' staging slots have one unless it could not be allocated).
// In place (one request, kOne): four resident waves per SIMD for massless
// events with at most 128 partons (kFour: 128 registers, no spills), three
// with more partons or with quark masses.  Three for
// massless events in the serving epochs' cached staging slots (a few
// spilled registers, outweighed by the third wave: 4000 requests/s of the
// serving mix keep p99 below 40 ms instead of 80); two otherwise.
template <bool kInPlace, bool kMassive, bool kCached, bool kOne = false, bool kFour = false>
__global__ void __launch_bounds__(64, kFour ? 4 : (kInPlace || (kCached && !kMassive) ? 3 : 2))
    k_shower_flat(PersistArgs A) {
  static_assert(kInPlace || !kOne, "one request per launch only in place");
  static_assert(kOne || !kFour, "four waves need the single-request layout");
  // three waves in place: the shower weight in a register and the short
  // item list, so that 256-parton records fit twelve blocks per CU
  using SH = PersistShared<kMassive, kOne, kFour>;
  constexpr bool kRegW = SH::kRegW;
  __shared__ SH sh;
  const OneRequest one = kOne ? OneRequest{A.reqs[0].seed, A.reqs[0].first, A.reqs[0].cycle_limit}
                              : OneRequest{0ull, 0ull, 0u};
  const uint32_t lane = threadIdx.x;
  const uint32_t words = mask_words(A.slots.cap);
  const uint64_t L = (uint64_t)blockIdx.x * 64 + lane;
  EvState s = {};
  s.status = kDone;
  bool busy = false;
  bool drained = false;
  bool pend = false;
  Pending pd{};
  uint32_t req = 0;
  uint64_t ev = 0;
  uint64_t slot = L;
  uint32_t since = 0;
  while (true) {
    if (refill<(kInPlace ? 16u : 1u)>(A, busy, A.per_wave, lane, since, drained, req, ev)) {
      slot = kInPlace ? ev : L;
      start_event<kInPlace>(s, A, A.reqs[req], ev, slot);
      if constexpr (!kOne) sh.climit[lane] = A.reqs[req].cycle_limit;
      if constexpr (kRegW) s.wsh = 1.0;
      else sh.wsh[lane] = 1.0;
      mask_init(flat_gmask + (uint64_t)lane * words, flat_gmask + (uint64_t)(64 + lane) * words, words, A.slots,
                slot, s.n);
      busy = true;
    }
    if (!__any(busy)) break;
    flat_cycle<kCached, kMassive, kInPlace || kCached, kCached, kOne>(
        sh, one, flat_gmask, words, s, busy, pend, pd, A.slots, slot, A.cache, L - lane, lane, A.reqs[req].qm);
    if (busy && s.status != kRunning) {
      if constexpr (!kRegW) s.wsh = sh.wsh[lane];
      finish_event<kInPlace>(s, A, A.reqs[req], ev, slot);
      busy = false;
    }
    __syncthreads();
    ++since;
  }
}

// Writes a batch's request and segment descriptors (passed by value, so the
// launch carries them) and zeroes the work counter.
__global__ void k_setup(ReqDev* rd, ReqDev d, Segment* sd, Segment s, unsigned long long* counter) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    *rd = d;
    *sd = s;
    *counter = 0ull;
  }
}

__global__ void k_zero(double* p, uint32_t n) {
  const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0.0;
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
uint32_t persistent_lanes(const vsh_ctx* ctx) {
  const uint32_t waves = std::max<uint32_t>(1, ctx->tuned.pers_waves_per_cu) * (uint32_t)ctx->n_cu;
  return waves * 64;
}

uint64_t slots_bytes(uint64_t lanes, uint32_t cap) { return lanes * cap * (4 * 8 + 1 + 4 * 2) + 9 * 256; }

uint64_t request_out_bytes(uint64_t n, uint32_t cap, bool partners) {
  return n * cap * (4 * 8 + 1 + 2 * 2 + (partners ? 2 * 2 : 0)) + n * (kNSumD * 8 + kNSumI * 4 + 8) + 2 * n * 8 + 16 * 256 +
         kHistDoubles * 8;
}


Carver::Carver(void* base) : p(static_cast<char*>(base)) {}
char* Carver::take(uint64_t bytes) {
  char* q = p;
  p += align_up(bytes, 256);
  return q;
}

Records carve_slots(Carver& c, uint64_t lanes, uint32_t cap) {
  Records r;
  const uint64_t n = lanes * cap;
  r.E = (double*)c.take(n * 8);
  r.x = (double*)c.take(n * 8);
  r.y = (double*)c.take(n * 8);
  r.z = (double*)c.take(n * 8);
  r.pid = (int8_t*)c.take(n);
  r.col = (uint16_t*)c.take(n * 2);
  r.acol = (uint16_t*)c.take(n * 2);
  r.cpart = (uint16_t*)c.take(n * 2);
  r.apart = (uint16_t*)c.take(n * 2);
  r.stride = lanes;
  r.cap = cap;
  return r;
}

ReqBuffers carve_request(Carver& c, uint64_t n, uint32_t cap, bool partners) {
  ReqBuffers b;
  const uint64_t m = n * cap;
  b.out.E = (double*)c.take(m * 8);
  b.out.x = (double*)c.take(m * 8);
  b.out.y = (double*)c.take(m * 8);
  b.out.z = (double*)c.take(m * 8);
  b.out.pid = (int8_t*)c.take(m);
  b.out.col = (uint16_t*)c.take(m * 2);
  b.out.acol = (uint16_t*)c.take(m * 2);
  b.out.cpart = partners ? (uint16_t*)c.take(m * 2) : nullptr;
  b.out.apart = partners ? (uint16_t*)c.take(m * 2) : nullptr;
  b.out.stride = n;
  b.out.cap = cap;
  // the results in one span, in the order the serving drain copies them
  // back: histogram, integer fields, then the doubles (weight first), hash
  b.hist = (double*)c.take(kHistDoubles * 8);
  b.sum.i = (int32_t*)c.take(kNSumI * n * 4);
  b.sum.d = (double*)c.take(kNSumD * n * 8);
  b.sum.hash = (uint64_t*)c.take(n * 8);
  b.sum.stride = n;
  b.ecm = (double*)c.take(n * 8);
  b.tcut = (double*)c.take(n * 8);
  return b;
}

Scratch carve_scratch(Carver& c, uint64_t n, uint32_t cap) { return carve_obs_scratch(c.p, n, cap); }

// Lanes of the largest persistent grid (16 waves on each of 256 CUs): the
// stride of a batch's end-coefficient cache, whatever the tuning.
constexpr uint64_t kCacheLanes = 16ull * 256 * 64;

uint64_t cache_bytes(uint32_t cap, bool massive) {
  return align_up(kCacheLanes * cap * cache_words(massive) * 8, 256);
}

// A batch is one request, showered in place in its output records.
uint64_t batch_bytes(uint64_t n, uint32_t cap, bool massive) {
  return request_out_bytes(n, cap, true) + cache_bytes(cap, massive) + obs_scratch_bytes(n, cap) + 4096 +
         sizeof(ReqDev) + sizeof(Segment) + 1024;
}

BatchLayout carve_batch(void* base, uint64_t n, uint32_t cap, bool massive) {
  Carver c(base);
  BatchLayout L;
  L.buf = carve_request(c, n, cap, true);
  L.cache.rec = (uint64_t*)c.take(kCacheLanes * cap * cache_words(massive) * 8);
  L.cache.cap = cap;
  L.sc = carve_scratch(c, n, cap);
  L.counter = (unsigned long long*)c.take(256);
  L.reqs = (ReqDev*)c.take(sizeof(ReqDev));
  L.segs = (Segment*)c.take(sizeof(Segment));
  L.end = c.p;
  return L;
}

// The kernel of a mapping, in place or not, for requests with or without
// quark masses; the flattened mapping with or without an end cache (in place
// always has one).
const void* persistent_kernel(uint32_t mapping, bool in_place, bool massive, bool cached, uint32_t cap) {
  if (mapping == kMapFlat) {
    if (in_place && massive) return (const void*)k_shower_flat<true, true, true, true>;
    if (in_place)  // four-wave build up to 128 partons (LDS-bound above)
      return cap > kFourMaxCap ? (const void*)k_shower_flat<true, false, true, true>
                               : (const void*)k_shower_flat<true, false, true, true, true>;
    if (cached)
      return massive ? (const void*)k_shower_flat<false, true, true> : (const void*)k_shower_flat<false, false, true>;
    return massive ? (const void*)k_shower_flat<false, true, false> : (const void*)k_shower_flat<false, false, false>;
  }
  if (massive)
    return in_place ? (const void*)k_shower_persistent<true, true> : (const void*)k_shower_persistent<false, true>;
  return in_place ? (const void*)k_shower_persistent<true> : (const void*)k_shower_persistent<false>;
}

uint32_t persistent_block(uint32_t mapping, uint32_t block) { return mapping == kMapFlat ? 64u : block; }

uint32_t persistent_per_wave(uint64_t total, uint64_t lanes, uint32_t mapping, bool in_place, uint32_t cap,
                             bool massive, uint32_t n_cu) {
  if (mapping != kMapFlat) return 64;
  const FlatKind kind = in_place ? FlatKind::kInPlace : FlatKind::kStaged;
  return events_per_wave(total, std::min<uint64_t>(lanes / 64, flat_waves(n_cu, cap, massive, kind)));
}

// Blocks of a persistent launch: no more waves than the first claims serve.
uint32_t persistent_grid(const PersistArgs& A, uint64_t lanes, uint32_t block, uint32_t mapping) {
  const uint64_t all = lanes / block;
  return (uint32_t)(mapping == kMapFlat ? std::min<uint64_t>(all, (A.total + A.per_wave - 1) / A.per_wave) : all);
}

void launch_persistent(const PersistArgs& A, uint64_t lanes, uint32_t block, uint32_t mapping, bool in_place,
                       bool massive, hipStream_t st) {
  block = persistent_block(mapping, block);
  const dim3 grid(persistent_grid(A, lanes, block, mapping));
  const size_t lds = mapping == kMapFlat ? flat_lds_bytes(A.slots.cap) : 0;
  void* args[] = {const_cast<PersistArgs*>(&A)};
  (void)hipLaunchKernel(persistent_kernel(mapping, in_place, massive, A.cache.rec != nullptr, A.slots.cap), grid,
                        dim3(block), args, lds, st);
}

void launch_setup(ReqDev* rd, const ReqDev& d, Segment* sd, const Segment& s, unsigned long long* counter,
                  hipStream_t st) {
  hipLaunchKernelGGL(k_setup, dim3(1), dim3(64), 0, st, rd, d, sd, s, counter);
}

void launch_zero(double* p, uint32_t n, hipStream_t st) {
  hipLaunchKernelGGL(k_zero, dim3((n + 255) / 256), dim3(256), 0, st, p, n);
}

static void fill_request_desc(ReqDev& d, const ReqBuffers& b, const vsh_request* req, uint64_t first_idx,
                              const double* ecm_dev, const double* tcut_dev) {
  d.out = b.out;
  d.sum = b.sum;
  d.ecm = ecm_dev;
  d.tcut = tcut_dev;
  d.ecm0 = req->ecm;
  d.tcut0 = req->t_cut;
  d.seed = req->seed;
  d.first = req->first_event + first_idx;
  d.count = b.sum.stride;
  d.cycle_limit = effective_cycle_limit(req->cycle_limit);
  d.t_over = req->t_over;
  d.qm = request_masses(*req);
  d.massive = request_massive(*req);
}

// One batch of `n` events of req (starting at request index first_idx)
// through the persistent form on stream st, with the batch's buffers in the
// workspace at `base`.  Inputs: per-event arrays already on the device (or
// null).  Writes the histogram into hist (accumulates), the summary fields
// into the arrays that `out` names, [field][n], and the workspace's for others.
// The kernels are launched one by one: the same sequence as an instantiated
// graph took 25 us longer a call (its event nodes set anew each time), and 60
// where a caller's buffers change from call to call.
vsh_status run_batch(vsh_ctx* ctx, const vsh_request* req, uint64_t first_idx, uint64_t n,
                            hipStream_t st, void* base, const double* ecm_dev, const double* tcut_dev,
                            double* hist, const Summary* out, BatchLayout* out_layout) {
  const uint32_t cap = req->max_partons;
  const uint64_t lanes = persistent_lanes(ctx);
  const uint32_t mapping = ctx->tuned.mapping;
  const uint32_t block = persistent_block(mapping, ctx->tuned.pers_block);
  if (lanes > kCacheLanes) {
    set_error(ctx, "persistent grid of %llu lanes exceeds the %llu the batch layout holds",
              (unsigned long long)lanes, (unsigned long long)kCacheLanes);
    return VSH_E_INTERNAL;
  }
  BatchLayout L = carve_batch(base, n, cap, request_massive(*req) != 0);
  if (out && out->d) L.buf.sum.d = out->d;
  if (out && out->i) L.buf.sum.i = out->i;
  if (out && out->hash) L.buf.sum.hash = out->hash;
  if (out_layout) *out_layout = L;
  ReqDev d;
  fill_request_desc(d, L.buf, req, first_idx, ecm_dev, tcut_dev);
  Segment sg{0, 0, 0, n, 0};
  hipError_t err;
  PersistArgs A;
  A.slots = L.buf.out;  // in place
  A.reqs = L.reqs;
  A.segs = L.segs;
  A.n_segs = 1;
  A.total = n;
  A.next = L.counter;
  A.threshold = ctx->tuned.refill_threshold;
  A.period = ctx->tuned.refill_period;
  A.per_wave = persistent_per_wave(n, lanes, mapping, true, cap, request_massive(*req) != 0, (uint32_t)ctx->n_cu);
  A.cache = L.cache;
  EventInputs in{};
  in.ecm = ecm_dev;
  in.tcut = tcut_dev;
  in.ecm0 = req->ecm;
  in.tcut0 = req->t_cut;
  in.seed = req->seed;
  in.first = req->first_event + first_idx;
  in.cycle_limit = effective_cycle_limit(req->cycle_limit);
  in.t_over = req->t_over;
  in.qm = request_masses(*req);
  in.massive = request_massive(*req);
  in.fixed_hist = (req->flags & VSH_HIST_FIXEDPOINT) ? 1u : 0u;
  hipEvent_t* tev = timing_slot(ctx);
  if (tev) (void)hipEventRecord(tev[0], st);
  launch_setup(L.reqs, d, L.segs, sg, L.counter, st);
  launch_me(L.buf.out, L.buf.sum, in, (uint32_t)n, st, L.buf.hist);
  if (tev) (void)hipEventRecord(tev[1], st);
  launch_persistent(A, lanes, block, mapping, true, in.massive != 0, st);
  if (tev) (void)hipEventRecord(tev[2], st);
  launch_obs(L.buf.out, L.buf.sum, in, L.sc, (uint32_t)n, hist, L.buf.hist, st);
  if (tev) (void)hipEventRecord(tev[3], st);
  err = hipGetLastError();
  if (err != hipSuccess) return hip_fail(ctx, err, "kernel launch");
  return VSH_OK;
}

uint64_t persistent_workspace_bytes_ctx(const vsh_ctx* ctx, const vsh_request* req) {
  return batch_bytes(req->n_events, req->max_partons, request_massive(*req) != 0);
}

uint64_t persistent_workspace_bytes(const vsh_request* req) {
  return batch_bytes(req->n_events, req->max_partons, request_massive(*req) != 0);
}

vsh_status persistent_into(vsh_ctx* ctx, const vsh_request* req, hipStream_t st, void* ws, double* dev_hist,
                           double* dev_sum_d, int32_t* dev_sum_i, uint64_t* dev_hash) {
  const Summary out{dev_sum_d, dev_sum_i, dev_hash, req->n_events};
  return run_batch(ctx, req, 0, req->n_events, st, ws, req->ecm_per_event, req->tcut_per_event, dev_hist, &out,
                   nullptr);
}

vsh_status generate_persistent(vsh_ctx* ctx, const vsh_request* req, vsh_result** out) {
  const auto t0 = std::chrono::steady_clock::now();
  const uint32_t cap = req->max_partons;
  const uint64_t lanes = persistent_lanes(ctx);
  // chunk so that a batch fits the budget (half of it when records are returned)
  uint64_t budget = ctx->budget;
  if (req->flags & VSH_RECORDS) budget /= 2;
  if (lanes > kCacheLanes) {
    set_error(ctx, "persistent grid of %llu lanes exceeds the %llu the batch layout holds",
              (unsigned long long)lanes, (unsigned long long)kCacheLanes);
    return VSH_E_INTERNAL;
  }
  const uint64_t fixed = 64 * 1024 + cache_bytes(cap, request_massive(*req) != 0);
  if (budget <= fixed + request_out_bytes(64, cap, true) + obs_scratch_bytes(64, cap)) {
    set_error(ctx, "memory budget too small for the persistent form at %u partons", cap);
    return VSH_E_NOMEM;
  }
  const uint64_t per_event = request_out_bytes(1, cap, true) + 64 + (uint64_t)cap * 32;
  uint64_t chunk = std::min<uint64_t>(req->n_events, (budget - fixed) / per_event);
  chunk = std::min<uint64_t>(chunk, 1ull << 27);
  ResultBox* box = new_call_result(ctx, req, chunk >= req->n_events);
  if (!box) return VSH_E_NOMEM;
  hipStream_t st = ctx->stream;
  float t_me = 0, t_sh = 0, t_obs = 0;
  for (uint64_t a = 0; a < req->n_events; a += chunk) {
    const uint64_t n = std::min(chunk, req->n_events - a);
    vsh_status rc = ctx->arena.reserve(ctx, batch_bytes(n, cap, request_massive(*req) != 0));
    if (rc) {
      drop_result(ctx, box);
      return rc;
    }
    BatchLayout L = carve_batch(ctx->arena.ptr, n, cap, request_massive(*req) != 0);
    hipError_t err;
    const double* ecm_dev = nullptr;
    const double* tcut_dev = nullptr;
    if (req->ecm_per_event) {
      err = hipMemcpyAsync(L.buf.ecm, req->ecm_per_event + a, n * 8, hipMemcpyHostToDevice, st);
      if (err != hipSuccess) { drop_result(ctx, box); return hip_fail(ctx, err, "input copy"); }
      ecm_dev = L.buf.ecm;
    }
    if (req->tcut_per_event) {
      err = hipMemcpyAsync(L.buf.tcut, req->tcut_per_event + a, n * 8, hipMemcpyHostToDevice, st);
      if (err != hipSuccess) { drop_result(ctx, box); return hip_fail(ctx, err, "input copy"); }
      tcut_dev = L.buf.tcut;
    }
    (void)hipEventRecord(ctx->ev[0], st);
    PersistArgs A;
    ReqDev d;
    fill_request_desc(d, L.buf, req, a, ecm_dev, tcut_dev);
    const Segment sg{0, 0, 0, n, 0};
    launch_setup(L.reqs, d, L.segs, sg, L.counter, st);
    EventInputs in{};
    in.ecm = ecm_dev;
    in.tcut = tcut_dev;
    in.ecm0 = req->ecm;
    in.tcut0 = req->t_cut;
    in.seed = req->seed;
    in.first = req->first_event + a;
    in.cycle_limit = effective_cycle_limit(req->cycle_limit);
    in.t_over = req->t_over;
    in.qm = request_masses(*req);
    in.massive = request_massive(*req);
    in.fixed_hist = (req->flags & VSH_HIST_FIXEDPOINT) ? 1u : 0u;
    launch_me(L.buf.out, L.buf.sum, in, (uint32_t)n, st, L.buf.hist);
    A.slots = L.buf.out;  // in place
    A.reqs = L.reqs;
    A.segs = L.segs;
    A.n_segs = 1;
    A.total = n;
    A.next = L.counter;
    A.threshold = ctx->tuned.refill_threshold;
    A.period = ctx->tuned.refill_period;
    A.per_wave = persistent_per_wave(n, lanes, ctx->tuned.mapping, true, cap, in.massive != 0, (uint32_t)ctx->n_cu);
    A.cache = L.cache;
    (void)hipEventRecord(ctx->ev[1], st);
    launch_persistent(A, lanes, ctx->tuned.pers_block, ctx->tuned.mapping, true, in.massive != 0, st);
    (void)hipEventRecord(ctx->ev[2], st);
    launch_obs(L.buf.out, L.buf.sum, in, L.sc, (uint32_t)n, L.buf.hist, nullptr, st);
    (void)hipEventRecord(ctx->ev[3], st);
    err = hipGetLastError();
    if (err != hipSuccess) { drop_result(ctx, box); return hip_fail(ctx, err, "kernel launch"); }
    const int32_t* n_host = nullptr;
    rc = copy_back_chunk(ctx, st, L.buf.hist, L.buf.sum, n, req->flags, box, a, &n_host);
    if (rc) {
      drop_result(ctx, box);
      return rc;
    }
    float ms;
    if (hipEventElapsedTime(&ms, ctx->ev[0], ctx->ev[1]) == hipSuccess) t_me += ms;
    if (hipEventElapsedTime(&ms, ctx->ev[1], ctx->ev[2]) == hipSuccess) t_sh += ms;
    if (hipEventElapsedTime(&ms, ctx->ev[2], ctx->ev[3]) == hipSuccess) t_obs += ms;
    if (req->flags & VSH_RECORDS) {
      vsh_status rc2 = gather_records(ctx, L.buf.out, n_host, n, box);
      if (rc2) {
        drop_result(ctx, box);
        return rc2;
      }
    }
  }
  box->pub.t_me_ms = t_me;
  box->pub.t_shower_ms = t_sh;
  box->pub.t_obs_ms = t_obs;
  box->pub.t_total_ms =
      std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
  finish_result(box);
  *out = &box->pub;
  return VSH_OK;
}

}  // namespace vsh
