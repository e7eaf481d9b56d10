// vsh_kernels.hip -- the plain form of the shower hot path for gfx950 and the
// observables pass shared by both forms.
//
//   k_me             LO matrix element and event initialisation (App. B)
//   k_load_records   caller-supplied initial states into records, checked
//   k_shower_plain   thread per event, the whole veto loop in one launch
//                    (App. A / C: select winner, cutoff, alpha_s, veto, split)
//   k_obs            validation, Durham y23/y34, thrust, C, rho_H, B_T/B_W
//                    (Sec. 3.1) and histograms reduced in LDS before the
//                    global atomics
#include <algorithm>

#include "vsh_observables.hpp"
#include "vsh_shower.hpp"

namespace vsh {

// zero_hist (optional): a histogram set to clear on the way (the first block
// clears it), saving its own launch.
__global__ void __launch_bounds__(256) k_me(Records r, Summary s, EventInputs in, uint32_t n, double* zero_hist) {
  const uint32_t e = blockIdx.x * blockDim.x + threadIdx.x;
  if (zero_hist && blockIdx.x == 0)
    for (uint32_t a = threadIdx.x; a < (uint32_t)kHistDoubles; a += blockDim.x) zero_hist[a] = 0.0;
  if (e >= n) return;
  const MEOut m = me_event(r, e, make_keyed(in.seed, in.first + e), in.ecm_of(e), in.qm, in.massive != 0);
  s.d[kSdW * s.stride + e] = m.w;
  s.d[kSdCos * s.stride + e] = m.c;
  s.d[kSdPhi * s.stride + e] = m.phi;
  s.i[kSiN * s.stride + e] = 2;
  s.i[kSiFlavour * s.stride + e] = m.f;
}

// Caller-supplied starts (CSR arrays, as the caller laid them out) into the
// slot-major records, kLoadLanes lanes per event: flavours and colours
// checked, partner links from the colour labels, the event's sqrt(s) as the
// sum of its energies in order.  Done on the host this was a pass over
// capacity x events of mostly empty slots, their upload, and two label tables
// cleared per event: 23 of the 26 ms of a 20011-event call.  *bad: the first
// event that fails a check (its record is not used then); offsets have been
// checked by the host.
__global__ void __launch_bounds__(256) k_load_records(Records r, Summary s, CsrStarts in, uint32_t n, double* ecm,
                                                      unsigned long long* bad, double* zero_hist) {
  for (uint32_t a = blockIdx.x * 256 + threadIdx.x; a < (uint32_t)kHistDoubles; a += gridDim.x * 256) zero_hist[a] = 0.0;
  const uint32_t e = (blockIdx.x * 256 + threadIdx.x) / kLoadLanes, lane = threadIdx.x % kLoadLanes;
  if (e >= n) return;
  const uint64_t o = in.off[e] - in.off[0];
  const int np = (int)(in.off[e + 1] - in.off[e]);
  bool ok = true;
  for (int a = (int)lane; a < np; a += (int)kLoadLanes) {
    const int f = in.pid[o + a];
    const uint32_t ca = in.col[o + a], aa = in.acol[o + a];
    const bool q = f >= 1 && f <= 5, qb = f <= -1 && f >= -5, g = f == kGluon;
    if (!(q || qb || g) || (q && (ca == 0 || aa != 0)) || (qb && (ca != 0 || aa == 0)) || (g && (ca == 0 || aa == 0)) ||
        ca > 2 * kMaxCount || aa > 2 * kMaxCount)
      ok = false;
    // every colour line has exactly one start and one end
    uint32_t starts_c = 0, ends_c = 0, starts_a = 0, ends_a = 0;
    uint16_t cp = kNoPartner, ap = kNoPartner;
    for (int b = 0; b < np; ++b) {
      const uint32_t cb = in.col[o + b], ab = in.acol[o + b];
      starts_c += cb == ca;
      ends_c += ab == ca;
      starts_a += cb == aa;
      ends_a += ab == aa;
      if (b != a && ca != 0 && ab == ca && cp == kNoPartner) cp = (uint16_t)b;
      if (b != a && aa != 0 && cb == aa && ap == kNoPartner) ap = (uint16_t)b;
    }
    if ((ca != 0 && (starts_c != 1 || ends_c != 1)) || (aa != 0 && (starts_a != 1 || ends_a != 1))) ok = false;
    const double* p = in.p + 4 * (o + a);
    const uint64_t to = (uint64_t)a * r.stride + e;
    r.E[to] = p[0];
    r.x[to] = p[1];
    r.y[to] = p[2];
    r.z[to] = p[3];
    r.pid[to] = (int8_t)f;
    r.col[to] = (uint16_t)ca;
    r.acol[to] = (uint16_t)aa;
    r.cpart[to] = cp;
    r.apart[to] = ap;
  }
  if (lane == 0) {
    double sum = 0.0;
    for (int a = 0; a < np; ++a) sum += in.p[4 * (o + a)];
    if (!(sum > 0.0)) ok = false;
    ecm[e] = sum;
    s.d[kSdW * s.stride + e] = 1.0;
    s.d[kSdCos * s.stride + e] = 0.0;
    s.d[kSdPhi * s.stride + e] = 0.0;
    s.i[kSiN * s.stride + e] = np;
    s.i[kSiFlavour * s.stride + e] = 0;
  }
  if (!ok) atomicMin(bad, (unsigned long long)e);
}

// Plain form: each thread evolves its event to the cutoff in one launch.
// Compiled for 2, 3 and 4 resident waves per SIMD (register budgets 256,
// 168 and 128); the autotuner picks by timing.  kMassive: each kernel with
// its own massive phase space (requests with quark masses).
template <int kWaves, bool kMassive = false>
__global__ void __launch_bounds__(256, kWaves) k_shower_plain(Records r, Summary sm, EventInputs in,
                                                              uint32_t n) {
  const uint32_t e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  EvState s;
  init_state(s, r, e, make_keyed(in.seed, in.first + e), in.ecm_of(e), in.tcut_of(e), in.t_over,
             sm.i[kSiN * sm.stride + e], (int)r.cap);
  while (s.status == kRunning) {
    if constexpr (kMassive) veto_cycle_massive(s, r, e, in.qm);
    else veto_cycle(s, r, e);
    if (s.cycle >= in.cycle_limit && s.status == kRunning) s.status = kCycleLimitHit;
  }
  write_state(s, sm, e);
}

// ---------------------------------------------------------------------------
// Observables pass.  Events are sorted by parton count (largest first) with a
// counting sort, so the lanes of a wave work on events of the same size;
// each thread copies its event into its scratch column (coalesced in every
// later pass), computes the observables and fills an LDS histogram that is
// added to the global one once per block.
// ---------------------------------------------------------------------------
// A launch of the pass works on one request (its job in the kernel arguments)
// or, in serving, on all that an epoch finishes (a table of jobs; each has a
// range of blocks).  f(job, block within the job, the job's blocks).
template <bool kMulti>
struct ObsArgs;
template <>
struct ObsArgs<false> {
  ObsJob job;
};
template <>
struct ObsArgs<true> {
  const ObsJob* jobs;
  uint32_t count;
};
template <bool kMulti, class F>
__device__ __forceinline__ void with_job(const ObsArgs<kMulti>& A, int stage, F&& f) {
  if constexpr (!kMulti) {
    f(A.job, blockIdx.x, gridDim.x);
  } else {
    uint32_t lo = 0, hi = A.count;  // the last job that begins at or before this block
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) / 2;
      if (A.jobs[mid].at[stage] <= blockIdx.x) lo = mid;
      else hi = mid;
    }
    const uint32_t from = A.jobs[lo].at[stage], to = lo + 1 < A.count ? A.jobs[lo + 1].at[stage] : gridDim.x;
    f(A.jobs[lo], blockIdx.x - from, to - from);
  }
}

// Zero the counting sort's counters, the histogram copies and, for fixed-point histograms, the
// integer cells and the largest-weight word (a kernel, not a memset, so the
// sequence can be captured in a graph).
template <bool kMulti>
__global__ void __launch_bounds__(256) k_obs_reset(ObsArgs<kMulti> A) {
  with_job(A, kObsStageHist, [&](const ObsJob& J, uint32_t blk, uint32_t grid) {
    (void)grid;
    const uint32_t nb = J.r.cap + 1;
    uint32_t* cnt = J.sc.cnt;
    double* hcopy = J.sc.hcopy;
    unsigned long long* ihist = J.in.fixed_hist ? J.sc.ihist : nullptr;
    unsigned long long* wmax = J.in.fixed_hist ? J.sc.wmax : nullptr;
    const uint32_t i = blk * blockDim.x + threadIdx.x;
    if (i < nb) cnt[i] = 0u;
    if (i < kHistCopies * (uint32_t)kHistDoubles) {
      hcopy[i] = 0.0;
      if (ihist) ihist[i] = 0ull;
    }
    if (wmax && i == 0) *wmax = 0ull;
  });
}

// The largest |w| of the launch's events (the bits of non-negative doubles
// order like the integers), one atomic per wave.
__device__ __forceinline__ void wave_max_weight(double w, unsigned long long* wmax) {
  const uint64_t m = wave_max_u64((uint64_t)__double_as_longlong(w));
  if (__lane_id() == 0 && m) atomicMax(wmax, (unsigned long long)m);
}

// Per-block counts in LDS over kObsSortPer events per thread, one global
// atomic per non-empty count per block (few blocks, so that the atomics of
// the handful of occupied counts do not queue up); with wmax, also the
// largest |w| of the events (the bits of non-negative doubles order like the
// integers, so the maximum does not depend on order).
template <bool kMulti>
__global__ void __launch_bounds__(256) k_obs_count(ObsArgs<kMulti> A) {
  with_job(A, kObsStageSort, [&](const ObsJob& J, uint32_t blk, uint32_t grid) {
    (void)grid;
    const Summary sm = J.sm;
    const uint32_t n = J.n, cap = J.r.cap;
    uint32_t* cnt = J.sc.cnt;
    unsigned long long* wmax = J.in.fixed_hist ? J.sc.wmax : nullptr;
    __shared__ uint32_t lc[kMaxCount + 1];
    const uint32_t nb = cap + 1;
    for (uint32_t k = threadIdx.x; k < nb; k += blockDim.x) lc[k] = 0u;
    double w = 0.0;
    __syncthreads();
    const uint64_t e0 = (uint64_t)blk * blockDim.x * kObsSortPer;
    const uint64_t e1 = e0 + (uint64_t)blockDim.x * kObsSortPer < n ? e0 + (uint64_t)blockDim.x * kObsSortPer : n;
    for (uint64_t e = e0 + threadIdx.x; e < e1; e += blockDim.x) {
      const uint32_t np = (uint32_t)sm.i[kSiN * sm.stride + e];
      atomicAdd(&lc[cap - (np < cap ? np : cap)], 1u);
      if (wmax) w = fmax(w, fabs(sm.d[kSdW * sm.stride + e]));
    }
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < nb; k += blockDim.x)
      if (lc[k]) atomicAdd(&cnt[k], lc[k]);
    if (wmax) wave_max_weight(w, wmax);
  });
}

// The histogram copies into the caller's histogram (accumulated), one cell
// per thread with its kHistCopies loads in flight together (five blocks: 3 us
// against 7 us for one block of 256 threads).  Fixed point: the copies'
// integer cells summed (exactly, in any order), then sum w and sum w^2 scaled
// back by their powers of two, entries as they are, so the result does not
// depend on the order of the events.
template <bool kMulti>
__global__ void __launch_bounds__(256) k_hist_finalize(ObsArgs<kMulti> A) {
  with_job(A, kObsStageSum, [&](const ObsJob& J, uint32_t blk, uint32_t grid) {
    (void)grid;
    const Scratch sc = J.sc;
    double* hist = J.hist;
    const bool fixed = J.in.fixed_hist != 0;
    const uint32_t a = blk * 256 + threadIdx.x;
    if (a >= (uint32_t)kHistDoubles) return;
    if (fixed) {
      const FixScale fx = fix_scale(sc);
      unsigned long long s = 0;
#pragma unroll
      for (uint32_t c = 0; c < kHistCopies; ++c) s += sc.ihist[c * kHistDoubles + a];
      const double q = (double)(long long)s;
      const int col = (int)(a % 3);
      hist[a] += col == 0 ? ldexp(q, -fx.fw) : (col == 1 ? ldexp(q, -fx.fw2) : q);
    } else {
      double v = 0.0;
#pragma unroll
      for (uint32_t c = 0; c < kHistCopies; ++c) v += sc.hcopy[c * kHistDoubles + a];
      hist[a] += v;
    }
  });
}

// A small launch's histogram (collected in the workspace) into the caller's:
// 10 KB, a launch's latency (2 us of a call).
__global__ void __launch_bounds__(256) k_hist_add(const double* __restrict__ own, double* __restrict__ hist) {
  const uint32_t a = blockIdx.x * 256 + threadIdx.x;
  if (a < (uint32_t)kHistDoubles) hist[a] += own[a];
}

// exclusive prefix sum of nb counters, in place (one block)
template <bool kMulti>
__global__ void __launch_bounds__(256) k_obs_scan(ObsArgs<kMulti> A) {
  with_job(A, kObsStageScan, [&](const ObsJob& J, uint32_t blk, uint32_t grid) {
    (void)blk;
    (void)grid;
    uint32_t* cnt = J.sc.cnt;
    const uint32_t nb = J.r.cap + 1;
    __shared__ uint32_t part[256];
    const uint32_t t = threadIdx.x;
    const uint32_t per = (nb + 255) / 256;
    uint32_t sum = 0;
    for (uint32_t k = t * per; k < nb && k < (t + 1) * per; ++k) sum += cnt[k];
    part[t] = sum;
    __syncthreads();
    if (t == 0) {
      uint32_t run = 0;
      for (uint32_t k = 0; k < 256; ++k) {
        const uint32_t v = part[k];
        part[k] = run;
        run += v;
      }
    }
    __syncthreads();
    uint32_t run = part[t];
    for (uint32_t k = t * per; k < nb && k < (t + 1) * per; ++k) {
      const uint32_t v = cnt[k];
      cnt[k] = run;
      run += v;
    }
  });
}

// Each block (kObsSortPer events per thread, as k_obs_count) reserves one
// range per parton count with a single global atomic and places its events
// by their LDS rank inside the range.
template <bool kMulti>
__global__ void __launch_bounds__(256) k_obs_scatter(ObsArgs<kMulti> A) {
  with_job(A, kObsStageSort, [&](const ObsJob& J, uint32_t blk, uint32_t grid) {
    (void)grid;
    const Summary sm = J.sm;
    const uint32_t n = J.n, cap = J.r.cap;
    uint32_t *cnt = J.sc.cnt, *perm = J.sc.perm;
    __shared__ uint32_t lc[kMaxCount + 1];
    const uint32_t nb = cap + 1;
    for (uint32_t k = threadIdx.x; k < nb; k += blockDim.x) lc[k] = 0u;
    __syncthreads();
    const uint64_t e0 = (uint64_t)blk * blockDim.x * kObsSortPer;
    uint32_t bin[kObsSortPer], rank[kObsSortPer];
#pragma unroll
    for (uint32_t q = 0; q < kObsSortPer; ++q) {
      const uint64_t e = e0 + (uint64_t)q * blockDim.x + threadIdx.x;
      bin[q] = 0;
      rank[q] = 0;
      if (e < n) {
        const uint32_t np = (uint32_t)sm.i[kSiN * sm.stride + e];
        bin[q] = cap - (np < cap ? np : cap);
        rank[q] = atomicAdd(&lc[bin[q]], 1u);
      }
    }
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < nb; k += blockDim.x)
      if (lc[k]) lc[k] = atomicAdd(&cnt[k], lc[k]);
    __syncthreads();
#pragma unroll
    for (uint32_t q = 0; q < kObsSortPer; ++q) {
      const uint64_t e = e0 + (uint64_t)q * blockDim.x + threadIdx.x;
      if (e < n) perm[lc[bin[q]] + rank[q]] = (uint32_t)e;
    }
  });
}

// Orders a wave's LDS accesses on either side (the LDS takes them in program
// order; the compiler may not move them across).
__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <bool kMassive>
__device__ __forceinline__ void window_events(const Records& r, const Summary& sm, const EventInputs& in,
                                              const Scratch& sc, uint32_t n, double* __restrict__ hist, uint32_t blk,
                                              uint32_t grid) {
  __shared__ double lh[kHistDoubles];
  for (int a = threadIdx.x; a < kHistDoubles; a += blockDim.x) lh[a] = 0.0;
  const bool fixed = in.fixed_hist != 0;
  FixScale fxs{0, 0};
  if (fixed) fxs = fix_scale(sc);
  const FixScale* fx = fixed ? &fxs : nullptr;
  __syncthreads();
  const uint64_t t = (uint64_t)blk * blockDim.x + threadIdx.x;
  const uint64_t step = (uint64_t)grid * blockDim.x;
  const uint32_t cap = r.cap;
  // After k_obs_scatter, cnt[b] is the end of bin b (bin = cap - parton
  // count), so cnt[cap - m] counts the events with at least m partons; they
  // sit at the front of perm, largest first.
  const uint64_t n_big = sc.threshold <= cap ? sc.cnt[cap - sc.threshold] : 0u;  // done by k_obs_group
  const uint64_t n_mid = (uint32_t)kObsRegSlots < cap ? sc.cnt[cap - (kObsRegSlots + 1)] : n_big;
  // events of at most kObsRegSlots partons, in windows of consecutive events
  // (coalesced counts; the records of a window share cache lines), each
  // window ordered by parton count in LDS so that the 64 events a wave takes
  // at a time have nearly the same size and its loops stop at the largest.
  // A grid that covers the events has a window of 256 per block, 64 for each
  // wave.  A smaller one has windows of up to 256 per wave, which works
  // through all of its window: shared out over the block, the waves with the
  // small events waited for the one with the largest (36% of the issue slots
  // used; k_obs on 10^6 LEP events 427 and 304 us, 3 10^6 of mixed energies
  // 1197 and 711).
  constexpr uint32_t kWaves = 4;  // per block
  __shared__ uint8_t orders[kWaves][256];
  __shared__ uint32_t bins_n[kWaves][kObsRegSlots + 2];  // events per parton count, then the others
  const uint32_t chunks = (uint32_t)std::min<uint64_t>(4, ((uint64_t)n + grid * 256ull - 1) / (grid * 256ull));
  const bool shared = chunks == 1;  // one window, and one pass of the loop, for the block
  const uint32_t wave = shared ? 0 : threadIdx.x / 64, lane = shared ? threadIdx.x : threadIdx.x % 64;
  const uint32_t span = shared ? 256 : 64 * chunks, teams = shared ? 1 : kWaves;
  uint8_t* order = orders[wave];
  uint32_t* bin_n = bins_n[wave];
  auto fence = [&] {
    if (shared) __syncthreads();
    else wave_fence();
  };
  for (uint64_t w0 = ((uint64_t)blk * teams + wave) * span; w0 < n; w0 += (uint64_t)grid * teams * span) {
    if (lane < kObsRegSlots + 2) bin_n[lane] = 0;
    fence();
    uint32_t bin[4], rank[4];
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
      bin[q] = rank[q] = 0;
      if (q >= chunks) continue;
      const uint64_t e_own = w0 + q * 64 + lane;
      const int np_own = e_own < n ? sm.i[kSiN * sm.stride + e_own] : kObsRegSlots + 1;
      const bool mine = np_own <= kObsRegSlots && (uint32_t)np_own < sc.threshold;  // else the lane groups
      bin[q] = mine ? (uint32_t)np_own : kObsRegSlots + 1;
      rank[q] = atomicAdd(&bin_n[bin[q]], 1u);
    }
    fence();
#pragma unroll
    for (uint32_t q = 0; q < 4; ++q) {
      if (q >= chunks) continue;
      uint32_t start = 0;
      for (uint32_t b = 0; b < bin[q]; ++b) start += bin_n[b];
      order[start + rank[q]] = (uint8_t)(q * 64 + lane);
    }
    fence();
    for (uint32_t q = 0; q < chunks; ++q) {
      const uint64_t e = w0 + order[q * 64 + lane];
      const int np = e < n ? sm.i[kSiN * sm.stride + e] : kObsRegSlots + 1;
      const bool ok = np <= kObsRegSlots && (uint32_t)np < sc.threshold;
      const int wmax = (int)wave_max(ok ? (uint32_t)np : 0u);
      if (ok) {
        const int status = sm.i[kSiStatus * sm.stride + e];
        const ObsOut o = reg_observables<kObsRegSlots, kMassive>(r, e, np, wmax, in.ecm_of(e), status, in);
        if (o.status == kDone) hist_fill(lh, o, sm.d[kSdW * sm.stride + e], sm.d[kSdCos * sm.stride + e], fx);
        for (int h = 0; h < 7; ++h) sm.d[(kSdY23 + h) * sm.stride + e] = o.v[h];
        sm.i[kSiStatus * sm.stride + e] = o.status;
      }
    }
    fence();  // order and bin_n serve the next window
  }
  // the rest below the wave threshold, sorted by size, through the scratch
  for (uint64_t q = n_big + t; q < n_mid; q += step) {
    const uint64_t e = sc.perm[q];
    const int status = sm.i[kSiStatus * sm.stride + e];
    const int np = sm.i[kSiN * sm.stride + e];
    for (int a = 0; a < np; ++a) {
      const uint64_t from = (uint64_t)a * r.stride + e, to = (uint64_t)a * sc.stride + t;
      sc.E[to] = r.E[from];
      sc.x[to] = r.x[from];
      sc.y[to] = r.y[from];
      sc.z[to] = r.z[from];
    }
    const ObsOut o = scratch_observables<kMassive>(sc, t, np, in.ecm_of(e), status, in, r, e);
    if (o.status == kDone) hist_fill(lh, o, sm.d[kSdW * sm.stride + e], sm.d[kSdCos * sm.stride + e], fx);
    for (int h = 0; h < 7; ++h) sm.d[(kSdY23 + h) * sm.stride + e] = o.v[h];
    sm.i[kSiStatus * sm.stride + e] = o.status;
  }
  __syncthreads();
  hist_flush(lh, sc, fixed, threadIdx.x, blockDim.x, kHistCopies, hist);
}

template <bool kMassive>
__global__ void __launch_bounds__(256) k_obs(Records r, Summary sm, EventInputs in, Scratch sc, uint32_t n,
                                             double* __restrict__ hist) {
  window_events<kMassive>(r, sm, in, sc, n, hist, blockIdx.x, gridDim.x);
}

template <bool kMassive>
__global__ void __launch_bounds__(256) k_obs_jobs(ObsArgs<true> A) {
  with_job(A, kObsStageWindow, [&](const ObsJob& J, uint32_t blk, uint32_t grid) {
    window_events<kMassive>(J.r, J.sm, J.in, J.sc, J.n, J.hist, blk, grid);
  });
}

// ---------------------------------------------------------------------------
// Events of 9 partons and more: a group of G lanes per event (G = 16 for up
// to 31 partons, four events per wave; G = 64 beyond), the group's partons
// in LDS.  Thrust's candidate planes (i < j, four sign choices) and each
// Durham step's pair scan are spread over the group's lanes; ties go to the
// smallest index in the serial scan order (first maximum for thrust, first
// minimum for Durham, as in the one-thread-per-event path).  A block is one
// wave, whose LDS operations take effect in program order, so the groups
// (which may run different numbers of steps) need no barrier between them.
// ---------------------------------------------------------------------------
// Reductions over G = 16 or 64 lanes.  Within a row of 16 lanes as DPP
// rotations (by 8, 4, 2, 1: after each the values repeat with that period, so
// a rotation meets the same pairs as a butterfly) instead of shuffles through
// the LDS pipe, whose latency bound the groups: k_obs_group<16> on the
// 10^6-event stress batch 4.54 -> 4.47 ms.
template <int G>
__device__ __forceinline__ double group_sum(double v) {
  static_assert(G == 16 || G == 64, "a row of lanes or a wave");
  if constexpr (G == 64) {
    v += __shfl_xor(v, 32);
    v += __shfl_xor(v, 16);
  }
  v += row_ror<8>(v);
  v += row_ror<4>(v);
  v += row_ror<2>(v);
  v += row_ror<1>(v);
  return v;
}

// (value, index) -> largest (smallest) value, smallest index among equal values
template <int G>
__device__ __forceinline__ void group_argmax(double& v, uint32_t& idx) {
  if constexpr (G == 64) {  // DPP sequences (no value is NaN)
    const double m = wave_max_f64(v);
    idx = wave_min(v == m ? idx : 0xFFFFFFFFu);
    v = m;
  } else {
    auto take = [&](double ov, uint32_t oi) {
      if (ov > v || (ov == v && oi < idx)) {
        v = ov;
        idx = oi;
      }
    };
    take(row_ror<8>(v), row_ror<8>(idx));
    take(row_ror<4>(v), row_ror<4>(idx));
    take(row_ror<2>(v), row_ror<2>(idx));
    take(row_ror<1>(v), row_ror<1>(idx));
  }
}

template <int G>
__device__ __forceinline__ void group_argmin(double& v, uint32_t& idx) {
  if constexpr (G == 64) {  // DPP sequences (no value is NaN)
    const double m = wave_min_f64(v);
    idx = wave_min(v == m ? idx : 0xFFFFFFFFu);
    v = m;
  } else {
    auto take = [&](double ov, uint32_t oi) {
      if (ov < v || (ov == v && oi < idx)) {
        v = ov;
        idx = oi;
      }
    };
    take(row_ror<8>(v), row_ror<8>(idx));
    take(row_ror<4>(v), row_ror<4>(idx));
    take(row_ror<2>(v), row_ror<2>(idx));
    take(row_ror<1>(v), row_ror<1>(idx));
  }
}

// Walk over the pairs (i < j < n) in row-major order: start at linear
// index p, then advance by `by` indices at a time.
struct PairWalk {
  uint32_t i, r, n;  // row i, offset r within the row (j = i + 1 + r)
  __device__ __forceinline__ PairWalk(uint32_t p, uint32_t n_) : i(0), r(p), n(n_) { settle(); }
  __device__ __forceinline__ void settle() {
    while (i + 1 < n && r >= n - 1 - i) {
      r -= n - 1 - i;
      ++i;
    }
  }
  __device__ __forceinline__ void advance(uint32_t by) {
    r += by;
    settle();
  }
  __device__ __forceinline__ uint32_t j() const { return i + 1 + r; }
};

// LDS of one event: momenta and unit vectors (small events first keep |p|,
// 1/|p| and transverse momenta there), and the jet list, `slots` entries each.
struct EventLds {
  double *pE, *px, *py, *pz, *ux, *uy, *uz;
  uint16_t* list;
  __device__ __forceinline__ EventLds(double* base, uint32_t slots, uint16_t* jets)
      : pE(base), px(base + slots), py(base + 2 * slots), pz(base + 3 * slots), ux(base + 4 * slots),
        uy(base + 5 * slots), uz(base + 6 * slots), list(jets) {}
};

// Observables v of event e (np partons) by a group of P lanes of one wave,
// this lane being `lane` of group `grp`.  The sums over partons run over S <=
// P lanes (each S of the group's lanes make the same sums), thrust's planes
// and Durham's pairs over all P: maxima and minima do not depend on the
// split, so the results have the same bits for every P.  Returns the status.
template <int S, int P, int MV, bool kMassive>
__device__ __forceinline__ int group_observables(const Records& r, const EventInputs& in, uint64_t e, int np,
                                                 double ecm, int status, uint32_t lane, uint32_t grp,
                                                 const EventLds& L, double* v) {
  constexpr uint64_t kGroupBits = P == 64 ? ~0ull : ((1ull << (P % 64)) - 1ull);
  double *pE = L.pE, *px = L.px, *py = L.py, *pz = L.pz, *ux = L.ux, *uy = L.uy, *uz = L.uz;
  uint16_t* list = L.list;
  const uint32_t sub = lane % S;
  const double sh = ecm * ecm;
  // nonfin: partons with a non-finite component; offshell: finite partons
  // off their mass shell (kept apart: one non-finite parton makes the
  // event NONFINITE, any number of finite off-shell ones CONSERVATION)
  double tE = 0.0, tx = 0.0, ty = 0.0, tz = 0.0, nonfin = 0.0, offshell = 0.0, sum = 0.0;
  double mxx = 0.0, myy = 0.0, mzz = 0.0, mxy = 0.0, mxz = 0.0, myz = 0.0;
  for (int a = sub; a < np; a += S) {
    const uint64_t o = (uint64_t)a * r.stride + e;
    const P4 p{r.E[o], r.x[o], r.y[o], r.z[o]};
    pE[a] = p.e;
    px[a] = p.x;
    py[a] = p.y;
    pz[a] = p.z;
    if (!(isfinite(p.e) && isfinite(p.x) && isfinite(p.y) && isfinite(p.z))) nonfin += 1.0;
    else if (!(fabs(mdot(p, p) - shell2<kMassive>(in, r, a, e)) <= 1e-10 * sh)) offshell += 1.0;
    tE += p.e;
    tx += p.x;
    ty += p.y;
    tz += p.z;
    const double l = len3(p.x, p.y, p.z);
    sum += l;
    const double il = 1.0 / l;
    mxx = fma(p.x * p.x, il, mxx);
    myy = fma(p.y * p.y, il, myy);
    mzz = fma(p.z * p.z, il, mzz);
    mxy = fma(p.x * p.y, il, mxy);
    mxz = fma(p.x * p.z, il, mxz);
    myz = fma(p.y * p.z, il, myz);
  }
  tE = group_sum<S>(tE);
  tx = group_sum<S>(tx);
  ty = group_sum<S>(ty);
  tz = group_sum<S>(tz);
  nonfin = group_sum<S>(nonfin);
  offshell = group_sum<S>(offshell);
  if (status == kDone) {
    const double tol = 1e-10 * ecm;
    if (nonfin > 0.0) status = kNonFinite;
    else if (fabs(tE - ecm) > tol || fabs(tx) > tol || fabs(ty) > tol || fabs(tz) > tol || offshell > 0.0)
      status = kConservation;
  }
  if (status == kDone) {
    sum = group_sum<S>(sum);
    mxx = group_sum<S>(mxx);
    myy = group_sum<S>(myy);
    mzz = group_sum<S>(mzz);
    mxy = group_sum<S>(mxy);
    mxz = group_sum<S>(mxz);
    myz = group_sum<S>(myz);
    // thrust over the candidate planes
    const uint32_t npairs = (uint32_t)np * (np - 1) / 2;
    double best = -1.0;
    uint32_t bidx = 0xFFFFFFFFu;
    double bx = 0.0, by = 0.0, bz = 1.0;
    PairWalk pw(lane, (uint32_t)np);
    for (uint32_t pidx = lane; pidx < npairs; pidx += P, pw.advance(P)) {
      const uint32_t i = pw.i, j = pw.j();
      const double xi = px[i], yi = py[i], zi = pz[i], xj = px[j], yj = py[j], zj = pz[j];
      const double nx = det2(yi, zj, zi, yj), ny = det2(zi, xj, xi, zj), nz = det2(xi, yj, yi, xj);
      double vx = 0.0, vy = 0.0, vz = 0.0;
      for (int k = 0; k < np; ++k) {
        const double xk = px[k], yk = py[k], zk = pz[k];
        const double sk = side(dot3(xk, yk, zk, nx, ny, nz), k == (int)i || k == (int)j);
        vx = fma(sk, xk, vx);
        vy = fma(sk, yk, vy);
        vz = fma(sk, zk, vz);
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const double si = (c < 2) ? 1.0 : -1.0, sj = (c & 1) ? -1.0 : 1.0;
        const double wx = vx + si * xi + sj * xj, wy = vy + si * yi + sj * yj, wz = vz + si * zi + sj * zj;
        const double m2 = sq3(wx, wy, wz);
        if (m2 > best) { best = m2; bidx = 4 * pidx + c; bx = wx; by = wy; bz = wz; }
      }
    }
    double wbest = best;
    uint32_t widx = bidx;
    group_argmax<P>(wbest, widx);
    // the winning lane of the group broadcasts its vector
    const uint64_t who = __ballot(bidx == widx && best == wbest);
    const uint32_t src = (uint32_t)__ffsll((unsigned long long)((who >> (grp * P)) & kGroupBits)) - 1;
    bx = __shfl(bx, (int)src, P);
    by = __shfl(by, (int)src, P);
    bz = __shfl(bz, (int)src, P);
    const double lb = sqrt(wbest);
    double ax = 0.0, ay = 0.0, az = 1.0;
    if (lb > 0.0) { ax = bx / lb; ay = by / lb; az = bz / lb; }
    const double T = sum > 0.0 ? lb / sum : 0.0;
    const double tau = 1.0 - T;
    v[2] = tau > 0.0 ? tau : 0.0;
    v[3] = c_parameter(sum, mxx, myy, mzz, mxy, mxz, myz);
    // hemispheres
    double hpE = 0, hpx = 0, hpy = 0, hpz = 0, hmE = 0, hmx = 0, hmy = 0, hmz = 0, bp = 0, bm = 0;
    for (int a = sub; a < np; a += S) {
      const double x = px[a], y = py[a], z = pz[a], en = pE[a];
      const double d = dot3(x, y, z, ax, ay, az);
      const double kt = len3(det2(y, az, z, ay), det2(z, ax, x, az), det2(x, ay, y, ax));
      if (d >= 0.0) { hpE += en; hpx += x; hpy += y; hpz += z; bp += kt; }
      else { hmE += en; hmx += x; hmy += y; hmz += z; bm += kt; }
    }
    hpE = group_sum<S>(hpE); hpx = group_sum<S>(hpx); hpy = group_sum<S>(hpy); hpz = group_sum<S>(hpz);
    hmE = group_sum<S>(hmE); hmx = group_sum<S>(hmx); hmy = group_sum<S>(hmy); hmz = group_sum<S>(hmz);
    bp = group_sum<S>(bp); bm = group_sum<S>(bm);
    const double mp = mass2(hpE, hpx, hpy, hpz), mm = mass2(hmE, hmx, hmy, hmz);
    const double rho = (mp > mm ? mp : mm) / sh;
    v[4] = rho > 0.0 ? rho : 0.0;
    bp /= 2.0 * sum;
    bm /= 2.0 * sum;
    v[5] = bp + bm;
    v[6] = bp > bm ? bp : bm;
    // Durham: pair scan over the current jets each step
    const double inv_s = 1.0 / sh;
    for (int a = lane; a < np; a += P) {
      list[a] = (uint16_t)a;
      const double l = len3(px[a], py[a], pz[a]);
      ux[a] = px[a] / l;
      uy[a] = py[a] / l;
      uz[a] = pz[a] / l;
    }
    int m = np;
    while (m > 2) {
      const uint32_t mp2 = (uint32_t)m * (m - 1) / 2;
      double ymin = INFINITY;
      uint32_t yidx = 0xFFFFFFFFu;
      PairWalk dw(lane, (uint32_t)m);
      for (uint32_t pidx = lane; pidx < mp2; pidx += P, dw.advance(P)) {
        const int ja = list[dw.i], jb = list[dw.j()];
        const double dx = ux[ja] - ux[jb], dy = uy[ja] - uy[jb], dz = uz[ja] - uz[jb];
        const double y = jet_y(pE[ja] < pE[jb] ? pE[ja] : pE[jb], dx, dy, dz, inv_s);
        if (y < ymin) { ymin = y; yidx = (dw.i << 16) | dw.j(); }  // ordered like pidx
      }
      group_argmin<P>(ymin, yidx);
      const uint32_t ia = yidx >> 16, ib = yidx & 0xFFFFu;
      if (m == 4) v[1] = ymin;
      if (m == 3) {  // two jets are left
        v[0] = ymin;
        break;
      }
      const int ja = list[ia], jb = list[ib];
      const double en = pE[ja] + pE[jb], x = px[ja] + px[jb], y = py[ja] + py[jb], z = pz[ja] + pz[jb];
      const double l = len3(x, y, z);
      // one of E and the components per lane: one division instead of three in
      // the step's serial chain (stress batch 4.15 -> 4.06 ms)
      if (lane < 4) {
        const double c = lane == 0 ? x : lane == 1 ? y : z;
        (lane == 3 ? pE : lane == 0 ? px : lane == 1 ? py : pz)[ja] = lane == 3 ? en : c;
        if (lane < 3) (lane == 0 ? ux : lane == 1 ? uy : uz)[ja] = c / l;
      }
      // drop jet ib from the list: read the entries after it, then write them back one place down
      uint16_t mv[MV];
#pragma unroll
      for (uint32_t k = 0; k < MV; ++k) {
        const uint32_t a = ib + 1 + lane + P * k;
        mv[k] = a < (uint32_t)m ? list[a] : (uint16_t)0;
      }
#pragma unroll
      for (uint32_t k = 0; k < MV; ++k) {
        const uint32_t a = ib + 1 + lane + P * k;
        if (a < (uint32_t)m) list[a - 1] = mv[k];
      }
      --m;
    }
  }
  return status;
}

// Events of 9 to 31 partons (G = 16) or more (G = 64); `slots` (at most G *
// MV) LDS parton slots per group
// (four waves per SIMD: 126 or 127 registers, none spilled; stress 10^6 events
// 6.9 -> 6.0 ms against the three waves of the unconstrained build, LEP
// unchanged; five waves, 43 spilled, 5.7 ms on stress but 3% slower on LEP)
template <int G, int MV, bool kMassive>
__device__ __forceinline__ void group_events(const Records& r, const Summary& sm, const EventInputs& in,
                                             const Scratch& sc, uint32_t slots, uint32_t blk, uint32_t grid) {
  const uint32_t cap = r.cap;
  const uint32_t lo_n = G == 16 ? kObsWaveThreshold : kObsGroup64, hi_n = G == 16 ? kObsGroup64 : cap + 1;
  const uint32_t *perm = sc.perm, *cnt = sc.cnt;
  constexpr uint32_t kGroups = 64 / G;
  extern __shared__ double lds[];
  // this block's copy of the global histogram set (block b: copy b mod
  // kHistCopies), filled with each event's atomics directly: FP64 sums, or
  // the fixed-point integer cells.  A group block holds a few events, so an
  // LDS set would cost more to clear and flush than it saves (k_obs, with
  // 256 to 1024 events per block, keeps one)
  const uint32_t c0 = (blk % kHistCopies) * (uint32_t)kHistDoubles;
  const uint32_t lane = threadIdx.x % G, grp = threadIdx.x / G;
  const EventLds L(lds + (size_t)grp * 7 * slots, slots,
                   (uint16_t*)(lds + (size_t)kGroups * 7 * slots) + (size_t)grp * slots);
  // cnt[cap - m] counts the events with at least m partons (see k_obs)
  const uint32_t q_lo = hi_n <= cap ? cnt[cap - hi_n] : 0u;
  const uint32_t q_hi = lo_n <= cap ? cnt[cap - lo_n] : 0u;
  // the grid is sized for the worst case: blocks without an event of this
  // range leave at once (the whole block, before touching LDS)
  if (q_lo + blk * kGroups >= q_hi) return;
  const bool fixed = in.fixed_hist != 0;
  FixScale fxs{0, 0};
  if (fixed) fxs = fix_scale(sc);
  const FixScale* fx = fixed ? &fxs : nullptr;
  __syncthreads();
  for (uint32_t q = q_lo + blk * kGroups + grp; q < q_hi; q += grid * kGroups) {
    const uint64_t e = perm[q];
    const int np = sm.i[kSiN * sm.stride + e];
    const double ecm = in.ecm_of(e);
    double v[7] = {0, 0, 0, 0, 0, 0, 0};
    const int status = group_observables<G, G, MV, kMassive>(r, in, e, np, ecm, sm.i[kSiStatus * sm.stride + e], lane,
                                                             grp, L, v);
    if (status == kDone) {
      double* gh = fixed ? reinterpret_cast<double*>(sc.ihist + c0) : sc.hcopy + c0;
      if (lane == 0) hist_fill(gh, ObsOut{{v[0], v[1], v[2], v[3], v[4], v[5], v[6]}, status},
                                   sm.d[kSdW * sm.stride + e], sm.d[kSdCos * sm.stride + e], fx);
    }
#pragma unroll
    for (uint32_t h = 0; h < 7; ++h)  // the group's lanes share the seven stores
      if (h % G == lane) sm.d[(kSdY23 + h) * sm.stride + e] = v[h];
    if (lane == 0) sm.i[kSiStatus * sm.stride + e] = status;
  }
}

template <int G, int MV, bool kMassive>
__global__ void __launch_bounds__(64, 4) k_obs_group(Records r, Summary sm, EventInputs in, Scratch sc,
                                                     uint32_t slots) {
  group_events<G, MV, kMassive>(r, sm, in, sc, slots, blockIdx.x, gridDim.x);
}

template <int G, int MV, bool kMassive>
__global__ void __launch_bounds__(64, 4) k_obs_group_jobs(ObsArgs<true> A, uint32_t slots) {
  with_job(A, kObsStageGroup, [&](const ObsJob& J, uint32_t blk, uint32_t grid) {
    group_events<G, MV, kMassive>(J.r, J.sm, J.in, J.sc, slots, blk, grid);
  });
}

// Observables v of an event of at most kObsRegSlots partons by one wave: the
// quantities of reg_observables with its sums in its order (each lane makes
// them all, from LDS), one candidate plane of thrust and one pair of Durham
// per lane, so the same bits in a chain some six times shorter.  Returns the
// status.
template <bool kMassive>
__device__ __forceinline__ int small_observables(const Records& r, const EventInputs& in, uint64_t e, int np,
                                                 double ecm, int status, uint32_t lane, const EventLds& L, double* v) {
  static_assert(kObsRegSlots * (kObsRegSlots - 1) / 2 <= 64, "one pair per lane");
  double *E = L.pE, *X = L.px, *Y = L.py, *Z = L.pz;
  const double sh = ecm * ecm;
  if (status != kDone) return status;
  bool fine = true, shell = true;
  double l = 0.0;
  if (lane < (uint32_t)np) {
    const P4 p = r.load(lane, e);
    E[lane] = p.e;
    X[lane] = p.x;
    Y[lane] = p.y;
    Z[lane] = p.z;
    fine = isfinite(p.e) && isfinite(p.x) && isfinite(p.y) && isfinite(p.z);
    shell = fabs(mdot(p, p) - shell2<kMassive>(in, r, lane, e)) <= 1e-10 * sh;
    l = len3(p.x, p.y, p.z);
    L.ux[lane] = l;
    L.uy[lane] = 1.0 / l;
  }
  double tE = 0.0, tx = 0.0, ty = 0.0, tz = 0.0;
  double sum = 0.0, mxx = 0.0, myy = 0.0, mzz = 0.0, mxy = 0.0, mxz = 0.0, myz = 0.0;
  for (int a = 0; a < np; ++a) {
    const double x = X[a], y = Y[a], z = Z[a], il = L.uy[a];
    tE += E[a];
    tx += x;
    ty += y;
    tz += z;
    sum += L.ux[a];
    mxx = fma(x * x, il, mxx);
    myy = fma(y * y, il, myy);
    mzz = fma(z * z, il, mzz);
    mxy = fma(x * y, il, mxy);
    mxz = fma(x * z, il, mxz);
    myz = fma(y * z, il, myz);
  }
  const double tol = 1e-10 * ecm;
  if (__any(!fine)) return kNonFinite;
  if (fabs(tE - ecm) > tol || fabs(tx) > tol || fabs(ty) > tol || fabs(tz) > tol || __any(!shell)) return kConservation;
  // thrust: lane p takes the p-th pair (i < j); the first lane with the
  // largest candidate is the first in the serial scan
  const uint32_t npairs = (uint32_t)np * (np - 1) / 2;
  const PairWalk pw(lane < npairs ? lane : 0u, (uint32_t)np);
  const int i = (int)pw.i, j = (int)pw.j();
  double best = -1.0, bx = 0.0, by = 0.0, bz = 1.0;
  if (np < 3) {
    for (int mk = 0; mk < (1 << np); ++mk) {
      double vx = 0.0, vy = 0.0, vz = 0.0;
      for (int a = 0; a < np; ++a) {
        const double sg = (mk >> a & 1) ? -1.0 : 1.0;
        vx += sg * X[a];
        vy += sg * Y[a];
        vz += sg * Z[a];
      }
      const double m2 = sq3(vx, vy, vz);
      if (m2 > best) { best = m2; bx = vx; by = vy; bz = vz; }
    }
  } else {
    if (lane < npairs) {
      const double xi = X[i], yi = Y[i], zi = Z[i], xj = X[j], yj = Y[j], zj = Z[j];
      const double nx = det2(yi, zj, zi, yj), ny = det2(zi, xj, xi, zj), nz = det2(xi, yj, yi, xj);
      double vx = 0.0, vy = 0.0, vz = 0.0;
      for (int k = 0; k < np; ++k) {
        const double xk = X[k], yk = Y[k], zk = Z[k];
        const double sk = side(dot3(xk, yk, zk, nx, ny, nz), k == i || k == j);
        vx = fma(sk, xk, vx);
        vy = fma(sk, yk, vy);
        vz = fma(sk, zk, vz);
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const double si = (c < 2) ? 1.0 : -1.0, sj = (c & 1) ? -1.0 : 1.0;
        const double wx = vx + si * xi + sj * xj, wy = vy + si * yi + sj * yj, wz = vz + si * zi + sj * zj;
        const double m2 = sq3(wx, wy, wz);
        if (m2 > best) { best = m2; bx = wx; by = wy; bz = wz; }
      }
    }
    const double most = wave_max_f64(best);
    const int src = __ffsll((unsigned long long)__ballot(best == most)) - 1;
    best = most;
    bx = lane_value(bx, src);
    by = lane_value(by, src);
    bz = lane_value(bz, src);
  }
  const double lb = sqrt(best);
  double ax = 0.0, ay = 0.0, az = 1.0;
  if (lb > 0.0) { ax = bx / lb; ay = by / lb; az = bz / lb; }
  const double T = sum > 0.0 ? lb / sum : 0.0;
  const double tau = 1.0 - T;
  v[2] = tau > 0.0 ? tau : 0.0;
  v[3] = c_parameter(sum, mxx, myy, mzz, mxy, mxz, myz);
  // hemispheres
  bool plus = false;
  if (lane < (uint32_t)np) {
    const P4 p{E[lane], X[lane], Y[lane], Z[lane]};
    plus = dot3(p.x, p.y, p.z, ax, ay, az) >= 0.0;
    L.uz[lane] = len3(det2(p.y, az, p.z, ay), det2(p.z, ax, p.x, az), det2(p.x, ay, p.y, ax));
  }
  const uint64_t in_plus = __ballot(plus);
  P4 hp{0, 0, 0, 0}, hm{0, 0, 0, 0};
  double bp = 0.0, bm = 0.0;
  for (int a = 0; a < np; ++a) {
    const P4 p{E[a], X[a], Y[a], Z[a]};
    const double kt = L.uz[a];
    if (in_plus >> a & 1ull) { hp.e += p.e; hp.x += p.x; hp.y += p.y; hp.z += p.z; bp += kt; }
    else { hm.e += p.e; hm.x += p.x; hm.y += p.y; hm.z += p.z; bm += kt; }
  }
  const double mp = mass2(hp.e, hp.x, hp.y, hp.z), mm = mass2(hm.e, hm.x, hm.y, hm.z);
  const double rho = (mp > mm ? mp : mm) / sh;
  v[4] = rho > 0.0 ? rho : 0.0;
  bp /= 2.0 * sum;
  bm /= 2.0 * sum;
  v[5] = bp + bm;
  v[6] = bp > bm ? bp : bm;
  if (np < 3) return status;
  // Durham: lane p keeps the y of its pair, computed again when a merge
  // touches one of its jets
  const double inv_s = 1.0 / sh;
  if (lane < (uint32_t)np) {
    L.ux[lane] = X[lane] / l;
    L.uy[lane] = Y[lane] / l;
    L.uz[lane] = Z[lane] / l;
  }
  uint32_t alive = (1u << np) - 1u;
  double y = 0.0;
  bool stale = true;
  for (int m = np; m > 2; --m) {
    const bool live = lane < npairs && (alive >> i & 1u) && (alive >> j & 1u);
    if (live && stale) {
      const double dx = L.ux[i] - L.ux[j], dy = L.uy[i] - L.uy[j], dz = L.uz[i] - L.uz[j];
      const double ei = E[i], ej = E[j];
      y = jet_y(ei < ej ? ei : ej, dx, dy, dz, inv_s);
    }
    // the serial scan takes the first pair and then any smaller one: a NaN
    // stays only if it comes first
    const int first = __ffsll((unsigned long long)__ballot(live)) - 1;
    const double y0 = lane_value(y, first);
    const double least = wave_min_f64(live && y == y ? y : INFINITY);
    const bool keep = !(y0 == y0);
    const double ymin = keep ? y0 : least;
    const int win = keep ? first : __ffsll((unsigned long long)__ballot(live && y == least)) - 1;
    if (m == 4) v[1] = ymin;
    if (m == 3) v[0] = ymin;
    if (m == 3) break;
    const int ia = __builtin_amdgcn_readlane(i, win), ib = __builtin_amdgcn_readlane(j, win);
    const double en = E[ia] + E[ib], x = X[ia] + X[ib], yy = Y[ia] + Y[ib], z = Z[ia] + Z[ib];
    const double lj = len3(x, yy, z);
    const double ux = x / lj, uy = yy / lj, uz = z / lj;
    E[ia] = en;  // the same values from every lane
    X[ia] = x;
    Y[ia] = yy;
    Z[ia] = z;
    L.ux[ia] = ux;
    L.uy[ia] = uy;
    L.uz[ia] = uz;
    alive &= ~(1u << ib);
    stale = i == ia || j == ia;
  }
  return status;
}

__global__ void __launch_bounds__(256) k_obs_wmax(Summary sm, uint32_t n, unsigned long long* wmax) {
  double w = 0.0;
  for (uint32_t e = blockIdx.x * 256 + threadIdx.x; e < n; e += gridDim.x * 256)
    w = fmax(w, fabs(sm.d[kSdW * sm.stride + e]));
  wave_max_weight(w, wmax);
}

// Small launches: one wave per event of any size, in event order, a block's
// waves (up to four) sharing an LDS histogram set, which ends in one of
// `copies` copies of the global set (0: in hist itself).
// With few events the general path is bound by its chain of eight launches
// and by one lane's (or sixteen lanes') scan over all of an event's planes and
// pairs: 100 LEP events took 118 us; spread over a wave, 27 us.  Four waves per
// SIMD: 128 registers with 32 spilled (36 with quark masses); two, three and
// four took 5003 LEP events 55.6, 47.6 and 49.6 us, 20000 124, 96 and 91.
// `slots`: LDS parton slots per wave (at least the capacity).
template <bool kMassive>
__global__ void __launch_bounds__(256, 4) k_obs_few(Records r, Summary sm, EventInputs in, Scratch sc,
                                                                  uint32_t n, uint32_t slots, uint32_t copies,
                                                                  double* __restrict__ hist) {
  extern __shared__ double lds[];
  __shared__ double lh[kHistDoubles];
  for (int a = threadIdx.x; a < kHistDoubles; a += blockDim.x) lh[a] = 0.0;
  const bool fixed = in.fixed_hist != 0;
  FixScale fxs{0, 0};
  if (fixed) fxs = fix_scale(sc);
  __syncthreads();
  const uint32_t lane = threadIdx.x % 64, w = threadIdx.x / 64, waves = blockDim.x / 64;
  const EventLds L(lds + (size_t)w * 7 * slots, slots,
                   (uint16_t*)(lds + (size_t)waves * 7 * slots) + (size_t)w * slots);
  for (uint64_t e = (uint64_t)blockIdx.x * waves + w; e < n; e += (uint64_t)gridDim.x * waves) {
    const int np = __builtin_amdgcn_readfirstlane(sm.i[kSiN * sm.stride + e]);
    int status = __builtin_amdgcn_readfirstlane(sm.i[kSiStatus * sm.stride + e]);
    const double ecm = in.ecm_of(e);
    double v[7] = {0, 0, 0, 0, 0, 0, 0};
    if (np <= kObsRegSlots) status = small_observables<kMassive>(r, in, e, np, ecm, status, lane, L, v);
    else if (np < (int)kObsGroup64)
      status = group_observables<16, 64, 1, kMassive>(r, in, e, np, ecm, status, lane, 0, L, v);
    else
      status = group_observables<64, 64, kObsWaveMaxCap / 64, kMassive>(r, in, e, np, ecm, status, lane, 0, L, v);
    double mine = sm.d[kSdCos * sm.stride + e];  // lane h: quantity h (7: cos theta)
#pragma unroll
    for (uint32_t h = 0; h < 7; ++h)
      if (lane == h) mine = v[h];
    if (status == kDone && lane < (uint32_t)kNObs)
      hist_add(lh, (int)lane, mine, sm.d[kSdW * sm.stride + e], fixed ? &fxs : nullptr);
    if (lane < 7) sm.d[(kSdY23 + lane) * sm.stride + e] = mine;
    if (lane == 0) sm.i[kSiStatus * sm.stride + e] = status;
  }
  __syncthreads();
  hist_flush(lh, sc, fixed, threadIdx.x, blockDim.x, copies, hist);
}

static inline uint32_t blocks_for(uint64_t n, uint32_t b) { return (uint32_t)((n + b - 1) / b); }

// the one-wave-per-event launch of small requests
struct ObsFewLaunch {
  uint32_t blocks, threads, slots, lds, copies;
};

static size_t obs_group_lds(uint32_t g, uint32_t slots) {
  return (size_t)(64 / g) * slots * (7 * 8 + 2) + 64;
}

// One wave per event up to kObsFew events (kObsFewBig with records above 128
// partons, whose events are larger); kObsWaveMaxCap bounds the LDS.  Observables
// of a plain call, general path and this one: 100 LEP events 118 and 27 us,
// 5003 148 and 54, 20000 166 and 95, 50000 170 and 193; at 200 GeV and t_C =
// 0.5, 30000 events 279 and 255, 60000 283 and 467; at 500 GeV and t_C = 0.5,
// 10000 events 598 and 340, 100000 644 and 1831.  FP64 sums go straight into
// one histogram of the library's: copies would add two launches, and the
// additions of up to 2048 blocks do not queue up.  A caller's histogram gets
// that one added by plain loads and stores, as k_hist_finalize does (one launch
// more): hardware FP64 atomics lose additions where the memory is not ordinary
// device memory (pinned host or managed).
static bool obs_few_launch(uint64_t n, uint32_t cap, bool fixed, ObsFewLaunch* out) {
  if (cap > kObsWaveMaxCap || n > (cap > 128 ? kObsFewBig : kObsFew)) return false;
  const uint32_t waves = cap <= 128 ? 4 : cap <= 256 ? 2 : 1;  // at most 30 KB of LDS
  out->threads = 64 * waves;
  out->blocks = (uint32_t)std::min<uint64_t>((n + waves - 1) / waves, kObsFewBlocks);
  out->slots = std::max<uint32_t>(cap, kObsRegSlots);
  out->lds = waves * out->slots * (7 * 8 + 2);
  out->copies = fixed ? kHistCopies : 0u;
  return true;
}

static uint32_t obs_wmax_blocks(uint64_t n) { return (uint32_t)std::min<uint64_t>(blocks_for(n, 256), 256); }

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
void launch_me(const Records& r, const Summary& s, const EventInputs& in, uint32_t n,
               hipStream_t st, double* zero_hist) {
  if (!n) return;
  hipLaunchKernelGGL(k_me, dim3(blocks_for(n, 256)), dim3(256), 0, st, r, s, in, n, zero_hist);
}

void launch_load_records(const Records& r, const Summary& s, const CsrStarts& in, uint32_t n, double* ecm,
                         unsigned long long* bad, double* zero_hist, hipStream_t st) {
  if (!n) return;
  hipLaunchKernelGGL(k_load_records, dim3(blocks_for((uint64_t)n * kLoadLanes, 256)), dim3(256), 0, st, r, s, in, n,
                     ecm, bad, zero_hist);
}

void launch_shower_plain(const Records& r, const Summary& s, const EventInputs& in, uint32_t n,
                         uint32_t block, uint32_t waves, hipStream_t st) {
  if (!n) return;
  if (block == 0 || block > 256) block = 256;
  const dim3 g(blocks_for(n, block)), b(block);
  if (in.massive) hipLaunchKernelGGL((k_shower_plain<2, true>), g, b, 0, st, r, s, in, n);
  else if (waves >= 4) hipLaunchKernelGGL(k_shower_plain<4>, g, b, 0, st, r, s, in, n);
  else if (waves == 3) hipLaunchKernelGGL(k_shower_plain<3>, g, b, 0, st, r, s, in, n);
  else hipLaunchKernelGGL(k_shower_plain<2>, g, b, 0, st, r, s, in, n);
}

// Parton slots of Durham scratch per thread of the one-thread-per-event
// pass: it only sees events below the wave threshold when the wave pass
// runs, else every event up to cap.
static uint32_t thread_slots(uint32_t cap) {
  return (cap <= kObsWaveMaxCap && kObsWaveThreshold <= cap) ? kObsWaveThreshold - 1 : cap;
}

// at most 2^24 parton slots of scratch (1.1 GB) and 2^18 threads (about
// the resident threads of the pass), at most n
uint64_t obs_threads(uint64_t n, uint32_t cap) {
  const uint64_t most =
      std::max<uint64_t>(256, std::min<uint64_t>(1ull << 18, ((1ull << 24) / thread_slots(cap)) / 256 * 256));
  const uint64_t t = ((n + 255) / 256) * 256;
  return t < most ? t : most;
}

static inline uint64_t al256(uint64_t v) { return (v + 255) / 256 * 256; }

uint64_t obs_scratch_bytes(uint64_t n, uint32_t cap) {
  const uint64_t m = obs_threads(n, cap) * thread_slots(cap);
  return 8 * al256(m * 8) + al256(m * 2) + al256(m) + al256(n * 4) + al256((cap + 2) * 4) +
         2 * al256(kHistCopies * kHistDoubles * 8) + al256(8) + 256;
}

// the part of the scratch that every request's pass needs
static void carve_lists(Scratch& s, char*& p, uint64_t n, uint32_t cap) {
  auto take = [&](uint64_t bytes) {
    char* q = p;
    p += al256(bytes);
    return q;
  };
  s.perm = (uint32_t*)take(n * 4);
  s.cnt = (uint32_t*)take((cap + 2) * 4);
  s.hcopy = (double*)take(kHistCopies * kHistDoubles * 8);
  s.ihist = (unsigned long long*)take(kHistCopies * kHistDoubles * 8);
  s.wmax = (unsigned long long*)take(8);
  s.lbits = 0;
  while ((1ull << s.lbits) < n) ++s.lbits;
  // events with at least `threshold` partons go to lane groups (LDS holds up
  // to kObsWaveMaxCap partons); smaller ones to one thread each
  s.threshold = cap <= kObsWaveMaxCap ? kObsWaveThreshold : 0xFFFFFFFFu;
}

Scratch carve_obs_scratch(char*& p, uint64_t n, uint32_t cap) {
  Scratch s;
  s.stride = obs_threads(n, cap);
  const uint64_t m = s.stride * thread_slots(cap);
  auto take = [&](uint64_t bytes) {
    char* q = p;
    p += al256(bytes);
    return q;
  };
  s.E = (double*)take(m * 8);
  s.x = (double*)take(m * 8);
  s.y = (double*)take(m * 8);
  s.z = (double*)take(m * 8);
  s.ux = (double*)take(m * 8);
  s.uy = (double*)take(m * 8);
  s.uz = (double*)take(m * 8);
  s.dn = (double*)take(m * 8);
  s.nn = (uint16_t*)take(m * 2);
  s.dead = (uint8_t*)take(m);
  carve_lists(s, p, n, cap);
  return s;
}

// Most blocks of the 64-lane groups: where a call has no event that large, 32768
// blocks that leave at once take 8.4 us, 4096 take 4.8 (10^6 events at 500 GeV:
// 363 and 362 us).
constexpr uint32_t kObsGroup64Blocks = 4096;

// The pass over one job or a table of jobs, `blocks` in each stage in all;
// records of at most `cap` partons.
template <bool kMulti>
static void launch_general(const ObsArgs<kMulti>& A, const uint32_t* blocks, uint32_t cap, bool massive,
                           hipStream_t st) {
  const dim3 b256(256), b64(64);
  hipLaunchKernelGGL(k_obs_reset<kMulti>, dim3(blocks[kObsStageHist]), b256, 0, st, A);
  hipLaunchKernelGGL(k_obs_count<kMulti>, dim3(blocks[kObsStageSort]), b256, 0, st, A);
  hipLaunchKernelGGL(k_obs_scan<kMulti>, dim3(blocks[kObsStageScan]), b256, 0, st, A);
  hipLaunchKernelGGL(k_obs_scatter<kMulti>, dim3(blocks[kObsStageSort]), b256, 0, st, A);
  if constexpr (kMulti) {
    hipLaunchKernelGGL(massive ? k_obs_jobs<true> : k_obs_jobs<false>, dim3(blocks[kObsStageWindow]), b256, 0, st, A);
  } else {
    const ObsJob& j = A.job;
    hipLaunchKernelGGL(massive ? k_obs<true> : k_obs<false>, dim3(blocks[kObsStageWindow]), b256, 0, st, j.r, j.sm, j.in,
                       j.sc, j.n, j.hist);
  }
  if (cap <= kObsWaveMaxCap && cap >= kObsWaveThreshold) {
    const uint32_t slots = std::min<uint32_t>(kObsGroup64 - 1, cap);
    const dim3 gb(blocks[kObsStageGroup]);
    constexpr int kMv = kObsWaveMaxCap / 64;
    if constexpr (kMulti) {
      const auto g16 = massive ? k_obs_group_jobs<16, 2, true> : k_obs_group_jobs<16, 2, false>;
      const auto g64 = massive ? k_obs_group_jobs<64, kMv, true> : k_obs_group_jobs<64, kMv, false>;
      hipLaunchKernelGGL(g16, gb, b64, obs_group_lds(16, slots), st, A, slots);
      if (cap >= kObsGroup64) hipLaunchKernelGGL(g64, gb, b64, obs_group_lds(64, cap), st, A, cap);
    } else {
      const ObsJob& j = A.job;
      const auto g16 = massive ? k_obs_group<16, 2, true> : k_obs_group<16, 2, false>;
      const auto g64 = massive ? k_obs_group<64, kMv, true> : k_obs_group<64, kMv, false>;
      hipLaunchKernelGGL(g16, gb, b64, obs_group_lds(16, slots), st, j.r, j.sm, j.in, j.sc, slots);
      const dim3 gb64(std::min(blocks[kObsStageGroup], kObsGroup64Blocks));
      if (cap >= kObsGroup64)
        hipLaunchKernelGGL(g64, gb64, b64, obs_group_lds(64, cap), st, j.r, j.sm, j.in, j.sc, cap);
    }
  }
  hipLaunchKernelGGL(k_hist_finalize<kMulti>, dim3(blocks[kObsStageSum]), b256, 0, st, A);
}

// `all`: the events of every job of the launch.  k_obs takes 64 events per wave
// up to two rounds of the 2048 resident waves, then 192 or 256 ordered together
// (window_events derives the number from the grid).  The whole pass, 64 per
// wave and more: 140000 events at 200 GeV 310 and 340 us, 262144 at LEP 219
// and 203, 300000 261 and 235.
static void job_blocks(const ObsJob& j, uint64_t all, uint32_t most_groups, uint32_t* blocks) {
  const uint64_t per = 256 * (all <= 262144 ? 1 : std::min<uint64_t>(4, (all + 131071) / 131072));
  blocks[kObsStageHist] = blocks_for(std::max<uint32_t>(j.r.cap + 1, kHistCopies * kHistDoubles), 256);
  blocks[kObsStageSort] = blocks_for(j.n, 256u * kObsSortPer);
  blocks[kObsStageScan] = 1;
  blocks[kObsStageWindow] = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(j.sc.stride / 256, (j.n + per - 1) / per));
  blocks[kObsStageGroup] = std::min<uint32_t>(j.n, most_groups);
  blocks[kObsStageSum] = kHistBlocks;
}

void launch_obs(const Records& r, const Summary& s, const EventInputs& in, const Scratch& sc,
                uint32_t n, double* hist, double* own, hipStream_t st) {
  if (!n) return;
  const bool fixed = in.fixed_hist != 0, massive = in.massive != 0;
  const ObsArgs<false> A{ObsJob{r, s, in, sc, hist, n, {}}};
  uint32_t blocks[kObsStages];
  job_blocks(A.job, n, kObsWaveBlocks, blocks);
  ObsFewLaunch few;
  if (obs_few_launch(n, r.cap, fixed, &few)) {
    const dim3 b256(256);
    if (few.copies) hipLaunchKernelGGL(k_obs_reset<false>, dim3(blocks[kObsStageHist]), b256, 0, st, A);
    if (fixed) hipLaunchKernelGGL(k_obs_wmax, dim3(obs_wmax_blocks(n)), b256, 0, st, s, n, sc.wmax);
    hipLaunchKernelGGL(massive ? k_obs_few<true> : k_obs_few<false>, dim3(few.blocks), dim3(few.threads), few.lds, st,
                       r, s, in, sc, n, few.slots, few.copies, own ? own : hist);
    if (few.copies) hipLaunchKernelGGL(k_hist_finalize<false>, dim3(kHistBlocks), b256, 0, st, A);
    else if (own) hipLaunchKernelGGL(k_hist_add, dim3(kHistBlocks), b256, 0, st, own, hist);
    return;
  }
  launch_general(A, blocks, r.cap, massive, st);
}

uint64_t obs_job_bytes(uint64_t n, uint32_t cap) {
  return al256(n * 4) + al256((cap + 2) * 4) + 2 * al256(kHistCopies * kHistDoubles * 8) + al256(8);
}

Scratch carve_obs_job(char*& p, uint64_t n, uint32_t cap) {
  Scratch s{};
  s.stride = (n + 255) / 256 * 256;
  carve_lists(s, p, n, cap);
  return s;
}

void plan_obs_jobs(ObsJob* jobs, uint32_t count, ObsPlan* plan) {
  *plan = ObsPlan{};
  uint64_t all = 0;
  for (uint32_t q = 0; q < count; ++q) all += jobs[q].n;
  for (uint32_t q = 0; q < count; ++q) {
    uint32_t blocks[kObsStages];
    job_blocks(jobs[q], all, kObsJobGroupBlocks, blocks);
    for (int k = 0; k < kObsStages; ++k) {
      jobs[q].at[k] = plan->blocks[k];
      plan->blocks[k] += blocks[k];
    }
    plan->cap = std::max(plan->cap, jobs[q].r.cap);
    plan->massive |= jobs[q].in.massive != 0;
  }
  plan->count = count;
}

void launch_obs_jobs(const ObsJob* jobs_dev, const ObsPlan& plan, hipStream_t st) {
  launch_general(ObsArgs<true>{jobs_dev, plan.count}, plan.blocks, plan.cap, plan.massive, st);
}

}  // namespace vsh
