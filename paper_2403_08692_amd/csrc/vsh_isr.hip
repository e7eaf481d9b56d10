// vsh_isr.hip -- the initial-state shower: Drell-Yan q qbar -> V at a hadron
// collider with backward evolution of the incoming lines and the ratio of
// parton densities in the veto (the step to hadron colliders that the
// paper's conclusions name), a few lanes per event.
//
// No parton-density set is available here, so a closed-form density stands
// in for one: every light quark and antiquark flavour has
// f(x) = (63/128) x^(-1/2) (1 - x)^3 (the ten carry half the momentum; a
// gluon density 3 x^(-1) (1 - x)^5 carries the other half and is not
// needed by this branch), independent of the scale.
//
// Per event: flavour uniform over d, u, s, c, b, the quark from either beam,
// the rapidity of V uniform in |y| < ln(sqrt(S)/Q); x_A x_B = Q^2/S; weight
// (arbitrary units) 10 (2Y) tau f(x_A) f(x_B).  Each incoming line (the
// other incoming parton its spectator) makes one trial per cycle with the
// overestimate 2 C_F x^(-1/2)/(1 - z) of the backward-evolution density
// (alpha_s/2 pi) (dt/t) (dz/z) P_qq(z) f(x/z)/f(x) over x < z < z_max(t_C);
// the largest trial above t_C wins (App. A's competition between trials);
// the veto keeps it with probability alpha_s(t)/alpha_s(t_C) times density
// over overestimate, where (1 - z)^2 >= 4 t z / s~ leaves room for it.  An
// accepted emission uses the Catani-Seymour initial-initial map: the emitter
// becomes p_a/z, the gluon (1 - z - v) p_a/z + v p_b + kT (kT^2 = t, the
// smaller root of v(1 - z - v) = t z / s~) and the final state is carried by
// the Lorentz transformation from the old final-state total to the new one.
// Emitted gluons do not radiate.  The arithmetic is FP64 throughout.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <mutex>

#include "../../include/vsh.h"
#include "vsh_internal.hpp"
#include "vsh_math.hpp"

namespace vsh {

struct IsrInputs {
  uint64_t seed, first;
  double sqrt_s, q, tcut;
};

// the stand-in density and its ratio f(x/z)/f(x) as the veto takes it
__device__ __forceinline__ double isr_pdf(double x) {
  return (63.0 / 128.0) / sqrt(x) * ((1.0 - x) * (1.0 - x) * (1.0 - x));
}

constexpr int kIsrHist = 4 * kNHCol * 3;  // the histogram's used rows
constexpr uint32_t kIsrEmitDiv = 2;  // pending emissions are built once one running event in two has one
constexpr int kIsrKernel = 16;  // the emission hash's kernel id of an initial-state q -> q g

// histogram ranges of the branch: log10(p_T,V / GeV), y_V, emitted gluons,
// log10(p_T / GeV) of the hardest gluon (rows 4-7 unused)
__device__ __forceinline__ double isr_lo(int h) { return h == 1 ? -5.0 : (h == 3 || h == 0 ? -1.0 : 0.0); }
__device__ __forceinline__ double isr_hi(int h) { return h == 1 ? 5.0 : (h == 2 ? 50.0 : (h < 4 ? 3.0 : 1.0)); }

__device__ __forceinline__ int isr_bin(double x, double lo, double hi) {
  if (x != x) return kNBins + 1;
  if (x < lo) return 0;
  if (x >= hi) return kNBins + 1;
  const int b = 1 + (int)((x - lo) / (hi - lo) * kNBins);
  return b > kNBins ? kNBins : b;
}

__device__ __forceinline__ double isr_zmax(double a) { return 1.0 + 2.0 * a - 2.0 * sqrt(a + a * a); }

// a value that every lane holds alike, kept in scalar registers
__device__ __forceinline__ double uniform(double x) { return lane_value(x, 0); }

// x of the lane below (within a row of 16)
__device__ __forceinline__ double lane_below(double x) {
  return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), 0x111, 0xf, 0xf, false),
                          __builtin_amdgcn_update_dpp(0, __double2loint(x), 0x111, 0xf, 0xf, false));
}

// One line's trial coefficient over the range of its overestimate; false
// when the line has no phase space above the cutoff.
struct IsrLine {
  double L, c;
  bool open;
};
__device__ __forceinline__ IsrLine isr_line(double x, double zmax, double cfac) {
  IsrLine l{0.0, 1.0, zmax > x};
  if (l.open) {
    l.L = log_fast((1.0 - x) / (1.0 - zmax));
    l.c = cfac * ((2.0 * kCF) / sqrt(x) * l.L);
  }
  return l;
}

// K lanes per event.  Between emissions a line's trial coefficient stays and
// a cycle's draws are keyed by the cycle alone, so lane k of a group makes
// the trials of cycle c + k; the lanes add the winners' ln(R)/c in cycle order
// (a cycle's scale is the one before plus its own, whichever lane adds them),
// make their cutoff and veto tests, and the first lane whose cycle ends the
// sequence (cutoff or emission) is what the event takes; the cycles after it
// are drawn again, under the same keys, after the emission.  Its final-state
// momenta are transformed by the group's lanes together.  With one lane per
// event the kernel spent its time on emissions that a few lanes of the wave
// built in nearly every cycle, and on coefficients that only an emission
// changes; a few events took as long as their longest chain of cycles.  Three
// waves per SIMD (160 registers, none spilled).
template <int K>  // 2, 4, 8 or 16
__global__ void __launch_bounds__(256, 3) k_isr(Records r, Summary sm, IsrInputs in, uint32_t n, double* hist) {
  constexpr uint32_t kPerBlock = 256 / K;
  constexpr uint64_t kGroup = (1ull << K) - 1ull;
  __shared__ double lh[kIsrHist], lw[kPerBlock];
  for (int a = threadIdx.x; a < kIsrHist; a += blockDim.x) lh[a] = 0.0;
  __syncthreads();
  const uint32_t lane = threadIdx.x % K, shift = __lane_id() / K * K;
  const double ltc = uniform(log_fast(in.tcut));
  const double asmax = uniform(alpha_s_of_log(ltc));
  const double cfac = uniform(asmax / (2.0 * kPi));
  const double lts = uniform(log_fast(in.q * in.q));
  const double Y = uniform(log(in.sqrt_s / in.q));
  const double tau = uniform(in.q * in.q / (in.sqrt_s * in.sqrt_s));
  const double sqrt_tau = uniform(sqrt(tau));
  for (uint64_t e0 = (uint64_t)blockIdx.x * kPerBlock; e0 < n; e0 += (uint64_t)gridDim.x * kPerBlock) {
    const uint64_t e = e0 + threadIdx.x / K;
    const bool mine = e < n;
    const Keyed key = make_keyed(in.seed, in.first + e);
    // --- the Drell-Yan start
    const U4 m0 = key.draw(0, kPurposeME, 0);
    const int f = 1 + (int)(((uint64_t)m0.x * 5u) >> 32);
    const bool qa = (m0.y & 1u) == 0u;
    const double y0 = -Y + 2.0 * Y * unit(m0.z, m0.w);
    double x[2] = {sqrt_tau * exp(y0), sqrt_tau * exp(-y0)};
    const double eb = 0.5 * in.sqrt_s;
    double ea = x[0] * eb, ebm = x[1] * eb;  // the incoming partons (E, 0, 0, +-E) from beams A and B
    P4 own{x[0] * eb + x[1] * eb, 0.0, 0.0, x[0] * eb - x[1] * eb};  // final-state parton 2 + lane (V: lane 0)
    uint16_t tag[2] = {1, 1};  // the incoming lines' open colour labels
    if (mine && lane == 0) {  // what the evolution does not change
      const double w = 10.0 * (2.0 * Y) * tau * isr_pdf(x[0]) * isr_pdf(x[1]);
      lw[threadIdx.x / K] = w;  // for the histograms (sm may lie in host memory: written, never read)
      sm.d[kSdW * sm.stride + e] = w;
      sm.i[kSiFlavour * sm.stride + e] = qa ? f : -f;
      const uint64_t s1 = r.stride, s2 = 2 * r.stride;
      r.pid[e] = (int8_t)(qa ? f : -f);
      r.pid[s1 + e] = (int8_t)(qa ? -f : f);
      r.pid[s2 + e] = 23;
      (qa ? r.acol : r.col)[e] = 0;
      (qa ? r.col : r.acol)[s1 + e] = 0;
      r.col[s2 + e] = 0;
      r.acol[s2 + e] = 0;
    }
    // --- backward evolution of the two incoming lines
    double lt = lts;
    int np = 3, status = mine ? kRunning : kDone;
    uint32_t cycle = 0, trials = 0;  // one trial per open line and cycle
    uint64_t hash = kFnvOffset;
    double st = 2.0 * mdot(P4{ea, 0.0, 0.0, ea}, P4{ebm, 0.0, 0.0, -ebm});
    double zmax = isr_zmax(in.tcut / st);
    IsrLine line[2] = {isr_line(x[0], zmax, cfac), isr_line(x[1], zmax, cfac)};
    bool pend = false;  // an accepted emission waits to be built
    double t = 0.0, z = 0.0, disc = 0.0;
    int wl = -1;
    while (__any(status == kRunning)) {
      if (status == kRunning && !pend) {
        const uint32_t this_cycle = cycle + lane;
        // the cycle's winner: the larger ln(R)/c, the first line on ties
        double v = -INFINITY;
        wl = -1;
#pragma unroll
        for (int l = 0; l < 2; ++l) {
          if (!line[l].open) continue;
          const U4 d = key.draw(this_cycle, kPurposeTrial, trial_slot((uint32_t)l, (uint32_t)(1 - l), 0));
          const double vl = log_fast(unit(d.x, d.y)) / line[l].c;
          if (wl < 0 || vl > v) {
            v = vl;
            wl = l;
          }
        }
        double my_lt = lt + v;  // this lane's cycle's scale: the one before it plus its own
#pragma unroll
        for (uint32_t q = 1; q < K; ++q) {
          const double before = lane_below(my_lt);
          if (lane == q) my_lt = before + v;
        }
        bool done = wl < 0 || !(my_lt > ltc), accept = false;
        if (!done) {
          t = exp(my_lt);
          const double xl = wl == 0 ? x[0] : x[1], wL = wl == 0 ? line[0].L : line[1].L;
          const U4 acc = key.draw(this_cycle, kPurposeAccept, 0);
          z = 1.0 - (1.0 - xl) * exp(-unit(acc.x, acc.y) * wL);
          disc = (1.0 - z) * (1.0 - z) - 4.0 * t * z / st;
          if (disc >= 0.0 && z > xl) {  // else no room for the emission at this t
            const double dens = kCF * (1.0 + z * z) / (1.0 - z) / z * isr_pdf(xl / z) / isr_pdf(xl);
            const double over = 2.0 * kCF / sqrt(xl) / (1.0 - z);
            const double prob = alpha_s_of_log(my_lt) / asmax * (dens / over);
            accept = unit(acc.z, acc.w) < prob;
          }
        }
        // the group's first cycle that ends the sequence, else all K
        const uint64_t stop = (__ballot(done || accept) >> shift) & kGroup;
        const int at = stop ? __ffsll((unsigned long long)stop) - 1 : K - 1;
        cycle += (uint32_t)at + 1u;
        trials += ((line[0].open ? 1u : 0u) + (line[1].open ? 1u : 0u)) * ((uint32_t)at + 1u);
        lt = __shfl(my_lt, at, K);
        if (stop) {
          t = __shfl(t, at, K);
          z = __shfl(z, at, K);
          disc = __shfl(disc, at, K);
          wl = __shfl(wl, at, K);
          done = __shfl((int)done, at, K) != 0;
          if (done) status = kDone;
          else if (np == (int)r.cap) status = kOverflow;
          else pend = true;
        }
      }
      // the emissions of the wave's events together, once half of the running
      // ones have one (a third and a quarter 1 to 7% slower, at once 33%)
      const uint32_t n_pend = __popcll(__ballot(pend)), n_run = __popcll(__ballot(status == kRunning));
      if (kIsrEmitDiv * n_pend < n_run || !pend) continue;
      pend = false;
      // --- the emission: initial-initial map and the final state's transformation
      const U4 sd = key.draw(cycle - 1u, kPurposeSplit, 0);
      const double phi = 2.0 * kPi * unit(sd.x, sd.y);
      double sphi, cphi;
      sincos(phi, &sphi, &cphi);
      const P4 pa{ea, 0.0, 0.0, ea}, pb{ebm, 0.0, 0.0, -ebm};
      const P4 pe = wl == 0 ? pa : pb, ps = wl == 0 ? pb : pa;  // the emitter and the other incoming parton
      const double vv = 0.5 * ((1.0 - z) - sqrt(disc));
      const P4 na{pe.e / z, pe.x / z, pe.y / z, pe.z / z};
      const double kt = sqrt(t);
      const double c1 = 1.0 - z - vv;
      const P4 pj{c1 * na.e + vv * ps.e, c1 * na.x + vv * ps.x + kt * cphi, c1 * na.y + vv * ps.y + kt * sphi,
                  c1 * na.z + vv * ps.z};
      const P4 Kt{pe.e + ps.e, pe.x + ps.x, pe.y + ps.y, pe.z + ps.z};
      const P4 Kn{na.e + ps.e - pj.e, na.x + ps.x - pj.x, na.y + ps.y - pj.y, na.z + ps.z - pj.z};
      const P4 S{Kn.e + Kt.e, Kn.x + Kt.x, Kn.y + Kt.y, Kn.z + Kt.z};
      const double s2n = mdot(S, S), kt2 = mdot(Kt, Kt);
      for (int q = 2 + (int)lane; q < np; q += K) {
        const P4 k = q - 2 < K ? own : r.load((uint32_t)q, e);
        const double sx = mdot(S, k), kx = mdot(Kt, k);
        const double cs = 2.0 * sx / s2n, ck = 2.0 * kx / kt2;
        const P4 to{k.e - cs * S.e + ck * Kn.e, k.x - cs * S.x + ck * Kn.x, k.y - cs * S.y + ck * Kn.y,
                    k.z - cs * S.z + ck * Kn.z};
        if (q - 2 < K) own = to;
        else r.store((uint32_t)q, e, to);
      }
      const uint16_t m = (uint16_t)(np - 1);  // the next unused label
      if ((int)lane == (np - 2) % K) {
        if (np - 2 < K) own = pj;
        else r.store((uint32_t)np, e, pj);
        // the gluon goes onto the emitter's colour line (the quark's colour,
        // the antiquark's anticolour)
        const uint64_t oj = (uint64_t)np * r.stride + e;
        const bool quark = (wl == 0) == qa;
        const uint16_t was = wl == 0 ? tag[0] : tag[1];
        r.pid[oj] = (int8_t)kGluon;
        r.col[oj] = quark ? was : m;
        r.acol[oj] = quark ? m : was;
      }
      hash = fnv_step(fnv_step(fnv_step(hash, (uint32_t)kIsrKernel), (uint32_t)wl), (uint32_t)(1 - wl));
      ++np;
      if (cycle >= kCycleLimit) status = kCycleLimitHit;
      if (wl == 0) {
        ea = na.e;
        x[0] = x[0] / z;
        tag[0] = m;
      } else {
        ebm = na.e;
        x[1] = x[1] / z;
        tag[1] = m;
      }
      st = 2.0 * mdot(P4{ea, 0.0, 0.0, ea}, P4{ebm, 0.0, 0.0, -ebm});
      zmax = isr_zmax(in.tcut / st);
      line[0] = isr_line(x[0], zmax, cfac);
      line[1] = isr_line(x[1], zmax, cfac);
    }
    // --- validation: finite; the final state carries the incoming total;
    // V on its mass shell, the others massless
    const P4 pa{ea, 0.0, 0.0, ea}, pb{ebm, 0.0, 0.0, -ebm};
    const P4 tin{pa.e + pb.e, pa.x + pb.x, pa.y + pb.y, pa.z + pb.z};
    const double s_in = mdot(tin, tin);
    P4 tout{0.0, 0.0, 0.0, 0.0};
    double ptg = 0.0;
    bool finite = true, shell = true;
    if (mine) {
      auto check = [&](const P4& p, double m2) {
        finite = finite && isfinite(p.e) && isfinite(p.x) && isfinite(p.y) && isfinite(p.z);
        shell = shell && fabs(mdot(p, p) - m2) <= 1e-10 * s_in;
      };
      if (lane == 0) {
        check(pa, 0.0);
        check(pb, 0.0);
        r.store(0, e, pa);
        r.store(1, e, pb);
        (qa ? r.col : r.acol)[e] = tag[0];
        (qa ? r.acol : r.col)[r.stride + e] = tag[1];
      }
      for (int q = 2 + (int)lane; q < np; q += K) {
        P4 p = own;
        if (q - 2 < K) r.store((uint32_t)q, e, p);
        else p = r.load((uint32_t)q, e);
        check(p, q == 2 ? in.q * in.q : 0.0);
        tout.e += p.e;
        tout.x += p.x;
        tout.y += p.y;
        tout.z += p.z;
        if (q >= 3) {
          const double pt = sqrt(p.x * p.x + p.y * p.y);
          if (pt > ptg) ptg = pt;
        }
      }
    }
#pragma unroll
    for (int d = K / 2; d >= 1; d >>= 1) {
      tout.e += __shfl_xor(tout.e, d, K);
      tout.x += __shfl_xor(tout.x, d, K);
      tout.y += __shfl_xor(tout.y, d, K);
      tout.z += __shfl_xor(tout.z, d, K);
      ptg = fmax(ptg, __shfl_xor(ptg, d, K));
    }
    finite = !((__ballot(!finite) >> shift) & kGroup);
    shell = !((__ballot(!shell) >> shift) & kGroup);
    if (status == kDone) {
      const double tol = 1e-10 * tin.e;
      if (!finite) status = kNonFinite;
      else if (fabs(tout.e - tin.e) > tol || fabs(tout.x - tin.x) > tol || fabs(tout.y - tin.y) > tol ||
               fabs(tout.z - tin.z) > tol || !shell)
        status = kConservation;
    }
    if (mine && lane == 0) {  // V is this lane's
      const double ptv = sqrt(own.x * own.x + own.y * own.y);
      const double yv = 0.5 * log((own.e + own.z) / (own.e - own.z));
      if (status == kDone) {
        const double w = lw[threadIdx.x / K];
        const double vals[4] = {ptv > 0.0 ? log10(ptv) : -INFINITY, yv, (double)(np - 3),
                                ptg > 0.0 ? log10(ptg) : -INFINITY};
#pragma unroll
        for (int h = 0; h < 4; ++h) {
          double* cell = &lh[3 * (kNHCol * h + isr_bin(vals[h], isr_lo(h), isr_hi(h)))];
          atomicAdd(&cell[0], w);
          atomicAdd(&cell[1], w * w);
          atomicAdd(&cell[2], 1.0);
        }
      }
      const double dv[kNSumD] = {0.0, yv, ptv, x[0], x[1], ptg, 0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int k = kSdW + 1; k < kNSumD; ++k) sm.d[k * sm.stride + e] = dv[k];
      sm.i[kSiN * sm.stride + e] = np;
      sm.i[kSiStatus * sm.stride + e] = status;
      sm.i[kSiCycles * sm.stride + e] = (int32_t)cycle;
      sm.i[kSiEmit * sm.stride + e] = np - 3;
      sm.i[kSiTrials * sm.stride + e] = (int32_t)trials;
      sm.i[kSiEnds * sm.stride + e] = (int32_t)trials;
      sm.hash[e] = hash;
    }
  }
  __syncthreads();
  for (int a = threadIdx.x; a < kIsrHist; a += blockDim.x) {
    const double v = lh[a];
    if (v != 0.0) unsafeAtomicAdd(&hist[a], v);
  }
}

// Lanes per event: as many as leave every event resident.  k_isr alone, one
// lane per event as before and this rule: 100 events 347 and 40 us, 5000 452
// and 65, 20000 463 and 111, 50000 455 and 199, 200003 1161 and 566, 10^6
// 4396 and 2385 (sixteen lanes there: 4252), on 256 compute units.
static void launch_isr(const Records& r, const Summary& sm, const IsrInputs& in, uint32_t n, double* hist,
                       uint32_t n_cu, hipStream_t st) {
  const uint32_t K = n <= 16 * n_cu ? 16 : n <= 128 * n_cu ? 8 : n <= 512 * n_cu ? 4 : 2;
  // events past the grid's are taken in further rounds of its blocks, so
  // that their histograms are not flushed too often
  const dim3 g((uint32_t)std::min<uint64_t>(((uint64_t)n * K + 255) / 256, 8192)), b(256);
  if (K == 16) hipLaunchKernelGGL(k_isr<16>, g, b, 0, st, r, sm, in, n, hist);
  else if (K == 8) hipLaunchKernelGGL(k_isr<8>, g, b, 0, st, r, sm, in, n, hist);
  else if (K == 4) hipLaunchKernelGGL(k_isr<4>, g, b, 0, st, r, sm, in, n, hist);
  else hipLaunchKernelGGL(k_isr<2>, g, b, 0, st, r, sm, in, n, hist);
}

// The kernel writes each field of a wave's events side by side, 64 to 256
// bytes at a time, and reads none back: with the result's pinned block ready
// and no records to gather by the counts, it writes straight into the block,
// so that the transfer passes while other waves compute (the kernel takes 1.1
// times as long).  Calls of 200000 events 1026 -> 873 us, 10^6 4.47 -> 3.59 ms,
// 20000 and below unchanged.
static bool summary_in_block(vsh_ctx* ctx, const vsh_request* req, const ResultBox* box, Summary* sm) {
  if (!box->sum_block.ptr || (req->flags & VSH_RECORDS)) return false;
  void* dev = device_address(box->sum_block.ptr);
  if (!dev) return false;
  const ResultSpan sp(req->n_events);
  sm->i = (int32_t*)((char*)dev + sp.i);
  sm->d = (double*)((char*)dev + sp.d);
  sm->hash = (uint64_t*)((char*)dev + sp.hash);
  return true;
}

}  // namespace vsh

using namespace vsh;

extern "C" vsh_status vsh_generate_isr(vsh_ctx* ctx, const vsh_request* req, double sqrt_s_hadron,
                                       vsh_result** out) {
  if (!ctx || !out) return VSH_E_INVALID;
  std::lock_guard<std::mutex> lk(ctx->mu);
  *out = nullptr;
  vsh_status rc = validate_request(ctx, req, true);
  if (rc) return rc;
  if (req->max_partons < 3) {
    set_error(ctx, "Drell-Yan records hold the two incoming partons and V: max_partons must be >= 3");
    return VSH_E_INVALID;
  }
  if (req->flags & ~(VSH_SUMMARY | VSH_RECORDS)) {
    set_error(ctx, "vsh_generate_isr takes VSH_SUMMARY and VSH_RECORDS only");
    return VSH_E_INVALID;
  }
  if (req->ecm_per_event || req->tcut_per_event || req->cycle_limit || req->t_over != 0.0 || req->mass_c != 0.0 ||
      req->mass_b != 0.0) {
    set_error(ctx, "vsh_generate_isr takes one Q (ecm) and t_cut, no per-event arrays, tail cut, t_over or masses");
    return VSH_E_INVALID;
  }
  if (!(sqrt_s_hadron > req->ecm) || !std::isfinite(sqrt_s_hadron)) {
    set_error(ctx, "sqrt_s_hadron (%g) must be finite and above Q = ecm (%g)", sqrt_s_hadron, req->ecm);
    return VSH_E_INVALID;
  }
  if (!(req->t_cut < 0.25 * req->ecm * req->ecm)) {
    set_error(ctx, "t_cut must lie below Q^2 / 4");
    return VSH_E_INVALID;
  }
  (void)hipSetDevice(ctx->device);
  const auto t0 = std::chrono::steady_clock::now();
  const uint32_t cap = req->max_partons;
  const uint64_t per_event = (uint64_t)cap * (4 * 8 + 1 + 2 * 2) + kNSumD * 8 + kNSumI * 4 + 8;
  uint64_t budget = ctx->budget;
  if (req->flags & VSH_RECORDS) budget /= 2;
  uint64_t chunk = std::min<uint64_t>(req->n_events, std::min<uint64_t>(budget / (per_event + 64), 1ull << 26));
  if (chunk < req->n_events) chunk &= ~63ull;
  if (chunk == 0) {
    set_error(ctx, "memory budget cannot hold one event of %u partons", cap);
    return VSH_E_NOMEM;
  }
  ResultBox* box = new_call_result(ctx, req, chunk >= req->n_events);
  if (!box) return VSH_E_NOMEM;
  static const double L[kNObs] = {-1.0, -5.0, 0.0, -1.0, 0.0, 0.0, 0.0, 0.0};
  static const double H[kNObs] = {3.0, 5.0, 50.0, 3.0, 1.0, 1.0, 1.0, 1.0};
  for (int h = 0; h < kNObs; ++h) {
    box->lo[h] = L[h];
    box->hi[h] = H[h];
  }
  hipStream_t st = ctx->stream;
  float t_sh = 0.0f;
  for (uint64_t a = 0; a < req->n_events; a += chunk) {
    const uint64_t count = std::min(chunk, req->n_events - a);
    const uint64_t stride = align_up(count, 64);
    const uint64_t slots = (uint64_t)cap * stride;
    const uint64_t need = slots * (4 * 8 + 1 + 2 * 2) + stride * (kNSumD * 8 + kNSumI * 4 + 8) + kHistDoubles * 8 +
                          16 * 256;
    rc = ctx->arena.reserve(ctx, need);
    if (rc) {
      drop_result(ctx, box);
      return rc;
    }
    Carver c(ctx->arena.ptr);
    Records r{};
    r.E = (double*)c.take(slots * 8);
    r.x = (double*)c.take(slots * 8);
    r.y = (double*)c.take(slots * 8);
    r.z = (double*)c.take(slots * 8);
    r.pid = (int8_t*)c.take(slots);
    r.col = (uint16_t*)c.take(slots * 2);
    r.acol = (uint16_t*)c.take(slots * 2);
    r.cpart = r.apart = nullptr;
    r.stride = stride;
    r.cap = cap;
    Summary sm{};
    double* hist = (double*)c.take(kHistDoubles * 8);
    sm.i = (int32_t*)c.take(kNSumI * count * 4);
    sm.d = (double*)c.take(kNSumD * count * 8);
    sm.hash = (uint64_t*)c.take(count * 8);
    sm.stride = count;
    const bool direct = summary_in_block(ctx, req, box, &sm);
    launch_zero(hist, kHistDoubles, st);
    const IsrInputs in{req->seed, req->first_event + a, sqrt_s_hadron, req->ecm, req->t_cut};
    (void)hipEventRecord(ctx->ev[1], st);
    launch_isr(r, sm, in, (uint32_t)count, hist, (uint32_t)ctx->n_cu, st);
    (void)hipEventRecord(ctx->ev[2], st);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) {
      drop_result(ctx, box);
      return hip_fail(ctx, err, "k_isr launch");
    }
    const int32_t* n_host = nullptr;
    rc = copy_back_chunk(ctx, st, hist, sm, count, req->flags, box, a, &n_host, direct);
    if (rc) {
      drop_result(ctx, box);
      return rc;
    }
    float ms = 0.0f;
    if (hipEventElapsedTime(&ms, ctx->ev[1], ctx->ev[2]) == hipSuccess) t_sh += ms;
    if (req->flags & VSH_RECORDS) {
      rc = gather_records(ctx, r, n_host, count, box);
      if (rc) {
        drop_result(ctx, box);
        return rc;
      }
    }
  }
  box->pub.t_shower_ms = t_sh;
  box->pub.t_total_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
  finish_result(box);
  *out = &box->pub;
  return VSH_OK;
}
