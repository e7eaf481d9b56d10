// vsh_kernels.hpp -- data layout and kernel declarations of the shower engine.
//
// Layout in HBM (structure of arrays, slot-major so that lane e of a wave
// touching parton slot a of its event reads element [a][e]: consecutive lanes,
// consecutive addresses):
//   E, x, y, z      double   [cap][stride]   four-momenta
//   pid             int8     [cap][stride]
//   col, acol       uint16   [cap][stride]   colour / anticolour line, 0 = none
//   cpart, apart    uint16   [cap][stride]   index of the parton holding the
//                                            other end of this parton's colour
//                                            (anticolour) line, 0xFFFF = none
// plus per-event summaries [field][stride] (see vsh.h for the fields).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "vsh_device.hpp"

namespace vsh {

constexpr int kNSumD = 10;
constexpr int kNSumI = 7;
constexpr int kNObs = 8;
constexpr int kNBins = 50;
constexpr int kNHCol = kNBins + 2;
constexpr int kHistDoubles = kNObs * kNHCol * 3;
constexpr uint32_t kMaxCount = 1024;  // largest record capacity

// summary field indices
enum { kSdW = 0, kSdCos = 1, kSdY23 = 2, kSdY34 = 3, kSdTau = 4, kSdC = 5, kSdRho = 6, kSdBT = 7,
       kSdBW = 8, kSdPhi = 9 };
enum { kSiN = 0, kSiStatus = 1, kSiCycles = 2, kSiEmit = 3, kSiFlavour = 4, kSiTrials = 5, kSiEnds = 6 };

struct Records {
  double *E, *x, *y, *z;
  int8_t *pid;
  uint16_t *col, *acol, *cpart, *apart;
  uint64_t stride;  // elements per slot row (>= events in the launch)
  uint32_t cap;

  __device__ __forceinline__ P4 load(uint32_t a, uint64_t e) const {
    const uint64_t o = (uint64_t)a * stride + e;
    return P4{E[o], x[o], y[o], z[o]};
  }
  __device__ __forceinline__ void store(uint32_t a, uint64_t e, const P4& p) const {
    const uint64_t o = (uint64_t)a * stride + e;
    E[o] = p.e;
    x[o] = p.x;
    y[o] = p.y;
    z[o] = p.z;
  }
};

struct Summary {
  double *d;       // [kNSumD][stride]
  int32_t *i;      // [kNSumI][stride]
  uint64_t *hash;  // [stride]
  uint64_t stride;
};

struct EventInputs {
  const double *ecm;   // [n] or null -> ecm0
  const double *tcut;  // [n] or null -> tcut0
  double ecm0, tcut0;
  uint64_t seed, first;
  uint32_t cycle_limit;  // veto cycles after which a running event is given up (>= 1)
  double t_over;         // scale of alpha_s in the trial density, 0 = the event's t_C
  QuarkMasses qm;        // quark masses (massive kernels only when `massive`)
  uint32_t massive;      // any quark mass above zero
  uint32_t fixed_hist;   // histogram sums in int64 fixed point (order-independent)
  __device__ __forceinline__ double ecm_of(uint64_t e) const { return ecm ? ecm[e] : ecm0; }
  __device__ __forceinline__ double tcut_of(uint64_t e) const { return tcut ? tcut[e] : tcut0; }
};

// caller-supplied starts of a chunk of events on the device: parton a of
// event e at index off[e] - off[0] + a of the others
struct CsrStarts {
  const uint64_t* off;  // [n + 1]
  const double* p;      // [total][4]
  const int8_t* pid;
  const uint16_t *col, *acol;
};
constexpr uint32_t kLoadLanes = 16;  // lanes per event of k_load_records

struct HistRanges {
  double lo[kNObs], hi[kNObs];
};

// Scratch of the observables pass: thread slot t keeps its current event's
// partons (and Durham's jets) at element [a][t]; the events are visited in
// order of decreasing parton count (perm), so a wave's lanes hold events of
// the same size.
struct Scratch {
  double *E, *x, *y, *z;    // momenta; Durham merges jets in place
  double *ux, *uy, *uz;     // unit three-vectors of the current jets
  double *dn;               // forward nearest-neighbour y
  uint16_t *nn;             // forward nearest neighbour, 0xFFFF none
  uint8_t *dead;            // merged-away jets
  uint64_t stride;          // thread slots
  uint32_t *perm;           // event indices by decreasing parton count [n]
  uint32_t *cnt;            // per-count offsets [cap + 2]
  uint32_t threshold;       // events with at least this many partons: one wave each
  // the blocks' histograms meet in kHistCopies copies (block b adds into
  // copy b mod kHistCopies, so that no cell's atomics queue up behind every
  // block's), summed into the caller's histogram by k_hist_finalize: FP64
  // cells, or (requests with VSH_HIST_FIXEDPOINT) the cells' int64 sums; the
  // largest |w| of the launch's events (as the bits of a non-negative double,
  // which order like the integers) and L = ceil(log2 n)
  double *hcopy;              // [kHistCopies][kHistDoubles]
  unsigned long long *ihist;  // [kHistCopies][kHistDoubles]
  unsigned long long *wmax;   // [1]
  uint32_t lbits;
};

// One request's observables as the kernels of the pass take it, and where its
// blocks begin in the launches that serve several requests at once.
enum { kObsStageHist, kObsStageSort, kObsStageScan, kObsStageWindow, kObsStageGroup, kObsStageSum, kObsStages };
struct ObsJob {
  Records r;
  Summary sm;
  EventInputs in;
  Scratch sc;
  double* hist;
  uint32_t n;
  uint32_t at[kObsStages];
};
struct ObsPlan {
  uint32_t blocks[kObsStages] = {};
  uint32_t count = 0, cap = 0;
  bool massive = false;  // any of the jobs
};

constexpr uint32_t kObsWaveThreshold = 9;
constexpr int kObsRegSlots = 8;  // events of at most this many partons: observables in registers
constexpr uint32_t kObsWaveMaxCap = 512;
constexpr uint32_t kObsSortPer = 16;  // events per thread of the counting sort by parton count
constexpr uint32_t kHistCopies = 16;  // copies of the histogram set that the blocks' atomics spread over
constexpr uint32_t kHistBlocks = (kHistDoubles + 255) / 256;  // blocks of k_hist_finalize
constexpr uint32_t kObsGroup64 = 32;     // events from this many partons: 64 lanes each
constexpr uint32_t kObsFew = 32768, kObsFewBig = 16384;  // most events of k_obs_few (obs_few_launch)
constexpr uint32_t kObsFewBlocks = 2048;
// blocks of the group launches (each block's groups stride over the events
// of their size range): many short blocks end more evenly than a grid of
// one or a few rounds of resident blocks (stress, 10^6 events: 8192 blocks
// 7.3 ms, 32768 blocks 6.9 ms; empty blocks leave at once)
constexpr uint32_t kObsWaveBlocks = 32768;
constexpr uint32_t kObsJobGroupBlocks = 4096;  // the same for each of several requests in one launch

}  // namespace vsh

// host-side launchers (vsh_kernels.hip)
namespace vsh {
// The observables pass runs a grid-stride loop over obs_threads(n, cap)
// threads (at most 2^25 parton slots of scratch in all).
uint64_t obs_threads(uint64_t n, uint32_t cap);
uint64_t obs_scratch_bytes(uint64_t n, uint32_t cap);
Scratch carve_obs_scratch(char*& p, uint64_t n, uint32_t cap);
void launch_me(const Records& r, const Summary& s, const EventInputs& in, uint32_t n,
               hipStream_t st, double* zero_hist = nullptr);
void launch_shower_plain(const Records& r, const Summary& s, const EventInputs& in, uint32_t n,
                         uint32_t block, uint32_t waves, hipStream_t st);
// hist is accumulated into.  The kernels' FP64 atomics reach only memory that
// the library lays out: where hist is the caller's, `own` is a cleared histogram
// of the workspace that small launches collect in first.
void launch_obs(const Records& r, const Summary& s, const EventInputs& in, const Scratch& sc,
                uint32_t n, double* hist, double* own, hipStream_t st);
// the pass over several requests (records of at most kObsWaveMaxCap partons,
// each with a scratch of its own from carve_obs_job) in one set of launches
uint64_t obs_job_bytes(uint64_t n, uint32_t cap);
Scratch carve_obs_job(char*& p, uint64_t n, uint32_t cap);
void plan_obs_jobs(ObsJob* jobs, uint32_t count, ObsPlan* plan);
void launch_obs_jobs(const ObsJob* jobs_dev, const ObsPlan& plan, hipStream_t st);
void launch_load_records(const Records& r, const Summary& s, const CsrStarts& in, uint32_t n, double* ecm,
                         unsigned long long* bad, double* zero_hist, hipStream_t st);
}  // namespace vsh
