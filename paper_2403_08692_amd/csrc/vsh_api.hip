// vsh_api.hip -- the C ABI of libvsh (include/vsh.h): contexts, the device
// arena, request validation, the blocking and device-side generation calls
// and the caller-supplied-start shower.  Serving lives in vsh_serve.hip.
#include <hip/hip_runtime.h>
#include <pthread.h>
#include <sys/mman.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "../../include/vsh.h"
#include "vsh_internal.hpp"

namespace vsh {

thread_local std::string g_create_error;

void set_error(vsh_ctx* ctx, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  if (ctx) ctx->error = buf;
  else g_create_error = buf;
}

vsh_status hip_fail(vsh_ctx* ctx, hipError_t err, const char* what) {
  set_error(ctx, "%s: %s", what, hipGetErrorString(err));
  return VSH_E_DEVICE;
}

vsh_status validate_request(vsh_ctx* ctx, const vsh_request* req, bool need_energy) {
  if (!req) {
    set_error(ctx, "request is NULL");
    return VSH_E_INVALID;
  }
  if (req->n_events == 0) {
    set_error(ctx, "n_events must be >= 1");
    return VSH_E_INVALID;
  }
  if (req->n_events > (1ull << 32) - 1) {
    set_error(ctx, "n_events must be < 2^32 per request");
    return VSH_E_INVALID;
  }
  if (req->max_partons < 2 || req->max_partons > kMaxCap) {
    set_error(ctx, "max_partons must be in 2..%u (got %u)", kMaxCap, req->max_partons);
    return VSH_E_INVALID;
  }
  const uint32_t known = VSH_SUMMARY | VSH_RECORDS | VSH_FORM_PERSISTENT | VSH_INPUTS_ON_DEVICE | VSH_HIST_FIXEDPOINT;
  if (req->flags & ~known) {
    set_error(ctx, "unknown request flags 0x%x", req->flags & ~known);
    return VSH_E_INVALID;
  }
  const bool dev = req->flags & VSH_INPUTS_ON_DEVICE;
  if (need_energy && !req->ecm_per_event && !(req->ecm > 0.0)) {
    set_error(ctx, "ecm must be > 0 (got %g)", req->ecm);
    return VSH_E_INVALID;
  }
  if (!req->tcut_per_event && !(req->t_cut > kMinTcut)) {
    set_error(ctx, "t_cut must be > %g GeV^2 (got %g)", kMinTcut, req->t_cut);
    return VSH_E_INVALID;
  }
  if (!(req->mass_c >= 0.0 && std::isfinite(req->mass_c) && req->mass_b >= 0.0 && std::isfinite(req->mass_b))) {
    set_error(ctx, "quark masses must be finite and >= 0 (got c %g, b %g)", req->mass_c, req->mass_b);
    return VSH_E_INVALID;
  }
  if (!(req->t_over == 0.0 || (req->t_over > kMinTcut && std::isfinite(req->t_over)))) {
    set_error(ctx, "t_over must be 0 or a finite value > %g GeV^2 (got %g)", kMinTcut, req->t_over);
    return VSH_E_INVALID;
  }
  if (!dev) {
    if (need_energy && req->ecm_per_event)
      for (uint64_t e = 0; e < req->n_events; ++e)
        if (!(req->ecm_per_event[e] > 0.0)) {
          set_error(ctx, "ecm_per_event[%llu] must be > 0", (unsigned long long)e);
          return VSH_E_INVALID;
        }
    if (req->tcut_per_event)
      for (uint64_t e = 0; e < req->n_events; ++e)
        if (!(req->tcut_per_event[e] > kMinTcut)) {
          set_error(ctx, "tcut_per_event[%llu] must be > %g", (unsigned long long)e, kMinTcut);
          return VSH_E_INVALID;
        }
  }
  return VSH_OK;
}

// ---------------------------------------------------------------------------
// Plain-form device layout of a chunk of n events with capacity cap: records
// (columns of n rounded up to 64), Durham scratch, the results' span, per-event
// inputs.
// ---------------------------------------------------------------------------
uint64_t plain_bytes_per_event(uint32_t cap, bool massive) {
  return (uint64_t)cap * (4 * 8 + 1 + 4 * 2 + cache_words(massive) * 8) + kNSumD * 8 + kNSumI * 4 + 8 + 2 * 8;
}

uint64_t plain_layout_bytes(uint64_t stride, uint32_t cap, bool massive) {
  return align_up(plain_bytes_per_event(cap, massive) * stride + obs_scratch_bytes(stride, cap) + 20 * 256 +
                      kHistDoubles * 8, 256);
}

PlainLayout carve_plain(void* base, uint64_t n, uint32_t cap, bool massive) {
  PlainLayout L;
  const uint64_t stride = align_up(n, 64);
  char* p = static_cast<char*>(base);
  auto take = [&](uint64_t bytes) {
    char* q = p;
    p += align_up(bytes, 256);
    return q;
  };
  const uint64_t slots = (uint64_t)cap * stride;
  L.rec.E = (double*)take(slots * 8);
  L.rec.x = (double*)take(slots * 8);
  L.rec.y = (double*)take(slots * 8);
  L.rec.z = (double*)take(slots * 8);
  L.rec.pid = (int8_t*)take(slots);
  L.rec.col = (uint16_t*)take(slots * 2);
  L.rec.acol = (uint16_t*)take(slots * 2);
  L.rec.cpart = (uint16_t*)take(slots * 2);
  L.rec.apart = (uint16_t*)take(slots * 2);
  L.rec.stride = stride;
  L.rec.cap = cap;
  L.cache = (uint64_t*)take(slots * cache_words(massive) * 8);
  {
    char* q = p;
    L.sc = carve_obs_scratch(q, stride, cap);
    p = q;
  }
  L.hist = (double*)take(kHistDoubles * 8);
  L.sum.i = (int32_t*)take(kNSumI * n * 4);
  L.sum.d = (double*)take(kNSumD * n * 8);
  L.sum.hash = (uint64_t*)take(n * 8);
  L.sum.stride = n;
  L.ecm = (double*)take(n * 8);
  L.tcut = (double*)take(n * 8);
  L.end = p;
  return L;
}

vsh_status Arena::reserve(vsh_ctx* ctx, uint64_t bytes) {
  if (bytes <= size) return VSH_OK;
  if (ptr) {
    (void)hipFree(ptr);
    ptr = nullptr;
    size = 0;
  }
  hipError_t err = hipMalloc(&ptr, bytes);
  if (err != hipSuccess) {
    ptr = nullptr;
    (void)hipGetLastError();
    set_error(ctx, "device arena of %llu bytes: %s", (unsigned long long)bytes, hipGetErrorString(err));
    return VSH_E_NOMEM;
  }
  size = bytes;
  return VSH_OK;
}

void Arena::release() {
  if (ptr) (void)hipFree(ptr);
  ptr = nullptr;
  size = 0;
}

vsh_status HostStage::reserve(vsh_ctx* ctx, uint64_t bytes) {
  if (bytes <= size) return VSH_OK;
  release();
  hipError_t err = hipHostMalloc(&ptr, bytes, 0);
  if (err != hipSuccess) {
    ptr = nullptr;
    (void)hipGetLastError();
    set_error(ctx, "pinned host staging of %llu bytes: %s", (unsigned long long)bytes, hipGetErrorString(err));
    return VSH_E_NOMEM;
  }
  size = bytes;
  return VSH_OK;
}

void HostStage::release() {
  if (ptr) (void)hipHostFree(ptr);
  ptr = nullptr;
  size = 0;
}

// The process's pools, and what becomes of their blocks in use when it forks:
// copied to ordinary memory before, the copies moved to the blocks' addresses
// in the child and dropped in the parent.  A block whose copy found no memory
// is missing in the child.
static std::mutex g_pools_mu;
static PinnedPool* g_pools = nullptr;

static void before_fork() {
  g_pools_mu.lock();
  for (PinnedPool* p = g_pools; p; p = p->after) {
    p->mu.lock();
    if (p->forked) continue;  // ordinary memory already
    for (PinnedBlock& b : p->used) {
      b.copy = mmap(nullptr, b.size, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
      if (b.copy == MAP_FAILED) b.copy = nullptr;
      else std::memcpy(b.copy, b.ptr, b.size);
    }
  }
}

static void after_fork_parent() {
  for (PinnedPool* p = g_pools; p; p = p->after) {
    for (PinnedBlock& b : p->used) {
      if (b.copy) (void)munmap(b.copy, b.size);
      b.copy = nullptr;
    }
    p->mu.unlock();
  }
  g_pools_mu.unlock();
}

static void after_fork_child() {
  for (PinnedPool* p = g_pools; p; p = p->after) {
    if (!p->forked) {
      size_t kept = 0;  // release() unmaps what is listed
      for (const PinnedBlock& b : p->used)
        if (b.copy && mremap(b.copy, b.size, b.size, MREMAP_MAYMOVE | MREMAP_FIXED, b.ptr) == b.ptr)
          p->used[kept++] = PinnedBlock{b.ptr, b.size, nullptr};
      p->used.resize(kept);
      p->idle.clear();
      p->forked = true;
    }
    p->mu.unlock();
  }
  g_pools_mu.unlock();
}

PinnedPool::PinnedPool() {
  static std::once_flag once;
  std::call_once(once, [] { (void)pthread_atfork(before_fork, after_fork_parent, after_fork_child); });
  std::lock_guard<std::mutex> lk(g_pools_mu);
  after = g_pools;
  if (after) after->before = this;
  g_pools = this;
}

PinnedPool::~PinnedPool() {
  std::lock_guard<std::mutex> lk(g_pools_mu);
  (before ? before->after : g_pools) = after;
  if (after) after->before = before;
}

PinnedBlock PinnedPool::acquire(uint64_t bytes) try {
  std::lock_guard<std::mutex> lk(mu);
  if (forked) return PinnedBlock{};
  if (used.size() == used.capacity()) used.reserve(2 * used.size() + 16);
  size_t best = idle.size();
  for (size_t k = 0; k < idle.size(); ++k)
    if (idle[k].size >= bytes && idle[k].size <= 2 * bytes + (1u << 20) &&
        (best == idle.size() || idle[k].size < idle[best].size))
      best = k;
  if (best < idle.size()) {
    const PinnedBlock b = idle[best];
    idle.erase(idle.begin() + (long)best);
    used.push_back(b);
    return b;
  }
  PinnedBlock b;
  const uint64_t size = align_up(bytes, 65536);
  uint64_t in_use = held;
  for (const PinnedBlock& k : idle) in_use -= k.size;
  if (in_use + size > kMost) return b;  // whatever of the idle ones went
  while (held + size > kMost && !idle.empty()) {  // make room: the oldest first
    (void)hipHostFree(idle.front().ptr);
    held -= idle.front().size;
    idle.erase(idle.begin());
  }
  idle.reserve(idle.size() + 64);  // release() never allocates
  if (hipHostMalloc(&b.ptr, size, 0) != hipSuccess) {
    (void)hipGetLastError();
    b.ptr = nullptr;
    return b;
  }
  b.size = size;
  held += size;
  used.push_back(b);
  return b;
} catch (const std::bad_alloc&) {  // of the lists, before anything was taken
  return PinnedBlock{};
}

void PinnedPool::release(PinnedBlock b) {
  if (!b.ptr) return;
  std::lock_guard<std::mutex> lk(mu);
  size_t k = 0;
  while (k < used.size() && used[k].ptr != b.ptr) ++k;
  const bool listed = k < used.size();
  if (listed) {
    used[k] = used.back();
    used.pop_back();
  }
  if (forked) {
    if (listed) (void)munmap(b.ptr, b.size);
    return;
  }
  if (closed || idle.size() == idle.capacity()) {
    (void)hipHostFree(b.ptr);
    held -= b.size;
  } else {
    idle.push_back(b);
  }
}

void PinnedPool::close() {
  std::lock_guard<std::mutex> lk(mu);
  closed = true;
  for (const PinnedBlock& b : idle) {
    (void)hipHostFree(b.ptr);
    held -= b.size;
  }
  idle.clear();
}

ResultBox::~ResultBox() {
  if (!pool) return;
  pool->release(sum_block);
  pool->release(rec_block);
}

// ---------------------------------------------------------------------------
// result assembly
// ---------------------------------------------------------------------------
ResultBox* new_result(uint64_t n_events, bool summary) try {
  std::unique_ptr<ResultBox> b(new ResultBox());
  b->hist.assign(kHistDoubles, 0.0);
  b->lo.assign(kNObs, 0.0);
  b->hi.assign(kNObs, 0.0);
  static const double L[kNObs] = {-4.3, -4.3, 0.0, 0.0, 0.0, 0.0, 0.0, -1.0};
  static const double H[kNObs] = {-0.3, -0.3, 0.5, 1.0, 0.5, 0.5, 0.35, 1.0};
  for (int h = 0; h < kNObs; ++h) {
    b->lo[h] = L[h];
    b->hi[h] = H[h];
  }
  if (summary) {
    b->sum_d.assign((size_t)kNSumD * n_events, 0.0);
    b->sum_i.assign((size_t)kNSumI * n_events, 0);
    b->hash.assign(n_events, 0);
  }
  std::memset(&b->pub, 0, sizeof b->pub);
  b->pub.n_events = n_events;
  b->pub.n_obs = kNObs;
  b->pub.n_bins = kNBins;
  return b.release();
} catch (const std::bad_alloc&) {
  return nullptr;
}

ResultBox* new_call_result(vsh_ctx* ctx, const vsh_request* req, bool whole) {
  const bool summary = req->flags & VSH_SUMMARY;
  PinnedBlock block;
  if (whole && summary) block = ctx->pool->acquire(ResultSpan(req->n_events).bytes);
  ResultBox* box = new_result(req->n_events, summary && !block.ptr);
  if (!box) {
    ctx->pool->release(block);
    set_error(ctx, "host allocation failed");
    return nullptr;
  }
  box->pool = ctx->pool;
  box->sum_block = block;
  return box;
}

void drop_result(vsh_ctx* ctx, ResultBox* box) {
  (void)hipStreamSynchronize(ctx->stream);
  (void)hipGetLastError();  // this call's, not the next one's
  delete box;
}

// CSR records in one span: offsets, momenta, flavours, colours, anticolours.
struct RecordSpan {
  uint64_t p, pid, col, acol, bytes;
  RecordSpan(uint64_t n, uint64_t total)
      : p(align_up((n + 1) * 8, 256)), pid(p + align_up(total * 32, 256)), col(pid + align_up(total, 256)),
        acol(col + align_up(total * 2, 256)), bytes(acol + align_up(total * 2, 256)) {}
};

void finish_result(ResultBox* b) {
  vsh_result& r = b->pub;
  r.hist_lo = b->lo.data();
  r.hist_hi = b->hi.data();
  r.hist = b->hist.data();
  r.sum_d = b->sum_d.empty() ? nullptr : b->sum_d.data();
  r.sum_i = b->sum_i.empty() ? nullptr : b->sum_i.data();
  r.sum_hash = b->hash.empty() ? nullptr : b->hash.data();
  if (b->sum_block.ptr) {
    const ResultSpan sp(r.n_events);
    const char* p = static_cast<const char*>(b->sum_block.ptr);
    r.sum_i = reinterpret_cast<const int32_t*>(p + sp.i);
    r.sum_d = reinterpret_cast<const double*>(p + sp.d);
    r.sum_hash = reinterpret_cast<const uint64_t*>(p + sp.hash);
  }
  if (b->rec_block.ptr) {
    const uint64_t* off = static_cast<const uint64_t*>(b->rec_block.ptr);
    const RecordSpan sp(r.n_events, off[r.n_events]);
    const char* p = static_cast<const char*>(b->rec_block.ptr);
    r.rec_offsets = off;
    r.rec_p = reinterpret_cast<const double*>(p + sp.p);
    r.rec_pid = reinterpret_cast<const int8_t*>(p + sp.pid);
    r.rec_col = reinterpret_cast<const uint16_t*>(p + sp.col);
    r.rec_acol = reinterpret_cast<const uint16_t*>(p + sp.acol);
  } else if (!b->rec_offsets.empty()) {
    r.rec_offsets = b->rec_offsets.data();
    r.rec_p = b->rec_p.data();
    r.rec_pid = b->rec_pid.data();
    r.rec_col = b->rec_col.data();
    r.rec_acol = b->rec_acol.data();
  }
}

// The counts and sums of count events from the integer summary fields
// kSiStatus .. kSiEnds (field f at si0[(f - kSiStatus) * stride]) and the
// weights w.
void tally_fields(ResultBox* b, const int32_t* si0, uint64_t stride, const double* w, uint64_t count) {
  // In registers (the arrays could overlap b's fields) and unrolled: the plain
  // loop's time hung on the address that it came to lie at (200000 events 250 or
  // 320 us; so 220).
  vsh_result r = b->pub;
#pragma clang loop unroll_count(4)
  for (uint64_t e = 0; e < count; ++e) {
    const int s_ = si0[e];
    r.n_done += s_ == kDone;
    r.n_overflow += s_ == kOverflow;
    r.n_nonfinite += s_ == kNonFinite;
    r.n_conservation += s_ == kConservation;
    r.n_cycle_limit += s_ == kCycleLimitHit;
    r.sum_w += w[e];
    r.sum_w2 += w[e] * w[e];
    const uint32_t cyc = (uint32_t)si0[(kSiCycles - kSiStatus) * stride + e];
    r.total_cycles += cyc;
    r.max_cycles = std::max(r.max_cycles, cyc);
    r.total_trials += (uint32_t)si0[(kSiTrials - kSiStatus) * stride + e];
    r.total_ends += (uint32_t)si0[(kSiEnds - kSiStatus) * stride + e];
    r.total_emissions += (uint32_t)si0[(kSiEmit - kSiStatus) * stride + e];
  }
  b->pub = r;
}

void* device_address(void* host) {
  void* dev = nullptr;
  if (hipHostGetDevicePointer(&dev, host, 0) == hipSuccess) return dev;
  (void)hipGetLastError();  // handled here: not the next launch's
  return nullptr;
}

// n words, to host memory: in line with the kernels before it, without the
// wait that a copy starts with (calls of 100 events 172 -> 157 us).
__global__ void __launch_bounds__(256) k_copy_out(const uint64_t* __restrict__ from, uint64_t* __restrict__ to,
                                                  uint32_t n) {
  const uint32_t k = blockIdx.x * 256 + threadIdx.x;
  if (k < n) to[k] = from[k];
}

// Copy a chunk's results (one device span from dev_hist on, ResultSpan) back,
// add up the counts and the histogram, and with summaries place the fields in
// the result: in its own pinned block, the counts made from the span's head
// while the rest arrives, or through the staging buffer.  *n_host (optional)
// points at the parton counts.  direct: the kernels wrote the fields into the
// pinned block themselves, only the histogram is copied.
vsh_status copy_back_chunk(vsh_ctx* ctx, hipStream_t st, const double* dev_hist, const Summary& dev_sum,
                           uint64_t count, uint32_t flags, ResultBox* box, uint64_t first_idx,
                           const int32_t** n_host, bool direct) {
  static_assert(kSiStatus == 1 && kSiEnds == kNSumI - 1 && kSdW == 0, "the counts read the span's head");
  const ResultSpan sp(count);
  const char* dev = reinterpret_cast<const char*>(dev_hist);
  const bool span = reinterpret_cast<const char*>(dev_sum.i) == dev + sp.i &&
                    reinterpret_cast<const char*>(dev_sum.d) == dev + sp.d &&
                    reinterpret_cast<const char*>(dev_sum.hash) == dev + sp.hash && dev_sum.stride == count;
  if (direct ? !box->sum_block.ptr : !span) {
    set_error(ctx, "results are not in one span (internal error)");
    return VSH_E_INTERNAL;
  }
  const uint64_t bytes = direct ? kHistDoubles * 8 : (flags & VSH_SUMMARY) ? sp.bytes : sp.head;
  char* host = static_cast<char*>(box->sum_block.ptr);
  if (!host) {
    vsh_status rc = ctx->stage.reserve(ctx, bytes);
    if (rc) return rc;
    host = static_cast<char*>(ctx->stage.ptr);
  }
  // small results in one copy
  const uint64_t first = bytes <= (1u << 18) ? bytes : sp.head;
  hipError_t err = hipSuccess;
  void* host_dev = first == bytes && first <= (1u << 18) ? device_address(host) : nullptr;
  if (host_dev) {
    hipLaunchKernelGGL(k_copy_out, dim3((uint32_t)((first / 8 + 255) / 256)), dim3(256), 0, st, (const uint64_t*)dev,
                       (uint64_t*)host_dev, (uint32_t)(first / 8));
    err = hipGetLastError();
  } else {
    err = hipMemcpyAsync(host, dev, first, hipMemcpyDeviceToHost, st);
  }
  if (err == hipSuccess && first < bytes) {
    err = hipEventRecord(ctx->head_ev, st);
    if (err == hipSuccess) err = hipMemcpyAsync(host + first, dev + first, bytes - first, hipMemcpyDeviceToHost, st);
    if (err == hipSuccess) err = hipEventSynchronize(ctx->head_ev);
  } else if (err == hipSuccess) {
    err = hipStreamSynchronize(st);
  }
  if (err != hipSuccess) return hip_fail(ctx, err, "result copy");
  const double* hh = reinterpret_cast<const double*>(host);
  const int32_t* si = reinterpret_cast<const int32_t*>(host + sp.i);
  const double* sd = reinterpret_cast<const double*>(host + sp.d);
  for (int a = 0; a < kHistDoubles; ++a) box->hist[a] += hh[a];
  tally_fields(box, si + kSiStatus * count, count, sd + kSdW * count, count);
  if (first < bytes) {
    err = hipStreamSynchronize(st);
    if (err != hipSuccess) return hip_fail(ctx, err, "result copy");
  }
  if ((flags & VSH_SUMMARY) && !box->sum_block.ptr) {
    const uint64_t N = box->pub.n_events;
    for (int f = 0; f < kNSumD; ++f) std::memcpy(&box->sum_d[f * N + first_idx], &sd[f * count], count * 8);
    for (int f = 0; f < kNSumI; ++f) std::memcpy(&box->sum_i[f * N + first_idx], &si[f * count], count * 4);
    std::memcpy(&box->hash[first_idx], host + sp.hash, count * 8);
  }
  if (n_host) *n_host = si + kSiN * count;
  return VSH_OK;
}

// gather the final partons of a chunk into CSR order
// A block takes the records of kGatherEvents consecutive events, one stretch
// of each output array, and writes it in order: the output may lie in host
// memory, where only whole lines pass at the link's rate.
constexpr uint32_t kGatherEvents = 128;
__global__ void __launch_bounds__(256) k_gather_records(Records r, const uint64_t* __restrict__ off, uint32_t n,
                                                        double* __restrict__ p, int8_t* __restrict__ pid,
                                                        uint16_t* __restrict__ col, uint16_t* __restrict__ acol) {
  __shared__ uint32_t at[kGatherEvents + 1];  // the events' first partons in the stretch, and its end
  const uint32_t e0 = blockIdx.x * kGatherEvents, ne = n - e0 < kGatherEvents ? n - e0 : kGatherEvents;
  const uint64_t o0 = off[e0];
  for (uint32_t q = threadIdx.x; q <= ne; q += 256) at[q] = (uint32_t)(off[e0 + q] - o0);
  __syncthreads();
  const uint32_t total = at[ne];
  // record column and slot of the stretch's k-th parton
  auto place = [&](uint32_t k) -> uint64_t {
    uint32_t lo = 0, hi = ne;  // at[lo] <= k < at[hi]
    while (hi - lo > 1) {
      const uint32_t mid = (lo + hi) / 2;
      if (at[mid] <= k) lo = mid;
      else hi = mid;
    }
    return (uint64_t)(k - at[lo]) * r.stride + e0 + lo;
  };
  for (uint32_t d = threadIdx.x; d < 4 * total; d += 256) {
    const uint64_t s = place(d / 4);
    const uint32_t c = d % 4;
    p[4 * o0 + d] = (c == 0 ? r.E : c == 1 ? r.x : c == 2 ? r.y : r.z)[s];
  }
  for (uint32_t k = threadIdx.x; k < total; k += 256) {
    const uint64_t s = place(k);
    pid[o0 + k] = r.pid[s];
    col[o0 + k] = r.col[s];
    acol[o0 + k] = r.acol[s];
  }
}

// The final partons of `count` events held slot-major in r (parton counts
// n_host) as CSR records: the whole result's
// (first_idx 0, all its events) in a pinned block of its own, a chunk's
// appended to box's vectors.
vsh_status gather_records(vsh_ctx* ctx, const Records& r, const int32_t* n_host, uint64_t count, ResultBox* box) {
  hipStream_t st = ctx->stream;
  uint64_t total = 0;
  for (uint64_t e = 0; e < count; ++e) total += (uint64_t)n_host[e];
  const RecordSpan sp(count, total);
  PinnedBlock block;
  if (count == box->pub.n_events) block = ctx->pool->acquire(sp.bytes);
  box->rec_block = block;  // released with the result
  // Up to kDirectRecords the kernel reads the offsets from the block and writes
  // the records into it: two copies less (calls of 1000 events 259 -> 236 us,
  // 20000 591 -> 572; 200000 the same, 10^6 1% slower than by the copy engine).
  constexpr uint64_t kDirectRecords = 32u << 20;
  void* dev = block.ptr && sp.bytes <= kDirectRecords ? device_address(block.ptr) : nullptr;
  const bool direct = dev != nullptr;
  char* q = (char*)dev;
  if (!direct) {
    vsh_status rc = ctx->arena2.reserve(ctx, sp.bytes + 256);
    if (rc) return rc;
    q = (char*)ctx->arena2.ptr;
  }
  std::vector<uint64_t> own;
  if (!block.ptr) own.resize(count + 1);
  uint64_t* off = block.ptr ? static_cast<uint64_t*>(block.ptr) : own.data();
  off[0] = 0;
  for (uint64_t e = 0; e < count; ++e) off[e + 1] = off[e] + (uint64_t)n_host[e];
  uint64_t* d_off = (uint64_t*)q;
  double* d_p = (double*)(q + sp.p);
  int8_t* d_pid = (int8_t*)(q + sp.pid);
  uint16_t* d_col = (uint16_t*)(q + sp.col);
  uint16_t* d_acol = (uint16_t*)(q + sp.acol);
  hipError_t err = hipSuccess;
  if (!direct) err = hipMemcpyAsync(d_off, off, (count + 1) * 8, hipMemcpyHostToDevice, st);
  if (err != hipSuccess) return hip_fail(ctx, err, "offset copy");
  hipLaunchKernelGGL(k_gather_records, dim3((uint32_t)((count + kGatherEvents - 1) / kGatherEvents)), dim3(256), 0, st,
                     r, (const uint64_t*)d_off, (uint32_t)count, d_p, d_pid, d_col, d_acol);
  err = hipGetLastError();
  if (err != hipSuccess) return hip_fail(ctx, err, "k_gather_records");
  if (block.ptr) {
    if (!direct && total)
      err = hipMemcpyAsync(static_cast<char*>(block.ptr) + sp.p, q + sp.p, sp.bytes - sp.p, hipMemcpyDeviceToHost, st);
    if (err != hipSuccess) return hip_fail(ctx, err, "record copy");
  } else {
    const uint64_t base = box->rec_offsets.empty() ? 0 : box->rec_offsets.back();
    if (box->rec_offsets.empty()) box->rec_offsets.push_back(0);
    for (uint64_t e = 0; e < count; ++e) box->rec_offsets.push_back(base + off[e + 1]);
    box->rec_p.resize((base + total) * 4);
    box->rec_pid.resize(base + total);
    box->rec_col.resize(base + total);
    box->rec_acol.resize(base + total);
    if (total) {
      err = hipMemcpyAsync(&box->rec_p[base * 4], d_p, total * 32, hipMemcpyDeviceToHost, st);
      if (err == hipSuccess) err = hipMemcpyAsync(&box->rec_pid[base], d_pid, total, hipMemcpyDeviceToHost, st);
      if (err == hipSuccess) err = hipMemcpyAsync(&box->rec_col[base], d_col, total * 2, hipMemcpyDeviceToHost, st);
      if (err == hipSuccess) err = hipMemcpyAsync(&box->rec_acol[base], d_acol, total * 2, hipMemcpyDeviceToHost, st);
      if (err != hipSuccess) return hip_fail(ctx, err, "record copy");
    }
  }
  err = hipStreamSynchronize(st);
  if (err != hipSuccess) return hip_fail(ctx, err, "hipStreamSynchronize");
  return VSH_OK;
}

// ---------------------------------------------------------------------------
// One chunk through the plain pipeline on ctx->stream.
// ---------------------------------------------------------------------------
struct ChunkTimes {
  float me = 0, shower = 0, obs = 0;
};

// Caller-supplied starts (checked offsets) into the chunk's records through
// pinned staging and k_load_records; the device copy of the CSR arrays lies
// where the end cache and the observables' scratch come to work afterwards.
// VSH_E_INVALID (no message) when an event fails a check.
static vsh_status load_records(vsh_ctx* ctx, const PlainLayout& L, const uint64_t* offsets, const double* p,
                               const int8_t* pid, const uint16_t* col, const uint16_t* acol, uint64_t count,
                               hipStream_t st) {
  const uint64_t base = offsets[0], total = offsets[count] - base;
  struct Part {
    const void* from;
    uint64_t bytes, at;
  } parts[] = {{offsets, (count + 1) * 8, 0}, {p + 4 * base, total * 32, 0}, {pid + base, total, 0},
               {col + base, total * 2, 0}, {acol + base, total * 2, 0}};
  uint64_t bytes = 256;  // the first word: the first event that fails
  for (Part& q : parts) {
    q.at = bytes;
    bytes += align_up(q.bytes, 256);
  }
  char* dev = reinterpret_cast<char*>(L.cache);
  if (bytes > (uint64_t)(reinterpret_cast<char*>(L.hist) - dev)) {
    set_error(ctx, "caller-supplied starts of %llu bytes exceed the workspace", (unsigned long long)bytes);
    return VSH_E_INTERNAL;
  }
  vsh_status rc = ctx->stage.reserve(ctx, bytes);
  if (rc) return rc;
  char* host = static_cast<char*>(ctx->stage.ptr);
  unsigned long long* bad = reinterpret_cast<unsigned long long*>(host);
  *bad = ~0ull;
  for (const Part& q : parts) std::memcpy(host + q.at, q.from, q.bytes);
  hipError_t err = hipMemcpyAsync(dev, host, bytes, hipMemcpyHostToDevice, st);
  if (err != hipSuccess) return hip_fail(ctx, err, "starts copy");
  const CsrStarts in{(const uint64_t*)(dev + parts[0].at), (const double*)(dev + parts[1].at),
                     (const int8_t*)(dev + parts[2].at), (const uint16_t*)(dev + parts[3].at),
                     (const uint16_t*)(dev + parts[4].at)};
  launch_load_records(L.rec, L.sum, in, (uint32_t)count, L.ecm, (unsigned long long*)dev, L.hist, st);
  err = hipGetLastError();
  if (err == hipSuccess) err = hipMemcpyAsync(bad, dev, 8, hipMemcpyDeviceToHost, st);
  if (err == hipSuccess) err = hipStreamSynchronize(st);
  if (err != hipSuccess) return hip_fail(ctx, err, "starts");
  return *bad == ~0ull ? VSH_OK : VSH_E_INVALID;
}

static vsh_status run_plain_chunk(vsh_ctx* ctx, const vsh_request* req, uint64_t first_idx,
                                  uint64_t count, const uint64_t* caller_offsets,
                                  const double* cp, const int8_t* cpid, const uint16_t* ccol,
                                  const uint16_t* cacol, ResultBox* box, ChunkTimes& tm) {
  hipStream_t st = ctx->stream;
  const uint32_t cap = req->max_partons;
  const bool massive = request_massive(*req) != 0;
  vsh_status rc = ctx->arena.reserve(ctx, plain_layout_bytes(align_up(count, 64), cap, massive));
  if (rc) return rc;
  PlainLayout L = carve_plain(ctx->arena.ptr, count, cap, massive);
  hipError_t err;
#define HIPCHK(x)                                 \
  do {                                            \
    err = (x);                                    \
    if (err != hipSuccess) return hip_fail(ctx, err, #x); \
  } while (0)
  EventInputs in{};
  in.seed = req->seed;
  in.first = req->first_event + first_idx;
  in.cycle_limit = effective_cycle_limit(req->cycle_limit);
  in.t_over = req->t_over;
  in.qm = request_masses(*req);
  in.massive = request_massive(*req);
  in.fixed_hist = (req->flags & VSH_HIST_FIXEDPOINT) ? 1u : 0u;
  in.ecm0 = req->ecm;
  in.tcut0 = req->t_cut;
  const bool from_records = caller_offsets != nullptr;
  if (from_records) {
    in.ecm = L.ecm;
  } else if (req->ecm_per_event) {
    HIPCHK(hipMemcpyAsync(L.ecm, req->ecm_per_event + first_idx, count * 8, hipMemcpyHostToDevice, st));
    in.ecm = L.ecm;
  }
  if (req->tcut_per_event) {
    HIPCHK(hipMemcpyAsync(L.tcut, req->tcut_per_event + first_idx, count * 8, hipMemcpyHostToDevice, st));
    in.tcut = L.tcut;
  }
  HIPCHK(hipEventRecord(ctx->ev[0], st));
  if (from_records) {
    rc = load_records(ctx, L, caller_offsets + first_idx, cp, cpid, ccol, cacol, count, st);
    if (rc) return rc;
  } else {
    launch_me(L.rec, L.sum, in, (uint32_t)count, st, L.hist);
  }
  HIPCHK(hipGetLastError());
  HIPCHK(hipEventRecord(ctx->ev[1], st));
  if (ctx->tuned.plain_mapping == kMapFlat)
    launch_shower_plain_flat(L.rec, L.sum, in, (uint32_t)count, L.cache, (uint32_t)ctx->n_cu, st);
  else launch_shower_plain(L.rec, L.sum, in, (uint32_t)count, ctx->tuned.plain_block, ctx->tuned.plain_waves, st);
  HIPCHK(hipGetLastError());
  HIPCHK(hipEventRecord(ctx->ev[2], st));
  launch_obs(L.rec, L.sum, in, L.sc, (uint32_t)count, L.hist, nullptr, st);
  HIPCHK(hipGetLastError());
  HIPCHK(hipEventRecord(ctx->ev[3], st));
  const int32_t* n_host = nullptr;
  rc = copy_back_chunk(ctx, st, L.hist, L.sum, count, req->flags, box, first_idx, &n_host);
  if (rc) return rc;
  float ms;
  HIPCHK(hipEventElapsedTime(&ms, ctx->ev[0], ctx->ev[1]));
  tm.me += ms;
  HIPCHK(hipEventElapsedTime(&ms, ctx->ev[1], ctx->ev[2]));
  tm.shower += ms;
  HIPCHK(hipEventElapsedTime(&ms, ctx->ev[2], ctx->ev[3]));
  tm.obs += ms;
  if (req->flags & VSH_RECORDS) {
    rc = gather_records(ctx, L.rec, n_host, count, box);
    if (rc) return rc;
  }
#undef HIPCHK
  return VSH_OK;
}

uint64_t chunk_events(vsh_ctx* ctx, const vsh_request* req) {
  const uint64_t per = plain_bytes_per_event(req->max_partons, request_massive(*req) != 0);
  uint64_t budget = ctx->budget;
  // leave room for the record-gather buffer when records are returned
  if (req->flags & VSH_RECORDS) budget = budget / 2;
  uint64_t n = budget / (per + 64);
  n = std::min<uint64_t>(n, 1ull << 26);
  if (n >= req->n_events) return req->n_events;  // the whole request in one piece
  return n & ~63ull ? n & ~63ull : n;
}

vsh_status generate_plain(vsh_ctx* ctx, const vsh_request* req, const uint64_t* offsets,
                          const double* p, const int8_t* pid, const uint16_t* col,
                          const uint16_t* acol, vsh_result** out) {
  const auto t0 = std::chrono::steady_clock::now();
  const uint64_t chunk = chunk_events(ctx, req);
  if (chunk == 0) {
    set_error(ctx, "memory budget of %llu bytes cannot hold one event of %u partons",
              (unsigned long long)ctx->budget, req->max_partons);
    return VSH_E_NOMEM;
  }
  ResultBox* box = new_call_result(ctx, req, chunk >= req->n_events);
  if (!box) return VSH_E_NOMEM;
  ChunkTimes tm;
  for (uint64_t a = 0; a < req->n_events; a += chunk) {
    const uint64_t count = std::min(chunk, req->n_events - a);
    vsh_status rc = run_plain_chunk(ctx, req, a, count, offsets, p, pid, col, acol, box, tm);
    if (rc) {
      drop_result(ctx, box);
      return rc;
    }
  }
  box->pub.t_me_ms = tm.me;
  box->pub.t_shower_ms = tm.shower;
  box->pub.t_obs_ms = tm.obs;
  box->pub.t_total_ms =
      std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
  finish_result(box);
  *out = &box->pub;
  return VSH_OK;
}

// events of the next timed vsh_generate_into call, or null when not timing
hipEvent_t* timing_slot(vsh_ctx* ctx) {
  if (!ctx->timing || ctx->timing_calls >= VSH_TIMING_MAX_CALLS) return nullptr;
  const size_t need = 4 * (size_t)(ctx->timing_calls + 1);
  while (ctx->timing_ev.size() < need) {
    hipEvent_t e;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    ctx->timing_ev.push_back(e);
  }
  return &ctx->timing_ev[4 * (size_t)ctx->timing_calls++];
}

// The plain-form launch sequence of vsh_generate_into on stream st with the
// workspace at `ws` (at least vsh_workspace_size bytes; nothing in it needs
// to start at zero): matrix element, shower, observables and histogram
// accumulated into dev_hist, the kernels working in the caller's [field][n]
// summary buffers directly (in the workspace's where the caller gave none).
// `timed`: record the stage events of vsh_timing_start.
// Launches only.
vsh_status plain_into(vsh_ctx* ctx, const vsh_request* req, hipStream_t st, void* ws, double* dev_hist,
                      double* dev_sum_d, int32_t* dev_sum_i, uint64_t* dev_hash, bool timed) {
  const uint64_t n = req->n_events;
  PlainLayout L = carve_plain(ws, n, req->max_partons, request_massive(*req) != 0);
  EventInputs in{};
  in.seed = req->seed;
  in.first = req->first_event;
  in.cycle_limit = effective_cycle_limit(req->cycle_limit);
  in.t_over = req->t_over;
  in.qm = request_masses(*req);
  in.massive = request_massive(*req);
  in.fixed_hist = (req->flags & VSH_HIST_FIXEDPOINT) ? 1u : 0u;
  in.ecm0 = req->ecm;
  in.tcut0 = req->t_cut;
  in.ecm = req->ecm_per_event;
  in.tcut = req->tcut_per_event;
  Summary sum = L.sum;
  if (dev_sum_d) sum.d = dev_sum_d;
  if (dev_sum_i) sum.i = dev_sum_i;
  if (dev_hash) sum.hash = dev_hash;
  hipEvent_t* tev = timed ? timing_slot(ctx) : nullptr;
  if (tev) (void)hipEventRecord(tev[0], st);
  launch_me(L.rec, sum, in, (uint32_t)n, st, L.hist);
  if (tev) (void)hipEventRecord(tev[1], st);
  if (ctx->tuned.plain_mapping == kMapFlat)
    launch_shower_plain_flat(L.rec, sum, in, (uint32_t)n, L.cache, (uint32_t)ctx->n_cu, st);
  else launch_shower_plain(L.rec, sum, in, (uint32_t)n, ctx->tuned.plain_block, ctx->tuned.plain_waves, st);
  if (tev) (void)hipEventRecord(tev[2], st);
  launch_obs(L.rec, sum, in, L.sc, (uint32_t)n, dev_hist, L.hist, st);
  if (tev) (void)hipEventRecord(tev[3], st);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return hip_fail(ctx, err, "kernel launch");
  return VSH_OK;
}

// The message for the first fault of caller-supplied starts.
static vsh_status explain_starts(vsh_ctx* ctx, const vsh_request* req, const uint64_t* offsets, const double* p,
                                 const int8_t* pid, const uint16_t* col, const uint16_t* acol) {
  for (uint64_t e = 0; e < req->n_events; ++e) {
    if (offsets[e + 1] < offsets[e] || offsets[e + 1] - offsets[e] > req->max_partons ||
        offsets[e + 1] - offsets[e] < 2) {
      set_error(ctx, "event %llu: parton count must be in 2..max_partons", (unsigned long long)e);
      return VSH_E_INVALID;
    }
    // every colour line must have exactly one start and one end
    std::vector<int> seen_c(kMaxCap * 2 + 2, 0), seen_a(kMaxCap * 2 + 2, 0);
    double E = 0.0;
    for (uint64_t a = offsets[e]; a < offsets[e + 1]; ++a) {
      const int f = pid[a];
      const bool q = f >= 1 && f <= 5, qb = f <= -1 && f >= -5, g = f == 21;
      if (!(q || qb || g) || (q && (col[a] == 0 || acol[a] != 0)) || (qb && (col[a] != 0 || acol[a] == 0)) ||
          (g && (col[a] == 0 || acol[a] == 0)) || col[a] > 2 * kMaxCap || acol[a] > 2 * kMaxCap) {
        set_error(ctx, "event %llu parton %llu: bad flavour/colour", (unsigned long long)e,
                  (unsigned long long)(a - offsets[e]));
        return VSH_E_INVALID;
      }
      if (col[a]) seen_c[col[a]]++;
      if (acol[a]) seen_a[acol[a]]++;
      E += p[4 * a];
    }
    for (size_t c = 0; c < seen_c.size(); ++c)
      if (seen_c[c] != seen_a[c] || seen_c[c] > 1) {
        set_error(ctx, "event %llu: colour line %zu is not closed once", (unsigned long long)e, c);
        return VSH_E_INVALID;
      }
    if (!(E > 0.0)) {
      set_error(ctx, "event %llu: total energy must be > 0", (unsigned long long)e);
      return VSH_E_INVALID;
    }
  }
  set_error(ctx, "inconsistent initial states");  // not reached: the device makes the same checks
  return VSH_E_INVALID;
}

}  // namespace vsh

using namespace vsh;

extern "C" {

vsh_status vsh_create(const vsh_ctx_opts* opts, vsh_ctx** out) {
  if (!out) {
    set_error(nullptr, "out is NULL");
    return VSH_E_INVALID;
  }
  *out = nullptr;
  const int dev = opts ? opts->device : 0;
  int count = 0;
  hipError_t err = hipGetDeviceCount(&count);
  if (err != hipSuccess || count == 0) {
    (void)hipGetLastError();
    set_error(nullptr, "no HIP device available (%s)", hipGetErrorString(err));
    return VSH_E_DEVICE;
  }
  if (dev < 0 || dev >= count) {
    set_error(nullptr, "device %d out of range (%d devices)", dev, count);
    return VSH_E_INVALID;
  }
  hipDeviceProp_t prop;
  err = hipGetDeviceProperties(&prop, dev);
  if (err != hipSuccess) return hip_fail(nullptr, err, "hipGetDeviceProperties");
  if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0) {
    set_error(nullptr, "device %d is %s; libvsh is built for gfx950 only", dev, prop.gcnArchName);
    return VSH_E_DEVICE;
  }
  err = hipSetDevice(dev);
  if (err != hipSuccess) return hip_fail(nullptr, err, "hipSetDevice");
  vsh_ctx* ctx = new (std::nothrow) vsh_ctx();
  if (!ctx) {
    set_error(nullptr, "host allocation failed");
    return VSH_E_NOMEM;
  }
  ctx->device = dev;
  ctx->n_cu = prop.multiProcessorCount;
  try {
    ctx->pool = std::make_shared<PinnedPool>();
  } catch (const std::bad_alloc&) {
    delete ctx;
    set_error(nullptr, "host allocation failed");
    return VSH_E_NOMEM;
  }
  size_t free_b = 0, total_b = 0;
  err = hipMemGetInfo(&free_b, &total_b);
  if (err != hipSuccess) {
    delete ctx;
    return hip_fail(nullptr, err, "hipMemGetInfo");
  }
  ctx->budget = (opts && opts->mem_budget_bytes) ? opts->mem_budget_bytes : (uint64_t)(0.8 * (double)free_b);
  if (opts && opts->tuner_cache_path) ctx->tuner_cache_path = opts->tuner_cache_path;
  err = hipStreamCreateWithFlags(&ctx->stream, hipStreamNonBlocking);
  if (err != hipSuccess) {
    delete ctx;
    return hip_fail(nullptr, err, "hipStreamCreate");
  }
  // the stage events only take times: without the caches' write-back to the
  // system between the kernels (calls of 100 events 2% shorter)
  for (auto& e : ctx->ev) {
    err = hipEventCreateWithFlags(&e, hipEventDisableSystemFence);
    if (err != hipSuccess) {
      delete ctx;
      return hip_fail(nullptr, err, "hipEventCreate");
    }
  }
  err = hipEventCreateWithFlags(&ctx->head_ev, hipEventDisableTiming);
  if (err != hipSuccess) {
    delete ctx;
    return hip_fail(nullptr, err, "hipEventCreate");
  }
  // the static workspace's address on this device (vsh_generate_into_static
  // looks it up itself if this fails; nothing else depends on it)
  (void)static_scratch_init(ctx);
  ctx->error.clear();
  *out = ctx;
  return VSH_OK;
}

void vsh_destroy(vsh_ctx* ctx) {
  if (!ctx) return;
  serve_shutdown(ctx);
  (void)hipSetDevice(ctx->device);
  if (ctx->stream) (void)hipStreamSynchronize(ctx->stream);
  ctx->arena.release();
  ctx->arena2.release();
  ctx->stage.release();
  ctx->pool->close();  // results still held free their blocks themselves
  if (ctx->head_ev) (void)hipEventDestroy(ctx->head_ev);
  for (auto& e : ctx->timing_ev) (void)hipEventDestroy(e);
  for (auto& e : ctx->ev)
    if (e) (void)hipEventDestroy(e);
  if (ctx->stream) (void)hipStreamDestroy(ctx->stream);
  delete ctx;
}

const char* vsh_last_error(const vsh_ctx* ctx) {
  if (!ctx) return g_create_error.c_str();
  return ctx->error.c_str();
}

vsh_status vsh_generate(vsh_ctx* ctx, const vsh_request* req, vsh_result** out) {
  if (!ctx || !out) return VSH_E_INVALID;
  std::lock_guard<std::mutex> lk(ctx->mu);
  *out = nullptr;
  vsh_status rc = validate_request(ctx, req, true);
  if (rc) return rc;
  if (req->flags & VSH_INPUTS_ON_DEVICE) {
    set_error(ctx, "VSH_INPUTS_ON_DEVICE is for vsh_generate_into only");
    return VSH_E_INVALID;
  }
  (void)hipSetDevice(ctx->device);
  if (req->flags & VSH_FORM_PERSISTENT) return generate_persistent(ctx, req, out);
  return generate_plain(ctx, req, nullptr, nullptr, nullptr, nullptr, nullptr, out);
}

void vsh_result_free(vsh_result* res) {
  if (!res) return;
  delete reinterpret_cast<ResultBox*>(reinterpret_cast<char*>(res) - offsetof(ResultBox, pub));
}

vsh_status vsh_shower_records(vsh_ctx* ctx, const vsh_request* req, const uint64_t* offsets,
                              const double* p, const int8_t* pid, const uint16_t* col,
                              const uint16_t* acol, vsh_result** out) {
  if (!ctx || !out) return VSH_E_INVALID;
  std::lock_guard<std::mutex> lk(ctx->mu);
  *out = nullptr;
  vsh_status rc = validate_request(ctx, req, false);
  if (rc) return rc;
  if (!offsets || !p || !pid || !col || !acol) {
    set_error(ctx, "offsets, p, pid, col and acol are required");
    return VSH_E_INVALID;
  }
  if (req->flags & (VSH_INPUTS_ON_DEVICE | VSH_FORM_PERSISTENT)) {
    set_error(ctx, "vsh_shower_records runs the plain form with host inputs");
    return VSH_E_INVALID;
  }
  // the counts here, flavours and colours on the device as the events are
  // loaded; a request that fails either is gone through again for its first
  // fault
  bool counts = true;
  for (uint64_t e = 0; e < req->n_events; ++e)
    counts = counts && offsets[e + 1] >= offsets[e] && offsets[e + 1] - offsets[e] <= req->max_partons &&
             offsets[e + 1] - offsets[e] >= 2;
  if (!counts) return explain_starts(ctx, req, offsets, p, pid, col, acol);
  (void)hipSetDevice(ctx->device);
  rc = generate_plain(ctx, req, offsets, p, pid, col, acol, out);
  return rc == VSH_E_INVALID ? explain_starts(ctx, req, offsets, p, pid, col, acol) : rc;
}

uint64_t vsh_workspace_size(const vsh_request* req) {
  if (!req || req->n_events == 0 || req->max_partons < 2 || req->max_partons > kMaxCap) return 0;
  if (req->flags & VSH_FORM_PERSISTENT) return persistent_workspace_bytes(req);
  return plain_layout_bytes(align_up(req->n_events, 64), req->max_partons, request_massive(*req) != 0);
}

vsh_status vsh_generate_into(vsh_ctx* ctx, const vsh_request* req, void* stream, void* workspace,
                             uint64_t workspace_bytes, double* dev_hist, double* dev_sum_d,
                             int32_t* dev_sum_i, uint64_t* dev_hash) {
  if (!ctx) return VSH_E_INVALID;
  std::lock_guard<std::mutex> lk(ctx->mu);
  vsh_status rc = validate_request(ctx, req, true);
  if (rc) return rc;
  if (!workspace || !dev_hist) {
    set_error(ctx, "workspace and dev_hist are required");
    return VSH_E_INVALID;
  }
  if (req->flags & VSH_RECORDS) {
    set_error(ctx, "vsh_generate_into returns summaries and histograms only");
    return VSH_E_INVALID;
  }
  const uint64_t need = vsh_workspace_size(req);
  if (workspace_bytes < need) {
    set_error(ctx, "workspace of %llu bytes is smaller than the %llu needed", (unsigned long long)workspace_bytes,
              (unsigned long long)need);
    return VSH_E_INVALID;
  }
  const bool dev_inputs = req->flags & VSH_INPUTS_ON_DEVICE;
  if (!dev_inputs && (req->ecm_per_event || req->tcut_per_event)) {
    set_error(ctx, "per-event arrays of vsh_generate_into must be device pointers (VSH_INPUTS_ON_DEVICE)");
    return VSH_E_INVALID;
  }
  (void)hipSetDevice(ctx->device);
  hipStream_t st = (hipStream_t)stream;
  if (req->flags & VSH_FORM_PERSISTENT)
    return persistent_into(ctx, req, st, workspace, dev_hist, dev_sum_d, dev_sum_i, dev_hash);
  return plain_into(ctx, req, st, workspace, dev_hist, dev_sum_d, dev_sum_i, dev_hash, true);
}

vsh_status vsh_timing_start(vsh_ctx* ctx) {
  if (!ctx) return VSH_E_INVALID;
  std::lock_guard<std::mutex> lk(ctx->mu);
  ctx->timing = true;
  ctx->timing_calls = 0;
  return VSH_OK;
}

vsh_status vsh_timing_read(vsh_ctx* ctx, float* ms, uint32_t max_calls, uint32_t* n_calls) {
  if (!ctx) return VSH_E_INVALID;
  std::lock_guard<std::mutex> lk(ctx->mu);
  if (!ctx->timing) {
    set_error(ctx, "vsh_timing_read without vsh_timing_start");
    return VSH_E_INVALID;
  }
  const uint32_t n = std::min(ctx->timing_calls, max_calls);
  for (uint32_t c = 0; c < n; ++c) {
    hipEvent_t* e = &ctx->timing_ev[4 * (size_t)c];
    hipError_t err = hipEventSynchronize(e[3]);
    if (err != hipSuccess) return hip_fail(ctx, err, "hipEventSynchronize");
    for (int k = 0; k < 3; ++k) {
      float v = 0.0f;
      err = hipEventElapsedTime(&v, e[k], e[k + 1]);
      if (err != hipSuccess) return hip_fail(ctx, err, "hipEventElapsedTime");
      if (ms) ms[3 * c + k] = v;
    }
  }
  if (n_calls) *n_calls = n;
  ctx->timing = false;
  ctx->timing_calls = 0;
  return VSH_OK;
}

}  // extern "C"
