// host_paths.cpp -- one scenario of the library's host code per run (argv[1]),
// on the fake runtime.  Exit status 0: as it should be.
#include <sys/wait.h>
#include <unistd.h>

#include <new>

#include "fake_hip.hpp"
#include "vsh.h"

void* operator new(size_t n) {
  if (fake::fail_new > 0 && --fake::fail_new == 0) throw std::bad_alloc();
  if (void* p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

#define CHECK(x)                                                \
  do {                                                          \
    if (!(x)) {                                                 \
      std::fprintf(stderr, "line %d: %s\n", __LINE__, #x);      \
      _exit(1);                                                 \
    }                                                           \
  } while (0)

static vsh_ctx* context(uint64_t budget = 0) {
  vsh_ctx_opts o{};
  o.mem_budget_bytes = budget;
  vsh_ctx* c = nullptr;
  CHECK(vsh_create(&o, &c) == VSH_OK);
  return c;
}

static vsh_request request(uint64_t n, uint32_t flags) {
  vsh_request r{};
  r.n_events = n;
  r.seed = 1;
  r.ecm = 91.2;
  r.t_cut = 1.0;
  r.max_partons = 16;
  r.flags = flags;
  return r;
}

static vsh_result* generate(vsh_ctx* c, uint64_t n, uint32_t flags) {
  const vsh_request r = request(n, flags);
  vsh_result* out = nullptr;
  CHECK(vsh_generate(c, &r, &out) == VSH_OK);
  return out;
}

// A forked child reads, writes and frees the results that its parent holds;
// the parent's stay as they were and its blocks go on serving.
static void forked_child() {
  vsh_ctx* c = context();
  const uint64_t n = 5000;
  vsh_result* r = generate(c, n, VSH_SUMMARY | VSH_RECORDS);
  double* d = const_cast<double*>(r->sum_d);
  for (uint64_t k = 0; k < VSH_NSUM_D * n; ++k) d[k] = 0.5 * (double)k;
  for (int round = 0; round < 2; ++round) {
    const pid_t pid = fork();
    CHECK(pid >= 0);
    if (pid == 0) {
      for (uint64_t k = 0; k < VSH_NSUM_D * n; ++k) CHECK(d[k] == 0.5 * (double)k);
      CHECK(r->rec_offsets[n] == 0);
      d[7] = -1.0;
      const pid_t sub = fork();  // a child's child too
      CHECK(sub >= 0);
      if (sub == 0) {
        CHECK(d[7] == -1.0 && d[8] == 4.0);
        _exit(0);
      }
      int s = 0;
      CHECK(waitpid(sub, &s, 0) == sub && s == 0);
      vsh_result_free(r);
      _exit(0);
    }
    int status = 0;
    CHECK(waitpid(pid, &status, 0) == pid);
    CHECK(WIFEXITED(status) && WEXITSTATUS(status) == 0);
    CHECK(d[7] == 3.5);
  }
  vsh_result_free(r);
  vsh_result_free(generate(c, n, VSH_SUMMARY));
  vsh_destroy(c);
}

// A served request with little device memory left: the observables' scratch is
// no larger than it has to be.
static void serving_little_memory() {
  vsh_ctx* c = context((uint64_t)256 << 20);
  const vsh_request r = request(200, 0);
  vsh_result* out = nullptr;
  uint64_t t = 0;
  CHECK(vsh_test_fail_epochs(c, 1) == VSH_OK);  // allocates an epoch's memory, ends before its scratch
  CHECK(vsh_submit(c, &r, &t) == VSH_OK);
  CHECK(vsh_wait(c, t, &out) == VSH_E_DEVICE);
  {
    fake::Lock l(fake::st().mu);
    fake::st().dev_limit = fake::st().dev_bytes + ((size_t)2 << 20);
  }
  CHECK(vsh_submit(c, &r, &t) == VSH_OK);
  CHECK(vsh_wait(c, t, &out) == VSH_OK);
  vsh_result_free(out);
  // many requests finished by one epoch, whose scratch together does not fit
  {
    fake::Lock l(fake::st().mu);
    fake::st().running = true;
  }
  std::vector<uint64_t> tickets(200);
  for (uint64_t& q : tickets) CHECK(vsh_submit(c, &r, &q) == VSH_OK);
  {
    fake::Lock l(fake::st().mu);
    fake::st().running = false;
  }
  for (uint64_t q : tickets) {
    CHECK(vsh_wait(c, q, &out) == VSH_OK);
    vsh_result_free(out);
  }
  vsh_destroy(c);
}

// Whichever runtime call fails, a failed call leaves nothing in flight (its
// memory serves the next one) and the next call works.
static void failing_calls() {
  int failed = 0;
  for (const uint64_t n : {(uint64_t)100, (uint64_t)5000}) {
    std::vector<uint64_t> off(n + 1);
    std::vector<double> p(8 * n, 1.0);
    std::vector<int8_t> pid(2 * n);
    std::vector<uint16_t> col(2 * n), acol(2 * n);
    for (uint64_t k = 0; k <= n; ++k) off[k] = 2 * k;
    for (uint64_t k = 0; k < n; ++k) {
      pid[2 * k] = col[2 * k] = acol[2 * k + 1] = 1;
      pid[2 * k + 1] = -1;
    }
    for (int call = 0; call < 4; ++call) {
      vsh_ctx* c = context();  // its memory starts at zero, and no kernel writes it
      for (const uint32_t flags : {VSH_SUMMARY, VSH_SUMMARY | VSH_RECORDS, 0u}) {
        const vsh_request r = request(n, flags | (call == 1 ? VSH_FORM_PERSISTENT : 0u));
        auto run = [&](vsh_result** out) {
          if (call == 2) return vsh_generate_isr(c, &r, 1960.0, out);
          if (call == 3) return vsh_shower_records(c, &r, off.data(), p.data(), pid.data(), col.data(), acol.data(), out);
          return vsh_generate(c, &r, out);
        };
        for (const char* name : {"hipMemcpyAsync", "hipEventRecord", "hipLaunchKernel", "hipStreamSynchronize",
                                 "hipEventSynchronize", "hipHostMalloc", "hipHostGetDevicePointer"})
          for (int k = 1;; ++k) {
            vsh_result* out = nullptr;
            fake::st().fail[name] = k;
            const vsh_status rc = run(&out);
            const bool hit = !fake::st().fail.count(name);
            fake::st().fail.clear();
            if (rc == VSH_OK) vsh_result_free(out);
            else {
              ++failed;
              const bool idle = fake::st().queue.empty();
              const bool next = run(&out) == VSH_OK;
              if (!idle || !next)
                std::fprintf(stderr, "call %d of %d events, flags %u, %s number %d: %s\n", call, (int)n, flags, name, k,
                             vsh_last_error(c));
              CHECK(idle && next);
              vsh_result_free(out);
            }
            if (!hit) break;
          }
      }
      vsh_destroy(c);
    }
  }
  CHECK(failed > 100);
}

// Where the device address of pinned memory is not to be had, results come by
// copies instead: the calls work, and their errors end with them.
static void no_device_address() {
  vsh_ctx* c = context();
  for (const uint64_t n : {(uint64_t)100, (uint64_t)5000})
    for (const uint32_t flags : {VSH_SUMMARY, VSH_SUMMARY | VSH_RECORDS, 0u})
      for (int k = 1; k <= 2; ++k) {
        fake::st().fail["hipHostGetDevicePointer"] = k;
        vsh_result_free(generate(c, n, flags));
        fake::st().fail.clear();
        CHECK(hipGetLastError() == hipSuccess);
      }
  vsh_destroy(c);
}

// A result that the pool cannot hold, by itself or beside those in use, goes
// through the staging memory and leaves the pool's idle blocks where they are.
static void result_beyond_the_pool() {
  vsh_ctx* c = context();
  vsh_result_free(generate(c, 5000, VSH_SUMMARY));
  vsh_request r = request(9300000, VSH_SUMMARY);  // 1.08 GB of summaries
  r.max_partons = 2;
  vsh_result* out = nullptr;
  CHECK(vsh_generate(c, &r, &out) == VSH_OK);
  vsh_result_free(out);
  const int allocs = fake::st().pinned_allocs;
  vsh_result_free(generate(c, 5000, VSH_SUMMARY));
  CHECK(fake::st().pinned_allocs == allocs);
  r.n_events = 8000000;  // 0.93 GB
  CHECK(vsh_generate(c, &r, &out) == VSH_OK);
  r.n_events = 2000000;
  vsh_result* second = nullptr;
  CHECK(vsh_generate(c, &r, &second) == VSH_OK);  // no room beside the first
  const int more = fake::st().pinned_allocs;
  vsh_result_free(generate(c, 5000, VSH_SUMMARY));
  CHECK(fake::st().pinned_allocs == more);
  vsh_result_free(out);
  vsh_result_free(second);
  vsh_destroy(c);
}

// Where host memory runs out while a result is set up, the call says so (or
// does without a pinned block); no exception leaves it.
static void no_host_memory() {
  for (int call = 0; call < 3; ++call)
    for (int k = 1;; ++k) {
      vsh_ctx* c = context();
      const vsh_request r = request(5000, VSH_SUMMARY | (call == 1 ? VSH_FORM_PERSISTENT : 0u));
      vsh_result* out = nullptr;
      fake::fail_new = k;
      const vsh_status rc = call == 2 ? vsh_generate_isr(c, &r, 1960.0, &out) : vsh_generate(c, &r, &out);
      const bool hit = fake::fail_new == 0;
      fake::fail_new = 0;
      CHECK(rc == VSH_OK || rc == VSH_E_NOMEM);
      vsh_result_free(out);
      vsh_destroy(c);
      if (!hit) {
        CHECK(rc == VSH_OK && k > 3);
        break;
      }
    }
}

// blocks of the launch of the last kernel with `name` in its name
static uint32_t blocks_of(const char* name) {
  const auto& l = fake::st().launches;
  for (size_t k = l.size(); k-- > 0;)
    if (l[k].kernel.find(name) != std::string::npos) return l[k].blocks;
  CHECK(!"launched");
  return 0;
}

// A small launch's events are spread over the waves that the device's compute
// units hold at once, and no more: `resident` per CU, by the kernel's registers
// and its LDS of 1280-byte units.
static void waves_of_small_launches() {
  struct Case {
    uint32_t cap;
    bool massive, batched;
    uint32_t resident;
  };
  const Case cases[] = {{64, false, false, 16}, {128, false, false, 16}, {256, false, false, 12},
                        {512, false, false, 9}, {1024, false, false, 6}, {128, false, true, 16},
                        {256, false, true, 12}, {512, false, true, 9},   {1024, false, true, 6},
                        {64, true, false, 12},  {128, true, false, 12},  {256, true, false, 10},
                        {512, true, false, 8},  {1024, true, false, 6},  {64, true, true, 12},
                        {256, true, true, 11},  {512, true, true, 9},    {1024, true, true, 6}};
  for (const int cus : {256, 32}) {
    fake::st().cus = cus;
    vsh_ctx* c = context();
    for (const Case& k : cases)
      for (const uint32_t per : {1u, 3u}) {
        vsh_request r = request((uint64_t)per * k.resident * (uint32_t)cus, k.batched ? VSH_FORM_PERSISTENT : 0u);
        r.max_partons = k.cap;
        if (k.massive) r.mass_b = 4.8;
        vsh_result* out = nullptr;
        CHECK(vsh_generate(c, &r, &out) == VSH_OK);
        vsh_result_free(out);
        const uint32_t blocks = blocks_of(k.batched ? "k_shower_flat" : "k_shower_plain_flat");
        const uint32_t most = k.resident * (uint32_t)cus;
        if (blocks > most || 2 * blocks < most)
          std::fprintf(stderr, "%d CUs, cap %u, massive %d, batched %d: %u blocks of %u\n", cus, k.cap, k.massive,
                       k.batched, blocks, most);
        CHECK(blocks <= most && 2 * blocks >= most);
      }
    // the initial-state shower: as many lanes per event as leave all resident
    const vsh_request r = request(40 * (uint64_t)cus, 0);
    vsh_result* out = nullptr;
    CHECK(vsh_generate_isr(c, &r, 1960.0, &out) == VSH_OK);
    vsh_result_free(out);
    CHECK(blocks_of("k_isr") == 40u * 8u * (uint32_t)cus / 256u);
    vsh_destroy(c);
  }
}

int main(int argc, char** argv) {
  const std::map<std::string, void (*)()> scenarios{{"forked child", forked_child},
                                                        {"serving, little memory", serving_little_memory},
                                                        {"failing calls", failing_calls},
                                                        {"no device address", no_device_address},
                                                        {"result beyond the pool", result_beyond_the_pool},
                                                        {"no host memory", no_host_memory},
                                                        {"waves of small launches", waves_of_small_launches}};
  CHECK(argc == 2 && scenarios.count(argv[1]));
  scenarios.at(argv[1])();
  return 0;
}
