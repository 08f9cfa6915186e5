// The drain (gsys_wait, gsys_stats_get, gsys_unregister_buffer,
// gsys_shutdown) of a device context whose device is this file: the few HIP
// functions that capi.cpp calls work on host memory, and the kernel that hands
// the ticket counter over does what a test says.  The counter is device memory
// in a real context; here host threads claim tickets from it and publish
// requests as the GPU does.  One scenario per run, named by argv[1]; exit 0
// when its checks pass.
//
// Build: g++ over this file, capi.cpp and host_pool.cpp (no HIP device needed;
// the definitions here take the place of the runtime's).
#include <errno.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <time.h>

#include <atomic>
#include <mutex>
#include <thread>
#include <vector>

#include <hip/hip_runtime.h>

#include "gsys.h"
#include "gsys_abi.h"

namespace {

enum Mode { kStores, kNever, kFails, kEndsSilently, kQueryFails };
std::atomic<int> mode{kStores};
std::mutex late_mu;
std::vector<uint64_t*> late;  // words of stores that were queued and not made
std::atomic<bool> kernel_runs{false}, watchdog{false};  // a "kernel" that waits for a result

uint64_t now_ns() {
  timespec ts;
  clock_gettime(CLOCK_MONOTONIC, &ts);
  return (uint64_t)ts.tv_sec * 1000000000ull + (uint64_t)ts.tv_nsec;
}

void sleep_ms(long ms) {
  timespec ts{ms / 1000, (ms % 1000) * 1000000};
  nanosleep(&ts, nullptr);
}

void store(uint64_t* out, uint64_t v) { __atomic_store_n(out, v, __ATOMIC_RELEASE); }

}  // namespace

// ------------------------------------------------------------ the fake device
namespace gsys_internal {
int serve_scratch_setup(int) { return 0; }
bool launch_read_tail(const unsigned long long* tail, uint64_t out, hipStream_t) {
  const int m = mode.load();
  if (m == kFails) return false;
  if (m == kStores) {
    store((uint64_t*)out, __atomic_load_n(tail, __ATOMIC_ACQUIRE));
  } else {
    std::lock_guard<std::mutex> g(late_mu);
    late.push_back((uint64_t*)out);
  }
  return true;
}
}  // namespace gsys_internal

extern "C" {
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  memset(p, 0, sizeof *p);
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = 100000, hipSuccess; }
hipError_t hipDeviceSynchronize() {
  for (int i = 0; i < 3000 && kernel_runs; ++i) sleep_ms(1);
  watchdog = true;  // the kernel's own bound on its wait
  while (kernel_runs) sleep_ms(1);
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return *s = (hipStream_t)8, hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t) {
  const int m = mode.load();
  return m == kEndsSilently ? hipSuccess : m == kQueryFails ? hipErrorUnknown : hipErrorNotReady;
}
hipError_t hipMalloc(void** p, size_t n) { return (*p = calloc(1, n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { return free(p), hipSuccess; }
hipError_t hipMemset(void* p, int v, size_t n) { return memset(p, v, n), hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  return posix_memalign(p, 4096, n) ? hipErrorOutOfMemory : hipSuccess;
}
hipError_t hipHostFree(void* p) { return free(p), hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) { return *d = h, hipSuccess; }
}

// ------------------------------------------------------------------ scenarios
namespace {

#define CHECK(x)                                                          \
  do {                                                                    \
    if (!(x)) {                                                           \
      fprintf(stderr, "FAIL line %d: %s\n", __LINE__, #x);                \
      exit(1);                                                            \
    }                                                                     \
  } while (0)

gsys_ctx* make(gsys_dev_ctx* d) {
  gsys_config cfg;
  memset(&cfg, 0, sizeof cfg);
  cfg.abi_version = GSYS_ABI_VERSION;
  cfg.ring_slots = 4096;
  cfg.service_threads = 2;
  cfg.first_cpu = -1;
  gsys_ctx* c = nullptr;
  CHECK(gsys_init(&cfg, &c) == 0);
  CHECK(gsys_device_ctx(c, d) == 0);
  return c;
}

uint64_t claim(const gsys_dev_ctx& d, uint64_t n) { return __atomic_fetch_add(d.tail, n, __ATOMIC_RELAXED); }

// publish ticket t: a pread of a descriptor that is not allowed (-EBADF)
void publish(const gsys_dev_ctx& d, uint64_t t) {
  gsys_slot* s = d.ring + (t & d.ring_mask);
  s->nr = GSYS_NR_PREAD64;
  s->flags = 0;
  s->grp_n = 1;
  s->grp_off = 0;
  for (auto& a : s->args) a = 0;
  s->args[0] = 77777;
  __atomic_store_n(&s->ctl, GSYS_CTL(t, GSYS_ST_READY), __ATOMIC_RELEASE);
}

// result of ticket t once its completion record says so, else INT64_MIN
int64_t result(const gsys_dev_ctx& d, uint64_t t) {
  const gsys_comp* c = &d.comp[t & d.comp_mask];
  if (__atomic_load_n(&c->stamp, __ATOMIC_ACQUIRE) != GSYS_STAMP(t, 1)) return INT64_MIN;
  return __atomic_load_n(&c->ret, __ATOMIC_RELAXED);
}

struct Timed {
  uint64_t t0 = now_ns();
  double ms() const { return (double)(now_ns() - t0) * 1e-6; }
};

// the counter never arrives: every call ends by its own bound
void never(gsys_ctx* c, const gsys_dev_ctx& d) {
  publish(d, claim(d, 1));
  CHECK(gsys_wait(c, 1000000000) == 0);
  mode = kNever;
  Timed a;
  CHECK(gsys_wait(c, 300000000) == -ETIMEDOUT);
  CHECK(a.ms() > 250 && a.ms() < 1500);
  // and while another thread reads, which has no bound of its own
  std::thread forever([&] { CHECK(gsys_wait(c, 0) == 0); });
  sleep_ms(50);
  Timed b;
  CHECK(gsys_wait(c, 300000000) == -ETIMEDOUT);
  CHECK(b.ms() > 250 && b.ms() < 1500);
  // what the host has seen in the ring
  gsys_stats st;
  Timed e;
  CHECK(gsys_stats_get(c, &st, 0) == 0);
  CHECK(e.ms() < 4000 && st.claimed == 1 && st.requests == 1);
  mode = kStores;
  {
    std::lock_guard<std::mutex> g(late_mu);
    CHECK(!late.empty());
    store(late[0], 1);
  }
  forever.join();
  CHECK(gsys_shutdown(c, 1000000000) == 0);
}

// a store that comes after its read was given up answers no later read
void late_store(gsys_ctx* c, const gsys_dev_ctx& d) {
  mode = kNever;
  CHECK(gsys_wait(c, 150000000) == -ETIMEDOUT);
  mode = kStores;
  const uint64_t t = claim(d, 1);  // after the read that is owed: 0 tickets then
  std::thread arrives([&] {
    sleep_ms(100);
    std::lock_guard<std::mutex> g(late_mu);
    store(late[0], 0);
  });
  // one ticket is claimed and not published: the drain may not report success
  CHECK(gsys_wait(c, 400000000) == -ETIMEDOUT);
  arrives.join();
  publish(d, t);
  CHECK(gsys_wait(c, 1000000000) == 0);
  CHECK(result(d, t) == -EBADF);
  CHECK(gsys_shutdown(c, 1000000000) == 0);
}

// a launch that fails, a stream that ends without the store or fails: errors,
// not a drain that saw no tickets
void errors(gsys_ctx* c, const gsys_dev_ctx& d) {
  uint32_t id = 0;
  static uint8_t mem[4096] __attribute__((aligned(4096)));
  CHECK(gsys_register_buffer(c, (uint64_t)mem, mem, sizeof mem, GSYS_BUF_HOST, &id) == 0);
  const uint64_t t = claim(d, 1);
  for (int m : {kFails, kEndsSilently, kQueryFails}) {
    mode = m;
    CHECK(gsys_wait(c, 1000000000) == -ENODEV);
    CHECK(gsys_wait(c, 0) == -ENODEV);
    gsys_stats st;
    CHECK(gsys_stats_get(c, &st, 0) == -ENODEV);
    CHECK(gsys_unregister_buffer(c, id) == -EBUSY);
    if (m == kQueryFails) {  // those stores may still come
      std::lock_guard<std::mutex> g(late_mu);
      store(late.back(), 0);
    }
  }
  mode = kStores;
  CHECK(gsys_wait(c, 200000000) == -ETIMEDOUT);
  publish(d, t);
  CHECK(gsys_wait(c, 1000000000) == 0);
  CHECK(gsys_unregister_buffer(c, id) == 0);
  CHECK(gsys_shutdown(c, 1000000000) == 0);
}

// shutdown answers a request that waits even if the counter cannot be read
void release(gsys_ctx* c, const gsys_dev_ctx& d, Mode m, int want) {
  // earlier tickets that are never published keep the pool from the later one
  const uint64_t t = claim(d, 3000) + 2900;
  publish(d, t);
  sleep_ms(20);
  CHECK(result(d, t) == INT64_MIN);
  mode = m;
  watchdog = false;  // gsys_init synchronised
  kernel_runs = true;
  int64_t seen = INT64_MIN;
  std::thread kernel([&] {
    while (!watchdog && seen == INT64_MIN) seen = result(d, t);
    kernel_runs = false;
  });
  Timed a;
  const int rc = gsys_shutdown(c, 100000000);
  kernel.join();
  CHECK(seen == -ESHUTDOWN);
  CHECK(rc == want);
  CHECK(a.ms() < 6000);
}

}  // namespace

int main(int argc, char** argv) {
  const char* what = argc > 1 ? argv[1] : "";
  gsys_dev_ctx d;
  gsys_ctx* c = make(&d);
  if (!strcmp(what, "never")) never(c, d);
  else if (!strcmp(what, "late")) late_store(c, d);
  else if (!strcmp(what, "errors")) errors(c, d);
  else if (!strcmp(what, "release_read")) release(c, d, kStores, -ETIMEDOUT);
  else if (!strcmp(what, "release_never")) release(c, d, kNever, -ETIMEDOUT);
  else if (!strcmp(what, "release_fails")) release(c, d, kFails, -ENODEV);
  else return 2;
  printf("%s ok\n", what);
  return 0;
}
