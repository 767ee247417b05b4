// amg_solve_batch's host side on the CPU: the program defines the HIP runtime calls that the library makes (they take
// the place of the runtime's), so every launch, copy and wait of a call is seen, can be made to fail, and moves no data
// but the convergence scalars. The hierarchies hold the shapes that planning and launching read and no values.
#include <hip/hip_runtime.h>

#include <dlfcn.h>
#include <pthread.h>

#include <atomic>
#include <cerrno>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <vector>

#include "qa_internal.hpp"

namespace {

std::mutex g_mu;
std::map<hipStream_t, long> g_pending;       // launches on a stream since it was last waited for
std::vector<amg_hierarchy *> g_hs;
long g_launches = 0, g_fail_at = -1;         // the launch that fails, counted from 0 (-1: none)
hipError_t g_error = hipSuccess;             // what hipGetLastError returns next

struct Config {
  dim3 grid, block;
  size_t lds;
  hipStream_t s;
};
thread_local Config g_config;

std::atomic<bool> g_no_threads{false};
std::atomic<long> g_new{0}, g_new_fail_at{-1};  // allocations since g_new was cleared, and the one that fails

hipError_t launched(hipStream_t s) {
  std::lock_guard<std::mutex> lock(g_mu);
  if (g_launches++ == g_fail_at) return g_error = hipErrorLaunchFailure;
  g_pending[s]++;
  return hipSuccess;
}

}  // namespace

void *operator new(size_t n) {
  if (g_new++ == g_new_fail_at) throw std::bad_alloc();
  if (void *p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

extern "C" {
int pthread_create(pthread_t *t, const pthread_attr_t *a, void *(*f)(void *), void *arg) {
  using Create = int (*)(pthread_t *, const pthread_attr_t *, void *(*)(void *), void *);
  static const Create real = reinterpret_cast<Create>(dlsym(RTLD_NEXT, "pthread_create"));
  return g_no_threads ? EAGAIN : real(t, a, f, arg);
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) {
  g_config = Config{grid, block, lds, s};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *s) {
  *grid = g_config.grid, *block = g_config.block, *lds = g_config.lds, *s = g_config.s;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t s) { return launched(s); }
hipError_t hipGetLastError() {
  std::lock_guard<std::mutex> lock(g_mu);
  const hipError_t e = g_error;
  g_error = hipSuccess;
  return e;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
  std::lock_guard<std::mutex> lock(g_mu);
  g_pending[s] = 0;
  for (amg_hierarchy *h : g_hs) {  // |b| = 1, and every residual zero: converged after one iteration
    for (int i = 0; i < 9; i++) h->host_scal[i] = 0.0;
    h->host_scal[8] = 1.0;
  }
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) { return *v = 160 * 1024, hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipFuncGetAttributes(hipFuncAttributes *a, const void *) { return *a = hipFuncAttributes{}, hipSuccess; }
hipError_t hipMemPoolCreate(hipMemPool_t *p, const hipMemPoolProps *) {
  return *p = reinterpret_cast<hipMemPool_t>(1), hipSuccess;
}
hipError_t hipMemPoolSetAttribute(hipMemPool_t, hipMemPoolAttr, void *) { return hipSuccess; }
hipError_t hipMallocFromPoolAsync(void **p, size_t n, hipMemPool_t, hipStream_t) {
  return (*p = std::calloc(n, 1)) ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFreeAsync(void *p, hipStream_t) { return std::free(p), hipSuccess; }
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind, hipStream_t) {
  return std::memcpy(dst, src, n), hipSuccess;
}
hipError_t hipMemsetAsync(void *dst, int v, size_t n, hipStream_t) { return std::memset(dst, v, n), hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) {
  static double scratch[1 << 17];
  return *p = scratch, hipSuccess;
}
}

namespace {

// the caller's allocator: blocks taken on another thread than the caller's
const std::thread::id g_caller = std::this_thread::get_id();
std::atomic<long> g_blocks{0}, g_foreign{0};
void *own_alloc(size_t n, void *) {
  g_blocks++;
  if (std::this_thread::get_id() != g_caller) g_foreign++;
  return std::calloc(n, 1);
}
void own_free(void *p, void *) {
  if (std::this_thread::get_id() != g_caller) g_foreign++;
  std::free(p);
}

// a hierarchy of n unknowns on quadtree levels k = 5, 4, 3 (1,024 < n <= 4,096), FP32 preconditioner, on its own stream
amg_hierarchy *make(int64_t n, bool allocator = false) {
  amg_hierarchy *h = new amg_hierarchy;
  amg_default_options(&h->opt);
  if (allocator) h->opt.alloc = own_alloc, h->opt.dealloc = own_free;
  h->stream = reinterpret_cast<hipStream_t>(0x1000 + 16 * g_hs.size());
  h->n = h->fine.n = n;
  h->L = 5, h->kc = 3, h->nlev = 4, h->nc = 64;
  h->precision = 1;
  h->lev.resize(4);
  for (int l = 1; l < 4; l++) h->lev[l].k = 6 - l, h->lev[l].n = int64_t(1) << (2 * (6 - l));
  qa::FineLevel &F = h->fine;
  F.nnz = 7 * n;
  F.nslices = (n + 63) / 64;
  F.nwin = 16;
  for (int c = 0; c <= 4; c++) {
    F.color_row[c] = n * c / 4;
    F.color_slice[c] = F.nslices * c / 4;
    F.color_win[c] = 4 * c;
  }
  F.win_ent_max = 100;
  h->use_engine = 1;
  h->host_scal = static_cast<double *>(std::calloc(qa::kScalars, sizeof(double)));
  if (qa::alloc_workspaces(h) != AMG_OK || qa::plan_engine(h) != AMG_OK || qa::plan_wg(h) != AMG_OK) std::exit(3);
  g_hs.push_back(h);
  g_pending[h->stream] = 0;
  return h;
}

amg_status call(bool noalloc, std::vector<amg_info> &info) {
  const int m = static_cast<int>(g_hs.size());
  static double b[4096], x[4096];
  std::vector<const double *> bs(m, b);
  std::vector<double *> xs(m, x);
  std::vector<double> tol(m, 1e-8);
  info.assign(m, amg_info{});
  return (noalloc ? amg_solve_batch_noalloc : amg_solve_batch)(g_hs.data(), bs.data(), xs.data(), tol.data(), m,
                                                               info.data());
}

// a launch fails at each place of a call in turn: the call says so and leaves nothing queued
int drain(bool noalloc) {
  make(3000), make(3500), make(4000);
  std::vector<amg_info> info;
  g_launches = 0;
  if (call(noalloc, info) != AMG_OK) return 4;
  const long total = g_launches;
  long bad = 0, queued = 0;
  for (long at = 0; at < total; at++) {
    g_launches = 0, g_fail_at = at;
    const amg_status st = call(noalloc, info);
    g_fail_at = -1;
    if (st != AMG_ERR_DEVICE) bad++;
    for (const auto &p : g_pending) queued += p.second;
    g_pending.clear();
    if (call(noalloc, info) != AMG_OK) bad++;  // the next call is whole
  }
  std::printf("launches %ld bad %ld queued %ld\n", total, bad, queued);
  return 0;
}

// a whole-solve system with the caller's allocator beside one that runs in step
int allocator() {
  make(2000, true), make(3000);
  std::vector<amg_info> info;
  const long before = g_blocks;
  const amg_status st = call(false, info);
  std::printf("status %d blocks %ld foreign %ld\n", static_cast<int>(st), g_blocks - before, g_foreign.load());
  return 0;
}

// every route at once: two in-step systems, a whole-solve one, one that runs as its own amg_solve
void every_route() {
  make(3000), make(3500), make(2000);
  make(4000)->use_batch = 0;
}

// no thread can be started: the routes run one after another
int no_threads() {
  every_route();
  std::vector<amg_info> info;
  g_no_threads = true;
  const amg_status st = call(false, info);
  g_no_threads = false;
  long ok = 0;
  for (const amg_info &i : info) ok += i.status == AMG_OK;
  std::printf("status %d ok %ld\n", static_cast<int>(st), ok);
  return 0;
}

// each allocation of host memory of a call fails in turn
int no_memory(bool noalloc) {
  if (noalloc) make(3000), make(3500), make(2000);
  else every_route();
  std::vector<amg_info> info;
  if (call(noalloc, info) != AMG_OK) return 4;
  long bad = 0, queued = 0, refused = 0, at = 0;
  for (;; at++) {
    const int m = static_cast<int>(g_hs.size());
    static double b[4096], x[4096], tol[8];
    static const double *bs[8];
    static double *xs[8];
    static amg_info inf[8];
    for (int i = 0; i < m; i++) bs[i] = b, xs[i] = x, tol[i] = 1e-8;
    g_new = 0, g_new_fail_at = at;
    const amg_status st = (noalloc ? amg_solve_batch_noalloc : amg_solve_batch)(g_hs.data(), bs, xs, tol, m, inf);
    const bool reached = g_new > at;
    g_new_fail_at = -1;
    if (st != AMG_OK && st != AMG_ERR_NOMEM) bad++;
    if (st == AMG_ERR_NOMEM) refused++;
    for (const auto &p : g_pending) queued += p.second;
    g_pending.clear();
    if (call(noalloc, info) != AMG_OK) bad++;
    if (!reached) break;  // the call made fewer allocations than this
  }
  std::printf("allocations %ld bad %ld refused %ld queued %ld\n", at, bad, refused, queued);
  return 0;
}

// a system that planning would let run in step, whose iteration needs a kernel with no form for several systems (the
// general engine; the per-step path of the engine's levels): the recording is refused, nothing is launched by it, and the
// system becomes a whole-solve workgroup, one launch of a call
int refused(bool engine) {
  amg_hierarchy *h = make(3000);
  if (!h->in_step[1]) return 4;
  if (engine) h->use_engine = 0;
  else h->engine_top[1] = h->nlev;
  g_launches = 0;
  if (qa::plan_wg(h) != AMG_OK) return 5;
  const long planning = g_launches;
  std::vector<amg_info> info;
  const amg_status st = call(false, info);
  std::printf("planning %ld in_step %d status %d launches %ld\n", planning, h->in_step[1] ? 1 : 0, static_cast<int>(st),
              g_launches - planning);
  return 0;
}

// host memory that the first call without allocation takes
int heap_noalloc() {
  make(3000), make(3500), make(2000);
  static double b[4096], x[4096], tol[3] = {1e-8, 1e-8, 1e-8};
  static const double *bs[3] = {b, b, b};
  static double *xs[3] = {x, x, x};
  static amg_info info[3];
  g_new = 0;
  const amg_status st = amg_solve_batch_noalloc(g_hs.data(), bs, xs, tol, 3, info);
  std::printf("status %d allocations %ld\n", static_cast<int>(st), g_new.load());
  return 0;
}

}  // namespace

int main(int argc, char **argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  if (what == "drain") return drain(false);
  if (what == "drain-noalloc") return drain(true);
  if (what == "allocator") return allocator();
  if (what == "no-threads") return no_threads();
  if (what == "no-memory") return no_memory(false);
  if (what == "no-memory-noalloc") return no_memory(true);
  if (what == "refused-engine") return refused(true);
  if (what == "refused-top") return refused(false);
  if (what == "heap-noalloc") return heap_noalloc();
  return 2;
}
