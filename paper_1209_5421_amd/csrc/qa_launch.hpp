// Launches that can be recorded. The host code of a solve launches its kernels through launch(): directly, on the
// hierarchy's stream, or, while the hierarchy records, into a list of steps. The lists of several hierarchies are then
// run together, one launch per step for all the systems that are at that step (run_lists).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>
#include <type_traits>
#include <vector>

namespace qa {

// arguments of one kernel call
template <class... A>
struct KArgs;
template <class H>
struct KArgs<H> {
  H head;
  template <class F, class... B>
  __device__ __forceinline__ void call(F f, const B &...b) const {
    f(b..., head);
  }
};
template <class H, class... R>
struct KArgs<H, R...> {
  H head;
  KArgs<R...> rest;
  template <class F, class... B>
  __device__ __forceinline__ void call(F f, const B &...b) const {
    rest.call(f, b..., head);
  }
};
template <class H>
KArgs<H> kargs(H h) {
  return KArgs<H>{h};
}
template <class H, class R1, class... R>
KArgs<H, R1, R...> kargs(H h, R1 r1, R... r) {
  return KArgs<H, R1, R...>{h, kargs(r1, r...)};
}

// a call: the kernel's body and its arguments
template <class F, class... A>
struct KCall {
  F body;
  KArgs<A...> args;
  __device__ __forceinline__ void run() const { args.call(body); }
};

// The calls of up to many_cap systems, passed by value: at most 16,000 bytes of kernel arguments, and no device memory
// for them. (With at most 4,000, 64 systems of 3,844 unknowns took 6.2 ms for the 2.6 that they take so, and 64 of
// 63,504 took 16.7 for 13.1; 32,000 gave no more.) A call's workgroups are blockIdx.x < grid; a launch takes the largest grid, rounded up to a multiple of
// eight so that workgroup b of every system runs on XCD b mod 8.
template <class P>
constexpr int many_cap() {
  return std::max<int>(1, std::min<int>(64, 16000 / static_cast<int>(sizeof(P) + 4)));
}
template <class P>
struct Many {
  P call[many_cap<P>()];
  unsigned grid[many_cap<P>()];
};
template <int NT, class P>
__global__ void __launch_bounds__(NT) k_many(Many<P> m) {
  if (blockIdx.x >= m.grid[blockIdx.y]) return;
  m.call[blockIdx.y].run();
}

// Recorded calls: a step's arguments lie at `at` in the list's bytes.
struct LaunchStep {
  // one launch for the steps of `count` systems, given their arguments, grids and LDS
  hipError_t (*run)(const unsigned char *const *args, const LaunchStep *const *steps, int count, hipStream_t s);
  unsigned grid, lds;
  size_t at;
};
struct LaunchList {
  std::vector<LaunchStep> steps;
  std::vector<unsigned char> bytes;
  bool refused = false;  // it met a kernel that cannot be recorded
  void clear() { steps.clear(), bytes.clear(), refused = false; }
};

// dynamic LDS beyond the default limit has to be asked for, once per device: all that the kernel's static arrays leave
inline hipError_t lds_limit(const void *kernel, std::once_flag *once, hipError_t *err) {
  int dev = 0;
  const hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  std::call_once(once[dev], [&]() {
    int lds = 0;
    hipFuncAttributes at{};
    err[dev] = hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
    if (err[dev] == hipSuccess) err[dev] = hipFuncGetAttributes(&at, kernel);
    if (err[dev] == hipSuccess)
      err[dev] = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     lds - static_cast<int>(at.sharedSizeBytes));
  });
  return err[dev];
}

template <int NT, class P>
hipError_t run_many(const unsigned char *const *args, const LaunchStep *const *steps, int count, hipStream_t s) {
  constexpr int cap = many_cap<P>();
  static std::once_flag once[64];
  static hipError_t err[64];
  for (int i = 0; i < count; i += cap) {
    alignas(Many<P>) unsigned char buf[sizeof(Many<P>)];  // a body has no default constructor
    Many<P> &m = *reinterpret_cast<Many<P> *>(buf);
    const int k = std::min(cap, count - i);
    unsigned grid = 1, lds = 0;
    for (int j = 0; j < cap; j++) {  // places past the last system: no workgroup runs them
      const int l = i + std::min(j, k - 1);
      std::memcpy(static_cast<void *>(&m.call[j]), args[l], sizeof(P));
      m.grid[j] = j < k ? steps[l]->grid : 0;
      grid = std::max(grid, m.grid[j]);
      lds = std::max(lds, steps[l]->lds);
    }
    if (grid > 1) grid = (grid + 7) / 8 * 8;
    if (lds > 48 * 1024) {
      const hipError_t e = lds_limit(reinterpret_cast<const void *>(k_many<NT, P>), once, err);
      if (e != hipSuccess) return e;
    }
    k_many<NT, P><<<dim3(grid, static_cast<unsigned>(k)), NT, lds, s>>>(m);
  }
  return hipGetLastError();
}

template <int NT, class F, class... A>
void record(LaunchList &list, F body, unsigned grid, size_t lds, A... a) {
  using P = KCall<F, A...>;
  static_assert(std::is_trivially_copyable<P>::value, "arguments are copied as bytes");
  const P p{body, kargs(a...)};
  list.steps.push_back(LaunchStep{run_many<NT, P>, grid, static_cast<unsigned>(lds), list.bytes.size()});
  const unsigned char *b = reinterpret_cast<const unsigned char *>(&p);
  list.bytes.insert(list.bytes.end(), b, b + sizeof(P));
}

// Launch kernel K<TA> of NT threads for hierarchy h, or record the call of its body K_body<TA>. TA: QA_T(...) or empty.
// QA_ONCE launches a kernel that no recorded list needs (it has no form for several systems): a list that meets one is
// refused, so that nothing runs ahead of the list's own steps. QA_RUN_IF takes the one or the other by a constant.
#define QA_T(...) <__VA_ARGS__>
#define QA_RUN_IF(COND, h, NT, GRID, LDS, K, TA, ...)                                                           \
  ::qa::launch<NT, (COND)>(h, K TA, [] __device__(const auto &...a) { K##_body TA(a...); }, GRID, LDS, __VA_ARGS__)
#define QA_RUN(h, NT, GRID, LDS, K, TA, ...)                                                                  \
  ::qa::launch<NT, true>(h, K TA, [] __device__(const auto &...a) { K##_body TA(a...); }, GRID, LDS, __VA_ARGS__)
#define QA_ONCE(h, NT, GRID, LDS, K, TA, ...) ::qa::launch_once<NT>(h, K TA, GRID, LDS, __VA_ARGS__)
template <class H>
bool refuse_recording(H *h) {
  if (h->recording) h->recording->refused = true;
  return h->recording != nullptr;
}
template <int NT, class H, class K, class... A>
void launch_once(H *h, K kern, unsigned grid, size_t lds, A... a) {
  if (!refuse_recording(h)) kern<<<grid, NT, lds, h->stream>>>(a...);
}
template <int NT, bool SHARED, class H, class K, class F, class... A>
void launch(H *h, K kern, F body, unsigned grid, size_t lds, A... a) {
  if constexpr (SHARED)
    if (h->recording) return record<NT>(*h->recording, body, grid, lds, a...);
  launch_once<NT>(h, kern, grid, lds, a...);
}

// Run count lists on one stream, each in its own order. The system with the most steps left names the next kernel, and
// every system whose next step is that kernel joins the launch: systems of one depth go in step, and a shallower one
// waits where its deeper neighbour has more levels and joins it again below them. What a system computes does not
// depend on who joins.
struct ListCursor {
  const LaunchList *list;
  size_t next;
  size_t left() const { return list->steps.size() - next; }
};
// args, steps: room for `count` pointers
inline hipError_t run_lists(ListCursor *c, const unsigned char **args, const LaunchStep **steps, int count,
                            hipStream_t s) {
  for (;;) {
    int lead = 0;
    for (int i = 1; i < count; i++)
      if (c[i].left() > c[lead].left()) lead = i;
    if (count == 0 || c[lead].left() == 0) return hipSuccess;
    const auto run = c[lead].list->steps[c[lead].next].run;
    int k = 0;
    for (int i = 0; i < count; i++) {
      if (c[i].left() == 0) continue;
      const LaunchStep &t = c[i].list->steps[c[i].next];
      if (t.run != run) continue;
      args[k] = c[i].list->bytes.data() + t.at;
      steps[k++] = &t;
      c[i].next++;
    }
    const hipError_t e = run(args, steps, k, s);
    if (e != hipSuccess) return e;
  }
}

}  // namespace qa
