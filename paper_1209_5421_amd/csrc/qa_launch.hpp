// Launches that can be recorded. The host code of a solve launches its kernels through launch(): directly, on the
// hierarchy's stream, or, while the hierarchy records, into a list of steps. The lists of several hierarchies are then
// run together, one launch per step for all the systems that are at that step (run_lists).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstddef>
#include <cstring>
#include <mutex>
#include <type_traits>
#include <vector>

namespace qa {

// A pointer read from memory is taken to point anywhere (flat loads, which occupy the LDS path as well); of a kernel's
// own arguments it is known that they point to global memory. global_pointer says so for a pointer of a recorded call,
// and the classes that kernels take hold Ptrs, which say so where they are read: made on the host, never to name LDS.
template <class X>
__host__ __device__ __forceinline__ X *global_pointer(X *p) {
#ifdef __HIP_DEVICE_COMPILE__
  // by way of an integer: the cast to the global address space and back alone is folded away
  return (X *)(__attribute__((address_space(1))) X *)reinterpret_cast<uintptr_t>(p);
#else
  return p;
#endif
}
template <class X>
struct Ptr {
  X *p;
  Ptr() = default;
  __host__ __device__ Ptr(X *q) : p(q) {}
  __host__ __device__ operator X *() const { return global_pointer(p); }
};

// arguments of one kernel call
template <class... A>
struct KArgs;
template <class H>
struct KArgs<H> {
  H head;
  template <class F, class... B>
  __device__ __forceinline__ void call(F f, const B &...b) const {
    if constexpr (std::is_pointer<H>::value) f(b..., global_pointer(head));
    else f(b..., head);
  }
};
template <class H, class... R>
struct KArgs<H, R...> {
  H head;
  KArgs<R...> rest;
  template <class F, class... B>
  __device__ __forceinline__ void call(F f, const B &...b) const {
    if constexpr (std::is_pointer<H>::value) rest.call(f, b..., global_pointer(head));
    else rest.call(f, b..., head);
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

// The calls of up to kManySystems systems. Up to many_cap of them go by value, in at most 16,000 bytes of kernel
// arguments: a workgroup then has its call's arguments after one wait. A launch for more systems names where the arguments
// lie in device memory, each hierarchy's own, written at its setup. By value alone a step of 256 systems took four
// launches or more, one behind the other and each far from filling the chip: 7.0 ms instead of 3.0 for systems of 2,601
// unknowns (FP32 preconditioner), 22.3 instead of 13.7 for 10,000 (FP64); a whole-solve workgroup each takes 3.4 and 13.9.
// By address alone 64 systems of 63,504 unknowns took 13.5 ms instead of 13.2.
// A system's one word says its grid and which of the two it is: with the choice in a word of its own a workgroup waited
// twice before its arguments (2,601 unknowns: 64 systems 1.82 instead of 1.70 ms, 128 systems 2.20 instead of 2.09).
// A call's workgroups are blockIdx.x < grid. From kAlignGrid workgroups on, the launch's grid is rounded up to a multiple
// of eight, so that workgroup b of every system runs on XCD b mod 8; smaller grids are left as they are, since the empty
// places would leave XCDs idle (rounded too, the 256 systems of 2,601, of 3 to 12 workgroups a step, took 4.2 ms).
constexpr int kManySystems = 256;
constexpr unsigned kAlignGrid = 64;
template <class P>
constexpr int many_cap() {
  return std::max<int>(1, std::min<int>(64, 16000 / static_cast<int>(sizeof(P) + 4)));
}
template <class P>
struct Many {
  static constexpr int cap = many_cap<P>();
  static constexpr size_t calls = (4 * cap + 15) / 16 * 16;  // where the calls begin, by value,
  static constexpr size_t places = 4 * kManySystems;         // or their addresses
  static constexpr unsigned by_address = 1u << 31;
  // a word for each system, its grid and by_address; then the calls or their addresses
  alignas(16) unsigned char bytes[std::max(calls + cap * sizeof(P), places + kManySystems * sizeof(const P *))];
};
template <int NT, class P>
__global__ void __launch_bounds__(NT) k_many(Many<P>) {
  // read where the arguments lie (a copy of them would be indexed in scratch memory); constant for the launch in either
  // place, so scalar loads
  using Byte = const __attribute__((address_space(4))) unsigned char;
  using Word = const __attribute__((address_space(4))) unsigned;
  using Place = const __attribute__((address_space(4))) unsigned long long;
  Byte *m = (Byte *)__builtin_amdgcn_kernarg_segment_ptr();
  const unsigned y = blockIdx.y, w = *(Word *)(m + 4 * y);
  if (blockIdx.x >= (w & ~Many<P>::by_address)) return;
  Byte *call = m + Many<P>::calls + y * sizeof(P);
  if (w & Many<P>::by_address) call = (Byte *)*(Place *)(m + Many<P>::places + 8 * y);
  ((const P *)call)->run();
}

// Recorded calls: a step's arguments lie at `at` in the list's bytes, while it is recorded, and then in its copies on
// the host and on the device.
struct LaunchList;
struct LaunchStep {
  // one launch for the steps of `count` systems, each of a list
  hipError_t (*run)(const LaunchList *const *lists, const LaunchStep *const *steps, int count, hipStream_t s);
  unsigned grid, lds;
  size_t at;
};
struct LaunchList {
  std::vector<LaunchStep> steps;
  std::vector<unsigned char> bytes;
  const unsigned char *host = nullptr, *dev = nullptr;
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
hipError_t run_many(const LaunchList *const *lists, const LaunchStep *const *steps, int count, hipStream_t s) {
  static std::once_flag once[64];
  static hipError_t err[64];
  for (int i = 0; i < count; i += kManySystems) {
    Many<P> m;
    const int k = std::min(kManySystems, count - i);
    const bool by_value = k <= Many<P>::cap;
    unsigned grid = 1, lds = 0;
    for (int j = 0; j < k; j++) {
      const LaunchStep &t = *steps[i + j];
      const unsigned word = t.grid | (by_value ? 0 : Many<P>::by_address);
      std::memcpy(m.bytes + 4 * j, &word, 4);
      if (by_value) {
        std::memcpy(m.bytes + Many<P>::calls + j * sizeof(P), lists[i + j]->host + t.at, sizeof(P));
      } else {
        const unsigned char *at = lists[i + j]->dev + t.at;
        std::memcpy(m.bytes + Many<P>::places + j * sizeof(at), &at, sizeof(at));
      }
      grid = std::max(grid, t.grid);
      lds = std::max(lds, t.lds);
    }
    if (grid >= kAlignGrid) grid = (grid + 7) / 8 * 8;
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
  list.bytes.resize((list.bytes.size() + 15) / 16 * 16);
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
// lists, steps: room for `count` pointers
inline hipError_t run_lists(ListCursor *c, const LaunchList **lists, const LaunchStep **steps, int count,
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
      lists[k] = c[i].list;
      steps[k++] = &t;
      c[i].next++;
    }
    const hipError_t e = run(lists, steps, k, s);
    if (e != hipSuccess) return e;
  }
}

}  // namespace qa
