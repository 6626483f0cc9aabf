// Stand-in for the HIP runtime header in the host build of ff_relax.h: the
// device functions become host functions, a wavefront's cross-lane operations,
// memory operations and clock go to the simulator (relax_host.cpp).
#pragma once
#include <stdint.h>
#include "hip_runtime_api.h"

#define __host__
#define __device__
#define __forceinline__ inline
#define address_space(n)

namespace sim {
struct Idx {
  unsigned x;
};
Idx thread_idx();
uint64_t collective(uint64_t v, int lane);   // the value of `lane` (-1: a bit per lane with a non-zero value)
void memory();                               // a memory operation: the other workgroups may run before it
void sleep(int n);
uint64_t clock();
template <class T>
T load(T* p) {
  memory();
  return *p;
}
template <class T>
void store(T* p, T v) {
  memory();
  *p = v;
}
template <class T>
T add(T* p, T v) {
  memory();
  const T old = *p;
  *p = old + v;
  return old;
}
template <class T>
T exchange(T* p, T v) {
  memory();
  const T old = *p;
  *p = v;
  return old;
}
template <class T>
bool compare_exchange(T* p, T* want, T v) {
  memory();
  if (*p == *want) {
    *p = v;
    return true;
  }
  *want = *p;
  return false;
}
}  // namespace sim

#define threadIdx sim::thread_idx()
#define __hip_atomic_load(p, order, scope) sim::load(p)
#define __hip_atomic_store(p, v, order, scope) sim::store(p, v)
#define __hip_atomic_fetch_add(p, v, order, scope) sim::add(p, v)
#define __hip_atomic_exchange(p, v, order, scope) sim::exchange(p, v)
#define __hip_atomic_compare_exchange_strong(p, want, v, o1, o2, scope) sim::compare_exchange(p, want, v)
#define __HIP_MEMORY_SCOPE_AGENT 0

inline int __builtin_amdgcn_readfirstlane(int v) { return (int)sim::collective((uint64_t)(uint32_t)v, 0); }
inline int __builtin_amdgcn_readlane(int v, int lane) { return (int)sim::collective((uint64_t)(uint32_t)v, lane); }
inline uint64_t __ballot(int p) { return sim::collective(p != 0, -1); }
inline int __popcll(uint64_t v) { return __builtin_popcountll(v); }
inline int __ffsll(unsigned long long v) { return __builtin_ffsll((long long)v); }
inline void __builtin_amdgcn_s_waitcnt(int) {}   // a memory operation here is complete when it returns
inline void __builtin_amdgcn_s_sleep(int n) { sim::sleep(n); }
inline uint64_t __builtin_amdgcn_s_memrealtime() { return sim::clock(); }
