// Runs a device function of one block on the host, one thread per lane, for bounds and race checks.
//
// Included before the device headers of the library.  It supplies what they take from the compiler's
// device mode: thread indices, the block barrier, the wave-uniform reads (the identity here), buffer
// descriptors, and empty register fences.  Memory checks come from the host's sanitizers, with every
// buffer in an allocation of its exact size.  A raw buffer load is checked against both readings of the
// range check that the scalar offset may have (left out of the check, or taken from the record count,
// which must not go below zero): a load that one of them lets through past the records is an error.
#pragma once

#include <pthread.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <limits>
#include <memory>
#include <thread>
#include <type_traits>
#include <vector>

#include <hip/hip_runtime.h>

using std::max;
using std::min;

struct HostLane {
  unsigned x;
};
inline thread_local HostLane threadIdx{0}, blockIdx{0}, gridDim{1};
inline pthread_barrier_t host_barrier;
inline void __syncthreads() { pthread_barrier_wait(&host_barrier); }

inline int host_readfirstlane(int v) { return v; }
inline void host_sched_barrier(int) {}

struct __amdgpu_buffer_rsrc_t {
  const char* base;
  int64_t records;
};
template <class T>
__amdgpu_buffer_rsrc_t host_make_buffer_rsrc(T* p, short, int records, int) {
  if (records < 0) {
    std::fprintf(stderr, "buffer descriptor of %d bytes\n", records);
    std::abort();
  }
  return {reinterpret_cast<const char*>(p), records};
}
template <class U>
U host_buffer_load(const __amdgpu_buffer_rsrc_t& r, int voff, int soff) {
  const int64_t v = uint32_t(voff), s = uint32_t(soff), n = int64_t(sizeof(U));
  const bool in = v + s + n <= r.records;
  if (s > r.records || (v + n <= r.records && !in)) {
    std::fprintf(stderr, "buffer load at offset %lld + %lld (scalar) of %lld bytes\n", (long long)v, (long long)s,
                (long long)r.records);
    std::abort();
  }
  U u = 0;
  if (in) std::memcpy(&u, r.base + v + s, sizeof(U));
  return u;
}
inline uint64_t host_buffer_load_b64(const __amdgpu_buffer_rsrc_t& r, int v, int s, int) {
  return host_buffer_load<uint64_t>(r, v, s);
}
inline uint32_t host_buffer_load_b32(const __amdgpu_buffer_rsrc_t& r, int v, int s, int) {
  return host_buffer_load<uint32_t>(r, v, s);
}

#define __builtin_amdgcn_readfirstlane host_readfirstlane
#define __builtin_amdgcn_sched_barrier host_sched_barrier
#define __builtin_amdgcn_make_buffer_rsrc host_make_buffer_rsrc
#define __builtin_amdgcn_raw_buffer_load_b64 host_buffer_load_b64
#define __builtin_amdgcn_raw_buffer_load_b32 host_buffer_load_b32

// an array in an allocation of exactly its size
template <class T>
struct Exact {
  T* p;
  size_t n;
  explicit Exact(size_t n_, T v = T(0)) : p(static_cast<T*>(std::malloc(n_ * sizeof(T)))), n(n_) {
    std::fill(p, p + n, v);
  }
  Exact(const Exact&) = delete;
  ~Exact() { std::free(p); }
};

// body(block) by every lane of `nblocks` blocks of `threads` lanes, one block after the other;
// before(block) by one lane ahead of each
inline void run_blocks(int threads, int64_t nblocks, const std::function<void(int64_t)>& before,
                       const std::function<void(int64_t)>& body) {
  pthread_barrier_init(&host_barrier, nullptr, unsigned(threads));
  std::vector<std::thread> lanes;
  for (int t = 0; t < threads; ++t)
    lanes.emplace_back([&, t] {
      threadIdx.x = unsigned(t);
      for (int64_t b = 0; b < nblocks; ++b) {
        if (t == 0) before(b);
        __syncthreads();
        body(b);
        __syncthreads();
      }
    });
  for (auto& l : lanes) l.join();
  pthread_barrier_destroy(&host_barrier);
}

// What only the device compiler understands in the headers that follow: register fences
// (`asm volatile("" : ...)`), address spaces, launch bounds, register budgets, kernel launches
#define asm
#define volatile(...)
#define __attribute__(...)
#define __launch_bounds__(...)
#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(...)
