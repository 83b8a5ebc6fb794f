// A wavefront on the CPU, for tests of the integration kernels' control flow:
// 64 lanes as coroutines, each wave operation (ballot, first lane, lane moves)
// a point that all lanes reach before any goes on.  The kernels' own source is
// compiled against this header in place of the HIP one; what they do not use
// outside kernels that synchronise a workgroup is not here.
#pragma once
#include <ucontext.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <functional>

#define __global__
#define __device__
#define __host__
#define __shared__ static
#define __launch_bounds__(...)
#define hipLaunchKernelGGL(...) ((void)0)

struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
using hipStream_t = void*;
using hipError_t = int;
enum { hipSuccess = 0, hipMemcpyHostToDevice, hipDeviceAttributeMultiprocessorCount };
inline const char* hipGetErrorString(hipError_t) { return ""; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipGetDevice(int* d) { return *d = 0; }
inline hipError_t hipDeviceGetAttribute(int* v, int, int) { return *v = 256, hipSuccess; }
inline hipError_t hipMemcpyAsync(void*, const void*, size_t, int, hipStream_t) { return hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }

namespace wave {
struct Lane {
  ucontext_t ctx;
  char* stack = nullptr;
  bool done = false;
};
inline Lane lanes[64];
inline ucontext_t back;
inline int cur;                        // the lane that runs
inline unsigned long long slot[64];    // the lanes' values of a wave operation
inline const std::function<void()>* body;
inline dim3 block_idx, block_dim, grid_dim;

inline void yield() { swapcontext(&lanes[cur].ctx, &back); }
inline void entry() {
  (*body)();
  lanes[cur].done = true;
  for (;;) yield();
}
// every lane's value, once all have given theirs
inline void exchange(unsigned long long v, unsigned long long out[64]) {
  slot[cur] = v;
  yield();
  std::memcpy(out, slot, sizeof(slot));
  yield();
}
// Runs f on 64 lanes; false if they have not ended after `limit` wave operations.
inline bool run(const std::function<void()>& f, long long limit) {
  constexpr size_t STACK = 256 << 10;
  body = &f;
  for (Lane& l : lanes) {
    if (!l.stack) l.stack = static_cast<char*>(std::malloc(STACK));
    getcontext(&l.ctx);
    l.ctx.uc_stack.ss_sp = l.stack;
    l.ctx.uc_stack.ss_size = STACK;
    l.ctx.uc_link = nullptr;
    l.done = false;
    makecontext(&l.ctx, entry, 0);
  }
  for (long long op = 0; op < 2 * limit; ++op) {
    int ended = 0;
    for (cur = 0; cur < 64; ++cur) {
      swapcontext(&back, &lanes[cur].ctx);
      ended += lanes[cur].done;
    }
    if (ended == 64) return true;
    if (ended) std::abort();  // lanes part at a wave operation
  }
  return false;
}
}  // namespace wave

struct ThreadIdx {
  struct {
    operator unsigned() const { return static_cast<unsigned>(wave::cur); }
  } x;
};
inline ThreadIdx threadIdx;
#define blockIdx wave::block_idx
#define blockDim wave::block_dim
#define gridDim wave::grid_dim

inline unsigned long long __builtin_amdgcn_ballot_w64(bool b) {
  unsigned long long o[64], r = 0;
  wave::exchange(b, o);
  for (int l = 0; l < 64; ++l) r |= o[l] << l;
  return r;
}
inline bool __builtin_amdgcn_inverse_ballot_w64(unsigned long long m) { return m >> wave::cur & 1; }
inline void __builtin_amdgcn_wave_barrier() {}
inline void __builtin_amdgcn_sched_barrier(int) {}
inline int __any(bool b) { return __builtin_amdgcn_ballot_w64(b) != 0; }
inline int __all(bool b) { return __builtin_amdgcn_ballot_w64(b) == ~0ull; }
inline int __builtin_amdgcn_readlane(int x, int l) {
  unsigned long long o[64];
  wave::exchange(static_cast<unsigned>(x), o);
  return static_cast<int>(o[l]);
}
inline int __builtin_amdgcn_readfirstlane(int x) { return __builtin_amdgcn_readlane(x, 0); }
// the lane moves in use: row_shr, row_bcast:15, row_bcast:31, the identity
inline int __builtin_amdgcn_update_dpp(int old, int src, int ctrl, int rows, int, bool) {
  unsigned long long o[64];
  wave::exchange(static_cast<unsigned>(src), o);
  const int l = wave::cur, row = l / 16;
  if (!(rows >> row & 1)) return old;
  if (ctrl == 0xe4) return src;
  if (ctrl == 0x142) return row ? static_cast<int>(o[16 * row - 1]) : old;
  if (ctrl == 0x143) return row >= 2 ? static_cast<int>(o[31]) : old;
  if (ctrl <= 0x110 || ctrl > 0x11f) std::abort();
  return l % 16 >= ctrl - 0x110 ? static_cast<int>(o[l - (ctrl - 0x110)]) : old;
}
// (named in kernels that synchronise a workgroup, which are not run here)
template <class T>
T __shfl_up(T, int) {
  std::abort();
}
template <class T>
T __shfl(T, int) {
  std::abort();
}
inline unsigned long long __ballot(bool b) { return __builtin_amdgcn_ballot_w64(b); }
inline int __popcll(unsigned long long x) { return __builtin_popcountll(x); }
inline int __ffsll(long long x) { return __builtin_ffsll(x); }
inline void __syncthreads() { std::abort(); }
template <class T, class U>
T atomicAdd(T* p, U v) {
  const T o = *p;
  *p += v;
  return o;
}
inline long long __double_as_longlong(double d) {
  long long r;
  std::memcpy(&r, &d, sizeof(r));
  return r;
}
inline double __longlong_as_double(long long b) {
  double r;
  std::memcpy(&r, &b, sizeof(r));
  return r;
}
inline float __builtin_amdgcn_cosf(float x) { return cosf(6.2831853f * x); }
inline float __builtin_amdgcn_sinf(float x) { return sinf(6.2831853f * x); }
inline float __builtin_amdgcn_logf(float x) { return log2f(x); }
inline float __builtin_amdgcn_sqrtf(float x) { return sqrtf(x); }
using std::max;
using std::min;
