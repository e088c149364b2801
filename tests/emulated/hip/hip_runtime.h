// A stand-in for the HIP headers that lets clang compile the library's selection sources for the CPU (test
// infrastructure, not part of libsts.so). A workgroup is one operating-system thread, its work-items
// are fibers on it; a cross-lane operation waits for the 64 lanes of its wave and a barrier for the workgroup's
// waves, as on the device, and between those points the order of the waves is the schedule's to choose. An
// ordering that the code does not enforce can so be taken on purpose: one wave of one part is held back
// until nothing else in its workgroup can go on.
#pragma once
#include <math.h>
#include <stddef.h>
#include <stdint.h>

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline __attribute__((always_inline))
#define __launch_bounds__(...)
#define __shared__ static thread_local

struct dim3 {
  unsigned x, y, z;
  dim3(unsigned x_ = 1, unsigned y_ = 1, unsigned z_ = 1) : x(x_), y(y_), z(z_) {}
};
enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1 };
enum hipDeviceAttribute_t { hipDeviceAttributeMultiprocessorCount };
typedef struct emu_stream *hipStream_t;
typedef struct emu_event *hipEvent_t;
hipError_t hipGetDevice(int *);
hipError_t hipDeviceGetAttribute(int *, hipDeviceAttribute_t, int);
inline hipError_t hipEventCreate(hipEvent_t *) { return hipErrorInvalidValue; }
inline hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return hipErrorInvalidValue; }
inline hipError_t hipEventElapsedTime(float *, hipEvent_t, hipEvent_t) { return hipErrorInvalidValue; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t) { return hipErrorInvalidValue; }
inline hipError_t hipExtLaunchKernel(const void *, dim3, dim3, void **, size_t, hipStream_t, hipEvent_t, hipEvent_t, int) { return hipErrorInvalidValue; }

namespace emu {
struct Lane {
  dim3 thread, block;
};
extern thread_local Lane *lane;                       // of the work-item that runs now
const uint32_t *exchange(uint32_t v);                 // the values of the wave's 64 lanes (0: a lane that has ended)
uint64_t live();                                      // lanes of the wave that have not ended
void barrier();
void sleep();
void launch(void (*body)(void *), void *arg, dim3 grid, dim3 block);
bool noted(const char *kernel);                       // true: the launch is noted down and not run

inline int lane_id() { return (int)(lane->thread.x & 63u); }
inline int readlane(int v, int l) { return (int)exchange((uint32_t)v)[l & 63]; }
inline int readfirstlane(int v) {
  const uint32_t *x = exchange((uint32_t)v);
  return (int)x[__builtin_ctzll(live())];
}
inline uint64_t ballot(bool p) {
  const uint32_t *x = exchange(p ? 1u : 0u);
  uint64_t m = 0;
  for (int i = 0; i < 64; ++i) m |= (uint64_t)(x[i] & 1u) << i;
  return m;
}
inline uint32_t mbcnt_lo(uint32_t mask, uint32_t base) {
  const int l = lane_id();
  return base + (uint32_t)__builtin_popcount(l >= 32 ? mask : mask & ((1u << l) - 1u));
}
inline uint32_t mbcnt_hi(uint32_t mask, uint32_t base) {
  const int l = lane_id();
  return base + (l < 32 ? 0u : (uint32_t)__builtin_popcount(mask & (uint32_t)((1ull << (l - 32)) - 1ull)));
}
// row_shl / row_shr inside a row of 16 lanes, and the broadcasts of lanes 15 and 31 into the next rows
inline int update_dpp(int old, int v, int ctrl, int row_mask, int, bool zero) {
  const uint32_t *x = exchange((uint32_t)v);
  const int l = lane_id(), row = l >> 4;
  int src = -1;
  if (ctrl > 0x100 && ctrl < 0x110) src = (l & 15) + (ctrl & 15) < 16 ? l + (ctrl & 15) : -1;
  else if (ctrl > 0x110 && ctrl < 0x120) src = (l & 15) >= (ctrl & 15) ? l - (ctrl & 15) : -1;
  else if (ctrl == 0x142) src = row > 0 ? 16 * row - 1 : -1;
  else if (ctrl == 0x143) src = row > 1 ? 31 : -1;
  else __builtin_trap();
  if (!((row_mask >> row) & 1)) return old;
  return src < 0 ? (zero ? 0 : old) : (int)x[src];
}
extern thread_local uint64_t loaded;
extern thread_local const void *recent[128];
inline void count_load(const void *p, size_t n) {
  const void *&r = recent[reinterpret_cast<uintptr_t>(p) * 0x9e3779b97f4a7c15ull >> 57];
  if (p != r) loaded += n;
  r = p;
}
template <class F>
void run(F body, dim3 grid, dim3 block) {
  launch([](void *f) { (*static_cast<F *>(f))(); }, &body, grid, block);
}
}  // namespace emu

#define threadIdx (emu::lane->thread)
#define blockIdx (emu::lane->block)
#define __syncthreads emu::barrier
#define __builtin_amdgcn_readlane emu::readlane
#define __builtin_amdgcn_readfirstlane emu::readfirstlane
#define __builtin_amdgcn_ballot_w64 emu::ballot
#define __builtin_amdgcn_mbcnt_lo emu::mbcnt_lo
#define __builtin_amdgcn_mbcnt_hi emu::mbcnt_hi
#define __builtin_amdgcn_update_dpp emu::update_dpp
#define __builtin_amdgcn_exp2f exp2f
#define __builtin_amdgcn_s_sleep(n) emu::sleep()
// the loads of scores: their bytes are counted (what was asked for just before costs no memory)
#define __builtin_nontemporal_load(p) (emu::count_load((p), sizeof(*(p))), *(p))
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, order, scope) __atomic_load_n(p, __ATOMIC_SEQ_CST)
#define __hip_atomic_store(p, v, order, scope) __atomic_store_n(p, v, __ATOMIC_SEQ_CST)

inline int __shfl_xor(int v, int off, int) { return (int)emu::exchange((uint32_t)v)[emu::lane_id() ^ off]; }
inline int __shfl_down(int v, int off, int) { return (int)emu::exchange((uint32_t)v)[emu::lane_id() + off < 64 ? emu::lane_id() + off : emu::lane_id()]; }
inline int __shfl_up(int v, int off, int) { return (int)emu::exchange((uint32_t)v)[emu::lane_id() >= off ? emu::lane_id() - off : emu::lane_id()]; }
inline int __clz(int v) { return v ? __builtin_clz((unsigned)v) : 32; }
template <class T, class V> inline T atomicAdd(T *p, V v) { return __atomic_fetch_add(p, (T)v, __ATOMIC_SEQ_CST); }
template <class T, class V> inline T atomicOr(T *p, V v) { return __atomic_fetch_or(p, (T)v, __ATOMIC_SEQ_CST); }
template <class T, class V> inline T atomicMax(T *p, V v) { return __atomic_fetch_max(p, (T)v, __ATOMIC_SEQ_CST); }
#define EMU_MINMAX(T) \
  inline T min(T a, T b) { return b < a ? b : a; } \
  inline T max(T a, T b) { return a < b ? b : a; }
EMU_MINMAX(int)
EMU_MINMAX(uint32_t)
EMU_MINMAX(long)
EMU_MINMAX(unsigned long)
EMU_MINMAX(float)
inline uint32_t min(uint32_t a, int b) { return min(a, (uint32_t)b); }
inline uint32_t min(int a, uint32_t b) { return min((uint32_t)a, b); }
inline uint32_t max(uint32_t a, int b) { return max(a, (uint32_t)b); }
inline uint32_t max(int a, uint32_t b) { return max((uint32_t)a, b); }
