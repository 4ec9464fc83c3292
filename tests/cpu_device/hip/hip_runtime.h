// The part of HIP that the library's sources use, on the CPU: a kernel launch runs its workgroups
// one after another, every thread a fiber, every wave of 64 in step at its cross-lane operations.
//
// Which wave runs is the schedule's choice (emu::order), at every point where a wave is free to go
// on, so a schedule can let one wave run as far ahead of the others as the barriers allow. That
// makes a missing barrier a failing test without a GPU. What is not modelled: memory latency and
// ordering (every access is done at once), caches, the rate of anything.
//
// - __shared__ variables are statics. The program is linked at a fixed address below 4 GiB, since
//   the kernels keep LDS addresses in 32-bit registers.
// - Every buffer access, and any global access made through emu::Buffers' memory, is bounds
//   checked: buffers lie between unmapped pages.
// - Within a wave, lanes run one after another between two cross-lane operations. Code that hands
//   values from lane to lane through LDS has to have one in between: a matrix instruction syncs the
//   wave before its operands are formed, the transposed LDS read before it reads.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

struct dim3 {
  unsigned x = 1, y = 1, z = 1;
  dim3(unsigned x_ = 1, unsigned y_ = 1, unsigned z_ = 1) : x(x_), y(y_), z(z_) {}
};
struct uint2 {
  unsigned x, y;
};
struct uint4 {
  unsigned x, y, z, w;
};
inline uint2 make_uint2(unsigned x, unsigned y) { return uint2{x, y}; }
using std::max;
using std::min;

// ---- host API
typedef int hipError_t;
typedef void* hipStream_t;
typedef void* hipEvent_t;
constexpr hipError_t hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorInvalidDevice = 101, hipErrorInvalidSymbol = 13;
enum { hipDeviceAttributeMultiprocessorCount, hipMemcpyDeviceToHost };

namespace emu {
inline int compute_units = 256;
inline std::vector<std::pair<const void*, unsigned>> launches;  // kernel, grid

enum State { kRunning, kWave, kBarrier, kDone };
struct Fiber {
  void* sp = nullptr;
  State state = kRunning;
  dim3 tid;
};
inline Fiber* cur = nullptr;
inline dim3 block_idx, block_dim, grid_dim;

// 0: the lowest wave that can run, 1: the highest, otherwise a pseudo-random one (the seed)
inline unsigned order = 0;

void run(const void* kernel_at, dim3 grid, dim3 block, const std::function<void()>& kernel);
void wave_sync(const char* what);  // every live lane of the wave arrives
void barrier();
void yield();                      // the wave has nothing to do until another wave has run
void assembly(const char* text);
[[noreturn]] void fail(const std::string& what);

inline int lane() { return cur->tid.x & 63; }
// One 64-bit value of each lane, exchanged. Two buffers: a lane may be at the next exchange before
// another has read this one.
uint64_t* exchange(uint64_t mine, const char* what);
template <typename T>
inline T from(const uint64_t* all, int l) {
  T v;
  std::memcpy(&v, all + l, sizeof(T));
  return v;
}
template <typename T>
inline uint64_t bits(T v) {
  static_assert(sizeof(T) <= 8, "one exchange word");
  uint64_t b = 0;
  std::memcpy(&b, &v, sizeof(T));
  return b;
}
// A matrix product's operands: up to 16 bytes a lane.
struct Operands {
  unsigned char a[64][16], b[64][16];
};
Operands* operands(const void* a, const void* b, size_t bytes, const char* what);
}  // namespace emu

inline hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
inline hipError_t hipDeviceGetAttribute(int* v, int, int) { return *v = emu::compute_units, hipSuccess; }
template <typename K>
inline hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, K, int, size_t) {
  return *n = 1, hipSuccess;
}
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
inline hipError_t hipMemcpy(void* d, const void* s, size_t n, int) { return std::memcpy(d, s, n), hipSuccess; }
#define HIP_SYMBOL(x) (&x)
template <typename T>
inline hipError_t hipGetSymbolAddress(void** p, T* symbol) {
  return *p = (void*)symbol, hipSuccess;
}
template <typename K, typename... A>
inline void emu_launch(K kernel, dim3 grid, dim3 block, A... args) {
  emu::run((const void*)kernel, grid, block, [&] { kernel(args...); });
}
#define hipLaunchKernelGGL(kernel, grid, block, shared, stream, ...) emu_launch(kernel, grid, block, __VA_ARGS__)
#define hipExtLaunchKernelGGL(kernel, grid, block, shared, stream, start, stop, flags, ...) \
  emu_launch(kernel, grid, block, __VA_ARGS__)

// ---- device language
#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static
#define __align__(n) __attribute__((aligned(n)))
#define threadIdx (emu::cur->tid)
#define blockIdx (emu::block_idx)
#define blockDim (emu::block_dim)
#define gridDim (emu::grid_dim)
#define __syncthreads() emu::barrier()
#define __HIP_MEMORY_SCOPE_WAVEFRONT 2
#define __HIP_MEMORY_SCOPE_WORKGROUP 3
#define __HIP_MEMORY_SCOPE_AGENT 4
#define __hip_atomic_load(p, ...) (*(p))
#define __hip_atomic_store(p, v, ...) (void)(*(p) = (v))
#define __hip_atomic_fetch_add(p, v, ...) emu_fetch_add(p, v)
template <typename T, typename V>
inline T emu_fetch_add(T* p, V v) {
  const T old = *p;
  *p = old + (T)v;
  return old;
}
inline unsigned atomicOr(unsigned* p, unsigned v) {
  const unsigned old = *p;
  *p = old | v;
  return old;
}

// ---- builtins
inline int __builtin_amdgcn_readfirstlane(int x) {
  const uint64_t* all = emu::exchange(emu::bits(x), "readfirstlane");
  const int v = emu::from<int>(all, 0);
  if (v != x) emu::fail("a value taken for the same in every lane is not");
  return v;
}
inline int __builtin_amdgcn_readlane(int x, int l) { return emu::from<int>(emu::exchange(emu::bits(x), "readlane"), l); }
inline uint64_t __builtin_amdgcn_ballot_w64(bool b) {
  const uint64_t* all = emu::exchange(b, "ballot");
  uint64_t m = 0;
  for (int l = 0; l < 64; ++l) m |= (all[l] & 1) << l;
  return m;
}
inline uint64_t __ballot(bool b) { return __builtin_amdgcn_ballot_w64(b); }
inline int __popcll(uint64_t x) { return __builtin_popcountll(x); }
inline int __ffsll(uint64_t x) { return __builtin_ffsll((long long)x); }
template <typename T>
inline T __shfl(T x, int l) {
  return emu::from<T>(emu::exchange(emu::bits(x), "shfl"), l & 63);
}
template <typename T>
inline T __shfl_xor(T x, int m) {
  return emu::from<T>(emu::exchange(emu::bits(x), "shfl_xor"), emu::lane() ^ m);
}
inline int __builtin_amdgcn_ds_swizzle(int x, int pattern) {  // bit-mask mode, inside 32 lanes
  const int l = emu::lane(), in = l & 31;
  const int src = ((in & (pattern & 31)) | ((pattern >> 5) & 31)) ^ ((pattern >> 10) & 31);
  return emu::from<int>(emu::exchange(emu::bits(x), "ds_swizzle"), (l & 32) | src);
}
inline int __builtin_amdgcn_ds_bpermute(int at, int x) {
  return emu::from<int>(emu::exchange(emu::bits(x), "ds_bpermute"), (at >> 2) & 63);
}
inline int __builtin_amdgcn_update_dpp(int old, int x, int ctrl, int row_mask, int, bool bound_ctrl) {
  const uint64_t* all = emu::exchange(emu::bits(x), "dpp");
  const int l = emu::lane(), row = l & 48, in = l & 15;
  int src = -1;
  if (ctrl < 0x100) src = (l & ~3) | ((ctrl >> (2 * (l & 3))) & 3);           // quad_perm
  else if (ctrl > 0x110 && ctrl < 0x120) src = in >= (ctrl & 15) ? l - (ctrl & 15) : -1;  // row_shr
  else if (ctrl == 0x140) src = row | (15 - in);                               // row_mirror
  else if (ctrl == 0x141) src = row | (in & 8) | (7 - (in & 7));               // row_half_mirror
  else if (ctrl == 0x142) src = row > 0 ? row - 1 : -1;                        // row_bcast:15
  else if (ctrl == 0x143) src = row >= 32 ? 31 : -1;                           // row_bcast:31
  else emu::fail("dpp control");
  if (!((row_mask >> (l >> 4)) & 1)) return old;
  return src >= 0 ? emu::from<int>(all, src) : (bound_ctrl ? 0 : old);
}
namespace emu {
typedef unsigned v2 __attribute__((ext_vector_type(2)));
// The odd groups of n lanes of a change places with the even ones of b.
inline v2 permlane_swap(unsigned a, unsigned b, int n) {
  const uint64_t* all = exchange(a | (uint64_t)b << 32, "permlane_swap");
  const int l = lane();
  return l & n ? v2{(unsigned)(all[l ^ n] >> 32), b} : v2{a, (unsigned)all[l ^ n]};
}
}  // namespace emu
inline emu::v2 __builtin_amdgcn_permlane16_swap(unsigned a, unsigned b, bool, bool) { return emu::permlane_swap(a, b, 16); }
inline emu::v2 __builtin_amdgcn_permlane32_swap(unsigned a, unsigned b, bool, bool) { return emu::permlane_swap(a, b, 32); }
template <typename V>
inline float __builtin_amdgcn_fdot2(V a, V b, float c, bool) { return std::fma((float)a[1], (float)b[1], std::fma((float)a[0], (float)b[0], c)); }
inline float __builtin_amdgcn_exp2f(float x) { return std::exp2(x); }
inline void __builtin_amdgcn_s_waitcnt(int) {}
inline void __builtin_amdgcn_s_sleep(int) { emu::yield(); }
inline void __builtin_amdgcn_wave_barrier() { emu::wave_sync("wave_barrier"); }
#define __builtin_amdgcn_fence(...) (void)0

struct __amdgpu_buffer_rsrc_t {
  char* base;
  uint32_t bytes;
};
inline __amdgpu_buffer_rsrc_t __builtin_amdgcn_make_buffer_rsrc(void* p, short, int bytes, int) {
  return {(char*)p, (uint32_t)bytes};
}
namespace emu {
typedef unsigned v4 __attribute__((ext_vector_type(4)));
template <typename T>
inline T load(__amdgpu_buffer_rsrc_t r, int off, int soff) {
  T v = {};
  const uint64_t at = (uint64_t)(uint32_t)off + (uint32_t)soff;
  if (at + sizeof(T) <= r.bytes) std::memcpy(&v, r.base + at, sizeof(T));
  return v;
}
template <typename T>
inline void store(T v, __amdgpu_buffer_rsrc_t r, int off, int soff) {
  const uint64_t at = (uint64_t)(uint32_t)off + (uint32_t)soff;
  if (at + sizeof(T) <= r.bytes) std::memcpy(r.base + at, &v, sizeof(T));
}
}  // namespace emu
inline unsigned __builtin_amdgcn_raw_buffer_load_b32(__amdgpu_buffer_rsrc_t r, int o, int s, int) { return emu::load<unsigned>(r, o, s); }
inline emu::v2 __builtin_amdgcn_raw_buffer_load_b64(__amdgpu_buffer_rsrc_t r, int o, int s, int) { return emu::load<emu::v2>(r, o, s); }
inline emu::v4 __builtin_amdgcn_raw_buffer_load_b128(__amdgpu_buffer_rsrc_t r, int o, int s, int) { return emu::load<emu::v4>(r, o, s); }
inline void __builtin_amdgcn_raw_buffer_store_b32(unsigned v, __amdgpu_buffer_rsrc_t r, int o, int s, int) { emu::store(v, r, o, s); }
inline void __builtin_amdgcn_raw_buffer_store_b128(emu::v4 v, __amdgpu_buffer_rsrc_t r, int o, int s, int) { emu::store(v, r, o, s); }

// Matrix products of 16 x K by K x 16: lane (grp, col) = (lane / 16, lane % 16) holds row col of the
// first and column col of the second operand at k = grp * (K / 4) + 0 .. K / 4 - 1, and rows
// 4 grp + 0 .. 3 of column col of the result. Sums are formed in order of k, in fp32.
namespace emu {
typedef float f4 __attribute__((ext_vector_type(4)));
template <typename T, int PER>
inline f4 mfma(const void* a, const void* b, f4 c) {
  const Operands* o = operands(a, b, PER * sizeof(T), "mfma");
  const int grp = lane() >> 4, col = lane() & 15;
  for (int r = 0; r < 4; ++r) {
    float s = c[r];
    for (int k = 0; k < 4 * PER; ++k) {
      T x, y;
      std::memcpy(&x, o->a[(k / PER) * 16 + 4 * grp + r] + (k % PER) * sizeof(T), sizeof(T));
      std::memcpy(&y, o->b[(k / PER) * 16 + col] + (k % PER) * sizeof(T), sizeof(T));
      s = std::fma((float)x, (float)y, s);
    }
    c[r] = s;
  }
  return c;
}
template <typename V>
inline f4 mfma_f16_k32(V a, V b, f4 c) { return mfma<_Float16, 8>(&a, &b, c); }
template <typename V>
inline f4 mfma_f16_k16(V a, V b, f4 c) { return mfma<_Float16, 4>(&a, &b, c); }
inline f4 mfma_f32_k4(float a, float b, f4 c) { return mfma<float, 1>(&a, &b, c); }
}  // namespace emu
#define __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, ...) (emu::wave_sync("mfma operands"), emu::mfma_f16_k32(a, b, c))
#define __builtin_amdgcn_mfma_f32_16x16x16f16(a, b, c, ...) (emu::wave_sync("mfma operands"), emu::mfma_f16_k16(a, b, c))
#define __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, ...) (emu::wave_sync("mfma operands"), emu::mfma_f32_k4(a, b, c))

// Transposed LDS read: inside 16 lanes, lane i receives element i % 4 of the four halves that lanes
// 4 j + i / 4 address, j = 0 .. 3.
typedef short emu_s4 __attribute__((ext_vector_type(4)));
template <typename PTR>
inline emu_s4 __builtin_amdgcn_ds_read_tr16_b64_v4i16(PTR p) {
  const uint64_t* all = emu::exchange((uint64_t)p, "ds_read_tr16");
  const int l = emu::lane(), i = l & 15;
  emu_s4 v;
  for (int j = 0; j < 4; ++j) v[j] = ((const short*)all[(l & 48) + 4 * j + i / 4])[i % 4];
  return v;
}

// Inline assembly: only what the text names matters here.
#define asm
#define volatile(...) emu::assembly(#__VA_ARGS__)
