// Internal helpers shared by the pvlm HIP sources (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>
#include <cstddef>

#include "layout.h"
#include "pvlm.h"

namespace pvlm {

// ------------------------------------------------------------------ host --
void set_hip_error(hipError_t e);
pvlm_status hip_check(hipError_t e);
#define PVLM_HIP(call)                               \
  do {                                               \
    hipError_t e_ = (call);                          \
    if (e_ != hipSuccess) return ::pvlm::hip_check(e_); \
  } while (0)
#define PVLM_LAUNCHED()                                        \
  do {                                                         \
    hipError_t e_ = hipGetLastError();                         \
    if (e_ != hipSuccess) return ::pvlm::hip_check(e_);        \
  } while (0)

// Compute-unit and XCD counts of the current device (queried once per
// device); with a stream, its compute-unit budget when it has one.
pvlm_status device_info(DeviceInfo* out);
pvlm_status device_info(DeviceInfo* out, hipStream_t stream);

// Raise a kernel's dynamic-LDS limit to `bytes` (done once per kernel and size).
hipError_t allow_dynamic_lds(const void* kernel, int bytes);

// PVLM_OK when `grid` workgroups of `kernel` (with `block` threads and `lds`
// dynamic LDS bytes) fit on the current device at once: the occupancy the
// runtime reports per compute unit, but at most `per_cu_most` (the runtime does
// not count registers that a waves-per-SIMD bound reserves beyond those used),
// times the compute units (the stream's budget when it has one).  A launch
// whose workgroups wait on each other (verify under stream capture) checks this
// before launching; that they do start together then rests on the caller's
// contract: the device not shared, or the budgets of overlapping streams within
// its compute units.
pvlm_status check_coresident(const void* kernel, int grid, int block, int lds, int per_cu_most,
                             hipStream_t stream);

// ---------------------------------------------------------------- device --
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf16_to_f32(uint16_t b) {
  return __uint_as_float(static_cast<uint32_t>(b) << 16);
}
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  __bf16 h = static_cast<__bf16>(f);
  return __builtin_bit_cast(uint16_t, h);
}

__device__ __forceinline__ void dev_flag(int32_t* status, int bit) {
  if (status) __hip_atomic_fetch_or(status, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Coherent (agent-scope) load and store of a pair that workgroups of one launch
// exchange, which may sit on different XCDs.  Each XCD has its own L2; a plain
// load can hit a stale line in the reader's L2 even after an acquire, so every
// read of another workgroup's data goes through these (they are independent
// loads and pipeline when issued back to back).
__device__ __forceinline__ void st_agent(float2* p, float2 v) {
  __hip_atomic_store(reinterpret_cast<uint64_t*>(p), __builtin_bit_cast(uint64_t, v),
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 ld_agent(const float2* p) {
  const uint64_t u = __hip_atomic_load(reinterpret_cast<const uint64_t*>(p), __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
  return __builtin_bit_cast(float2, u);
}

// Upper bound on polls of an inter-workgroup wait (each poll sleeps ~64
// clocks); a wait that exceeds it flags PVLM_DEV_TIMEOUT and gives up, so every
// wave always exits.
constexpr int kSpinLimit = 1 << 20;

// Workgroup barrier that orders LDS only: global loads and stores stay in
// flight across it (a full __syncthreads waits for every outstanding memory
// operation of the wave first).
__device__ __forceinline__ void lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ __forceinline__ uint64_t pack_bf16x4(float x, float y, float z, float w) {
  return (uint64_t)f32_to_bf16(x) | ((uint64_t)f32_to_bf16(y) << 16) | ((uint64_t)f32_to_bf16(z) << 32) |
         ((uint64_t)f32_to_bf16(w) << 48);
}

// The cache rows of one (batch, KV head): contiguous (base = the head's row
// 0, rows of D elements), or paged: pages of 2^shift rows (a multiple of the
// 32-row block) in a pool [n_pages][Hkv][2^shift][D]; base = the pool plus
// the head's offset inside a page, page_elems = elements of one page (all
// heads), table = the sequence's page-table row (logical page -> pool page).
// A kernel may stage the entries it will use in LDS (staged, from logical
// page page0), which takes the table load off each block's address path.
struct KvRows {
  const uint16_t* base;
  const int32_t* table;  // read only when paged
  const int32_t* staged; // LDS copy of the entries from logical page page0 (used when in_lds)
  int64_t page_elems;
  int64_t n_pages;
  int shift, page0;
  bool paged, in_lds;
};

// LDS byte address of a generic pointer into LDS: the shared aperture starts
// at a multiple of 2^32, so the address is the pointer's low 32 bits.
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>(p));
}

// log2 of a page size that is a power of two in [32, 2^20], else -1.
inline int page_shift_of(int page_size) {
  if (page_size < 32 || page_size > (1 << 20) || (page_size & (page_size - 1))) return -1;
  int s = 0;
  while ((1 << s) < page_size) ++s;
  return s;
}

// The address of row te, where te is the 32-row block start tb, or for a
// block past the chunk end c1 the start of the block holding row c1 - 1;
// rows te .. te + 31 are contiguous from it.  A page-table entry outside the
// pool is clamped into it (the kernel flags it separately).
template <int D>
__device__ __forceinline__ const uint16_t* kv_block(const KvRows& kv, int tb, int c1, int& te) {
  te = tb < c1 ? tb : ((c1 - 1) & ~31);
  if (!kv.paged) return kv.base + (size_t)te * D;
  int page;
  if (kv.in_lds) {
    page = kv.staged[(te >> kv.shift) - kv.page0];  // already clamped
  } else {
    page = kv.table[te >> kv.shift];
    page = page < 0 ? 0 : (page >= kv.n_pages ? (int)(kv.n_pages - 1) : page);
  }
  return kv.base + (size_t)page * kv.page_elems + (size_t)(te & ((1 << kv.shift) - 1)) * D;
}

// Cross-lane exchanges that stay in the VALU (no LDS crossbar round trip):
// DPP row operations and the gfx950 permlane swaps.
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf,
                                                               0xf, false));
}
__device__ __forceinline__ float lane_xor1(float x) { return dpp_mov<0xB1>(x); }   // quad_perm 1,0,3,2
__device__ __forceinline__ float lane_xor2(float x) { return dpp_mov<0x4E>(x); }   // quad_perm 2,3,0,1
__device__ __forceinline__ float lane_xor8(float x) { return dpp_mov<0x128>(x); }  // row_ror:8
// lane i of every 8 receives lane 7 - i (row_half_mirror): partners differ in bit 2
__device__ __forceinline__ float lane_mirror8(float x) { return dpp_mov<0x141>(x); }
// Sum / max over the four lanes l, l^16, l^32, l^48 (every lane gets the result).
__device__ __forceinline__ float rows4_sum(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float y = __uint_as_float(a[0]) + __uint_as_float(a[1]);  // lower row + upper row
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);            // lower half + upper half
}
__device__ __forceinline__ float rows4_max(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  const float y = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(y), __float_as_uint(y), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
// The value of lane l ^ 16 and of lane l ^ 32.
__device__ __forceinline__ float lane_xor16(float x) {
  const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float((threadIdx.x & 16) ? a[0] : a[1]);
}
__device__ __forceinline__ float lane_xor32(float x) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float((threadIdx.x & 32) ? a[0] : a[1]);
}

__device__ __forceinline__ float warp_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
__device__ __forceinline__ float warp_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ double warp_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

}  // namespace pvlm
