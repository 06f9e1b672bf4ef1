// Device helpers shared by the single- and multi-column chain kernels.
#pragma once
#include "internal.hpp"

namespace polfed {

__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// Orders the LDS accesses of a wavefront around a staging step.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Wave-uniform data of one segment (see the record layout).
template <int NH>
struct SegRec {
  int row0, len, lidx, flags, n_idle_h, d_join, d_pbc;
  double dhi;
  int dh[NH > 0 ? NH : 1];
};

template <int NH>
__device__ __forceinline__ SegRec<NH> load_rec(const int32_t* rec) {
  SegRec<NH> r;
  r.row0 = uniform(rec[0]);
  r.len = uniform(rec[1]);
  r.lidx = uniform(rec[2]);
  r.flags = uniform(rec[3]);
  r.n_idle_h = uniform(rec[4]) & 255;
  r.d_join = uniform(rec[5]);
  r.d_pbc = uniform(rec[6]);
  int dw[2] = {uniform(rec[8]), uniform(rec[9])};
  __builtin_memcpy(&r.dhi, dw, sizeof(double));
#pragma unroll
  for (int b = 0; b < NH; ++b) r.dh[b] = uniform(rec[10 + b]);
  return r;
}

// Buffer accesses: a 128-bit resource for each vector, a per-lane 32-bit
// byte offset (VGPR) and a wave-uniform byte offset (SGPR), so gathers at
// uniform row offsets need no per-lane address arithmetic.  Accesses beyond
// the resource's size return 0 / are dropped by the hardware.
using rsrc_t = __amdgpu_buffer_rsrc_t;
constexpr int kAuxNT = 2;  // non-temporal cache policy

__device__ __forceinline__ rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes,
                                           0x00020000);
}
template <typename T, int AUX = 0>
__device__ __forceinline__ T bload(rsrc_t r, uint32_t vo, uint32_t so) {
  if constexpr (sizeof(T) == 8)
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, vo, so, AUX));
  else
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, vo, so, AUX));
}
// Two consecutive elements in one 16-byte access (8-byte alignment suffices
// for buffer accesses).
template <typename T, int AUX = 0>
__device__ __forceinline__ void bload2(rsrc_t r, uint32_t vo, uint32_t so, T& x0, T& x1) {
  if constexpr (sizeof(T) == 8) {
    using d2 = __attribute__((ext_vector_type(2))) double;
    const d2 d = __builtin_bit_cast(d2, __builtin_amdgcn_raw_buffer_load_b128(r, vo, so, AUX));
    x0 = d[0];
    x1 = d[1];
  } else {
    using f2 = __attribute__((ext_vector_type(2))) float;
    const f2 d = __builtin_bit_cast(f2, __builtin_amdgcn_raw_buffer_load_b64(r, vo, so, AUX));
    x0 = d[0];
    x1 = d[1];
  }
}
// R consecutive elements, R = 1 or 2.
template <typename T, int R, int AUX = 0>
__device__ __forceinline__ void bload_rows(rsrc_t r, uint32_t vo, uint32_t so, T* x) {
  if constexpr (R == 2)
    bload2<T, AUX>(r, vo, so, x[0], x[1]);
  else
    x[0] = bload<T, AUX>(r, vo, so);
}
// R consecutive elements of a vector that is read once a launch, without a
// place in the caches if nt.
template <typename T, int R = 1>
__device__ __forceinline__ void bload_stream(rsrc_t r, uint32_t vo, uint32_t so, bool nt, T* x) {
  if (nt) {
    asm volatile("");  // two loads, not one with a policy chosen by select
    bload_rows<T, R, kAuxNT>(r, vo, so, x);
  } else {
    bload_rows<T, R>(r, vo, so, x);
  }
}
// Whether the vectors that a chain step streams (v and b_{i+2}, n elements in
// all the columns) are read past the caches.  While v, b_{i+1} and b_{i+2} are
// a few MB they compete with the gathered b_{i+1} for the L2s, and reading
// them past the caches is faster; beyond that it also denies them the 256 MB
// memory-side cache, which would hold them from step to step.  Measured, past
// the caches / through them, us a step of the best kernel: FP64 L = 20 (4.4 MB)
// 5.97 / 6.22, L = 21 (8.5 MB) 8.10 / 8.57, FP32 L = 22 (8.5 MB) 8.4 / 9.2,
// open FP32 L = 23, 10 up (13.7 MB) 10.5 / 11.1; FP32 L = 23, 11 up (16.2 MB)
// 12.5 / 11.3, FP64 L = 22 (16.9 MB) 10.5 / 9.7, L = 24 (65 MB) 29.5 / 26.7,
// L = 26 (250 MB) 113 / 102.
template <typename T>
__device__ __forceinline__ bool stream_nt(int64_t n) {
  return n * (int64_t)(3 * sizeof(T)) <= 15 * 1000 * 1000;
}
template <int AUX, typename T>
__device__ __forceinline__ void bstore2(T x0, T x1, rsrc_t r, uint32_t vo, uint32_t so) {
  if constexpr (sizeof(T) == 8) {
    using u4 = __attribute__((ext_vector_type(4))) unsigned int;
    using d2 = __attribute__((ext_vector_type(2))) double;
    const d2 d = {x0, x1};
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, d), r, vo, so, AUX);
  } else {
    using u2 = __attribute__((ext_vector_type(2))) unsigned int;
    using f2 = __attribute__((ext_vector_type(2))) float;
    const f2 d = {x0, x1};
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, d), r, vo, so, AUX);
  }
}
template <int AUX, typename T>
__device__ __forceinline__ void bstore(T x, rsrc_t r, uint32_t vo, uint32_t so) {
  using u2 = __attribute__((ext_vector_type(2))) unsigned int;
  if constexpr (sizeof(T) == 8)
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, x), r, vo, so, AUX);
  else
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, x), r, vo, so, AUX);
}
template <typename T, int R, int AUX>
__device__ __forceinline__ void bstore_rows(const T* x, rsrc_t r, uint32_t vo, uint32_t so) {
  if constexpr (R == 2)
    bstore2<AUX>(x[0], x[1], r, vo, so);
  else
    bstore<AUX>(x[0], r, vo, so);
}

// The element at a byte offset of the LDS image.
template <typename T>
__device__ __forceinline__ T lds_at(const unsigned char* smem, uint32_t off) {
  return *reinterpret_cast<const T*>(smem + off);
}

}  // namespace polfed
