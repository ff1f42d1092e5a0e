// Operand types of the convolution kernels (BF16 and OCP e4m3): packing,
// LDS and buffer reads, matrix instruction, stores of a lane's channels.
#pragma once
#include "bcts_internal.h"

namespace bcts {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(8))) int v8i;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

__device__ __forceinline__ unsigned bf2_pack(float a, float b) {
  const bf16x2 h = __builtin_convertvector(f32x2{a, b}, bf16x2);   // v_cvt_pk_bf16_f32 (RNE)
  return *reinterpret_cast<const unsigned*>(&h);
}
__device__ __forceinline__ unsigned fp8_pack4(float a, float b, float c, float d) {
  a = fminf(fmaxf(a, -448.f), 448.f);
  b = fminf(fmaxf(b, -448.f), 448.f);
  c = fminf(fmaxf(c, -448.f), 448.f);
  d = fminf(fmaxf(d, -448.f), 448.f);
  const int lo = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, 0, false);
  return (unsigned)__builtin_amdgcn_cvt_pk_fp8_f32(c, d, lo, true);
}

// Workgroup barrier for LDS hand-offs only.  __syncthreads() also waits for
// every outstanding global load (its workgroup fence drains vmcnt), which
// would cancel the frame and weight prefetches at each barrier; here only
// the LDS queue is drained before s_barrier, global loads stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __asm__ volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Keep global prefetch loads where they are issued: the scheduler may move
// ALU, MFMA and LDS instructions across this point, but no global read, so a
// prefetch is not sunk next to its first use.
__device__ __forceinline__ void pin_vmem_reads() { __builtin_amdgcn_sched_barrier(0x78F); }

// ---- operand traits ------------------------------------------------------
// EB: bytes per element; UB: bytes per 8-element unit (one lane's K group).
template <int P> struct Operand;
template <> struct Operand<P_BF16> {
  typedef uint16_t E;
  typedef bf16x8 V;
  static constexpr int EB = 2, UB = 16;
  __device__ static V ld(const void* p) { return *reinterpret_cast<const V*>(p); }
  // 8 pixels starting at a 4-byte-aligned LDS address (two 8-byte reads)
  __device__ static V ld_pix(const unsigned char* p) {
    uint4 u;
    const uint2 a = *reinterpret_cast<const uint2*>(p);
    const uint2 b = *reinterpret_cast<const uint2*>(p + 8);
    u.x = a.x; u.y = a.y; u.z = b.x; u.w = b.y;
    return *reinterpret_cast<const V*>(&u);
  }
  __device__ static f32x4 mma(V a, V b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
  // one lane's weight operand through a buffer resource: byte offset voff + soff
  __device__ static V ldw(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
    return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
  }
  // 16 raw pixels -> 16 operands in LDS (32 bytes)
  __device__ static void stage16(unsigned char* dst, uint4 raw, float) {
    const unsigned w[4] = {raw.x, raw.y, raw.z, raw.w};
    uint4 o0, o1;
    unsigned o[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[2 * i] = bf2_pack((float)(w[i] & 255u), (float)((w[i] >> 8) & 255u));
      o[2 * i + 1] = bf2_pack((float)((w[i] >> 16) & 255u), (float)(w[i] >> 24));
    }
    o0 = make_uint4(o[0], o[1], o[2], o[3]);
    o1 = make_uint4(o[4], o[5], o[6], o[7]);
    *reinterpret_cast<uint4*>(dst) = o0;
    *reinterpret_cast<uint4*>(dst + 16) = o1;
  }
  // 4 consecutive channels -> 8 bytes
  __device__ static void st4(void* p, float a, float b, float c, float d, float) {
    *reinterpret_cast<uint2*>(p) = make_uint2(bf2_pack(a, b), bf2_pack(c, d));
  }
  // 8 consecutive channels as two packed halves of 4 -> 16 bytes
  typedef uint2 PK;
  __device__ static PK pk4(float a, float b, float c, float d, float) {
    return make_uint2(bf2_pack(a, b), bf2_pack(c, d));
  }
  __device__ static void st8(void* p, PK lo, PK hi) {
    *reinterpret_cast<uint4*>(p) = make_uint4(lo.x, lo.y, hi.x, hi.y);
  }
};
template <> struct Operand<P_FP8> {
  typedef uint8_t E;
  typedef long V;
  static constexpr int EB = 1, UB = 8;
  __device__ static V ld(const void* p) { return *reinterpret_cast<const V*>(p); }
  __device__ static V ld_pix(const unsigned char* p) {
    const unsigned a = *reinterpret_cast<const unsigned*>(p);
    const unsigned b = *reinterpret_cast<const unsigned*>(p + 4);
    return (long)(((unsigned long long)b << 32) | a);
  }
  __device__ static f32x4 mma(V a, V b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_fp8_fp8(a, b, c, 0, 0, 0); }
  __device__ static V ldw(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
    return __builtin_bit_cast(V, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
  }
  __device__ static void stage16(unsigned char* dst, uint4 raw, float s8) {
    const unsigned w[4] = {raw.x, raw.y, raw.z, raw.w};
    unsigned o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      o[i] = fp8_pack4((float)(w[i] & 255u) * s8, (float)((w[i] >> 8) & 255u) * s8,
                       (float)((w[i] >> 16) & 255u) * s8, (float)(w[i] >> 24) * s8);
    *reinterpret_cast<uint4*>(dst) = make_uint4(o[0], o[1], o[2], o[3]);
  }
  __device__ static void st4(void* p, float a, float b, float c, float d, float s8) {
    *reinterpret_cast<unsigned*>(p) = fp8_pack4(a * s8, b * s8, c * s8, d * s8);
  }
  typedef unsigned PK;
  __device__ static PK pk4(float a, float b, float c, float d, float s8) {
    return fp8_pack4(a * s8, b * s8, c * s8, d * s8);
  }
  __device__ static void st8(void* p, PK lo, PK hi) { *reinterpret_cast<uint2*>(p) = make_uint2(lo, hi); }
};

}  // namespace
}  // namespace bcts
