// Device helpers shared by the attention kernels (gfx950).
#pragma once

#include "a2t_internal.h"

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace a2t {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
    typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
    const bf16x2 v = {(__bf16)a, (__bf16)b};   // v_cvt_pk_bf16_f32, round to nearest even
    return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ uint32_t pack_f16x2(float a, float b) {
    return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)a) |
           ((uint32_t)__builtin_bit_cast(uint16_t, (_Float16)b) << 16);
}
// s_waitcnt vmcnt(N) with expcnt and lgkmcnt left alone (gfx9 encoding)
template <int N>
__device__ __forceinline__ void wait_vmem() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}
// Stream of a workgroup, and the workgroup's place among the stream's.  Launches of uneven
// streams have no empty workgroups (place_workgroups): the dispatcher hands workgroups to the
// shader engines in turn, empty ones too, so that the real ones of small streams all went to
// one or two of an XCD's four engines where the largest stream had four or two query blocks (30
// streams of one row onto 2,500 keys beside one of 40, 90 or 400 rows, 8 KV heads of 128: 95,
// 69 and 168 us; without gaps 61, 68 and 73).
template <int N>
__device__ __forceinline__ int stream_of(const WgStart<N>& start, int count, int* place) {
    if (N == 1 || start.first[0] < 0) {
        *place = blockIdx.x;
        return blockIdx.z;
    }
    if (N <= 8) {   // scalar loads and compares
        int z = 0, at = 0;
#pragma unroll
        for (int i = 1; i < N; ++i) {
            const bool past = i < count && (int)blockIdx.x >= start.first[i];
            z = past ? i : z;
            at = past ? start.first[i] : at;
        }
        *place = (int)blockIdx.x - at;
        return z;
    }
    const int lane = threadIdx.x & 63;
    const int first = lane < count ? start.first[lane < N ? lane : 0] : 0x7fffffff;
    const int z = __builtin_popcountll(__ballot((int)blockIdx.x >= first)) - 1;
    *place = (int)blockIdx.x - __builtin_amdgcn_readlane(first, z);
    return z;
}
// workgroup barrier that the compiler may not move memory accesses across; no
// memory fence (the waits that make DMA'd data visible are explicit)
__device__ __forceinline__ void barrier_only() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}
__device__ __forceinline__ void dma16(const void* src, uint16_t* lds) {
    __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void*)lds, 16, 0, 0);
}
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)(p);
}
// Transposed LDS read issued as inline assembly: the compiler cannot tell which
// LDS the builtin form reads and would wait for every outstanding DMA before
// it.  The result is valid only after lds_wait_all() names it.
template <int OFF>
__device__ __forceinline__ uint2 lds_tr16_issue(uint32_t addr) {
    uint2 r;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "i"(OFF));
    return r;
}
// 16-byte LDS read issued as inline assembly (the compiler keeps only a few
// in flight and waits after each pair); valid only after k_wait() names it
template <int OFF>
__device__ __forceinline__ u32x4 lds_b128_issue(uint32_t addr) {
    u32x4 r;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "i"(OFF));
    return r;
}

}  // namespace
}  // namespace a2t
