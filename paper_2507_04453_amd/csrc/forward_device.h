// Device-side helpers shared by the kernels: register types, conversions, descriptor fetch, global-address-space
// pointers, LDS-only barrier, buffer loads, loads into LDS.
#pragma once
#include "essa_internal.h"

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(16))) int i32x16;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

namespace {

using essa_k::fwd_item;
using essa_k::stream_item;

__device__ __forceinline__ float bf16_bits_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }
__device__ __forceinline__ uint16_t f32_to_bf16_bits(float f) {
    // round to nearest even in one instruction (v_cvt_pk_bf16_f32)
    return __builtin_bit_cast(uint16_t, (__bf16)f);
}

// The descriptor of one item, fetched from the kernel arguments in one batch of scalar loads: left to itself the
// compiler loads every field where it is first used, and each of those loads is a separate wait on the way to the
// first tile.
template <class T>
__device__ __forceinline__ T fetch_item(const T& src) {
    constexpr int NW = sizeof(T) / 4;
    static_assert(sizeof(T) % 4 == 0, "descriptor is a whole number of words");
    int raw[NW];
    const int* p = reinterpret_cast<const int*>(&src);
#pragma unroll
    for (int i = 0; i < NW; ++i) raw[i] = p[i];
#pragma unroll
    for (int i = 0; i < NW; ++i) asm volatile("" : "+s"(raw[i]));      // all words are in scalar registers from here on
    T it;
    __builtin_memcpy(&it, raw, sizeof(T));
    return it;
}

// Pointers that come out of a descriptor are generic; memory instructions through them would be flat ones, which
// count against both the vector-memory and the LDS counter and force full waits.  These name the global address space.
template <class T> using gptr = __attribute__((address_space(1))) T*;
template <class T> __device__ __forceinline__ gptr<const T> as_global(const T* p) { return (gptr<const T>)p; }
template <class T> __device__ __forceinline__ gptr<T> as_global_w(T* p) { return (gptr<T>)p; }

// A workgroup barrier that orders LDS traffic only.  __syncthreads() also waits for every outstanding access to
// global memory (one counter serves loads and stores), which would put loads that are meant to fly across the
// barrier back on the critical path.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// N consecutive words of the kernel arguments in one batch of scalar loads.
template <int N>
__device__ __forceinline__ void fetch_words(const int* p, int (&out)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) out[i] = p[i];
#pragma unroll
    for (int i = 0; i < N; ++i) asm volatile("" : "+s"(out[i]));
}

// Buffer loads: (wave-uniform base in a resource descriptor) + (scalar offset) + (32-bit lane offset).  All address arithmetic
// that changes inside a loop is scalar, and the vector ALU, which the MFMAs also issue through, stays free.
typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const void* base_uniform) {
    // raw buffer (stride 0), 32-bit data format; 2 GB window: offsets used here are far below it
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base_uniform), 0, 0x7fffffff, 0x00020000);
}
__device__ __forceinline__ u32x4 load16(rsrc_t r, uint32_t lane_off, uint32_t scalar_off) {
    return __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, scalar_off, 0);
}


// ---- loads that go from memory into LDS without passing through registers ------------------------------------------
// A wave instruction moves 64 x 16 bytes: lane i's 16 bytes land at lds + 16 i, so the order in LDS is fixed and any
// permutation is made by the lanes' global addresses.  Written as one asm block because the compiler, which cannot tell
// the LDS stages apart, would otherwise wait for every such load in front of every LDS read; the waits are placed by hand.
typedef __attribute__((address_space(3))) unsigned char lds_byte;
__device__ __forceinline__ void load_lds16(uint32_t lds, uint32_t lane_off, i32x4 rsrc, uint32_t scalar_off) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :: "s"(lds), "v"(lane_off), "s"(rsrc), "s"(scalar_off) : "memory", "m0");
}
// the same with 4 bytes a lane
__device__ __forceinline__ void load_lds4(uint32_t lds, uint32_t lane_off, i32x4 rsrc, uint32_t scalar_off) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, %3 offen lds"
                 :: "s"(lds), "v"(lane_off), "s"(rsrc), "s"(scalar_off) : "memory", "m0");
}
__device__ __forceinline__ i32x4 buffer_words(const void* base) {
    const uint64_t p = reinterpret_cast<uint64_t>(base);
    i32x4 r;
    r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)p);
    r[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32)) & 0xffff;
    r[2] = 0x7fffffff;
    r[3] = 0x00020000;
    return r;
}
template <int N> __device__ __forceinline__ void wait_loads_and_meet() {
    // all but the last N loads of this wave have landed, this wave's LDS reads are done, and so are everybody else's
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(N) : "memory");
}

}  // namespace
