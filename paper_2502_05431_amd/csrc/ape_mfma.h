// Device helpers shared by the matrix-core kernels that are built on plain builtins (the tile kernels, the encode walk).
#pragma once

#include "ape_internal.h"

namespace ape {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;

constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;
constexpr float kUnset = -1.0e30f;           // softmax reference of a row that has not seen a token yet

// One direct global->LDS load: lane i's 16 bytes land at (wavefront-uniform) lds + 16 i.  Written as an
// instruction so that the compiler does not order it (it could only wait for all of them): the waits and
// barriers of the ring do.
__device__ __forceinline__ void load_lds16(const char* src, const char* lds) {
    const uint32_t m0v = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)lds;
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" :: "v"(src), "s"(m0v) : "m0");
}
// The same from a wavefront-uniform base and a 32-bit offset per lane.  Where the base comes from vector registers, the v_readfirstlane that
// writes its scalar registers must be five wait states ahead of the load that reads them.  The compiler keeps that distance for
// its own loads and does not look inside the statement, so they are in here: one for s_mov, four for s_nop 3 (and one of
// them is what M0 needs).
__device__ __forceinline__ void load_lds16(const char* base, uint32_t off, const char* lds) {
    const uint32_t m0v = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char*)lds;
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %0, %1" :: "v"(off), "s"(uniform_address(base)), "s"(m0v) : "m0");
}

// All but the youngest N vector-memory operations of this wavefront are complete (they complete in order).
template <int N>
__device__ __forceinline__ void wait_loads() {
    static_assert(N < 64, "vmcnt is a 6-bit counter");
    __builtin_amdgcn_s_waitcnt(0x0f70 | (N & 15) | ((N >> 4) << 14));
}
// Workgroup barrier that memory operations may not be moved across, without a wait for the loads in flight.
__device__ __forceinline__ void stage_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Over the two half-wavefronts: a query row lives in lanes l and l ^ 32.
__device__ __forceinline__ float max_halves(float x) {
    const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_halves(float x) {
    const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ bf16x4 lds_read_tr(const char* p) {
    s16x4 r = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p);
    return __builtin_bit_cast(bf16x4, r);
}
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));   // one instruction
}

}  // namespace
}  // namespace ape
