// Operands of the 16x16x32 matrix instructions staged through LDS: pieces of
// 16-bit data loaded straight from global memory, rows of 16 columns per slot
// with two sources (angles) side by side, read back transposed.
#pragma once

#include "tp_internal.h"

namespace tp {
namespace {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float f2_t __attribute__((ext_vector_type(2)));
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u4_t __attribute__((ext_vector_type(4)));
typedef short s4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s4_t* lds_s4_t;

// LDS layout of a tile of 16 columns: [slot][source of the pair][column], 64
// bytes per slot.  Four consecutive slots of one source lie in four different
// 64-byte quarters of a 256-byte line, in the half of each that belongs to the
// source: a read of 4 slots x 16 columns for two sources (32 lanes, 256 bytes)
// meets every bank once wherever the two windows start.
constexpr int kSlotBytes = 64;

// 8 slots of 16 columns from p (this lane's slot, source and columns),
// transposed: lane l of each 16 gets column l's values.
__device__ __forceinline__ u4_t read_slots(const unsigned char* p) {
    struct { s4_t lo, hi; } v;
    v.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_t)(p));
    v.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_t)(p + 4 * kSlotBytes));
    return __builtin_bit_cast(u4_t, v);
}

// The same from an LDS byte address.
__device__ __forceinline__ u4_t read_slots(uint32_t lds) {
    struct { s4_t lo, hi; } v;
    v.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_s4_t>(lds));
    v.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_s4_t>(lds + 4 * kSlotBytes));
    return __builtin_bit_cast(u4_t, v);
}
// An address the compiler takes as it is: reads at constant distances from it
// then carry them in the instruction.
__device__ __forceinline__ uint32_t opaque(uint32_t lds) {
    asm volatile("" : "+v"(lds));
    return lds;
}

// 16 bytes per lane from the lane's global address to LDS bytes lds .. lds +
// 1023, in lane order.  No register receives the data, so nothing waits for it
// but wait_loads(): for the builtin the compiler waits before the next LDS read
// of any kind, which ends the overlap with the products.
__device__ __forceinline__ void load_lds16(const void* p, uint32_t lds) {
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(p), "{m0}"(lds) : "memory");
}
// The same from a uniform base and a 32-bit byte offset per lane.
__device__ __forceinline__ void load_lds16(const void* base, uint32_t off, uint32_t lds) {
    asm volatile("s_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(off), "s"(base), "{m0}"(lds) : "memory");
}
__device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// LDS byte address of a shared object.
__device__ __forceinline__ uint32_t lds_address(unsigned char* p) {
    return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) unsigned char*)(p)));
}

// What lanes without a source read.
__device__ __align__(16) uint32_t g_zero[4];

__device__ __forceinline__ f4_t mfma16(u4_t a, u4_t b, f4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a), __builtin_bit_cast(half8_t, b), c, 0,
                                                  0, 0);
}

// x and y rounded to FP16, and what that misses (exact before it is rounded),
// each as a pair.  The differences are one mixed-precision FMA each, written out:
// from C they become a conversion and a subtraction.
__device__ __forceinline__ void split_pair(float x, float y, uint32_t& hi, uint32_t& lo) {
    hi = __builtin_bit_cast(uint32_t, __builtin_convertvector((f2_t{x, y}), half2_t));
    f2_t r;
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(r.x) : "v"(hi), "v"(x));
    asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(r.y) : "v"(hi), "v"(y));
    lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, half2_t));
}

// Data as two FP16 values (kLowScale).  Products of the second take weights
// 2^-11 times as large.
__device__ __forceinline__ void split_data(float x, float y, uint32_t& hi, uint32_t& lo) {
    const half2_t h = __builtin_convertvector((f2_t{x, y}), half2_t);
    const f2_t r{(x - static_cast<float>(h.x)) * kLowScale, (y - static_cast<float>(h.y)) * kLowScale};
    hi = __builtin_bit_cast(uint32_t, h);
    lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, half2_t));
}
// Weights in [0, 1] for the second values (below 2^-3 they round at 2^-25).
__device__ __forceinline__ uint32_t low_weights(uint32_t hi) {
    constexpr _Float16 s = static_cast<_Float16>(1.0f / kLowScale);
    return __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2_t, hi) * half2_t{s, s});
}

}  // namespace
}  // namespace tp
