// Device-side helpers for gfx950 (wave64): DPP lane exchanges, bf16 packing,
// wave-private LDS ordering.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "psa_trace.h"

namespace psa {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// ---- DPP: data-parallel-primitive lane permutations inside a row of 16 lanes
// quad_perm [1,0,3,2] = 0xB1, quad_perm [2,3,0,1] = 0x4E,
// row_half_mirror = 0x141 (lane i <-> 7-i in each 8).
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float x) {
    return __builtin_bit_cast(float,
        __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
}

// Sum over aligned groups of 8 lanes; every lane of the group gets the total.
__device__ __forceinline__ float group_sum8(float x) {
    x += dpp_mov<0xB1>(x);
    x += dpp_mov<0x4E>(x);
    x += dpp_mov<0x141>(x);
    return x;
}

// ---- bf16 <-> f32
__device__ __forceinline__ float bf16_lo(uint32_t pair) { return __uint_as_float(pair << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t pair) { return __uint_as_float(pair & 0xFFFF0000u); }
// round-to-nearest-even; NaN stays NaN
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    return (uint32_t)f32_to_bf16(lo) | ((uint32_t)f32_to_bf16(hi) << 16);
}

// two floats to a bf16 pair (lo in bits 0..15) with the hardware conversion, round-to-nearest-even
typedef float floatx2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t cvt_pk_bf16(float lo, float hi) {
    const floatx2 v = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// ---- ordering of LDS traffic between the lanes of ONE wave (no other wave
// touches the region): LDS executes a wave's instructions in order, so only
// the compiler has to be told not to move accesses across this point.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Work-group barrier that orders LDS traffic only.  __syncthreads() also waits
// for every outstanding global load of the wave (one counter covers loads and
// stores), which would serialise loads issued early on purpose; this one leaves
// them in flight.  Use it only where no global store needs to be seen by the
// other waves of the work-group.
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Exchange with the lane 32 away (the other half of the wave).
__device__ __forceinline__ float swap_half(float x) { return __shfl_xor(x, 32, 64); }

// Maximum over the lanes 32 apart, and over those 16 apart, in every lane: the swap instructions exchange half-waves
// (rows of 16) between two registers, here two copies of x, without the trip through the LDS unit a shuffle makes.
__device__ __forceinline__ float max_xor32(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float max_xor16(float x) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Sum of x and its value in the lane 32 (16) away, in every lane, the same way
__device__ __forceinline__ double sum_xor32(double x) {
    const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(x), __double2loint(x), false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(x), __double2hiint(x), false, false);
    return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
__device__ __forceinline__ double sum_xor16(double x) {
    const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(x), __double2loint(x), false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(x), __double2hiint(x), false, false);
    return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}

// ... and over those 8 apart: a rotation by 8 within each row of 16 lanes
__device__ __forceinline__ double sum_xor8(double x) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), 0x128, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), 0x128, 0xF, 0xF, false);
    return x + __hiloint2double(hi, lo);
}

// 2^x in float64 for x <= ~0 (anything below -1000, -inf included, gives 0; NaN stays NaN):
// x = n + f with |f| <= 1/2 by adding and taking away 1.5 * 2^52, 2^f by the polynomial of degree 6 with
// constant term 1 whose largest relative error on [-1/2, 1/2] is least (2.0e-9; 2^0 is exactly 1; the softmax weights need 1e-6, see
// the parity bound), scaled by adding n to the exponent field.  Vector instructions do not overlap with
// float64 matrix instructions on a SIMD, so every instruction here counts: a Taylor series of degree 7 (7.0e-9) with
// rint, a separate factor ln 2 and ldexp took 90 cycles per value, this one about 60.
// ABOVE: x may be anything; from 1024 on the exponent is set to that of infinity, which gives infinity or NaN where the
// exponent field would wrap to a finite value (two instructions more).
template <bool ABOVE = false>
__device__ __forceinline__ double exp2_f64(double x) {
    const double t = x + 6755399441055744.0;                 // the low word of t now holds n
    const double f = x - (t - 6755399441055744.0);
    double p = fma(f, 0.00015353361998437113, 0.0013398874452528137);
    p = fma(f, p, 0.009618437357635966);
    p = fma(f, p, 0.055503324710417745);
    p = fma(f, p, 0.24022647913627504);
    p = fma(f, p, 0.6931472028550949);
    p = fma(f, p, 1.0);
    int hi = __double2hiint(p) + (__double2loint(t) << 20);
    if (ABOVE) hi = x >= 1024.0 ? 0x7FF00000 : hi;
    const double y = __hiloint2double(hi, __double2loint(p));
    return x < -1000.0 ? 0.0 : y;
}

// Valid length of batch item b, clamped to [0, L].
__device__ __forceinline__ int valid_len(const int* lengths, int b, int L) {
    if (!lengths) return L;
    int n = lengths[b];
    return n < 0 ? 0 : (n > L ? L : n);
}

}  // namespace psa
