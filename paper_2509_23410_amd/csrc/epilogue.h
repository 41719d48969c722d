// Output stage shared by the product kernels: four consecutive features of one row, either as fp32 (the accumulator
// itself) or rounded to bf16 (round to nearest, ties to even: v_cvt_pk_bf16_f32).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace patch {

typedef float ep_f32x4 __attribute__((ext_vector_type(4)));

// bf16 bit pattern of an fp32 value, round to nearest even; a NaN stays a (quiet) NaN
__device__ __forceinline__ uint32_t bf16_rne_bits(float f) {
    const uint32_t u = __float_as_uint(f);
    const uint32_t nan = (u >> 16) | 0x40u, rne = (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;   // both computed: a select, no branch
    return (u & 0x7FFFFFFFu) > 0x7F800000u ? nan : rne;
}

typedef unsigned int ep_u32x2 __attribute__((ext_vector_type(2)));

// The same for two values at once, lo in the low half: v_cvt_pk_bf16_f32, which agrees with bf16_rne_bits on all 2^32 patterns
// (patch_test_bf16_mismatches compares them) in one instruction for about fourteen; a bf16 output stage of 256 x 256 spent 4 us on those (512 x 15360, K = 128: 17.9 -> 14.0 us; 65536 x 5120 at 1024 rows 454 -> 429).
typedef float ep_f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 ep_bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t bf16_pair(float lo, float hi) {
    const ep_bf16x2 r = __builtin_convertvector((ep_f32x2{lo, hi}), ep_bf16x2);
    return *reinterpret_cast<const uint32_t*>(&r);
}

#define PATCH_EP_GLOBAL __attribute__((address_space(1)))

// Store v at element offset `elem` of Y: fp32 (16 bytes) or bf16 (8 bytes).  `elem` is a multiple of 4.
// Y is device memory by contract; the store says so (address space 1).  The kernels pick Y with scalar selects from a
// by-value struct, after which the compiler no longer knows the address space and would emit flat stores.
__device__ __forceinline__ void store4(float* Y, int64_t elem, ep_f32x4 v, int ybf16) {
    if (ybf16) {
        ep_u32x2 p;
        p[0] = bf16_pair(v[0], v[1]);
        p[1] = bf16_pair(v[2], v[3]);
        PATCH_EP_GLOBAL uint16_t* Yh = reinterpret_cast<PATCH_EP_GLOBAL uint16_t*>(reinterpret_cast<uintptr_t>(Y));
        *reinterpret_cast<PATCH_EP_GLOBAL ep_u32x2*>(Yh + elem) = p;
    } else {
        PATCH_EP_GLOBAL float* Yg = reinterpret_cast<PATCH_EP_GLOBAL float*>(reinterpret_cast<uintptr_t>(Y));
        *reinterpret_cast<PATCH_EP_GLOBAL ep_f32x4*>(Yg + elem) = v;
    }
}

// read(0) + read(1) + ... + read(n - 1), added in that order: the partial sums of n wavefronts (n a multiple of 4) in LDS, four reads requested
// together: a loop over a run-time n reads one by one, each waiting its own LDS latency.
template <typename Read>
__device__ __forceinline__ ep_f32x4 sum_in_order(int n, Read read) {
    ep_f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    for (int i = 0; i < n; i += 4) {
        const ep_f32x4 v0 = read(i), v1 = read(i + 1), v2 = read(i + 2), v3 = read(i + 3);
        sum = i == 0 ? v0 : sum + v0;
        sum = sum + v1;
        sum = sum + v2;
        sum = sum + v3;
    }
    return sum;
}

}  // namespace patch
