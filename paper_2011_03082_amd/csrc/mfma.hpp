// mfma.hpp -- 16x16 CVAE layers on gfx950 matrix cores.
//
// Activations are kept feature-major: one 16 x 16 tile holds 16 features
// (rows) of 16 samples (columns).  For v_mfma_f32_16x16x16_bf16 the B
// operand and the D result of lane l both cover rows 4 (l / 16) + j,
// j = 0..3, of column l % 16, so the output of one layer, after its
// activation, is already the next layer's B operand: a whole MLP chains
// through registers with no data movement.  The A operand (the weights)
// covers row l % 16, columns 4 (l / 16) + j.
#pragma once

#include "device.hpp"

namespace msst {

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kTile = 16;

__device__ __forceinline__ f32x4 mfma_bf16(bf16x4 a, bf16x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ int frag_row() { return lane_id() & 15; }  // A row / B, D column
__device__ __forceinline__ int frag_k0() { return (lane_id() >> 4) * 4; } // first of 4 K (or D) rows

// Converted in pairs (four values at once, or one by one, the compiler converts
// each alone and then packs: six instructions instead of two).
__device__ __forceinline__ bf16x4 to_bf16x4(float a, float b, float c, float d) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const bf16x2 lo = __builtin_convertvector((f32x2){a, b}, bf16x2), hi = __builtin_convertvector((f32x2){c, d}, bf16x2);
    const uint2 u = make_uint2(__builtin_bit_cast(uint32_t, lo), __builtin_bit_cast(uint32_t, hi));
    return __builtin_bit_cast(bf16x4, u);
}
__device__ __forceinline__ bf16x4 to_bf16x4(f32x4 v) { return to_bf16x4(v[0], v[1], v[2], v[3]); }

// Intra-wave ordering of LDS traffic between lanes of the same wave.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A 16 x 16 tile of floats in LDS, row-major, from the D layout: this lane's
// rows k0..k0+3 of column c.
__device__ __forceinline__ void tile_store_d(float* t, f32x4 v) {
    const int c = frag_row(), k0 = frag_k0();
#pragma unroll
    for (int j = 0; j < 4; ++j) t[(k0 + j) * kTile + c] = v[j];
}

}  // namespace msst
