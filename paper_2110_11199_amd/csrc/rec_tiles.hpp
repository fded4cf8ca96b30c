// 16x16 MFMA tiles of the recurrent kernels that keep W_h in registers, and what they share with the split-contraction ones.
#pragma once
#include "gemm_core.hpp"

namespace adpsgd {

typedef __attribute__((ext_vector_type(4))) float f32x4_t;

template <typename T> __device__ inline void mma16_(f32x4_t& acc, const uint4& a, const uint4& b);
template <> __device__ inline void mma16_<bf16_t>(f32x4_t& acc, const uint4& a, const uint4& b) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), acc, 0, 0, 0);
}
template <> __device__ inline void mma16_<float>(f32x4_t& acc, const uint4& a, const uint4& b) {
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, a.x), __builtin_bit_cast(float, b.x), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, a.y), __builtin_bit_cast(float, b.y), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, a.z), __builtin_bit_cast(float, b.z), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, a.w), __builtin_bit_cast(float, b.w), acc, 0, 0, 0);
}

// EL consecutive rows of column `col` of a rows-contiguous matrix, as one fragment
__device__ inline uint4 column_frag_(const float* col, int64_t ld) {
    return make_uint4(__builtin_bit_cast(uint32_t, col[0]), __builtin_bit_cast(uint32_t, col[ld]),
                      __builtin_bit_cast(uint32_t, col[2 * ld]), __builtin_bit_cast(uint32_t, col[3 * ld]));
}
__device__ inline uint4 column_frag_(const bf16_t* col, int64_t ld) {
    uint32_t w[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = (uint32_t)col[(2 * j) * ld] | ((uint32_t)col[(2 * j + 1) * ld] << 16);
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// Barrier that waits for this wave's LDS accesses only: the stores of a frame's results stay in flight across it.  (The barrier is
// no memory access for the optimiser: an empty statement that is one stands on either side.)
__device__ inline void lds_barrier_() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

}  // namespace adpsgd
