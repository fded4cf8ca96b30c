// Column sums of a matrix (bias gradients) and the losses of the learners, as workgroups of a launch of their own (elementwise.hip) or
// beside the products that read the same matrix (gemm_multi.hip).
#pragma once
#include "kernels.hpp"

namespace adpsgd {

typedef float vf4_t __attribute__((ext_vector_type(4)));
typedef uint32_t vu2_t __attribute__((ext_vector_type(2)));
// ---- column sums -----------------------------------------------------------------
// Workgroup = 4 TX columns, four to a thread, x SL row slices; a slice's sums of four rows at a time and the slices are added in a
// fixed order (deterministic).  Bound by the read of the input once enough of it is in flight: with 64 columns x 4 slices, one
// column to a thread, 1050 rows took 33 us at any width (bf16 5 x 1050 x 120: 33 -> 5 us, x 3000: 35 -> 9).
// The workgroups behind the columns add the row losses of a learner, if asked for; a learner that took no part reports 0.
template <typename T> struct Quad;
template <> struct Quad<float> {
    __device__ static float4 load(const float* p) {
        const vf4_t v = __builtin_nontemporal_load((const vf4_t*)p);
        return make_float4(v.x, v.y, v.z, v.w);
    }
};
template <> struct Quad<bf16_t> {
    __device__ static float4 load(const bf16_t* p) {
        const vu2_t v = __builtin_nontemporal_load((const vu2_t*)p);
        return make_float4(__builtin_bit_cast(float, v.x << 16), __builtin_bit_cast(float, v.x & 0xffff0000u),
                           __builtin_bit_cast(float, v.y << 16), __builtin_bit_cast(float, v.y & 0xffff0000u));
    }
};
__device__ inline float4 add4_(const float4& a, const float4& b) { return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); }

// Workgroup x of a learner's columns, and those behind them (L_all of them, y = 0) of the row losses.
template <typename T, int SL, int TX>
__device__ __forceinline__ void colsum_block(const ColsumDesc& p, int x, int y, char* lds) {
    float4 (*sh)[TX] = (float4 (*)[TX])lds;                // [SL][TX]
    const int tid = threadIdx.x;
    if (x * 4 * TX >= p.N) {
        const int li = x - (p.N + 4 * TX - 1) / (4 * TX);
        if (y != 0) return;
        if (!((p.active_bits[li >> 5] >> (li & 31)) & 1u)) {
            if (tid == 0) p.loss[li] = 0.f;
            return;
        }
        float s = 0.f;
        for (int64_t r = tid; r < p.rows; r += TX * SL) s += p.row_loss[li * p.rows + r];
        float* f = (float*)sh;
        f[tid] = s;
        __syncthreads();
        for (int off = TX * SL / 2; off > 0; off >>= 1) {
            if (tid < off) f[tid] += f[tid + off];
            __syncthreads();
        }
        if (tid == 0) p.loss[li] = f[0] / (float)p.rows;
        return;
    }
    const int li = p.lmap.idx[y], tx = tid % TX, slice = tid / TX;
    const int col = x * 4 * TX + 4 * tx;
    const T* src = (const T*)p.in + li * p.sIi + col;
    float4 s[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) s[j] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (col < p.N) {
        int64_t r = slice;
        for (; r + 7 * SL < p.rows; r += 8 * SL) {
            float4 v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = Quad<T>::load(src + (r + j * SL) * p.ld);
#pragma unroll
            for (int j = 0; j < 8; ++j) s[j & 3] = add4_(s[j & 3], v[j]);
        }
        for (; r + 3 * SL < p.rows; r += 4 * SL) {
            float4 v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = Quad<T>::load(src + (r + j * SL) * p.ld);
#pragma unroll
            for (int j = 0; j < 4; ++j) s[j] = add4_(s[j], v[j]);
        }
        for (; r < p.rows; r += SL) s[0] = add4_(s[0], Quad<T>::load(src + r * p.ld));
    }
    sh[slice][tx] = add4_(add4_(s[0], s[1]), add4_(s[2], s[3]));
    __syncthreads();
    if (slice < 4) {                                       // a quarter of the slices each, then the quarters
        float4 t = sh[slice * (SL / 4)][tx];
#pragma unroll
        for (int j = 1; j < SL / 4; ++j) t = add4_(t, sh[slice * (SL / 4) + j][tx]);
        s[0] = t;
    }
    __syncthreads();
    if (slice < 4) sh[slice][tx] = s[0];
    __syncthreads();
    if (slice == 0 && col < p.N) *(float4*)(p.out + li * p.sOi + col) = add4_(add4_(sh[0][tx], sh[1][tx]), add4_(sh[2][tx], sh[3][tx]));
}

}  // namespace adpsgd
