// Bandwidth-bound helper kernels of the LSTM gradient: staging/casting of the
// minibatch and of the bf16 weight copy, softmax cross-entropy with its
// gradient, and the column sums that give the bias gradients.
#include "colsum.hpp"
#include "kernels.hpp"

namespace adpsgd {

// Rows of cols floats into rows of ld elements of the operand type, zero-padded; cols and ld multiples of 4, four elements to a thread
// (quad: of rows * ld / 4).  One element to a thread, with a 64-bit division each, took 58 us for the 16 x 4096 rows of 260 weights of the 512-cell
// model (126 MB) and a launch of its own beside the staging.
template <typename T> __device__ inline void copy_quad_(const float* src, T* dst, int64_t rows, int cols, int ld, int64_t first, int tid, bool wide) {
    const int per = ld / 4;
    const int64_t row0 = first / per;                      // (the same for the workgroup)
    const int x = (int)(first - row0 * per) + tid, dr = x / per, c = (x - dr * per) * 4;
    const int64_t row = row0 + dr;
    if (row >= rows) return;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    if (c < cols) {
        const float* p = src + row * cols + c;
        if (wide) v = *(const float4*)p;
        else { v.x = p[0]; v.y = p[1]; v.z = p[2]; v.w = p[3]; }
    }
    T* q = dst + row * ld + c;
    if constexpr (sizeof(T) == 2) *(uint2*)q = make_uint2(pack_bf16(v.x, v.y), pack_bf16(v.z, v.w));
    else *(float4*)q = v;
}

struct StageArgs {
    LearnerMap lmap;
    int64_t rows; int I, ldx;
    void* x0; int64_t sX0; int32_t* y; int64_t sY;
    const float* feats[128];
    const int32_t* labels[128];
    uint32_t* epoch; uint64_t* join; int64_t joins;
    int blocks;                                            // workgroups of the minibatch; those behind them pad weights
    const float* pad_src; int64_t pad_sS; bf16_t* pad_dst; int64_t pad_sD, pad_rows;
};

template <typename T>
__global__ __launch_bounds__(256) void stage_kernel(StageArgs p) {
    const int li = p.lmap.idx[blockIdx.y];
    if ((int)blockIdx.x >= p.blocks) {
        copy_quad_<bf16_t>(p.pad_src + li * p.pad_sS, p.pad_dst + li * p.pad_sD, p.pad_rows, p.I, p.ldx, (int64_t)((int)blockIdx.x - p.blocks) * 256, threadIdx.x, true);
        return;
    }
    const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const float* x = p.feats[li];
    copy_quad_<T>(x, (T*)p.x0 + li * p.sX0, p.rows, p.I, p.ldx, (int64_t)blockIdx.x * 256, threadIdx.x, ((uintptr_t)x & 15) == 0);
    if (idx < p.rows) p.y[li * p.sY + idx] = p.labels[li][idx];        // (a row is two quads at least)
    if (p.epoch && blockIdx.y == 0) {
        if (idx == 0) p.epoch[0] += 1u;
        for (int64_t i = idx; i < p.joins; i += (int64_t)p.blocks * 256) p.join[i] = 0ull;
    }
}

hipError_t launch_stage(const StageDesc& d, hipStream_t s) {
    if (d.L < 1 || d.L > 128 || d.I % 4 || d.ldx % 8 || (uintptr_t)d.pad_src % 16 || d.pad_sS % 4) return hipErrorInvalidValue;
    StageArgs a;
    a.lmap = d.lmap;
    a.rows = d.rows; a.I = d.I; a.ldx = d.ldx; a.x0 = d.x0; a.sX0 = d.sX0; a.y = d.y; a.sY = d.sY;
    for (int i = 0; i < 128; ++i) { a.feats[i] = d.feats[i]; a.labels[i] = d.labels[i]; }     // indexed by learner
    a.epoch = d.epoch; a.join = d.join; a.joins = d.joins;
    a.blocks = (int)((d.rows * (d.ldx / 4) + 255) / 256);
    a.pad_src = d.pad_src; a.pad_sS = d.pad_sS; a.pad_dst = d.pad_dst; a.pad_sD = d.pad_sD; a.pad_rows = d.pad_rows;
    const int64_t pad = d.pad_src ? (d.pad_rows * (d.ldx / 4) + 255) / 256 : 0;
    dim3 grid((unsigned)(a.blocks + pad), (unsigned)d.L);
    if (d.precision == 0) hipLaunchKernelGGL(stage_kernel<float>, grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL(stage_kernel<bf16_t>, grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

// n must be a multiple of 4 and both pointers 16-byte / 8-byte aligned.
__global__ __launch_bounds__(256) void cast_bf16_kernel(const float4* src, uint2* dst, int64_t n4) {
    int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (; i < n4; i += stride) {
        const float4 v = src[i];
        uint2 o;
        o.x = pack_bf16(v.x, v.y);
        o.y = pack_bf16(v.z, v.w);
        dst[i] = o;
    }
}

hipError_t launch_cast_bf16(const float* src, bf16_t* dst, int64_t n, hipStream_t s) {
    if (n % 4 != 0 || (uintptr_t)src % 16 != 0 || (uintptr_t)dst % 8 != 0) return hipErrorInvalidValue;
    const int64_t n4 = n / 4;
    int64_t blocks = (n4 + 255) / 256;
    if (blocks > 256 * 32) blocks = 256 * 32;
    hipLaunchKernelGGL(cast_bf16_kernel, dim3((unsigned)blocks), dim3(256), 0, s, (const float4*)src, (uint2*)dst, n4);
    return hipGetLastError();
}

// ---- softmax cross-entropy ---------------------------------------------------
// One workgroup per frame (row of logits).  loss_row = -(z_y - max - log sum exp(z - max));
// dlogits = (softmax - onehot) / rows   (mean over the B*T frames of the minibatch).
__device__ inline void lse_merge_(float& m, float& s, float m2, float s2) {
    const float mm = fmaxf(m, m2);
    s = s * expf(m - mm) + s2 * expf(m2 - mm);
    m = mm;
}

// Label of a frame.  A label outside [0, C) is reported through the status word (the host turns it
// into an error) and clamped, so that it is never used as an index.
__device__ inline int checked_label_(const SoftmaxDesc& p, int li, int64_t row) {
    const int y = p.y[li * p.sYi + row];
    if (y >= 0 && y < p.C) return y;
    if (threadIdx.x == 0 && p.status) raise_status_(p.status, kStatusBadLabel);
    return y < 0 ? 0 : p.C - 1;
}

template <typename T>
__global__ __launch_bounds__(256) void softmax_ce_kernel(SoftmaxDesc p) {
    const int li = p.lmap.idx[blockIdx.y];
    const int64_t row = blockIdx.x;
    const float* z = p.logits + li * p.sLi + row * p.ldl;
    T* dz = (T*)p.dlogits + li * p.sDi + row * p.ldd;
    const int y = checked_label_(p, li, row);
    float m = -INFINITY, s = 0.f;
    for (int c = threadIdx.x; c < p.C; c += 256) {
        const float v = z[c];
        if (v > m) { s = s * expf(m - v) + 1.f; m = v; }
        else s += expf(v - m);
    }
    // wave reduction, then across the 4 waves through LDS
    for (int off = 32; off > 0; off >>= 1) {
        const float m2 = __shfl_xor(m, off), s2 = __shfl_xor(s, off);
        if (m2 > -INFINITY || m > -INFINITY) lse_merge_(m, s, m2, s2);
    }
    __shared__ float sm[4], ss[4];
    if ((threadIdx.x & 63) == 0) { sm[threadIdx.x >> 6] = m; ss[threadIdx.x >> 6] = s; }
    __syncthreads();
    m = sm[0]; s = ss[0];
    for (int w = 1; w < 4; ++w) lse_merge_(m, s, sm[w], ss[w]);
    const float inv = 1.f / s;
    const float scale = 1.f / (float)p.rows;
    for (int c = threadIdx.x; c < p.C; c += 256) {
        float pr = expf(z[c] - m) * inv;
        if (c == y) pr -= 1.f;
        dz[c] = Elem<T>::from(pr * scale);
    }
    if (threadIdx.x == 0) p.row_loss[li * p.rows + row] = -((z[y] - m) - logf(s));
}

// Single-pass version: the whole row of logits lives in registers (NV float4 per thread, C <= 4*NT*NV),
// so the logits are read from HBM once.

template <typename T, int NV, int NT = 256>
__global__ __launch_bounds__(NT) void softmax_ce_row_kernel(SoftmaxDesc p) {
    const int li = p.lmap.idx[blockIdx.y];
    const int64_t row = blockIdx.x;
    const float4* z4 = (const float4*)(p.logits + li * p.sLi + row * p.ldl);
    T* dz = (T*)p.dlogits + li * p.sDi + row * p.ldd;
    const int C4 = p.C >> 2;
    const int y = checked_label_(p, li, row);
    float4 v[NV];
    float m = -INFINITY;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int c4 = threadIdx.x + NT * j;
        if (c4 < C4) {
            { const vf4_t t4 = __builtin_nontemporal_load((const vf4_t*)z4 + c4); v[j] = make_float4(t4.x, t4.y, t4.z, t4.w); }   // read once
            m = fmaxf(fmaxf(fmaxf(v[j].x, v[j].y), fmaxf(v[j].z, v[j].w)), m);
        }
    }
    __shared__ float red[2][NT / 64];
    for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    if ((threadIdx.x & 63) == 0) red[0][threadIdx.x >> 6] = m;
    __syncthreads();
    m = red[0][0];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) m = fmaxf(m, red[0][w]);
    float zy = 0.f;                      // logit of the label, picked up by the thread that holds it
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int c4 = threadIdx.x + NT * j;
        if (c4 < C4) {
            if ((y >> 2) == c4) zy = (y & 3) == 0 ? v[j].x : (y & 3) == 1 ? v[j].y : (y & 3) == 2 ? v[j].z : v[j].w;
            v[j].x = exp_fast_(v[j].x - m); v[j].y = exp_fast_(v[j].y - m); v[j].z = exp_fast_(v[j].z - m); v[j].w = exp_fast_(v[j].w - m);
            s += (v[j].x + v[j].y) + (v[j].z + v[j].w);
        }
    }
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off);
    if ((threadIdx.x & 63) == 0) red[1][threadIdx.x >> 6] = s;
    __syncthreads();
    s = red[1][0];
#pragma unroll
    for (int w = 1; w < NT / 64; ++w) s += red[1][w];
    const float inv = 1.f / s;
    const float scale = 1.f / (float)p.rows;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int c4 = threadIdx.x + NT * j;
        if (c4 < C4) {
            float4 pr = make_float4(v[j].x * inv, v[j].y * inv, v[j].z * inv, v[j].w * inv);
            if ((y >> 2) == c4) {
                if ((y & 3) == 0) pr.x -= 1.f; else if ((y & 3) == 1) pr.y -= 1.f; else if ((y & 3) == 2) pr.z -= 1.f; else pr.w -= 1.f;
            }
            pr.x *= scale; pr.y *= scale; pr.z *= scale; pr.w *= scale;
            if constexpr (sizeof(T) == 2) {
                uint2 o;
                o.x = pack_bf16(pr.x, pr.y);
                o.y = pack_bf16(pr.z, pr.w);
                { vu2_t o2; o2.x = o.x; o2.y = o.y; __builtin_nontemporal_store(o2, (vu2_t*)dz + c4); }
            } else {
                { vf4_t o4; o4.x = pr.x; o4.y = pr.y; o4.z = pr.z; o4.w = pr.w; __builtin_nontemporal_store(o4, (vf4_t*)dz + c4); }
            }
        }
    }
    if ((y >> 2) % NT == (int)threadIdx.x) p.row_loss[li * p.rows + row] = -((zy - m) - logf(s));
}

template <typename T>
static void launch_softmax_t(const SoftmaxDesc& d, hipStream_t s) {
    dim3 grid((unsigned)d.rows, (unsigned)d.L);
    const bool vec = d.C % 4 == 0 && d.ldl % 4 == 0 && d.sLi % 4 == 0 && d.ldd % 4 == 0 && d.sDi % 4 == 0 && (uintptr_t)d.logits % 16 == 0 &&
                     (uintptr_t)d.dlogits % 16 == 0;
    // long rows: 512 threads per row, so that a thread holds at most 16 float4 (measured on 32 000 classes:
    // 1.55 ms against 2.25 ms with 256 threads x 32 float4, whose 128 registers allow three waves per SIMD only, and
    // 1.78 ms with 1024 threads x 8 float4)
    if (vec && d.C <= 1024) hipLaunchKernelGGL((softmax_ce_row_kernel<T, 1>), grid, dim3(256), 0, s, d);
    else if (vec && d.C <= 4096) hipLaunchKernelGGL((softmax_ce_row_kernel<T, 4>), grid, dim3(256), 0, s, d);
    else if (vec && d.C <= 8192) hipLaunchKernelGGL((softmax_ce_row_kernel<T, 4, 512>), grid, dim3(512), 0, s, d);
    else if (vec && d.C <= 16384) hipLaunchKernelGGL((softmax_ce_row_kernel<T, 8, 512>), grid, dim3(512), 0, s, d);
    else if (vec && d.C <= 32768) hipLaunchKernelGGL((softmax_ce_row_kernel<T, 16, 512>), grid, dim3(512), 0, s, d);
    else hipLaunchKernelGGL(softmax_ce_kernel<T>, grid, dim3(256), 0, s, d);
}

hipError_t launch_softmax_ce(const SoftmaxDesc& d, hipStream_t s) {
    if (d.L < 1 || d.L > 128) return hipErrorInvalidValue;
    if (d.precision == 0) launch_softmax_t<float>(d, s);
    else launch_softmax_t<bf16_t>(d, s);
    return hipGetLastError();
}

// ---- column sums (colsum.hpp) -----------------------------------------------------
template <typename T, int SL>
__global__ __launch_bounds__(32 * SL) void colsum_kernel(ColsumDesc p) {
    __shared__ __attribute__((aligned(16))) char lds[SL * 32 * 16];
    colsum_block<T, SL, 32>(p, blockIdx.x, blockIdx.y, lds);
}

template <typename T> static void launch_colsum_t(const ColsumDesc& d, hipStream_t s) {
    const dim3 grid((unsigned)((d.N + 127) / 128 + (d.loss ? d.L_all : 0)), (unsigned)d.L);
    if (d.rows >= 128) hipLaunchKernelGGL((colsum_kernel<T, 32>), grid, dim3(1024), 0, s, d);
    else hipLaunchKernelGGL((colsum_kernel<T, 8>), grid, dim3(256), 0, s, d);
}

bool colsum_ok(const ColsumDesc& d) {
    // four columns at a time (every width and offset of the layout is a multiple of 4)
    const int quad = d.precision ? 8 : 16;
    return d.L >= 1 && d.L <= 128 && d.L_all <= 128 && d.N % 4 == 0 && d.ld % 4 == 0 && d.sIi % 4 == 0 && d.sOi % 4 == 0 && (uintptr_t)d.in % quad == 0 &&
           (uintptr_t)d.out % 16 == 0;
}

hipError_t launch_colsum(const ColsumDesc& d, hipStream_t s) {
    if (!colsum_ok(d)) return hipErrorInvalidValue;
    if (d.precision == 0) launch_colsum_t<float>(d, s);
    else launch_colsum_t<bf16_t>(d, s);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void zero_kernel(float* dst, int64_t sDi, int64_t n, LearnerMap lmap) {
    float* p = dst + lmap.idx[blockIdx.y] * sDi;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = 0.f;
}

hipError_t launch_zero(float* dst, int64_t sDi, int64_t n, int L, const LearnerMap& lmap, hipStream_t s) {
    if (L < 1 || L > 128 || n < 1) return hipErrorInvalidValue;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(zero_kernel, dim3((unsigned)blocks, (unsigned)L), dim3(256), 0, s, dst, sDi, n, lmap);
    return hipGetLastError();
}

}  // namespace adpsgd
