// Output layer and softmax cross-entropy of a small minibatch in one launch: logits = z W_o' + b_o, the losses and dlogits = (softmax - onehot) / rows.
//
// As two launches each is a few microseconds of latency (a launch, the first loads, the way of the logits through memory); the products
// are a microsecond or less.  Here a workgroup of W waves takes 16 frames of one learner through all their classes: wave w multiplies class tiles
// w, w + W, ... of 16, fragments straight from memory to registers (W_o of a learner lies in the L2, every workgroup reads all of it), and the
// logits stay in its accumulators: W_o is the first operand of the MFMAs, so that a lane holds four consecutive classes of one frame.  Maximum and sum
// go over the lanes of a frame, then over the waves through LDS.
//
// What bounds it: reading W_o, 16 bytes of 16 rows to an access.  Taken where W_o is up to 64 KB and its rows up to 1536 bytes, 2048 where every workgroup has a compute unit
// to itself: us an iteration, two launches / one (frames x classes x K x learners), fp32 80x100x64x4 67.0 / 63.5, 1280x100x64x16 146 / 126, 1280x256x64x8 126 / 118, 320x500x32x8 74.9 / 72.1, 5120x200x80x8 504 / 472; bf16
// 336x128x256x8 89 / 85, 2688x100x256x16 338 / 304, 336x500x64x8 66.2 / 62.4, 5120x500x64x16 382 / 323; and beyond fp32
// 640x500x64x8 98.9 / 98.9, bf16 336x500x256x8 92.5 / 94.7, 1344x100x1024x8 490 / 495, 336x500x1024x8 256 / 279.  Few classes are few tiles, for two or one of
// the waves, and a long row is a long chain, two chunks of it in flight: bf16 1344x32xKx8, K = 640 97.8 / 95.6, 768 99.5 / 98.9, 832 100.7 / 100.8, 896 102.2 / 103.4,
// 1024 107.1 / 110.3; 336x32xKx8, 1024 64.9 / 64.0, 80x32xKx4, 1024 52.5 / 52.0; 80x16x2048x4 60.8 / 63.9, 1344x16x2048x8 147.5 / 161.7, 1344x4x8192x8 419 / 486, 2688x4x8192x16 1364 / 1583.
//
// fp32: only contractions short enough for fp32 MFMAs in 64x64 tiles (gemm_plain_fp32), though two launches of the larger of these would multiply on the bf16 matrix
// units (gemm.hip: rows of logits are whole lines).  A 16x16x4 MFMA rounds a sum half as often as the 32x32x2 ones of the tiles.  Gradients of an iteration against
// 64 bits, two launches / one, 2-norm of b_o, W_o, b_p: 5120x200x80x8 1.42 / 1.42e-7, 1.27 / 1.27e-6, 1.42 / 1.43e-6, 5120x100x64x8 1.54 / 1.56e-7, 1.26 / 1.26e-6, 0.94 /
// 0.95e-6, 5120x256x64x8 1.44 / 1.43e-7, 1.29 / 1.29e-6, 1.50 / 1.51e-6.
#include <algorithm>
#include "gemm_tile.hpp"
#include "kernels.hpp"
#include "rec_tiles.hpp"

namespace adpsgd {
namespace {

template <typename T, int W, int NT>
__global__ __launch_bounds__(64 * W) void output_small_kernel(GemmDesc g, SoftmaxDesc p) {
    constexpr int EL = 16 / (int)sizeof(T), KC = 4 * EL, AHEAD = 2;          // elements of a fragment, of a chunk; chunks in flight
    __shared__ float red[2][W][16];
    const int li = __builtin_amdgcn_readfirstlane(p.lmap.idx[blockIdx.y]), m0 = (int)blockIdx.x * 16;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), r = lane & 15, quad = lane >> 4;
    const int rows = (int)p.rows, C = p.C, K = g.K, row = m0 + r;
    const buf_t z = make_buf_((const T*)g.A + li * g.sAi, (int64_t)rows * g.lda * sizeof(T));
    const buf_t w = make_buf_((const T*)g.B + li * g.sBi, (int64_t)C * g.ldb * sizeof(T));
    const buf_t bias = make_buf_(g.bias + li * g.sBiasI, (int64_t)C * 4);
    const buf_t dz = make_buf_((const T*)p.dlogits + li * p.sDi, (int64_t)rows * p.ldd * sizeof(T));

    const uint32_t vz = row < rows ? (uint32_t)(row * (int)g.lda + quad * EL) * (uint32_t)sizeof(T) : kOutOfRange;
    uint32_t vw[NT];
    f32x4_t acc[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int n0 = (wave + W * j) * 16;
        vw[j] = n0 + r < C ? (uint32_t)((n0 + r) * (int)g.ldb + quad * EL) * (uint32_t)sizeof(T) : kOutOfRange;
        acc[j] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(bias, n0 + 4 * quad < C ? (n0 + 4 * quad) * 4 : (int)kOutOfRange, 0, 0));   // (C: a multiple of 4)
    }
    const int chunks = (K + KC - 1) / KC;
    uint4 a[AHEAD], b[AHEAD][NT];
    auto load = [&](int c, uint4& x, uint4 (&y)[NT]) {     // (K is a multiple of EL: a fragment is whole or absent)
        const bool in = c * KC + quad * EL < K;
        const uint32_t k0 = (uint32_t)(c * KC) * (uint32_t)sizeof(T);
        x = buf_load16_(z, in ? vz : kOutOfRange, k0);
#pragma unroll
        for (int j = 0; j < NT; ++j) y[j] = buf_load16_(w, in ? vw[j] : kOutOfRange, k0);
    };
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) load(i, a[i], b[i]);
    for (int c0 = 0; c0 < chunks; c0 += AHEAD) {           // (chunks past the last read as zeros)
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
#pragma unroll
            for (int j = 0; j < NT; ++j) mma16_<T>(acc[j], b[i][j], a[i]);
            load(c0 + i + AHEAD, a[i], b[i]);
        }
    }

    // maximum and sum of a frame: this lane's classes, the four lanes of the frame, the waves
    float m = -INFINITY;
#pragma unroll
    for (int j = 0; j < NT; ++j)
        if ((wave + W * j) * 16 + 4 * quad < C) m = fmaxf(fmaxf(fmaxf(acc[j][0], acc[j][1]), fmaxf(acc[j][2], acc[j][3])), m);
    m = fmaxf(m, __shfl_xor(m, 16));
    m = fmaxf(m, __shfl_xor(m, 32));
    if (quad == 0) red[0][wave][r] = m;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < W; ++i) m = fmaxf(m, red[0][i][r]);
    int y = row < rows ? p.y[li * p.sYi + row] : 0;
    if (y < 0 || y >= C) {
        if (wave == 0 && quad == 0 && p.status) raise_status_(p.status, kStatusBadLabel);
        y = y < 0 ? 0 : C - 1;
    }
    float s = 0.f, zy = 0.f;
    bool mine = false;                                     // this lane holds the label's logit
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int n = (wave + W * j) * 16 + 4 * quad;
        if (n >= C) continue;
        if ((y >> 2) == (n >> 2)) {
            zy = (y & 3) == 0 ? acc[j][0] : (y & 3) == 1 ? acc[j][1] : (y & 3) == 2 ? acc[j][2] : acc[j][3];
            mine = true;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[j][i] = exp_fast_(acc[j][i] - m);
        s += (acc[j][0] + acc[j][1]) + (acc[j][2] + acc[j][3]);
    }
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    if (quad == 0) red[1][wave][r] = s;
    __syncthreads();
    s = red[1][0][r];
#pragma unroll
    for (int i = 1; i < W; ++i) s += red[1][i][r];
    const float inv = 1.f / s, scale = 1.f / (float)rows;
    if (mine && row < rows) p.row_loss[li * p.rows + row] = -((zy - m) - logf(s));
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int n = (wave + W * j) * 16 + 4 * quad;
        float pr[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            pr[i] = acc[j][i] * inv;
            if (n + i == y) pr[i] -= 1.f;
            pr[i] *= scale;
        }
        const uint32_t at = row < rows && n < C ? (uint32_t)(row * (int)p.ldd + n) * (uint32_t)sizeof(T) : kOutOfRange;
        if constexpr (sizeof(T) == 2) {
            const u32x2_t v = {pack_bf16(pr[0], pr[1]), pack_bf16(pr[2], pr[3])};
            __builtin_amdgcn_raw_buffer_store_b64(v, dz, (int)at, 0, 0);
        } else {
            const f32x4_t v = {pr[0], pr[1], pr[2], pr[3]};
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v), dz, (int)at, 0, 0);
        }
    }
}

template <typename T> void launch_t(const GemmDesc& g, const SoftmaxDesc& p, hipStream_t s) {
    const dim3 grid((unsigned)((p.rows + 15) / 16), (unsigned)p.L);
    if (p.C <= 128) hipLaunchKernelGGL((output_small_kernel<T, 4, 2>), grid, dim3(256), 0, s, g, p);
    else if (p.C <= 256) hipLaunchKernelGGL((output_small_kernel<T, 4, 4>), grid, dim3(256), 0, s, g, p);
    else hipLaunchKernelGGL((output_small_kernel<T, 8, 4>), grid, dim3(512), 0, s, g, p);
}

}  // namespace

bool output_small_supported(const GemmDesc& g, const SoftmaxDesc& p) {
    const int esz = g.precision ? 2 : 4;
    if (p.L < 1 || p.L > 128 || g.M < 1 || p.rows != g.M || p.C != g.N || g.groupsD != 1 || g.groupsI != p.L || !g.a_kc || !g.b_kc || !g.bias || g.tile != -1) return false;
    if (p.C % 4 != 0 || p.C > 512 || g.K * esz % 16 != 0 || g.lda * esz % 16 != 0 || g.ldb * esz % 16 != 0 || p.ldd * esz % 16 != 0) return false;
    if ((uintptr_t)g.A % 16 != 0 || (uintptr_t)g.B % 16 != 0 || (uintptr_t)p.dlogits % 16 != 0 || (uintptr_t)g.bias % 4 != 0) return false;
    if (g.sAi * esz % 16 != 0 || g.sBi * esz % 16 != 0 || p.sDi * esz % 16 != 0) return false;
    if ((int64_t)g.M * std::max(g.lda, p.ldd) * esz >= (int64_t)kOutOfRange || (int64_t)p.C * g.ldb * esz >= (int64_t)kOutOfRange) return false;     // buffer offsets
    if (!g.precision && !gemm_plain_fp32(g)) return false;
    if (g.K * esz > ((p.rows + 15) / 16 * p.L <= 256 ? 2048 : 1536)) return false;
    return (int64_t)p.C * g.K * esz <= 65536;
}

hipError_t launch_output_small(const GemmDesc& g, const SoftmaxDesc& p, hipStream_t s) {
    if (!output_small_supported(g, p)) return hipErrorInvalidValue;
    if (g.precision) launch_t<bf16_t>(g, p, s);
    else launch_t<float>(g, p, s);
    return hipGetLastError();
}

}  // namespace adpsgd
