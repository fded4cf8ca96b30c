// Recurrent LSTM kernels that keep W_h on one compute unit: all T frames of one layer in one launch, for hidden sizes up to 128.
//
// A step of such a model is a few hundred thousand multiply-adds per (learner, direction): launched frame by frame it is bound by
// the launch itself, by reading W_h again and by the latency of the reduction over the contraction.  us per frame
// (forward / backward), frame by frame against here: fp32 4 x 64 cells, batch 4: 8.2 / 6.4 -> 2.0 / 2.2; 16 x 128, 64: 9.9 / 8.6
// -> 6.0 / 6.6 (bound by the fp32 products of one compute unit, 3.5); 128 x 128, 128: 33 / 40 -> 26 / 32; bf16 16 x 128,
// 16: 5.8 / 5.9 -> 2.2 / 2.4, 128 x 128, 128: 19.8 / 25.0 -> 15.8 / 16.4 (the cell arithmetic of two waves per SIMD).  Batch rows do not depend on each other, so a
// workgroup here takes 16 batch rows of one (learner, direction) through ALL frames and needs nothing from any other
// workgroup: no launch, no global round trip and no wait between frames.
//
// One wave per 16 hidden units.  Its slice of W_h - the four gate rows of its units (forward, h W_h') or their unit columns
// (backward, da W_h) - stays in registers as MFMA B fragments for the whole launch (at most 128 registers: 128 units in
// fp32).  The frame's operand (h, or da) lies in LDS, double-buffered, and every wave reads all of it; the four
// gates of a unit end up in the same lane, so the cell update runs on the accumulators, the cell state (dL/dc) never
// leaves the registers, and a frame needs one barrier.  The pre-activations (the saved gates) of the next frame are
// requested before the products of the current one.
//
// MFMA operand mapping (16x16 tiles): lane (r = lane % 16, g = lane / 16) supplies 16 bytes of operand row r at
// k = chunk*KC + g*EL; accumulator element i of a lane is row 4*g + i, column r.  fp32: a chunk is four 16x16x4 products
// over k = 4g + j, j = 0..3; bf16: one 16x16x32.
#include "gemm_core.hpp"
#include "kernels.hpp"
#include "rec_tiles.hpp"

namespace adpsgd {
namespace {

constexpr int kRows = 16;                                 // batch rows of a workgroup

template <typename T, int NCH> struct Cu {
    static constexpr int EL = 16 / (int)sizeof(T), KC = 4 * EL, KP = NCH * KC;      // elements per fragment, per chunk, padded H
    // bytes of an operand row in LDS: 16 more than a multiple of 32, so that 16 rows at one chunk lie in different banks
    static constexpr int FWD_ROW = KP * (int)sizeof(T) + 16, BWD_ROW = 4 * KP * (int)sizeof(T) + 16;
};

// Guards are out-of-range buffer offsets, frames are unrolled by two and the frame past the last is a repeat of the last: so
// there is no branch between the request of a frame's inputs and their use, and the wait before their use leaves the
// stores that were issued in between in flight (with exec-masked accesses every frame waited for the stores of the one
// before: 5.7 us per frame at 64 cells).
//
// ---- forward ------------------------------------------------------------------------------------
//   a = W_x x_t + b + W_h h_{t'}     i,f,o = sigmoid(a), g = tanh(a)     c_t = f c_{t'} + i g     h_t = o tanh(c_t)
template <typename T, int NCH>
__global__ __launch_bounds__(512) void rec_forward_cu_kernel(RecDesc p) {
    typedef Cu<T, NCH> C;
    __shared__ __attribute__((aligned(16))) char lds[2 * kRows * C::FWD_ROW];
    const int D = p.D, H = p.H, B = p.B, Tn = p.T;
    const int li = __builtin_amdgcn_readfirstlane(p.lmap.idx[blockIdx.x / D]), d = blockIdx.x % D, b0 = blockIdx.y * kRows;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
    const int u = wave * 16 + r;
    const bool ok_u = u < H;
    const uint32_t DH = (uint32_t)(D * H), G4 = DH * 4;
    const buf_t gates = make_buf_(p.gates + li * p.sGi, (int64_t)Tn * B * G4 * 4);
    const buf_t cbuf = make_buf_(p.c + li * p.sCi + (int64_t)d * Tn * B * H, (int64_t)Tn * B * H * 4);
    const buf_t y = make_buf_((const T*)p.y + li * p.sYi, (int64_t)Tn * B * DH * sizeof(T));

    uint4 w[4][NCH];
    {
        const T* wrow = (const T*)p.wh + li * p.sWi + d * p.sWd + (int64_t)(ok_u ? u : 0) * H;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
                const int k = c * C::KC + g * C::EL;      // H is a multiple of EL: a fragment is whole or absent
                w[q][c] = ok_u && k < H ? *(const uint4*)(wrow + (int64_t)q * H * H + k) : make_uint4(0u, 0u, 0u, 0u);
            }
    }
    for (int i = threadIdx.x; i < (int)sizeof(lds) / 4; i += blockDim.x) ((uint32_t*)lds)[i] = 0u;   // k past H stays zero
    uint32_t vg[4], vc[4], vy[4];                         // byte offsets of this lane's four batch rows
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t row = b0 + 4 * g + i;
        const bool ok = ok_u && (int)row < B;
        vg[i] = ok ? (row * G4 + d * 4 * H + u) * 4u : kOutOfRange;
        vc[i] = ok ? (row * H + u) * 4u : kOutOfRange;
        vy[i] = ok ? (row * DH + d * H + u) * (uint32_t)sizeof(T) : kOutOfRange;
    }
    auto load_pre = [&](int s, float (&a)[4][4]) {
        const uint32_t m = (uint32_t)(d == 0 ? s : Tn - 1 - s) * B;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) a[q][i] = buf_load_(gates, vg[i], (m * G4 + q * H) * 4u);
    };
    float cs[4] = {0.f, 0.f, 0.f, 0.f};
    auto frame = [&](int s, const float (&pre)[4][4], float (&next)[4][4]) {
        const uint32_t m = (uint32_t)(d == 0 ? s : Tn - 1 - s) * B;
        f32x4_t acc[4];
        load_pre(s + 1 < Tn ? s + 1 : s, next);
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] = f32x4_t{pre[q][0], pre[q][1], pre[q][2], pre[q][3]};
        lds_barrier_();                                   // h of the frame before is complete (s = 0: the zero fill, h = 0)
        const char* hrow = lds + ((s + 1) & 1) * (kRows * C::FWD_ROW) + r * C::FWD_ROW + g * 16;
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            const uint4 a = *(const uint4*)(hrow + c * 64);
#pragma unroll
            for (int q = 0; q < 4; ++q) mma16_<T>(acc[q], a, w[q][c]);
        }
        T* hout = (T*)(lds + (s & 1) * (kRows * C::FWD_ROW)) + 4 * g * (C::FWD_ROW / (int)sizeof(T)) + (ok_u ? u : C::KP);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float ig = sigmoidf_(acc[0][i]), fg = sigmoidf_(acc[1][i]), gg = tanhf_(acc[2][i]), og = sigmoidf_(acc[3][i]);
            cs[i] = fg * cs[i] + ig * gg;
            const T h = Elem<T>::from(og * tanhf_(cs[i]));
            hout[i * (C::FWD_ROW / (int)sizeof(T))] = h;   // (rows past the batch are read by no valid row; units past H lie in the row's padding)
            buf_store_(ig, gates, vg[i], (m * G4 + 0 * H) * 4u);
            buf_store_(fg, gates, vg[i], (m * G4 + 1 * H) * 4u);
            buf_store_(gg, gates, vg[i], (m * G4 + 2 * H) * 4u);
            buf_store_(og, gates, vg[i], (m * G4 + 3 * H) * 4u);
            buf_store_(cs[i], cbuf, vc[i], m * H * 4u);
            buf_store_(h, y, vy[i], m * DH * (uint32_t)sizeof(T));
        }
    };
    float pa[4][4], pb[4][4];
    load_pre(0, pa);
    frame(0, pa, pb);                                     // (outside the loop, so that the loop is entered with its stores in flight)
    int s = 1;
    for (; s + 1 < Tn; s += 2) { frame(s, pb, pa); frame(s + 1, pa, pb); }
    if (s < Tn) frame(s, pb, pa);
}

// ---- backward -----------------------------------------------------------------------------------
//   dh_t = dY_t + da_{t''} W_h  (t'' = the frame handled before)
//   do = dh tanh(c_t)            dc = dc_rec + dh o (1 - tanh^2 c_t)
//   di = dc g, dg = dc i, df = dc c_{t'}, dc_rec <- dc f
//   da = (di i(1-i), df f(1-f), dg (1-g^2), do o(1-o))
// The column sums of da (bias gradients) run over all frames in registers: one row of partial sums per batch tile.
template <typename T, int NCH>
__global__ __launch_bounds__(512) void rec_backward_cu_kernel(RecDesc p) {
    typedef Cu<T, NCH> C;
    __shared__ __attribute__((aligned(16))) char lds[2 * kRows * C::BWD_ROW];
    const int D = p.D, H = p.H, B = p.B, Tn = p.T;
    const int li = __builtin_amdgcn_readfirstlane(p.lmap.idx[blockIdx.x / D]), d = blockIdx.x % D, b0 = blockIdx.y * kRows;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
    const int u = wave * 16 + r;
    const bool ok_u = u < H;
    const uint32_t DH = (uint32_t)(D * H), G4 = DH * 4;
    const buf_t gates = make_buf_(p.gates + li * p.sGi, (int64_t)Tn * B * G4 * 4);
    const buf_t cbuf = make_buf_(p.c + li * p.sCi + (int64_t)d * Tn * B * H, (int64_t)Tn * B * H * 4);
    const buf_t dy = make_buf_(p.dy + li * p.sDYi, (int64_t)Tn * B * DH * 4);
    const buf_t da = make_buf_((const T*)p.da + li * p.sDAi, (int64_t)Tn * B * G4 * sizeof(T));

    uint32_t vg[4], vc[4], vy[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t row = b0 + 4 * g + i;
        const bool ok = ok_u && (int)row < B;
        vg[i] = ok ? (row * G4 + d * 4 * H + u) * 4u : kOutOfRange;
        vc[i] = ok ? (row * H + u) * 4u : kOutOfRange;
        vy[i] = ok ? (row * DH + d * H + u) * 4u : kOutOfRange;
    }
    struct In { float dy[4], c[4], gate[4][4]; };
    auto load_in = [&](int s, In& in) {                    // s = T: the cell state before the first frame is 0
        const bool end = s >= Tn;
        const uint32_t m = (uint32_t)(d == 0 ? Tn - 1 - (end ? Tn - 1 : s) : (end ? Tn - 1 : s)) * B;   // reverse of the forward order
#pragma unroll
        for (int i = 0; i < 4; ++i) in.c[i] = buf_load_(cbuf, end ? kOutOfRange : vc[i], m * H * 4u);
#pragma unroll
        for (int i = 0; i < 4; ++i) in.dy[i] = buf_load_(dy, vy[i], m * DH * 4u);
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < 4; ++i) in.gate[q][i] = buf_load_(gates, vg[i], (m * G4 + q * H) * 4u);
    };
    In ia, ib;
    load_in(0, ia);
    uint4 w[4][NCH];
    {
        const T* wcol = (const T*)p.wh + li * p.sWi + d * p.sWd + (ok_u ? u : 0);      // W_h[k][u] at wcol[k*H]
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int c = 0; c < NCH; ++c) {
                const int k = c * C::KC + g * C::EL;
                w[q][c] = ok_u && k < H ? column_frag_(wcol + ((int64_t)q * H + k) * H, H) : make_uint4(0u, 0u, 0u, 0u);
            }
    }
    for (int i = threadIdx.x; i < (int)sizeof(lds) / 4; i += blockDim.x) ((uint32_t*)lds)[i] = 0u;

    float dcr[4] = {0.f, 0.f, 0.f, 0.f}, bs[4] = {0.f, 0.f, 0.f, 0.f};
    auto frame = [&](int s, const In& in, In& next) {
        const uint32_t m = (uint32_t)(d == 0 ? Tn - 1 - s : s) * B;
        load_in(s + 1, next);
        lds_barrier_();                                   // da of the frame before is complete (s = 0: the zero fill)
        const char* arow = lds + ((s + 1) & 1) * (kRows * C::BWD_ROW) + r * C::BWD_ROW + g * 16;
        f32x4_t part[4];                                  // one chain per gate
#pragma unroll
        for (int q = 0; q < 4; ++q) part[q] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < NCH; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q) mma16_<T>(part[q], *(const uint4*)(arow + (q * NCH + c) * 64), w[q][c]);
        const f32x4_t acc = (part[0] + part[1]) + (part[2] + part[3]);
        T* aout = (T*)(lds + (s & 1) * (kRows * C::BWD_ROW)) + 4 * g * (C::BWD_ROW / (int)sizeof(T)) + (ok_u ? u : 4 * C::KP);
        const int qs = ok_u ? C::KP : 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            // rows past the batch and units past H: all gates were read as 0, so all four results are 0
            const float dh = in.dy[i] + acc[i], ig = in.gate[0][i], fg = in.gate[1][i], gg = in.gate[2][i], og = in.gate[3][i];
            const float tc = tanhf_(in.c[i]);
            const float dov = dh * tc;
            const float dcv = dcr[i] + dh * og * (1.f - tc * tc);
            const float di = dcv * gg, dg = dcv * ig, df = dcv * next.c[i];            // next.c: the cell state before t
            dcr[i] = dcv * fg;
            const float a[4] = {di * ig * (1.f - ig), df * fg * (1.f - fg), dg * (1.f - gg * gg), dov * og * (1.f - og)};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                bs[q] += a[q];
                const T v = Elem<T>::from(a[q]);
                aout[i * (C::BWD_ROW / (int)sizeof(T)) + q * qs] = v;
                buf_store_(v, da, vg[i] == kOutOfRange ? kOutOfRange : vg[i] / (4u / (uint32_t)sizeof(T)), (m * G4 + q * H) * (uint32_t)sizeof(T));
            }
        }
    };
    frame(0, ia, ib);
    int s = 1;
    for (; s + 1 < Tn; s += 2) { frame(s, ib, ia); frame(s + 1, ia, ib); }
    if (s < Tn) frame(s, ib, ia);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float v = bs[q] + __shfl_xor(bs[q], 16);
        v += __shfl_xor(v, 32);
        if (g == 0 && ok_u) p.dbp[li * p.sDBi + (int64_t)blockIdx.y * G4 + (int64_t)d * 4 * H + (int64_t)q * H + u] = v;
    }
}

template <typename T, int NCH> void launch_cu_t(const RecDesc& d, bool backward, hipStream_t s) {
    const dim3 grid((unsigned)(d.L * d.D), (unsigned)((d.B + kRows - 1) / kRows)), block((unsigned)(64 * ((d.H + 15) / 16)));
    if (backward) hipLaunchKernelGGL((rec_backward_cu_kernel<T, NCH>), grid, block, 0, s, d);
    else hipLaunchKernelGGL((rec_forward_cu_kernel<T, NCH>), grid, block, 0, s, d);
}

}  // namespace

bool rec_resident_supported(const RecDesc& d) {
    // (every tensor of a learner below 2 GiB: the buffer offsets of the kernels)
    return d.direct && d.H <= 128 && rec_aligned(d) && (int64_t)d.T * d.B * d.D * d.H * 16 < (int64_t)kOutOfRange && d.L >= 1 && d.L <= 128 && d.D >= 1 && d.D <= 2 && d.B >= 1 && d.T >= 1;
}

int rec_resident_batch_tiles(const RecDesc& d) { return (d.B + kRows - 1) / kRows; }

hipError_t launch_rec_resident(const RecDesc& d, bool backward, hipStream_t s) {
    if (!rec_resident_supported(d)) return hipErrorInvalidValue;
    if (d.precision == 0) {
        if (d.H <= 32) launch_cu_t<float, 2>(d, backward, s);
        else if (d.H <= 64) launch_cu_t<float, 4>(d, backward, s);
        else if (d.H <= 96) launch_cu_t<float, 6>(d, backward, s);
        else launch_cu_t<float, 8>(d, backward, s);
    } else {
        if (d.H <= 32) launch_cu_t<bf16_t, 1>(d, backward, s);
        else if (d.H <= 64) launch_cu_t<bf16_t, 2>(d, backward, s);
        else if (d.H <= 96) launch_cu_t<bf16_t, 3>(d, backward, s);
        else launch_cu_t<bf16_t, 4>(d, backward, s);
    }
    return hipGetLastError();
}

}  // namespace adpsgd
