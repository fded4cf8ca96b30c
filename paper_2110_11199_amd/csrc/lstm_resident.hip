// Recurrent LSTM kernels that keep W_h on one compute unit: all T frames of one layer in one launch, for hidden sizes up to 128.
//
// A step of such a model is a few hundred thousand multiply-adds per (learner, direction): launched frame by frame it is bound by
// the launch itself, by reading W_h again and by the latency of the reduction over the contraction.  Batch rows do not depend
// on each other, so a workgroup here takes 16 batch rows of one (learner, direction) through ALL frames (or 4: the second pair
// of kernels) and needs nothing from any other workgroup: no launch, no global round trip and no wait between frames.  us per
// frame (forward / backward), frame by frame against here: four rows at a time fp32 4 x 64 cells, batch 4: 8.2 / 6.4 -> 0.9 / 1.1, 32 x
// 128, 64: 10 / 9 -> 3.9 / 4.3, bf16 16 x 128, 16: 5.8 / 5.9 -> 1.1 / 1.3; sixteen fp32 128 x 128, 128: 33 / 40 -> 26 / 32 (the fp32
// products of one compute unit, 3.5 a frame and block, four blocks to each), bf16 128 x 128, 128: 19.8 / 25.0 -> 15.8 / 16.4 (the
// cell arithmetic of two waves per SIMD).
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
#include <type_traits>
#include "gemm_core.hpp"
#include "kernels.hpp"
#include "rec_tiles.hpp"

namespace adpsgd {
namespace {

// ---- 16 batch rows to a workgroup ------------------------------------------------------------------
constexpr int kRows = 16;

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

// ---- four batch rows to a workgroup ---------------------------------------------------------------
// Small batches, and batches whose blocks of four rows still leave the chip free: a 16-row tile of 4 rows does 16 rows' products
// (fp32: 0.9 us of a 1.8 us frame at 64 cells), and its lanes finish four cells one after another.  Here the products are 4x4
// MFMAs of 16 blocks: one instruction multiplies four rows (the same for all blocks: cbsz = 4, abid picks the block that
// holds k) with 64 columns, a lane per column, and after a 4x4 transposition between lane groups a lane finishes ONE cell.
//   A: lane 4 b + i of register m holds row i at k = 16 m + b (bf16: k = 64 m + 4 b .. + 3)      B: lane = column
//   accumulator element i: row i, column = lane.
// Forward: the 64 columns of a wave are the four gates of its 16 units.  Backward: a wave multiplies the da of its own 16 units
// (which it has in registers: one lane permutation) with their 64 rows of W_h, and the waves' partial sums meet in LDS.
typedef __attribute__((ext_vector_type(4))) short s16x4_t;
template <int LO, int HI, class Fn> __device__ inline void for_(Fn&& f) {
    if constexpr (LO < HI) { f(std::integral_constant<int, LO>{}); for_<LO + 1, HI>(f); }
}

template <typename T, int KP> struct Row4 {                // KP: H rounded up to 32
    static constexpr bool F32 = sizeof(T) == 4;
    static constexpr int NB = (KP + 63) / 64;              // column blocks (backward), register pairs of A (bf16)
    static constexpr int NA = F32 ? KP / 16 : NB;          // A registers (pairs)
    static constexpr int NK = F32 ? KP : KP / 4;           // MFMAs of a contraction over KP
    // LDS bytes of h: fp32 a lane's NA words together; bf16 rows of NB * 128 bytes, 32 banks apart
    static constexpr int H_ROW = NB == 1 ? 128 : 384, H_BYTES = F32 ? 64 * NA * 4 : 4 * H_ROW;
};
template <typename T> struct Frag4;
template <> struct Frag4<float> { typedef float type; };
template <> struct Frag4<bf16_t> { typedef s16x4_t type; };
template <int ABID> __device__ inline void mma4_(f32x4_t& acc, float a, float b) { acc = __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, acc, 4, ABID, 0); }
template <int ABID> __device__ inline void mma4_(f32x4_t& acc, s16x4_t a, s16x4_t b) { acc = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(a, b, acc, 4, ABID, 0); }

// element i of lane group g  <->  element g of lane group i (groups of 16 lanes)
__device__ inline void transpose_groups_(float (&v)[4]) {
    auto swap = [](float& x, float& y, auto wide) {
        const auto r = [&] {
            if constexpr (decltype(wide)::value) return __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, y), false, false);
            else return __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, x), __builtin_bit_cast(uint32_t, y), false, false);
        }();
        x = __builtin_bit_cast(float, (uint32_t)r[0]); y = __builtin_bit_cast(float, (uint32_t)r[1]);
    };
    swap(v[0], v[2], std::true_type{}); swap(v[1], v[3], std::true_type{});
    swap(v[0], v[1], std::false_type{}); swap(v[2], v[3], std::false_type{});
}

template <typename T, int KP>
__global__ __launch_bounds__(512) void rec_forward_row4_kernel(RecDesc p) {
    typedef Row4<T, KP> C;
    typedef typename Frag4<T>::type frag_t;
    __shared__ __attribute__((aligned(16))) char lds[2 * C::H_BYTES];
    const int D = p.D, H = p.H, B = p.B, Tn = p.T;
    const int li = __builtin_amdgcn_readfirstlane(p.lmap.idx[blockIdx.x / D]), d = blockIdx.x % D, b0 = blockIdx.y * 4;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4, u = wave * 16 + (lane & 15);
    const bool ok_u = u < H, ok = ok_u && b0 + g < B;
    const uint32_t DH = (uint32_t)(D * H), G4 = DH * 4;
    const buf_t gates = make_buf_(p.gates + li * p.sGi, (int64_t)Tn * B * G4 * 4);
    const buf_t cbuf = make_buf_(p.c + li * p.sCi + (int64_t)d * Tn * B * H, (int64_t)Tn * B * H * 4);
    const buf_t y = make_buf_((const T*)p.y + li * p.sYi, (int64_t)Tn * B * DH * sizeof(T));

    frag_t wf[C::NK];                                      // row (gate g, unit u) of W_h: this lane's column of the products
    {
        const buf_t wh = make_buf_((const T*)p.wh + li * p.sWi + d * p.sWd, (int64_t)4 * H * H * sizeof(T));
        const uint32_t row = ok_u ? (uint32_t)((g * H + u) * H) * (uint32_t)sizeof(T) : kOutOfRange;
        constexpr int EL = 16 / (int)sizeof(T);
#pragma unroll
        for (int k = 0; k < KP; k += EL) {                 // H is a multiple of 4
            uint4 v = buf_load16_(wh, k < H ? row : kOutOfRange, (uint32_t)(k * (int)sizeof(T)));
            if (k + EL > H) v.z = v.w = 0u;                // bf16, H = 4 mod 8: half a chunk
            if constexpr (C::F32) {
                wf[k] = __builtin_bit_cast(float, v.x); wf[k + 1] = __builtin_bit_cast(float, v.y);
                wf[k + 2] = __builtin_bit_cast(float, v.z); wf[k + 3] = __builtin_bit_cast(float, v.w);
            } else {
                wf[k / 4] = __builtin_bit_cast(s16x4_t, make_uint2(v.x, v.y));
                wf[k / 4 + 1] = __builtin_bit_cast(s16x4_t, make_uint2(v.z, v.w));
            }
        }
    }
    for (int i = threadIdx.x; i < (int)sizeof(lds) / 4; i += blockDim.x) ((uint32_t*)lds)[i] = 0u;   // k past H stays zero
    // this lane's cell: row b0 + g, unit u
    const uint32_t vg = ok ? ((uint32_t)(b0 + g) * G4 + d * 4 * H + u) * 4u : kOutOfRange;
    const uint32_t vc = ok ? ((uint32_t)(b0 + g) * H + u) * 4u : kOutOfRange;
    const uint32_t vy = ok ? ((uint32_t)(b0 + g) * DH + d * H + u) * (uint32_t)sizeof(T) : kOutOfRange;
    auto load_pre = [&](int s, float (&a)[4]) {
        const uint32_t m = (uint32_t)(d == 0 ? s : Tn - 1 - s) * B;
#pragma unroll
        for (int q = 0; q < 4; ++q) a[q] = buf_load_(gates, vg, (m * G4 + q * H) * 4u);
    };
    float c = 0.f;
    auto frame = [&](int s, const float (&pre)[4], float (&next)[4]) {
        const uint32_t m = (uint32_t)(d == 0 ? s : Tn - 1 - s) * B;
        load_pre(s + 1 < Tn ? s + 1 : s, next);
        lds_barrier_();                                    // h of the frame before is complete (s = 0: the zero fill, h = 0)
        const char* hb = lds + ((s + 1) & 1) * C::H_BYTES;
        frag_t af[C::NA];
#pragma unroll
        for (int i = 0; i < C::NA; ++i) {
            if constexpr (C::F32) af[i] = ((const float*)hb)[lane * C::NA + i];
            else af[i] = *(const s16x4_t*)(hb + (lane & 3) * C::H_ROW + i * 128 + (lane >> 2) * 8);
        }
        f32x4_t acc[4];                                    // four chains
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        for_<0, C::NK>([&](auto k_) {
            constexpr int k = decltype(k_)::value;
            mma4_<k % 16>(acc[k & 3], af[k / 16], wf[k]);
        });
        const f32x4_t sum = (acc[0] + acc[1]) + (acc[2] + acc[3]);
        float a[4] = {sum[0], sum[1], sum[2], sum[3]};
        transpose_groups_(a);                              // rows of one gate -> gates of one row
        const float ig = sigmoidf_(pre[0] + a[0]), fg = sigmoidf_(pre[1] + a[1]), gg = tanhf_(pre[2] + a[2]), og = sigmoidf_(pre[3] + a[3]);
        c = fg * c + ig * gg;
        const T h = Elem<T>::from(og * tanhf_(c));         // (0 for units past H; rows past the batch are read by no valid row)
        char* ho = lds + (s & 1) * C::H_BYTES;
        if constexpr (C::F32) ((float*)ho)[((u & 15) * 4 + g) * C::NA + (u >> 4)] = h;
        else *(T*)(ho + g * C::H_ROW + u * 2) = h;
        buf_store_(ig, gates, vg, (m * G4 + 0 * H) * 4u);
        buf_store_(fg, gates, vg, (m * G4 + 1 * H) * 4u);
        buf_store_(gg, gates, vg, (m * G4 + 2 * H) * 4u);
        buf_store_(og, gates, vg, (m * G4 + 3 * H) * 4u);
        buf_store_(c, cbuf, vc, m * H * 4u);
        buf_store_(h, y, vy, m * DH * (uint32_t)sizeof(T));
    };
    float pa[4], pb[4];
    load_pre(0, pa);
    frame(0, pa, pb);                                      // (outside the loop, so that the loop is entered with its stores in flight)
    int s = 1;
    for (; s + 1 < Tn; s += 2) { frame(s, pb, pa); frame(s + 1, pa, pb); }
    if (s < Tn) frame(s, pb, pa);
}

template <typename T, int KP>
__global__ __launch_bounds__(512) void rec_backward_row4_kernel(RecDesc p) {
    typedef Row4<T, KP> C;
    typedef typename Frag4<T>::type frag_t;
    constexpr int NK = C::F32 ? 64 : 16;                   // MFMAs of a column block: k = 16 gate + unit; bf16: unit, its four gates
    __shared__ float4 red[2][KP / 16][C::NB * 64];         // partial dh of four rows: [frame parity][wave][column]
    const int D = p.D, H = p.H, B = p.B, Tn = p.T;
    const int li = __builtin_amdgcn_readfirstlane(p.lmap.idx[blockIdx.x / D]), d = blockIdx.x % D, b0 = blockIdx.y * 4;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, g = lane >> 4, u = wave * 16 + (lane & 15), waves = blockDim.x >> 6;
    const bool ok_u = u < H, ok = ok_u && b0 + g < B;
    const uint32_t DH = (uint32_t)(D * H), G4 = DH * 4;
    const buf_t gates = make_buf_(p.gates + li * p.sGi, (int64_t)Tn * B * G4 * 4);
    const buf_t cbuf = make_buf_(p.c + li * p.sCi + (int64_t)d * Tn * B * H, (int64_t)Tn * B * H * 4);
    const buf_t dy = make_buf_(p.dy + li * p.sDYi, (int64_t)Tn * B * DH * 4);
    const buf_t da = make_buf_((const T*)p.da + li * p.sDAi, (int64_t)Tn * B * G4 * sizeof(T));
    const uint32_t vg = ok ? ((uint32_t)(b0 + g) * G4 + d * 4 * H + u) * 4u : kOutOfRange;
    const uint32_t vc = ok ? ((uint32_t)(b0 + g) * H + u) * 4u : kOutOfRange;
    const uint32_t vy = ok ? ((uint32_t)(b0 + g) * DH + d * H + u) * 4u : kOutOfRange;
    const uint32_t va = ok ? vg / (4u / (uint32_t)sizeof(T)) : kOutOfRange;
    struct In { float dy, c, gate[4]; };
    auto load_in = [&](int s, In& in) {                    // s = T: the cell state before the first frame is 0
        const bool end = s >= Tn;
        const uint32_t m = (uint32_t)(d == 0 ? Tn - 1 - (end ? Tn - 1 : s) : (end ? Tn - 1 : s)) * B;   // reverse of the forward order
        in.c = buf_load_(cbuf, end ? kOutOfRange : vc, m * H * 4u);
        in.dy = buf_load_(dy, vy, m * DH * 4u);
#pragma unroll
        for (int q = 0; q < 4; ++q) in.gate[q] = buf_load_(gates, vg, (m * G4 + q * H) * 4u);
    };
    // Inputs are requested AHEAD frames before their use: a frame of 64 cells in fp32 is shorter than an access to memory (4 learners x 64 cells, batch
    // 4: 68.0 -> 66.1 us an iteration with 3 frames ahead, 8 x 2 x 128, batch 16, 101 frames 172 -> 164 a pass); in bf16 more frames of code
    // cost more than they bring (8 x 2 x 128, batch 16, 101 frames 96 -> 99), as they do forward.
    constexpr int AHEAD = C::F32 ? 3 : 1, R = AHEAD + 1;
    In in[R];                                              // frame s: in[s % R]
#pragma unroll
    for (int s = 0; s < AHEAD; ++s) load_in(s, in[s]);
    frag_t wf[C::NB][NK];                                  // rows of this wave's units, column 64 cb + lane
    {
        const buf_t wh = make_buf_((const T*)p.wh + li * p.sWi + d * p.sWd, (int64_t)4 * H * H * sizeof(T));
#pragma unroll
        for (int cb = 0; cb < C::NB; ++cb) {
            const int n = cb * 64 + lane;
            const uint32_t col = n < H ? (uint32_t)(wave * 16 * H + n) * (uint32_t)sizeof(T) : kOutOfRange;
#pragma unroll
            for (int b = 0; b < 16; ++b) {
                const uint32_t v = wave * 16 + b < H ? col : kOutOfRange;
                if constexpr (C::F32) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) wf[cb][q * 16 + b] = buf_load_(wh, v, (uint32_t)((q * H + b) * H) * 4u);
                } else {
                    uint32_t e[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) e[q] = buf_load2_(wh, v, (uint32_t)((q * H + b) * H) * 2u);
                    wf[cb][b] = __builtin_bit_cast(s16x4_t, make_uint2(e[0] | (e[1] << 16), e[2] | (e[3] << 16)));
                }
            }
        }
    }
    const int from = ((lane & 3) * 16 + (lane >> 2)) * 4;  // lane 4 b + i takes what lane 16 i + b holds
    float dcr = 0.f, bs[4] = {0.f, 0.f, 0.f, 0.f};
    auto frame = [&](int s, const In& in, const In& next, In& ahead) {
        const uint32_t m = (uint32_t)(d == 0 ? Tn - 1 - s : s) * B;
        load_in(s + AHEAD, ahead);
        float dh = in.dy;
        if (s > 0) {
            lds_barrier_();                                // the partial sums of the frame before are complete
            float part = 0.f;
#pragma unroll
            for (int w = 0; w < KP / 16; ++w)
                if (w < waves) part += ((const float*)red[(s + 1) & 1][w])[u * 4 + g];
            dh += part;
        }
        // rows past the batch and units past H: all gates were read as 0, so all four results are 0
        const float ig = in.gate[0], fg = in.gate[1], gg = in.gate[2], og = in.gate[3];
        const float tc = tanhf_(in.c);
        const float dov = dh * tc;
        const float dcv = dcr + dh * og * (1.f - tc * tc);
        const float di = dcv * gg, dg = dcv * ig, df = dcv * next.c;                   // next.c: the cell state before t
        dcr = dcv * fg;
        const float a[4] = {di * ig * (1.f - ig), df * fg * (1.f - fg), dg * (1.f - gg * gg), dov * og * (1.f - og)};
        frag_t af[C::F32 ? 4 : 1];
        if constexpr (C::F32) {
#pragma unroll
            for (int q = 0; q < 4; ++q) af[q] = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(from, __builtin_bit_cast(int, a[q])));
        } else {
            const uint32_t lo = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)pack_bf16(a[0], a[1]));
            const uint32_t hi = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)pack_bf16(a[2], a[3]));
            af[0] = __builtin_bit_cast(s16x4_t, make_uint2(lo, hi));
        }
        f32x4_t acc[C::NB][2];                             // two chains to a column block
#pragma unroll
        for (int cb = 0; cb < C::NB; ++cb)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[cb][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        for_<0, NK>([&](auto k_) {
            constexpr int k = decltype(k_)::value;
#pragma unroll
            for (int cb = 0; cb < C::NB; ++cb) mma4_<k % 16>(acc[cb][k & 1], af[k / 16], wf[cb][k]);
        });
#pragma unroll
        for (int cb = 0; cb < C::NB; ++cb) {
            const f32x4_t v = acc[cb][0] + acc[cb][1];
            red[s & 1][wave][cb * 64 + lane] = make_float4(v[0], v[1], v[2], v[3]);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            bs[q] += a[q];
            buf_store_(Elem<T>::from(a[q]), da, va, (m * G4 + q * H) * (uint32_t)sizeof(T));
        }
    };
    frame(0, in[0], in[1 % R], in[AHEAD]);
    int s = 1;
    for (; s + AHEAD < Tn; s += R) {
#pragma unroll
        for (int i = 0; i < R; ++i) frame(s + i, in[(1 + i) % R], in[(2 + i) % R], in[i]);
    }
#pragma unroll
    for (int i = 0; i < AHEAD; ++i)
        if (s + i < Tn) frame(s + i, in[(1 + i) % R], in[(2 + i) % R], in[i]);
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

template <typename T, int KP> void launch_row4_t(const RecDesc& d, bool backward, hipStream_t s) {
    const dim3 grid((unsigned)(d.L * d.D), (unsigned)((d.B + 3) / 4)), block((unsigned)(64 * ((d.H + 15) / 16)));
    if (backward) hipLaunchKernelGGL((rec_backward_row4_kernel<T, KP>), grid, block, 0, s, d);
    else hipLaunchKernelGGL((rec_forward_row4_kernel<T, KP>), grid, block, 0, s, d);
}
template <typename T> void launch_row4(const RecDesc& d, bool backward, hipStream_t s) {
    if (d.H <= 32) launch_row4_t<T, 32>(d, backward, s);
    else if (d.H <= 64) launch_row4_t<T, 64>(d, backward, s);
    else if (d.H <= 96) launch_row4_t<T, 96>(d, backward, s);
    else launch_row4_t<T, 128>(d, backward, s);
}

// Four rows to a workgroup up to three workgroups per compute unit.  us per frame, forward / backward, 16 rows against 4 (workgroups of
// four rows): fp32 4 x 64 cells, batch 4 (4) 1.9 / 2.2 against 0.9 / 1.1; 16 x 128, 16 (64) 5.7 / 6.3 against 2.0 / 2.1; 32 x 128, 64
// (512) 6.2 / 7.3 against 3.9 / 4.3; bf16 16 x 128, 16 (64) 2.1 / 2.5 against 1.1 / 1.3; 32 x 64, 64 (512) 1.5 / 1.6 against 1.2 / 1.3;
// 32 x 128, 160 (1280) 6.3 / 6.5 against 6.3 / 6.3; 64 x 128, 160 (2560) 10.6 / 10.8 against 13.1 / 12.4.
bool row4_blocks(const RecDesc& d) { return (int64_t)d.L * d.D * ((d.B + 3) / 4) <= 768; }

}  // namespace

// From two frames on: a single one needs no W_h, which a launch here begins with (64 x 112 cells, batch 32, fp32, 9.8 / 9.3 us frame by
// frame against 19.4 / 24.0), but where W_h's rows are not 16-byte aligned the kernels of a single frame are the longer all
// the same (64 x 4, 15, bf16: 10.2 against 6.5).  Two frames: 32 x 128, 64 15 / 14 against 17 / 19; 128 x 24, 123 23 / 23 against 12 / 12.
bool rec_resident_supported(const RecDesc& d) {
    // (every tensor of a learner below 2 GiB: the buffer offsets of the kernels)
    if (!rec_aligned(d) && !(rec_quad_aligned(d) && row4_blocks(d))) return false;
    if (rec_resident_batch_tiles(d) > 65535) return false;                             // the second dimension of a grid
    if (d.T < 1 || (d.T == 1 && rec_aligned(d))) return false;
    return d.direct && d.H <= 128 && (int64_t)d.T * d.B * d.D * d.H * 16 < (int64_t)kOutOfRange && d.L >= 1 && d.L <= 128 && d.D >= 1 && d.D <= 2 && d.B >= 1;
}

int rec_resident_batch_tiles(const RecDesc& d) { const int rows = row4_blocks(d) ? 4 : kRows; return (d.B + rows - 1) / rows; }

hipError_t launch_rec_resident(const RecDesc& d, bool backward, hipStream_t s) {
    if (!rec_resident_supported(d)) return hipErrorInvalidValue;
    if (row4_blocks(d)) {
        if (d.precision) launch_row4<bf16_t>(d, backward, s);
        else launch_row4<float>(d, backward, s);
        return hipGetLastError();
    }
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
