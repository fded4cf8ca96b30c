// Per-time-step LSTM kernels: the recurrent GEMM h_{t'} W_h' on MFMA with the
// gate non-linearities and the cell update fused into its epilogue (forward),
// and the recurrent gradient GEMM da W_h with the cell backward fused into its
// epilogue (backward through time).  One launch advances every learner and both
// directions of one layer by one frame.
//
// LSTM cell (vanilla, gate blocks i,f,g,o):
//   a = W_x x_t + b + W_h h_{t'}          i,f,o = sigmoid(a), g = tanh(a)
//   c_t = f c_{t'} + i g                  h_t = o tanh(c_t)
// with t' the previously processed frame (t-1 forward, t+1 backward direction)
// and h = c = 0 before the first processed frame of a segment.
//
// Each launch re-streams every learner's W_h from HBM (weights are not shared
// between learners), so these kernels are bound by HBM bandwidth and latency, not
// by MFMA: the bf16 versions feed LDS with direct global->LDS loads several stages
// ahead; the backward one reads W_h rows-contiguous (dh = da W_h contracts over the
// rows of W_h) and transposes on the LDS read.
#include "gemm_core.hpp"
#include "gemm_dma.hpp"
#include "kernels.hpp"

namespace adpsgd {

// ---- epilogues -------------------------------------------------------------------

// The gate, cell-state and dY tensors are touched once per launch and are far larger than the caches:
// their loads and stores carry the non-temporal hint, so that they do not displace the operands that
// are shared between workgroups (measured: -10 % forward, -8 % backward).  What the next launch reads
// back as a GEMM operand (h, da) is stored normally.
//
// Inputs of the forward epilogue, loaded BEFORE the recurrent GEMM so that their HBM
// latency hides behind it: the four pre-activations W_x x + b and c_{t'} of the 16
// (batch row, unit) positions a lane owns.
struct FwdInputs { float a[4][16]; float c_prev[16]; };

template <typename T, class Core>
__device__ inline void forward_prefetch(const RecDesc& p, FwdInputs& in, int li, int d, int t, int tp, int u0, int b0) {
    const int D = p.D, H = p.H, B = p.B;
    const int64_t G4 = (int64_t)D * 4 * H;
    const int n0c = Core::acc_col(0);
    const int u = u0 + 32 * (n0c >> 7) + (n0c & 31);
    const float* gates = p.gates + li * p.sGi;
    const float* cbuf = p.c + li * p.sCi + (int64_t)d * p.T * B * H;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int row = b0 + Core::acc_row(0, i);
        const bool ok = row < B && u < H;
        const float* gp = gates + ((int64_t)t * B + (ok ? row : 0)) * G4 + (int64_t)d * 4 * H + (ok ? u : 0);
#pragma unroll
        for (int g = 0; g < 4; ++g) in.a[g][i] = ok ? __builtin_nontemporal_load(gp + (int64_t)g * H) : 0.f;
        in.c_prev[i] = (ok && p.step > 0) ? __builtin_nontemporal_load(cbuf + ((int64_t)tp * B + row) * H + u) : 0.f;
    }
}

// acc[0][gate][i]: gate pre-activation contributions h W_h' for unit u (per lane) and
// batch rows Core::acc_row(0, i).
template <typename T, class Core>
__device__ inline void forward_epilogue(const RecDesc& p, f32x16_t (&acc)[1][4], FwdInputs& in, int li, int d,
                                        int t, int u0, int b0) {
    const int D = p.D, H = p.H, B = p.B;
    const int64_t DH = (int64_t)D * H, G4 = (int64_t)D * 4 * H;
    // tile column n = 128*wave_n + 32*gate + j holds gate `gate` of unit u0 + 32*wave_n + j
    const int n0c = Core::acc_col(0);
    const int u = u0 + 32 * (n0c >> 7) + (n0c & 31);
    if (u >= H) return;
    float* gates = p.gates + li * p.sGi;
    float* cbuf = p.c + li * p.sCi + (int64_t)d * p.T * B * H;
    T* y = (T*)p.y + li * p.sYi;
    // All results are computed first, each into a register of its own, and stored afterwards: a store
    // whose data register is reused by later arithmetic would have to complete before that arithmetic.
    float hv[16];
    uint32_t hb[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const float ig = sigmoidf_(in.a[0][i] + acc[0][0][i]);
        const float fg = sigmoidf_(in.a[1][i] + acc[0][1][i]);
        const float gg = tanhf_(in.a[2][i] + acc[0][2][i]);
        const float og = sigmoidf_(in.a[3][i] + acc[0][3][i]);
        const float cc = fg * in.c_prev[i] + ig * gg;
        acc[0][0][i] = ig; acc[0][1][i] = fg; acc[0][2][i] = gg; acc[0][3][i] = og;
        hv[i] = og * tanhf_(cc);
        if constexpr (sizeof(T) == 2) hb[i] = f32_to_bf16(hv[i]);
        in.c_prev[i] = cc;
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int row = b0 + Core::acc_row(0, i);
        if (row >= B) continue;
        float* gp = gates + ((int64_t)t * B + row) * G4 + (int64_t)d * 4 * H + u;
        __builtin_nontemporal_store(acc[0][0][i], gp); __builtin_nontemporal_store(acc[0][1][i], gp + H); __builtin_nontemporal_store(acc[0][2][i], gp + 2 * (int64_t)H); __builtin_nontemporal_store(acc[0][3][i], gp + 3 * (int64_t)H);
        __builtin_nontemporal_store(in.c_prev[i], cbuf + ((int64_t)t * B + row) * H + u);
        if constexpr (sizeof(T) == 2) y[((int64_t)t * B + row) * DH + (int64_t)d * H + u] = (bf16_t)hb[i];
        else y[((int64_t)t * B + row) * DH + (int64_t)d * H + u] = hv[i];
    }
}

// Backward through one frame: dh_t = dY_t + da_{t''} W_h (t'' = the frame
// processed just before in backward order; acc holds that product), then
//   do = dh tanh(c_t)            dc = dc_rec + dh o (1 - tanh^2 c_t)
//   di = dc g, dg = dc i, df = dc c_{t'}, dc_rec <- dc f
//   da = (di i(1-i), df f(1-f), dg (1-g^2), do o(1-o))
template <typename T, class Core, int FN>
__device__ inline void backward_epilogue(const RecDesc& p, f32x16_t (&acc)[1][FN], int li, int d, int t, int tp,
                                         int u0, int b0, char* lds) {
    const int D = p.D, H = p.H, B = p.B;
    const int64_t DH = (int64_t)D * H, G4 = (int64_t)D * 4 * H;
    const bool has_prev = tp >= 0 && tp < p.T;
    const float* gates = p.gates + li * p.sGi;
    const float* cbuf = p.c + li * p.sCi + (int64_t)d * p.T * B * H;
    const float* dy = p.dy + li * p.sDYi;
    float* dcb = p.dc + li * p.sDCi + (int64_t)d * B * H;
    T* da = (T*)p.da + li * p.sDAi;
    float cs[FN][4];                          // sums of the four da values over this lane's 16 rows
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
        cs[fn][0] = cs[fn][1] = cs[fn][2] = cs[fn][3] = 0.f;
        const int u = u0 + Core::acc_col(fn);
        if (u >= H) continue;
        // load everything, compute everything, store everything (see the forward epilogue)
        float dyv[16], gi[16], gf[16], gg[16], go[16], cv[16], cp[16], dcr[16];
        uint32_t pk0[16], pk1[16];            // bf16 results packed two per register (i,f) and (g,o)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int row = b0 + Core::acc_row(0, i);
            const bool ok = row < B;
            const int64_t m = (int64_t)t * B + (ok ? row : 0);
            const float* gp = gates + m * G4 + (int64_t)d * 4 * H + u;
            dyv[i] = ok ? __builtin_nontemporal_load(dy + m * DH + (int64_t)d * H + u) : 0.f;
            gi[i] = ok ? __builtin_nontemporal_load(gp) : 0.f; gf[i] = ok ? __builtin_nontemporal_load(gp + H) : 0.f;
            gg[i] = ok ? __builtin_nontemporal_load(gp + 2 * (int64_t)H) : 0.f; go[i] = ok ? __builtin_nontemporal_load(gp + 3 * (int64_t)H) : 0.f;
            cv[i] = ok ? __builtin_nontemporal_load(cbuf + m * H + u) : 0.f;
            cp[i] = (ok && has_prev) ? __builtin_nontemporal_load(cbuf + ((int64_t)tp * B + row) * H + u) : 0.f;
            dcr[i] = (ok && p.step > 0) ? __builtin_nontemporal_load(dcb + (int64_t)row * H + u) : 0.f;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            // rows past the batch: all gates read as 0, so all four results are 0 whatever the accumulator holds
            const float dh = dyv[i] + acc[0][fn][i];
            const float ig = gi[i], fg = gf[i], g2 = gg[i], og = go[i];
            const float tc = tanhf_(cv[i]);
            const float dov = dh * tc;
            const float dcv = dcr[i] + dh * og * (1.f - tc * tc);
            const float di = dcv * g2, dg = dcv * ig, df = dcv * cp[i];
            dcr[i] = dcv * fg;
            float a0 = di * ig * (1.f - ig), a1 = df * fg * (1.f - fg), a2 = dg * (1.f - g2 * g2), a3 = dov * og * (1.f - og);
            cs[fn][0] += a0; cs[fn][1] += a1; cs[fn][2] += a2; cs[fn][3] += a3;
            if constexpr (sizeof(T) == 2) {
                pk0[i] = pack_bf16(a0, a1);
                pk1[i] = pack_bf16(a2, a3);
            } else {
                gi[i] = a0; gf[i] = a1; gg[i] = a2; go[i] = a3;
            }
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int row = b0 + Core::acc_row(0, i);
            if (row >= B) continue;
            const int64_t m = (int64_t)t * B + row;
            __builtin_nontemporal_store(dcr[i], dcb + (int64_t)row * H + u);
            T* dp = da + m * G4 + (int64_t)d * 4 * H + u;
            if constexpr (sizeof(T) == 2) {
                dp[0] = (bf16_t)(pk0[i] & 0xffffu); dp[H] = (bf16_t)(pk0[i] >> 16);
                dp[2 * (int64_t)H] = (bf16_t)(pk1[i] & 0xffffu); dp[3 * (int64_t)H] = (bf16_t)(pk1[i] >> 16);
            } else {
                dp[0] = gi[i]; dp[H] = gf[i]; dp[2 * (int64_t)H] = gg[i]; dp[3 * (int64_t)H] = go[i];
            }
        }
    }
    // Bias gradient: the column sums of da over the rows of this tile, in a fixed order (lane pair, then
    // the waves along the rows through LDS), written as one row of partial sums per (frame, batch tile).
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    static_assert((Core::BN & (Core::BN - 1)) == 0, "the reduction indexing needs a power-of-two tile width");
    float* red = (float*)lds;                 // [kWM][BN][4]
    __syncthreads();                          // the stage buffers are no longer read
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float v = cs[fn][g] + __shfl_xor(cs[fn][g], 32);
            if (lane < 32) red[(((wave / Core::kWN) * Core::BN) + Core::acc_col(fn)) * 4 + g] = v;
        }
    }
    __syncthreads();
    float* out = p.dbp + li * p.sDBi + ((int64_t)t * gridDim.z + blockIdx.z) * G4 + (int64_t)d * 4 * H;
    for (int idx = threadIdx.x; idx < Core::BN * 4; idx += Core::NT) {
        const int col = idx & (Core::BN - 1), g = idx / Core::BN;
        float sum = red[col * 4 + g];
#pragma unroll
        for (int w = 1; w < Core::kWM; ++w) sum += red[(w * Core::BN + col) * 4 + g];
        if (u0 + col < H) out[(int64_t)g * H + u0 + col] = sum;
    }
}

template <int FN> __device__ inline void zero_acc(f32x16_t (&acc)[1][FN]) {
#pragma unroll
    for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[0][j][e] = 0.f;
}

// ---- register-staged versions (any operand type, any shape) ---------------------------

template <typename T, int WM, int WN, int VB>
__global__ __launch_bounds__(256) void rec_forward_kernel(RecDesc p) {
    typedef GemmCore<T, KcSrc<T>, GateSrc<T>, WM, WN, 1, 4, VB> Core;
    __shared__ __attribute__((aligned(16))) char lds[Core::LDS_BYTES];
    const int D = p.D, H = p.H, B = p.B;
    const int li = p.lmap.idx[blockIdx.x / D], d = blockIdx.x % D;      // groups on x: the tiles of one (learner, direction) share an XCD and its L2
    const int t = d == 0 ? p.step : p.T - 1 - p.step;
    const int tp = d == 0 ? t - 1 : t + 1;
    const int u0 = blockIdx.y * (32 * WN), b0 = blockIdx.z * (32 * WM);
    f32x16_t acc[1][4];
    zero_acc<4>(acc);
    FwdInputs in;
    forward_prefetch<T, Core>(p, in, li, d, t, tp, u0, b0);
    if (p.step > 0) {
        KcSrc<T> a;
        a.base = (const T*)p.y + li * p.sYi + ((int64_t)tp * B + b0) * ((int64_t)D * H) + (int64_t)d * H;
        a.ld = (int64_t)D * H; a.R = B - b0;
        GateSrc<T> b;
        b.base = (const T*)p.wh + li * p.sWi + d * p.sWd;
        b.ld = H; b.H = H; b.u0 = u0;
        Core::run(acc, a, b, H, lds);
    }
    forward_epilogue<T, Core>(p, acc, in, li, d, t, u0, b0);
}

template <typename T, int WM, int WN, int FN, int VB>
__global__ __launch_bounds__(256) void rec_backward_kernel(RecDesc p) {
    typedef GemmCore<T, KcSrc<T>, McSrc<T>, WM, WN, 1, FN, VB> Core;
    __shared__ __attribute__((aligned(16))) char lds[Core::LDS_BYTES];
    const int D = p.D, H = p.H, B = p.B;
    const int li = p.lmap.idx[blockIdx.x / D], d = blockIdx.x % D;      // groups on x: the tiles of one (learner, direction) share an XCD and its L2
    const int t = d == 0 ? p.T - 1 - p.step : p.step;     // reverse of the forward processing order
    const int tn = d == 0 ? t + 1 : t - 1;                 // frame handled by the previous launch
    const int tp = d == 0 ? t - 1 : t + 1;                 // frame the forward pass processed before t
    const int u0 = blockIdx.y * Core::BN, b0 = blockIdx.z * Core::BM;
    const int64_t G4 = (int64_t)D * 4 * H;
    f32x16_t acc[1][FN];
    zero_acc<FN>(acc);
    if (p.step > 0) {
        KcSrc<T> a;
        a.base = (const T*)p.da + li * p.sDAi + ((int64_t)tn * B + b0) * G4 + (int64_t)d * 4 * H;
        a.ld = G4; a.R = B - b0;
        McSrc<T> b;
        b.base = (const T*)p.wh + li * p.sWi + d * p.sWd + u0;
        b.ld = H; b.R = H - u0;
        Core::run(acc, a, b, 4 * H, lds);
    }
    backward_epilogue<T, Core, FN>(p, acc, li, d, t, tp, u0, b0, lds);
}

// ---- direct-to-LDS versions (16-byte aligned rows, H a multiple of 16 bytes) -----

// All workgroups of a launch start together and stream their W_h rows (a power-of-two pitch apart)
// at the same pace; walking K from the same offset they would all touch the same column block of
// every row, i.e. the same subset of memory channels, at the same time.  Workgroups therefore
// start their K loops at different stages (measured: 8 % faster backward step, 4 % forward).
// Forward: every tile its own rotation (its shared operand h is small and stays in L2).  Backward:
// one rotation per (learner, direction), so that the tiles of a group still read the same block of
// their shared operand da (1 MB per group) at the same time and fetch it from HBM once.
__device__ inline int stage_rotation_fwd(int nk) { return nk > 1 ? (int)((blockIdx.y * 5 + blockIdx.x * 3) % nk) : 0; }
__device__ inline int stage_rotation_bwd(int nk) { return nk > 1 ? (int)((blockIdx.x * 5) % nk) : 0; }

template <typename T, int WM, int WN, int SB, int NS>
__global__ __launch_bounds__(256) void rec_forward_dma_kernel(RecDesc p) {
    typedef GemmDma<T, KcSrc<T>, GateSrc<T>, WM, WN, 1, 4, SB, NS> Core;
    __shared__ __attribute__((aligned(1024))) char lds[Core::LDS_BYTES];
    const int D = p.D, H = p.H, B = p.B;
    const int li = p.lmap.idx[blockIdx.x / D], d = blockIdx.x % D;      // groups on x: the tiles of one (learner, direction) share an XCD and its L2
    const int t = d == 0 ? p.step : p.T - 1 - p.step;
    const int tp = d == 0 ? t - 1 : t + 1;
    const int u0 = blockIdx.y * (32 * WN), b0 = blockIdx.z * (32 * WM);
    f32x16_t acc[1][4];
    zero_acc<4>(acc);
    FwdInputs in;
    forward_prefetch<T, Core>(p, in, li, d, t, tp, u0, b0);
    if (p.step > 0) {
        KcSrc<T> a;
        a.base = (const T*)p.y + li * p.sYi + ((int64_t)tp * B + b0) * ((int64_t)D * H) + (int64_t)d * H;
        a.ld = (int64_t)D * H; a.R = B - b0;
        GateSrc<T> b;
        b.base = (const T*)p.wh + li * p.sWi + d * p.sWd;
        b.ld = H; b.H = H; b.u0 = u0;
        Core::run(acc, a, b, H, lds, stage_rotation_fwd(H / Core::KT));
    }
    forward_epilogue<T, Core>(p, acc, in, li, d, t, u0, b0);
}

// B operand = W_h itself read rows-contiguous: element (unit u, k = gate row j) at W_h[j*H + u];
// the transposition happens on the LDS read.
template <typename T, int WM, int WN, int FN, int SB, int NS>
__global__ __launch_bounds__(64 * WM * WN) void rec_backward_dma_kernel(RecDesc p) {
    typedef GemmDma<T, KcSrc<T>, McSrc<T>, WM, WN, 1, FN, SB, NS> Core;
    __shared__ __attribute__((aligned(1024))) char lds[Core::LDS_BYTES];
    const int D = p.D, H = p.H, B = p.B;
    const int li = p.lmap.idx[blockIdx.x / D], d = blockIdx.x % D;      // groups on x: the tiles of one (learner, direction) share an XCD and its L2
    const int t = d == 0 ? p.T - 1 - p.step : p.step;
    const int tn = d == 0 ? t + 1 : t - 1;
    const int tp = d == 0 ? t - 1 : t + 1;
    const int u0 = blockIdx.y * Core::BN, b0 = blockIdx.z * Core::BM;
    const int64_t G4 = (int64_t)D * 4 * H;
    f32x16_t acc[1][FN];
    zero_acc<FN>(acc);
    if (p.step > 0) {
        KcSrc<T> a;
        a.base = (const T*)p.da + li * p.sDAi + ((int64_t)tn * B + b0) * G4 + (int64_t)d * 4 * H;
        a.ld = G4; a.R = B - b0;
        McSrc<T> b;
        b.base = (const T*)p.wh + li * p.sWi + d * p.sWd + u0;
        b.ld = H; b.R = H - u0;
        Core::run(acc, a, b, 4 * H, lds, stage_rotation_bwd(4 * H / Core::KT));
    }
    backward_epilogue<T, Core, FN>(p, acc, li, d, t, tp, u0, b0, lds);
}

// ---- launchers ----------------------------------------------------------------------

template <typename T, int VB>
static hipError_t fwd_t(const RecDesc& d, hipStream_t s) {
    const unsigned groups = (unsigned)(d.L * d.D);
    if (d.B > 64) {
        dim3 grid(groups, (d.H + 31) / 32, (d.B + 127) / 128);
        hipLaunchKernelGGL((rec_forward_kernel<T, 4, 1, VB>), grid, dim3(256), 0, s, d);
    } else if (d.B > 32) {
        dim3 grid(groups, (d.H + 63) / 64, (d.B + 63) / 64);
        hipLaunchKernelGGL((rec_forward_kernel<T, 2, 2, VB>), grid, dim3(256), 0, s, d);
    } else {
        dim3 grid(groups, (d.H + 127) / 128, (d.B + 31) / 32);
        hipLaunchKernelGGL((rec_forward_kernel<T, 1, 4, VB>), grid, dim3(256), 0, s, d);
    }
    return hipGetLastError();
}

template <typename T, int VB>
static hipError_t bwd_t(const RecDesc& d, hipStream_t s) {
    const unsigned groups = (unsigned)(d.L * d.D);
    if (d.B > 64) {
        dim3 grid(groups, (d.H + 63) / 64, (d.B + 127) / 128);
        hipLaunchKernelGGL((rec_backward_kernel<T, 4, 1, 2, VB>), grid, dim3(256), 0, s, d);
    } else {
        dim3 grid(groups, (d.H + 127) / 128, (d.B + 31) / 32);
        hipLaunchKernelGGL((rec_backward_kernel<T, 1, 4, 1, VB>), grid, dim3(256), 0, s, d);
    }
    return hipGetLastError();
}

static bool rec_ok(const RecDesc& d) {
    return d.L >= 1 && d.L <= 128 && d.D >= 1 && d.D <= 2 && d.B >= 1 && d.H >= 4 && d.H % 4 == 0 && d.T >= 1 &&
           d.step >= 0 && d.step < d.T;
}

bool rec_aligned(const RecDesc& d) {
    const int epc = d.precision ? 8 : 4;
    return d.H % epc == 0 && (uintptr_t)d.wh % 16 == 0 && d.sWi % epc == 0 && d.sWd % epc == 0 && (uintptr_t)d.y % 16 == 0 &&
           d.sYi % epc == 0 && (uintptr_t)d.da % 16 == 0 && d.sDAi % epc == 0;
}

bool rec_quad_aligned(const RecDesc& d) {
    const int quad = d.precision ? 8 : 16;
    return d.H % 4 == 0 && (uintptr_t)d.wh % quad == 0 && d.sWi % 4 == 0 && d.sWd % 4 == 0;
}

// Which kernels a step runs on.
//   kSplit   32 x 32 tiles, contraction split over the waves (lstm_small.hip): as long as its workgroups fit the chip in
//            one round (two in fp32, whose other tiles are no faster), a step is bound by the latency of the K walk and this
//            one is the shortest.  us per frame (forward / backward), split against direct: fp32 6 x 320 cells, batch
//            64: 16.3 / 16.9 against 29.7 / 32.7; 16 x 256, 128 (512 workgroups): 23.4 / 25.9 against 25.9 / 29.4; bf16 10 x
//            360, 50: 8.4 / 11.4 against 15.0 / 17.4; and on the other side bf16 16 x 512, 64 (512 workgroups) 20.0 / 21.6
//            against 15.5 / 18.9, fp32 32 x 512, 64 (1024) 78 / 94 against 48 / 54.
//            Batches up to 32 leave the rows of a direct tile empty.  fp32 forward: split at any number of workgroups below
//            1024 cells (32 x 640, batch 2: 66 against 87, 32: 75 / 94; 128 x 512, 16: 161 / 229; but 48 x 1024, 1: 202 / 206, 8: 217 /
//            211; 32 x 1520, 2: 294 / 268).  bf16 backward, which reads W_h column by column: up to two rounds where
//            a column stays short (48 x 256, 16: 9.4 / 11.9) or the workgroups of a pair share an XCD and the batch is small
//            (24 x 512, 16: 14.2 / 16.0, 24: 17.0 / 16.7; 16 x 768, 8: 17.5 / 19.3; 8 x 1240, 8: 25 / 27;
//            20 x 768, 8: 27.3 / 19.5); the bf16 forward step is
//            the shorter on the direct kernel past 256 (24 x 512, 16: 15.7 / 13.4).
//   kDirect  the direct-to-LDS kernels.
//   kStaged  register-staged kernels: rows that are not 16-byte aligned, or forced (tuning).  fp32 6 x 320, 64: 31.0 /
//            91.6; 32 x 1024, 128: 317 / 700 against 277 / 299 direct.
//            The direct kernels address W_h of a (learner, direction) by a lane's 32-bit byte offset from its start: a matrix of
//            more than 4 GB (H > 16384 in fp32, 23170 with bf16 operands) is kStaged too, whose addresses have 64 bits.
enum RecKind { kStaged, kDirect, kSplit };

int rec_step_kind(int precision, bool backward, int pairs, int H, int B) {
    const int64_t split_wgs = (int64_t)pairs * ((H + 31) / 32) * ((B + 31) / 32);
    bool split = split_wgs <= (precision ? 256 : 512);
    if (B <= 32 && !precision && !backward) split = split || H < 1024;
    if (B <= 32 && precision && backward) split = split || (split_wgs <= 512 && (H <= 256 || (pairs % 8 == 0 && (H <= 768 ? B <= 16 : split_wgs <= 320 && B <= 8))));
    if (split) return kSplit;
    return (int64_t)4 * H * H * (precision ? 2 : 4) <= (int64_t)1 << 32 ? kDirect : kStaged;
}

static RecKind rec_kind(const RecDesc& d, bool backward) {
    if (!d.direct || !rec_aligned(d)) return kStaged;
    return (RecKind)rec_step_kind(d.precision, backward, d.L * d.D, d.H, d.B);
}

// Rows of a backward direct tile: 128 where that leaves three quarters of the chip a workgroup, else 32 (every batch tile
// reads its W_h slice again, but a launch that fills the chip matters more).  32 against 128 rows, us per frame:
// bf16 16 x 640 cells, batch 96 (80 workgroups of 128 rows): 23.8 against 38.9; fp32 32 x 512, 96 (128): 76 against 148; bf16
// 32 x 512, 128 (128): 35.6 against 44.4; 32 x 1024, 128 (256): 184 against 91, fp32 341 against 299.
// In bf16 the 32-row tiles also have to fit the chip at once, two workgroups to a compute unit (24 x 640, 128: 480 workgroups 38
// against 46; 40 x 512, 128: 640 56 against 49; 24 x 832, 128: 672 70 against 55), all W_h the memory-side cache, which
// serves them again (16 x 1024, 72, 134 MB: 41 against 48; 16 x 1280, 72, 210 MB: 69 against 57; 8 x 2048, 72, 268 MB: 93
// against 78), and the workgroups of a pair few XCDs (20 x 832, 72: 58 against 42; 12 x 1280, 72: 51 against 54).
static bool wide_backward_tile(const RecDesc& d) {
    if (d.B <= 64) return false;
    const int pairs = d.L * d.D;
    const int64_t units = (int64_t)pairs * ((d.H + 127) / 128);
    if (units * ((d.B + 127) / 128) >= 192) return true;
    return d.precision && (units * ((d.B + 31) / 32) > 512 || (int64_t)pairs * 8 * d.H * d.H > 160000000 || (pairs % 8 && pairs > 16));
}

int rec_backward_batch_tiles(const RecDesc& d) {
    const RecKind kind = rec_kind(d, true);
    const bool wide = kind == kStaged ? d.B > 64 : kind == kDirect && wide_backward_tile(d);
    return wide ? (d.B + 127) / 128 : (d.B + 31) / 32;
}

template <typename T> static void fwd_direct_t(const RecDesc& d, hipStream_t s) {
    const unsigned groups = (unsigned)(d.L * d.D);
    if (d.B > 64) {
        // two 32 KB stages (whole 128-byte lines per row and stage): 64 KB of LDS, two workgroups per CU
        dim3 grid(groups, (d.H + 31) / 32, (d.B + 127) / 128);
        hipLaunchKernelGGL((rec_forward_dma_kernel<T, 4, 1, 128, 2>), grid, dim3(256), 0, s, d);
    } else {
        dim3 grid(groups, (d.H + 63) / 64, (d.B + 63) / 64);
        hipLaunchKernelGGL((rec_forward_dma_kernel<T, 2, 2, 128, 3>), grid, dim3(256), 0, s, d);
    }
}
template <typename T> static void bwd_direct_t(const RecDesc& d, hipStream_t s) {
    const unsigned groups = (unsigned)(d.L * d.D);
    if (wide_backward_tile(d)) {
        dim3 grid(groups, (d.H + 127) / 128, (d.B + 127) / 128);
        hipLaunchKernelGGL((rec_backward_dma_kernel<T, 4, 2, 2, 128, 4>), grid, dim3(512), 0, s, d);
    } else {
        dim3 grid(groups, (d.H + 127) / 128, (d.B + 31) / 32);
        hipLaunchKernelGGL((rec_backward_dma_kernel<T, 1, 4, 1, 128, 4>), grid, dim3(256), 0, s, d);
    }
}

hipError_t launch_rec_forward(const RecDesc& d, hipStream_t s) {
    if (!rec_ok(d)) return hipErrorInvalidValue;
    const RecKind kind = rec_kind(d, false);
    if (kind == kSplit) return launch_rec_split(d, false, s);
    if (kind == kDirect) {
        if (d.precision == 0) fwd_direct_t<float>(d, s);
        else fwd_direct_t<bf16_t>(d, s);
        return hipGetLastError();
    }
    if (d.precision == 0) return fwd_t<float, 16>(d, s);
    return d.H % 8 == 0 ? fwd_t<bf16_t, 16>(d, s) : fwd_t<bf16_t, 8>(d, s);
}

hipError_t launch_rec_backward(const RecDesc& d, hipStream_t s) {
    if (!rec_ok(d)) return hipErrorInvalidValue;
    const RecKind kind = rec_kind(d, true);
    if (kind == kSplit) return launch_rec_split(d, true, s);
    if (kind == kDirect) {
        if (d.precision == 0) bwd_direct_t<float>(d, s);
        else bwd_direct_t<bf16_t>(d, s);
        return hipGetLastError();
    }
    if (d.precision == 0) return bwd_t<float, 16>(d, s);
    return d.H % 8 == 0 ? bwd_t<bf16_t, 16>(d, s) : bwd_t<bf16_t, 8>(d, s);
}

}  // namespace adpsgd
