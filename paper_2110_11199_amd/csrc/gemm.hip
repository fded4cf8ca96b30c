// Grouped MFMA GEMM kernels: the time-batched GEMMs of the LSTM gradient
// (input projections, output layers, weight gradients, input gradients).
//
// Seven tile configurations are built; 11-15 bring their operands in by direct global->LDS loads (no staging
// registers, no LDS store instructions), transpose an operand that is not K-contiguous (dW = dA' X, dX = dA W)
// on the LDS read, and run a main loop that is software-pipelined by hand (GemmDma::run_deep); they need
// 16-byte aligned rows and whole 16-byte chunks of K where an operand is K-contiguous:
//   12  256x256 tile on 4 waves (128x128 each, one wave per SIMD, accumulators in AGPRs), three 64-byte K
//       stages.  Large bf16 problems with a rows-contiguous operand (dW, dX).
//   11  the same with two 128-byte stages: when both operands are K-contiguous (input projections) their rows
//       are fetched in whole 128-byte lines, which 64-byte stages split in two requests (measured inside the
//       training step: 1.40 against 1.48 ms per input projection, and the reverse, 1.32 against 1.25 ms, for dX).
//   13  128x256 tile on 4 waves (64x128 each), three 64-byte stages, two workgroups per CU: K-contiguous
//       operands with K < 512 or a narrow output (output layer, layer-0 input projection), whose tiles spend
//       as long storing as computing; the second workgroup's loop runs during the first one's epilogue.
//   14  128x128 tile on 4 waves (64x64 each), two 128-byte stages.
//   15  64x64 tile on 4 waves (32x32 each), three 128-byte stages (smallest fp32 problems: four 64-byte ones).
//       14 and 15 are for problems with too few 256x256 tiles for the 256 CUs.  A small problem
//       is bound by the latency of its K loop (a 64x64 tile alone on its CU takes 5 ns per k, a 128x128 one 13)
//       and by how evenly its tiles cover the CUs, not by operand bytes per flop.  Against the register-staged
//       kernel 0, us: 336x256x1024x8 30.8 -> 8.4, 1050x720x2880x5 91 -> 38, 1050x120x3000x5 81 -> 18.
//       Other fp32 problems that meet the same conditions run in tiles of these two sizes on the bf16 matrix units (gemm_split.hpp).
//   5   256x256 tile on 8 waves (128x64 each) staged through registers, the transposition done between
//       the registers and LDS.  Large bf16 problems that miss the conditions of 11-15.
//   0   128x128 tile, 4 waves (64x64 each), 64-byte stages, staged through registers.  Small
//       problems that miss them.
// K need not be a multiple of a stage (GemmDma::run_tail), nor of 16 bytes where the rows are padded to that: 336x500 products with
// 256 columns, 8 of them, 19.6 and 17.9 us staged through registers, 8.7 and 8.1 here.  1344x1024x9000x16, bf16, 692 us on kernel 5, 486 on 13;
// 5120x1280x2016x8 354 -> 204.
// A 256x256 tile needs half the operand bytes per flop of a 128x128 one.
#include <type_traits>
#include "gemm_core.hpp"
#include "gemm_dma.hpp"
#include "gemm_tile.hpp"
#include "kernels.hpp"

namespace adpsgd {

template <typename T, bool AKC, bool BKC, int WM, int WN, int FM, int FN, int VB, int SB>
__global__ __launch_bounds__(64 * WM * WN) void gemm_kernel(GemmDesc p) {
    typedef typename std::conditional<AKC, KcSrc<T>, McSrc<T>>::type ASrc;
    typedef typename std::conditional<BKC, KcSrc<T>, McSrc<T>>::type BSrc;
    typedef GemmCore<T, ASrc, BSrc, WM, WN, FM, FN, VB, SB> Core;
    __shared__ __attribute__((aligned(16))) char lds[Core::LDS_BYTES];

    const int tiles_m = (p.M + Core::BM - 1) / Core::BM, tiles_n = (p.N + Core::BN - 1) / Core::BN;
    int grp, tm, tn;
    map_tile(blockIdx.x, gridDim.x, tiles_m, tiles_n, grp, tm, tn);
    const int gi = p.lmap.idx[grp / p.groupsD], gd = grp % p.groupsD;
    const int m0 = tm * Core::BM, n0 = tn * Core::BN;
    const T* A = (const T*)p.A + gi * p.sAi + gd * p.sAd;
    const T* B = (const T*)p.B + gi * p.sBi + gd * p.sBd;

    ASrc a; BSrc b;
    if constexpr (AKC) { a.base = A + (int64_t)m0 * p.lda; } else { a.base = A + m0; }
    a.ld = p.lda; a.R = p.M - m0;
    if constexpr (BKC) { b.base = B + (int64_t)n0 * p.ldb; } else { b.base = B + n0; }
    b.ld = p.ldb; b.R = p.N - n0;

    f32x16_t acc[FM][FN];
    zero_tile<FM, FN>(acc);
    Core::run(acc, a, b, p.K, lds);
    float bias[FN];          // (this register-staged loop has no registers to spare for an early load)
    load_bias<Core, FN>(bias, p, n0, gi, gd);
    store_tile<T, Core, FM, FN>(acc, bias, p, m0, n0, gi, gd);
}

template <typename T, bool AKC, bool BKC, int WM, int WN, int FM, int FN, int SB, int NS>
__global__ __launch_bounds__(64 * WM * WN, FM * FN <= 4 ? 3 : FM * FN == 8 ? 2 : 1) void gemm_dma_kernel(GemmDesc p) {
    typedef GemmDma<T, KcSrc<T>, KcSrc<T>, WM, WN, FM, FN, SB, NS> Core;
    __shared__ __attribute__((aligned(1024))) char lds[Core::LDS_BYTES];
    dma_tile<T, AKC, BKC, WM, WN, FM, FN, SB, NS>(p, blockIdx.x, gridDim.x, lds);
}

template <typename T, bool AKC, bool BKC, int WM, int WN, int FM, int FN, int VB, int SB>
static hipError_t launch_t(const GemmDesc& d, hipStream_t s) {
    constexpr int BM = 32 * FM * WM, BN = 32 * FN * WN;
    const int tiles_m = (d.M + BM - 1) / BM, tiles_n = (d.N + BN - 1) / BN;
    dim3 grid((unsigned)(tiles_m * tiles_n * d.groupsI * d.groupsD));
    hipLaunchKernelGGL((gemm_kernel<T, AKC, BKC, WM, WN, FM, FN, VB, SB>), grid, dim3(64 * WM * WN), 0, s, d);
    return hipGetLastError();
}

template <typename T, int WM, int WN, int FM, int FN, int VB, int SB>
static hipError_t launch_layout(const GemmDesc& d, hipStream_t s) {
    const int key = (d.a_kc ? 2 : 0) | (d.b_kc ? 1 : 0);
    switch (key) {
        case 0: return launch_t<T, false, false, WM, WN, FM, FN, VB, SB>(d, s);
        case 1: return launch_t<T, false, true, WM, WN, FM, FN, VB, SB>(d, s);
        case 2: return launch_t<T, true, false, WM, WN, FM, FN, VB, SB>(d, s);
        default: return launch_t<T, true, true, WM, WN, FM, FN, VB, SB>(d, s);
    }
}

template <typename T, bool AKC, bool BKC, int WM, int WN, int FM, int FN, int SB, int NS>
static hipError_t launch_dma_t(const GemmDesc& d, hipStream_t s) {
    constexpr int BM = 32 * FM * WM, BN = 32 * FN * WN;
    const int tiles_m = (d.M + BM - 1) / BM, tiles_n = (d.N + BN - 1) / BN;
    dim3 grid((unsigned)(tiles_m * tiles_n * d.groupsI * d.groupsD));
    hipLaunchKernelGGL((gemm_dma_kernel<T, AKC, BKC, WM, WN, FM, FN, SB, NS>), grid, dim3(64 * WM * WN), 0, s, d);
    return hipGetLastError();
}

template <typename T, int WM, int WN, int FM, int FN, int SB, int NS>
static hipError_t launch_dma(const GemmDesc& d, hipStream_t s) {
    const int key = (d.a_kc ? 2 : 0) | (d.b_kc ? 1 : 0);
    switch (key) {
        case 0: return launch_dma_t<T, false, false, WM, WN, FM, FN, SB, NS>(d, s);
        case 1: return launch_dma_t<T, false, true, WM, WN, FM, FN, SB, NS>(d, s);
        case 2: return launch_dma_t<T, true, false, WM, WN, FM, FN, SB, NS>(d, s);
        default: return launch_dma_t<T, true, true, WM, WN, FM, FN, SB, NS>(d, s);
    }
}

static bool aligned_to(const void* p, int64_t ld, int64_t s1, int64_t s2, int esz, int bytes) {
    return ((uintptr_t)p % bytes == 0) && ((ld * esz) % bytes == 0) && ((s1 * esz) % bytes == 0) &&
           ((s2 * esz) % bytes == 0);
}

// Time estimate of covering the problem with bm x bn tiles, for the choice between the smaller tiles: a CU works
// through its tiles at `rate` ns per k and tile, but a tile that has the CU to itself takes `latency` ns per k (its loads are not
// hidden by a second workgroup's MFMAs).
static double tile_time(const GemmDesc& d, int bm, int bn, double rate, double latency) {
    const int64_t tiles = (int64_t)((d.M + bm - 1) / bm) * ((d.N + bn - 1) / bn) * d.groupsI * d.groupsD;
    const double rounds = (double)((tiles + 255) / 256);
    return (rounds * rate > latency ? rounds * rate : latency) * d.K;
}

// The tile configuration of a problem (-1: not a valid problem), and whether its operands meet the rules of the direct loads.
int gemm_pick_tile(const GemmDesc& d, bool& dma) {
    if (d.M < 1 || d.N < 1 || d.K < 1 || d.groupsI < 1 || d.groupsI > 128 || d.groupsD < 1) return -1;
    if (d.tile != -1 && d.tile != 0 && d.tile != 5 && (d.tile < 11 || d.tile > 15)) return -1;
    // one-dimensional grid over all tiles of all groups (smallest tile 64 x 64)
    if ((int64_t)((d.M + 63) / 64) * ((d.N + 63) / 64) * d.groupsI * d.groupsD > 0x7fffffff) return -1;
    const int esz = d.precision ? 2 : 4, epc = 16 / esz;
    const int quad = 4 * esz;    // every operand must allow loads of 4 elements
    if (!aligned_to(d.A, d.lda, d.sAi, d.sAd, esz, quad) || !aligned_to(d.B, d.ldb, d.sBi, d.sBd, esz, quad))
        return -1;
    // Direct-to-LDS loads need 16-byte aligned rows, whole 16-byte chunks along the contiguous dimension (of K, or of
    // rows: the k-rows must be at least round_up(rows, chunk) long), and per-lane load offsets inside a tile that fit
    // 32 bits (row strides below 2^22 elements).
    const bool wide_a = aligned_to(d.A, d.lda, d.sAi, d.sAd, esz, 16), wide_b = aligned_to(d.B, d.ldb, d.sBi, d.sBd, esz, 16);
    dma = d.lda < (1 << 22) && d.ldb < (1 << 22) && wide_a && wide_b &&
          (d.a_kc ? d.K % epc == 0 || d.k_padded : d.lda >= (d.M + epc - 1) / epc * epc) &&
          (d.b_kc ? d.K % epc == 0 || d.k_padded : d.ldb >= (d.N + epc - 1) / epc * epc);
    int v = d.tile;
    if (d.precision == 0) {
        // ns per k of a tile, with others on its compute unit and alone on it, of the kernels that run it: what decides is how evenly the
        // tiles cover the compute units.  On the bf16 matrix units (gemm_split.hpp), us, 128x128 / 64x64: 672x2048x512x8 70 / 83, 1280x2000x320x6
        // 58 / 71, 1000x512x672x8 42 / 44; and 672x512x2048x8 98 / 85, 1280x320x1280x6 58 / 52, 2000x320x1280x6 91 / 75.  On fp32 MFMAs
        // (gemm_long_fp32): 672x1024x9000x8 1035 / 889, 672x1024x4096x8 474 / 406, 1344x1024x3000x8 521 / 509; 2688x1024x9000x4 1559 / 1654.
        if (v < 0) {
            const bool mfma = gemm_long_fp32(d);
            v = !dma ? 0 : tile_time(d, 64, 64, mfma ? 14.0 : 12.8, mfma ? 20.0 : 15.5) < tile_time(d, 128, 128, mfma ? 53.0 : 36.0, mfma ? 60.0 : 43.0) ? 15 : 14;
            // Short contractions are bound by how a tile starts and by its stores.  Where rows of C are not whole 64 bytes (widths of layers; rows of logits are) the
            // stores of 128x128 tiles take half as long again: of 1051 products of 20 to 360 columns, K = 40 to 112, eight are more than 5 per cent slower in 64x64 tiles, by up to
            // 1.5 us (2688x72x80x16 13.0 / 14.3; all 12250 / 8450).  Elsewhere 128x128 tiles pay once there are a few rounds of them.  us, 128x128 on the bf16 matrix units /
            // 64x64, up to 80 terms on fp32 MFMAs: 168x5000x40x12 20 / 19, 1344x3000x64x12 55 / 81, x80 62 / 90, x96 69 / 92, 5120x200x80x8 17.6 / 23.1, 2000x320x64x6
            // 12.3 / 9.8, 512x1024x40x8 9.1 / 8.6, 1280x1280x80x6 16.3 / 20.4, 3360x1280x80x8 42 / 59, 672x2048x40x16 26 / 31.  Against 64 bits, of the 2-norm at 64, 80, 96,
            // 112 terms: 128x128 1.1, 1.25, 1.4, 1.5e-7; 64x64 1.4, 1.6, 0.96, 1.06e-7.  (Gradients of an iteration behind either are as far from it, to 1 per cent.)
            const bool whole = d.ldc % 16 == 0;
            if (dma && d.K <= 80) v = whole && 2.6 * (gemm_tiles(d, 128, 128) + 256) < gemm_tiles(d, 64, 64) + 256 ? 14 : 15;
            else if (dma && d.K <= 112 && !whole) v = 15;
        }
        return v;
    }
    if (v < 0) {
        // 256x256 tiles once there are enough of them to fill the 256 CUs
        const int64_t big_tiles = (int64_t)((d.M + 255) / 256) * ((d.N + 255) / 256) * d.groupsI * d.groupsD;
        // Short contractions (a tile's first loads, stores and hand-over weigh as much as its loop) and row counts that
        // leave the last 256-row band mostly empty take the 128x256 tiles, two workgroups per CU, whatever the storage
        // order (16 x 1344-row problems with K <= 1344: 4.31 -> 4.07 ms over the 18 GEMMs of an iteration; only the
        // 2048 x 512 x 1344 weight-gradient problem is 5 % slower that way); long contractions keep the 256x256 tiles,
        // which move half the operand bytes per flop.
        const bool short_k = d.K <= 1536;
        const bool ragged_m = (int64_t)(((d.M + 255) / 256) * 256 - d.M) * 10 >= d.M;
        if (big_tiles < 128 && dma) {
            const double t64 = tile_time(d, 64, 64, 3.7, 5.0), t128 = tile_time(d, 128, 128, 8.0, 13.0), t256 = tile_time(d, 128, 256, 14.5, 14.5);
            v = t64 <= t128 && t64 <= t256 ? 15 : t128 <= t256 ? 14 : 13;
        } else v = big_tiles < 128 ? 0 : (short_k || ragged_m) ? 13 : !(d.a_kc && d.b_kc) ? 12 : (d.M >= 512 && d.N >= 512) ? 11 : 13;
    }
    return v;
}

// fp32 problems in 64x64 tiles with a short contraction stay on fp32 MFMAs, up to 192 terms in one round of the chip: there a launch costs the fetch
// of its instructions, of which the split kernels have several times as many (an iteration of the 4 x 64-unit model, five such launches: 74.6 us
// against 79.2), and a tile alone on its compute unit takes 20 ns per k here and 15.5 there; up to 80 terms in any number of rounds (split / here,
// us: 168x5000x40x12 21.7 / 19.2, 1008x256x40x16 10.7 / 8.5, 2000x320x64x6 10.7 / 9.8, 1344x3000x80x12 96 / 87).
bool gemm_plain_fp32(const GemmDesc& d) { return d.K <= 80 || (gemm_tiles(d, 64, 64) <= 256 && d.K <= 192); }

// fp32 contractions this long stay on fp32 MFMAs, for the sake of the results' continuity and not of their accuracy: results of the two
// kinds of kernels differ by 7.5e-7 of the 2-norm at K = 1024, 1.07e-6 at 2048 and 1.2e-6 at 2560, growing as the square root (each has rounding
// errors of its own: fp32 MFMAs 9.0e-7 against 64 bits at 2560, 1.14e-6 at 4096, the bf16 matrix units 7.9e-7 at 2560, 5.5e-7 in 64x64 tiles), and
// gradients with longer sums were seen to move by 1.4e-6 in all.
bool gemm_long_fp32(const GemmDesc& d) { return d.precision == 0 && d.K > 2560; }

hipError_t launch_gemm(const GemmDesc& d, hipStream_t s) {
    bool dma = false;
    const int v = gemm_pick_tile(d, dma);
    if (v < 0) return hipErrorInvalidValue;
    if (d.precision == 0) {
        if (v == 15 && dma && gemm_plain_fp32(d)) return launch_dma<float, 2, 2, 1, 1, 64, 4>(d, s);
        if (v >= 11 && dma && gemm_long_fp32(d)) return v == 15 ? launch_dma<float, 2, 2, 1, 1, 64, 4>(d, s) : launch_dma<float, 2, 2, 2, 2, 64, 3>(d, s);
        if (v >= 11 && dma) return launch_gemm_split(d, v != 15, s);
        return launch_layout<float, 2, 2, 2, 2, 16, 64>(d, s);
    }
    const bool wide_a = aligned_to(d.A, d.lda, d.sAi, d.sAd, 2, 16), wide_b = aligned_to(d.B, d.ldb, d.sBi, d.sBd, 2, 16);
    if ((d.a_kc && !wide_a) || (d.b_kc && !wide_b)) return launch_layout<bf16_t, 2, 2, 2, 2, 8, 64>(d, s);
    if (v == 15 && dma) return launch_dma<bf16_t, 2, 2, 1, 1, 128, 3>(d, s);
    if (v == 14 && dma) return launch_dma<bf16_t, 2, 2, 2, 2, 128, 2>(d, s);
    if (v == 13 && dma) return launch_dma<bf16_t, 2, 2, 2, 4, 64, 3>(d, s);
    if (v == 12 && dma) return launch_dma<bf16_t, 2, 2, 4, 4, 64, 3>(d, s);
    if (v == 11 && dma) return launch_dma<bf16_t, 2, 2, 4, 4, 128, 2>(d, s);
    if (v >= 5 && v < 14) return launch_layout<bf16_t, 2, 4, 4, 2, 16, 128>(d, s);
    return launch_layout<bf16_t, 2, 2, 2, 2, 16, 64>(d, s);
}

}  // namespace adpsgd
