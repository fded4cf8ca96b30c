// The products that read one gradient matrix - the gradient handed down (dX = dA W) and the weight gradients (dW = dA' X) - and its
// column sums, in one launch.
//
// None of them needs another's result.  One after the other each pays for a launch, for the latency of its contraction and for a last
// round of the chip that is partly empty: a small model's are all latency, a middle one's leave half of the 512 places of 128x256 tiles free (5
// learners of 2 x 360 cells: 135 tiles of dX 30 us, 240 of dW_x 28, 120 of dW_h 10, column sums 5).  In one launch the tiles of
// all follow each other; those of dX come first, and before them the column sums, which are bound by memory while the tiles are
// bound by the matrix units.  Every problem keeps the tile configuration it has alone (gemm.hip), but for one kind of dW (make_plan).
#include "colsum.hpp"
#include "gemm_split.hpp"
#include "gemm_tile.hpp"

namespace adpsgd {
namespace {

struct MultiArgs {
    GemmDesc d[3];                       // d[0]: A K-contiguous, B rows-contiguous (dX), if any; the others: both rows-contiguous
    int end[3];                          // workgroups up to the end of each (of none: 0)
    int tile[3];
    ColsumDesc cs;
    int cs_x, cs_blocks;                 // workgroups of the column sums: to a learner, in all (0: none)
};

struct Bf16Small {                       // tile configuration 15 throughout
    static constexpr int kLds = 3 * 128 * 128, kWaves = 3;
    template <bool AKC> __device__ __forceinline__ static void tile(const GemmDesc& d, int, int bid, int n, char* lds) { dma_tile<bf16_t, AKC, false, 2, 2, 1, 1, 128, 3>(d, bid, n, lds); }
};
struct Bf16Mid {                         // 13, 14, 15
    static constexpr int kLds = 3 * 384 * 64, kWaves = 2;
    template <bool AKC> __device__ __forceinline__ static void tile(const GemmDesc& d, int v, int bid, int n, char* lds) {
        if (v == 13) dma_tile<bf16_t, AKC, false, 2, 2, 2, 4, 64, 3>(d, bid, n, lds);
        else if (v == 14) dma_tile<bf16_t, AKC, false, 2, 2, 2, 2, 128, 2>(d, bid, n, lds);
        else dma_tile<bf16_t, AKC, false, 2, 2, 1, 1, 128, 3>(d, bid, n, lds);
    }
};
struct Bf16Large {                       // 12
    static constexpr int kLds = 3 * 512 * 64, kWaves = 1;
    template <bool AKC> __device__ __forceinline__ static void tile(const GemmDesc& d, int, int bid, int n, char* lds) { dma_tile<bf16_t, AKC, false, 2, 2, 4, 4, 64, 3>(d, bid, n, lds); }
};
struct Fp32Plain {                       // the smallest fp32 problems, and long contractions
    static constexpr int kLds = 4 * 128 * 64, kWaves = 3;
    template <bool AKC> __device__ __forceinline__ static void tile(const GemmDesc& d, int, int bid, int n, char* lds) { dma_tile<float, AKC, false, 2, 2, 1, 1, 64, 4>(d, bid, n, lds); }
};
struct Fp32Split {                       // 14, 15 on the bf16 matrix units
    static constexpr int kLds = SplitCore<false, false, 1>::LDS_BYTES, kWaves = 3;
    static_assert(SplitCore<true, false, 1>::LDS_BYTES == kLds && SplitCore<true, false, 2>::LDS_BYTES == kLds && SplitCore<false, false, 2>::LDS_BYTES == kLds, "LDS");
    template <bool AKC> __device__ __forceinline__ static void tile(const GemmDesc& d, int v, int bid, int n, char* lds) {
        if (v == 15) split_tile<AKC, false, 1>(d, bid, n, lds);
        else split_tile<AKC, false, 2>(d, bid, n, lds);
    }
};

template <class Kind>
__global__ __launch_bounds__(256, Kind::kWaves) void gemm_multi_kernel(MultiArgs p) {
    __shared__ __attribute__((aligned(1024))) char lds[Kind::kLds];
    static_assert(Kind::kLds >= 32 * 8 * 16, "column sums");
    int bid = (int)blockIdx.x;
    if (bid < p.cs_blocks) {
        const int x = bid % p.cs_x, y = bid / p.cs_x;
        const bool few = p.cs.rows < 128;
        if (p.cs.precision) { if (few) colsum_block<bf16_t, 8, 32>(p.cs, x, y, lds); else colsum_block<bf16_t, 32, 8>(p.cs, x, y, lds); }
        else { if (few) colsum_block<float, 8, 32>(p.cs, x, y, lds); else colsum_block<float, 32, 8>(p.cs, x, y, lds); }
        return;
    }
    bid -= p.cs_blocks;
    if (bid < p.end[0]) { Kind::template tile<true>(p.d[0], p.tile[0], bid, p.end[0], lds); return; }
    const int which = bid < p.end[1] ? 1 : 2, first = p.end[which - 1];
    Kind::template tile<false>(p.d[which], p.tile[which], bid - first, p.end[which] - first, lds);
}

template <class Kind> void launch_multi_t(const MultiArgs& a, hipStream_t s) {
    hipLaunchKernelGGL((gemm_multi_kernel<Kind>), dim3((unsigned)(a.cs_blocks + a.end[2])), dim3(256), 0, s, a);
}

// Problems of one family can share a launch.  Of the long fp32 contractions, on fp32 MFMAs, two weight gradients in 64x64 tiles do (us, an
// iteration with a launch each / with one: 4 x 128 cells in both directions, 4200 frames 1152 / 1081, 3 x 2 x 64, 3360 frames 495 / 377).
enum Family { kNone, kBf16Mid, kBf16Large, kFp32, kFp32Long };
Family family(const GemmDesc& d, bool dx, int& v) {
    bool dma = false;
    v = gemm_pick_tile(d, dma);
    if (v < 0 || !dma || d.b_kc || (d.a_kc != 0) != dx) return kNone;
    if (d.precision == 0 && gemm_long_fp32(d)) return v == 15 && !dx ? kFp32Long : kNone;
    if (d.precision == 0) return v >= 14 ? kFp32 : kNone;
    return v == 12 ? kBf16Large : v >= 13 ? kBf16Mid : kNone;
}

// What shares a launch: all, the weight gradients, or nothing.
struct Plan { Family fam; bool dx, dw, cs; int v[3]; };
Plan make_plan(const GradProducts& g) {
    Plan p{};
    Family f[3] = {kNone, kNone, kNone};
    if (g.has_dx) f[0] = family(g.dx, true, p.v[0]);
    for (int i = 0; i < g.ndw; ++i) f[1 + i] = family(g.dw[i], false, p.v[1 + i]);
    // 256x256 tiles of one weight gradient that leave a third of their rounds of the chip empty, beside a dX of smaller ones (an output
    // layer behind a bottleneck): 128x256 tiles, in dX's launch (8 learners, 2016 x 256 x 9000 and 9000 x 256 x 2016, 288 tiles: dX 153 us, dW 124,
    // column sums 71, one after the other; 299 together).  Not where dX has more than 128 blocks of 128 rows in 128x256 tiles: on half of the compute units its
    // tiles still have a compute unit each, on more they take each other's time.  Iterations of one layer of 64 cells in us, together / apart (blocks):
    // 8 x 9000 states, bottleneck 256 905 / 965 (128), 1045 / 1026 (136), 1504 / 1460 (216); 4 x 9000, 256 820 / 852 (112), 1057 / 987 (132);
    // 7 x 12000, 256 853 / 892 (126), 1026 / 952 (133); 6 x 12000, 200 850 / 916 (126), 991 / 962 (132); 4 x 9000, 512 900 / 923 (100), 1041 / 1039 (132).
    // Of 150 sizes up to 128 blocks four are slower, by 1.5 to 4 % (3 x 11600, 256, 4096 rows 809 / 775), most of the others faster, by up to 13 %.
    if (g.ndw == 1 && f[0] == kBf16Mid && f[1] == kBf16Large) {
        const int64_t tiles = gemm_tiles(g.dw[0], 256, 256), rounds = (tiles + 255) / 256, rows = (int64_t)((g.dx.M + 127) / 128) * g.dx.groupsI * g.dx.groupsD;
        if (3 * tiles <= 2 * 256 * rounds && (p.v[0] != 13 || rows <= 128)) { p.v[1] = 13; f[1] = kBf16Mid; }
    }
    if (g.ndw < 1 || f[1] == kNone || (g.ndw > 1 && f[2] != f[1])) return p;
    p.fam = f[1];
    p.dx = g.has_dx && f[0] == f[1];
    // (a large problem's one workgroup to a compute unit would leave the column sums too few loads in flight)
    p.cs = g.has_cs && p.fam != kBf16Large && p.fam != kFp32Long && colsum_ok(g.cs);
    p.dw = p.dx || p.cs || g.ndw > 1;
    int64_t blocks = p.cs ? (int64_t)((g.cs.N + 31) / 32 + g.cs.L_all) * g.cs.L : 0;
    if (p.dx) blocks += gemm_tiles(g.dx, 64, 64);
    for (int i = 0; i < g.ndw; ++i) blocks += gemm_tiles(g.dw[i], 64, 64);
    if (!p.dw || blocks > 0x7fffffff) return Plan{};
    return p;
}

int64_t tiles_of(const GemmDesc& d, int v) {
    return v == 12 ? gemm_tiles(d, 256, 256) : v == 13 ? gemm_tiles(d, 128, 256) : v == 14 ? gemm_tiles(d, 128, 128) : gemm_tiles(d, 64, 64);
}

}  // namespace

int grad_product_launches(const GradProducts& g, bool& colsum_apart) {
    const Plan p = make_plan(g);
    colsum_apart = g.has_cs && !(p.dw && p.cs);
    return p.dw ? 1 : g.ndw;
}

hipError_t launch_grad_products(const GradProducts& g, hipStream_t s) {
    const Plan p = make_plan(g);
    if (g.has_dx && !(p.dw && p.dx)) {
        const hipError_t e = launch_gemm(g.dx, s);
        if (e != hipSuccess) return e;
    }
    if (!p.dw) {
        for (int i = 0; i < g.ndw; ++i) {
            const hipError_t e = launch_gemm(g.dw[i], s);
            if (e != hipSuccess) return e;
        }
    } else {
        MultiArgs a{};
        a.d[0] = g.dx; a.d[1] = g.dw[0]; a.d[2] = g.dw[1];
        for (int i = 0; i < 3; ++i) a.tile[i] = p.v[i];
        a.end[0] = p.dx ? (int)tiles_of(g.dx, p.v[0]) : 0;
        a.end[1] = a.end[0] + (int)tiles_of(g.dw[0], p.v[1]);
        a.end[2] = a.end[1] + (g.ndw > 1 ? (int)tiles_of(g.dw[1], p.v[2]) : 0);
        if (p.cs) {
            a.cs = g.cs;
            const int cols = g.cs.rows < 128 ? 128 : 32;
            a.cs_x = (g.cs.N + cols - 1) / cols + (g.cs.loss ? g.cs.L_all : 0);
            a.cs_blocks = a.cs_x * g.cs.L;
        }
        if (p.fam == kFp32Long) {
            launch_multi_t<Fp32Plain>(a, s);
        } else if (p.fam == kFp32) {
            bool plain = (!p.dx || (p.v[0] == 15 && gemm_plain_fp32(g.dx)));
            for (int i = 0; i < g.ndw; ++i) plain = plain && p.v[1 + i] == 15 && gemm_plain_fp32(g.dw[i]);
            if (plain) launch_multi_t<Fp32Plain>(a, s);
            else launch_multi_t<Fp32Split>(a, s);
        } else if (p.fam == kBf16Large) {
            launch_multi_t<Bf16Large>(a, s);
        } else {
            bool small = !p.dx || p.v[0] == 15;
            for (int i = 0; i < g.ndw; ++i) small = small && p.v[1 + i] == 15;
            if (small) launch_multi_t<Bf16Small>(a, s);
            else launch_multi_t<Bf16Mid>(a, s);
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return g.has_cs && !(p.dw && p.cs) ? launch_colsum(g.cs, s) : hipSuccess;
}

}  // namespace adpsgd
