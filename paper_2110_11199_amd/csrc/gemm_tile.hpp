// What the GEMM kernels share around their main loops: which tile a workgroup takes, the bias and the stores of a tile.
#pragma once
#include <type_traits>
#include "gemm_core.hpp"
#include "gemm_dma.hpp"
#include "kernels.hpp"

namespace adpsgd {

// Workgroup ids are handed to the 8 XCDs round-robin; this maps them back so that each
// XCD (its own L2) works on a contiguous range of tiles.
__device__ inline int xcd_contiguous_id(int bid, int nb) {
    const int q = nb >> 3, r = nb & 7;
    const int xcd = bid & 7, local = bid >> 3;
    const int start = xcd < r ? xcd * (q + 1) : r * (q + 1) + (xcd - r) * q;
    return start + local;
}

// Workgroup -> (group, tile row, tile column).  The grid is one-dimensional over all tiles of all
// groups.  Each XCD (own L2, 32 CUs) owns a contiguous range of the ordered tile list, so it works on
// whole groups when there are enough of them instead of on a slice of every group; inside a group
// the tiles are ordered in bands of gm <= 8 tile rows walked column by column, so that the 32 tiles an
// XCD runs at one time form a gm x 32/gm patch that shares gm + 32/gm operand panels (an m-fastest
// walk of the whole group needs tiles_m + 32/tiles_m and re-reads every A panel in every round).
__device__ inline void map_tile(int bid, int total, int tiles_m, int tiles_n, int& grp, int& tm, int& tn) {
    const int id = xcd_contiguous_id(bid, total);
    const int per = tiles_m * tiles_n;
    grp = id / per;
    const int t = id - grp * per;
    const int nband = (tiles_m + 7) >> 3;
    const int gm = (tiles_m + nband - 1) / nband;
    const int band = t / (gm * tiles_n);
    const int first = band * gm;
    const int rows = tiles_m - first < gm ? tiles_m - first : gm;
    const int r = t - band * gm * tiles_n;
    tn = r / rows;
    tm = first + r - tn * rows;
}

// Epilogue shared by the GEMM kernels: C tile = acc (+ bias), fp32 or operand type.
// Every store reads its data from a register of its own (the bias is added in place, the
// bf16 values are converted into a separate array first): with one temporary register
// reused for all stores the compiler has to wait for each store before the next one.
// Bias of this lane's FN accumulator columns (0 without a bias or past the last column).  Loaded before the
// main loop: in the epilogue the load's latency would stand in front of the stores of every tile.
template <class Core, int FN>
__device__ inline void load_bias(float (&bv)[FN], const GemmDesc& p, int n0, int gi, int gd) {
    const float* bias = p.bias ? p.bias + gi * p.sBiasI + gd * p.sBiasD : nullptr;
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
        const int col = n0 + Core::acc_col(fn);
        bv[fn] = (bias && col < p.N) ? bias[col] : 0.f;
    }
}

template <typename T, class Core, int FM, int FN>
__device__ inline void store_tile(f32x16_t (&acc)[FM][FN], const float (&bias)[FN], const GemmDesc& p, int m0, int n0, int gi, int gd) {
    const int64_t coff = gi * p.sCi + gd * p.sCd;
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
        const int col = n0 + Core::acc_col(fn);
        if (col >= p.N) continue;
        const float bv = bias[fn];
#pragma unroll
        for (int fm = 0; fm < FM; ++fm) {
            const int row0 = m0 + Core::acc_row(fm, 0);          // rows of this lane: row0 + 8*(i/4) + i%4
            const int64_t o = coff + (int64_t)row0 * p.ldc + col;
            if (p.c_elem) {
                T* c = (T*)p.C + o;
                if constexpr (sizeof(T) == 2) {
                    uint32_t hb[16];
#pragma unroll
                    for (int i = 0; i < 16; ++i) hb[i] = f32_to_bf16(acc[fm][fn][i] + bv);
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int r = 8 * (i >> 2) + (i & 3);
                        if (row0 + r < p.M) c[(int64_t)r * p.ldc] = (bf16_t)hb[i];
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[fm][fn][i] += bv;
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int r = 8 * (i >> 2) + (i & 3);
                        if (row0 + r < p.M) c[(int64_t)r * p.ldc] = acc[fm][fn][i];
                    }
                }
            } else {
                float* c = (float*)p.C + o;
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[fm][fn][i] += bv;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int r = 8 * (i >> 2) + (i & 3);
                    // written once, read by a later kernel: keep it from displacing the operand panels in L2
                    if (row0 + r < p.M) __builtin_nontemporal_store(acc[fm][fn][i], c + (int64_t)r * p.ldc);
                }
            }
        }
    }
}

// Stores whose address is a wave-uniform 64-bit pointer (SGPR pair) plus a per-lane 32-bit byte offset.
// Written as inline asm because the compiler otherwise folds the uniform part into a 64-bit vector
// address and recomputes it with vector multiply-adds for every store.
__device__ inline void store_u_f32_(uint32_t off, float v, const void* base_uniform) {
    asm volatile("global_store_dword %0, %1, %2" :: "v"(off), "v"(v), "s"(base_uniform) : "memory");
}
__device__ inline void store_u_f32_nt_(uint32_t off, float v, const void* base_uniform) {
    asm volatile("global_store_dword %0, %1, %2 nt" :: "v"(off), "v"(v), "s"(base_uniform) : "memory");
}
__device__ inline void store_u_b16_(uint32_t off, uint32_t v, const void* base_uniform) {
    asm volatile("global_store_short %0, %1, %2" :: "v"(off), "v"(v), "s"(base_uniform) : "memory");
}

// The same for a tile that lies wholly inside C (no row or column guard): every store is one
// instruction whose address is a wave-uniform row pointer plus a per-lane byte offset that is the
// same for all stores of the lane, so the epilogue costs no vector address arithmetic and no branches.
// Needs (4 * ldc + 32) * 4 bytes to fit the 32-bit offset (checked by the caller).
template <typename T, class Core, int FM, int FN>
__device__ inline void store_tile_interior(f32x16_t (&acc)[FM][FN], const float (&bias)[FN], const GemmDesc& p, int m0, int n0, int gi, int gd) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wave_m = wave / Core::kWN, wave_n = wave % Core::kWN;
    const uint32_t lane_elem = (uint32_t)(4 * (lane >> 5)) * (uint32_t)p.ldc + (uint32_t)(lane & 31);
    const int64_t tile_off = gi * p.sCi + gd * p.sCd + (int64_t)(m0 + wave_m * FM * 32) * p.ldc + n0 + wave_n * FN * 32;
    const bool narrow = p.c_elem && sizeof(T) == 2;
    const int esz = narrow ? 2 : 4;
    const char* cbase = (const char*)p.C + tile_off * esz;
    const uint32_t lane_off = lane_elem * (uint32_t)esz;
    const int64_t row_bytes = (int64_t)p.ldc * esz;
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
        const float bv = bias[fn];
#pragma unroll
        for (int fm = 0; fm < FM; ++fm) {
            const char* fbase = cbase + (int64_t)(fm * 32) * row_bytes + fn * 32 * esz;
            if (narrow) {
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    store_u_b16_(lane_off, f32_to_bf16(acc[fm][fn][i] + bv), fbase + (8 * (i >> 2) + (i & 3)) * row_bytes);
            } else if (p.c_elem) {
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    store_u_f32_(lane_off, acc[fm][fn][i] + bv, fbase + (8 * (i >> 2) + (i & 3)) * row_bytes);
            } else {
#pragma unroll
                for (int i = 0; i < 16; ++i)   // written once, read by a later kernel: keep it out of L2
                    store_u_f32_nt_(lane_off, acc[fm][fn][i] + bv, fbase + (8 * (i >> 2) + (i & 3)) * row_bytes);
            }
        }
    }
}

template <int FM, int FN> __device__ inline void zero_tile(f32x16_t (&acc)[FM][FN]) {
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;
}

// Same tile bookkeeping with the direct-to-LDS main loop (16-byte aligned operands, whole 16-byte chunks of K where an
// operand is K-contiguous, or rows padded to them).
template <typename T, bool AKC, bool BKC, int WM, int WN, int FM, int FN, int SB, int NS>
__device__ __forceinline__ void dma_tile(const GemmDesc& p, int bid, int total, char* lds) {
    typedef typename std::conditional<AKC, KcSrc<T>, McSrc<T>>::type ASrc;
    typedef typename std::conditional<BKC, KcSrc<T>, McSrc<T>>::type BSrc;
    typedef GemmDma<T, ASrc, BSrc, WM, WN, FM, FN, SB, NS> Core;

    const int tiles_m = (p.M + Core::BM - 1) / Core::BM, tiles_n = (p.N + Core::BN - 1) / Core::BN;
    int grp, tm, tn;
    map_tile(bid, total, tiles_m, tiles_n, grp, tm, tn);
    const int gi = p.lmap.idx[grp / p.groupsD], gd = grp % p.groupsD;
    const int m0 = tm * Core::BM, n0 = tn * Core::BN;
    const T* A = (const T*)p.A + gi * p.sAi + gd * p.sAd;
    const T* B = (const T*)p.B + gi * p.sBi + gd * p.sBd;
    ASrc a; BSrc b;
    // A rows-contiguous operand is loaded in 16-byte chunks of rows: its row count is rounded up (its k-rows
    // are ld >= that many elements long, so the extra rows are readable; their products are never stored).
    constexpr int EPC = 16 / (int)sizeof(T);
    if constexpr (AKC) { a.base = A + (int64_t)m0 * p.lda; a.R = p.M - m0; } else { a.base = A + m0; a.R = (p.M - m0 + EPC - 1) & ~(EPC - 1); }
    a.ld = p.lda;
    if constexpr (BKC) { b.base = B + (int64_t)n0 * p.ldb; b.R = p.N - n0; } else { b.base = B + n0; b.R = (p.N - n0 + EPC - 1) & ~(EPC - 1); }
    b.ld = p.ldb;

    float bias[FN];
    load_bias<Core, FN>(bias, p, n0, gi, gd);
    f32x16_t acc[FM][FN];
    zero_tile<FM, FN>(acc);
    Core::run_deep(acc, a, b, p.K, lds);
    if (m0 + Core::BM <= p.M && n0 + Core::BN <= p.N && p.ldc < (1 << 26)) store_tile_interior<T, Core, FM, FN>(acc, bias, p, m0, n0, gi, gd);
    else store_tile<T, Core, FM, FN>(acc, bias, p, m0, n0, gi, gd);
}

// The tile configuration of a problem (see gemm.hip; -1: not a valid problem), whether its operands meet the rules of the direct
// loads, and whether an fp32 problem runs on fp32 MFMAs: the smallest ones in 64x64 tiles, long contractions in tiles of either size.
int gemm_pick_tile(const GemmDesc& d, bool& dma);
bool gemm_plain_fp32(const GemmDesc& d);
bool gemm_long_fp32(const GemmDesc& d);
inline int64_t gemm_tiles(const GemmDesc& d, int bm, int bn) {
    return (int64_t)((d.M + bm - 1) / bm) * ((d.N + bn - 1) / bn) * d.groupsI * d.groupsD;
}

// fp32 operands on the bf16 matrix units (gemm_split.hpp), in 128x128 (large) or 64x64 tiles; operands as for the direct-to-LDS kernels.
hipError_t launch_gemm_split(const GemmDesc& d, bool large, hipStream_t s);

}  // namespace adpsgd
