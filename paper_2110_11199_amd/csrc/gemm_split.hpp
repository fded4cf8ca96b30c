// fp32 products on the bf16 matrix units (G. Henry, P. T. P. Tang, A. Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For
// Higher-Precision Computations", 2019).
//
// An fp32 value is the sum of three bf16 values: x1 = bf16(x), x2 = bf16(x - x1), x3 = bf16(x - x1 - x2), 8 bits of the 24
// each, both differences exact.  Of the nine products of two such sums six are taken, x1 y1, x1 y2, x2 y1, x2 y2, x1 y3, x3 y1; the
// other three are below 2^-26 of |x y|, an eighth of the rounding of one fp32 addition.  Six bf16 MFMAs replace eight fp32 ones that
// take 64 cycles each where a bf16 one takes 32 for the same 16 k: the matrix pipe's share of a 32x32x16 block falls from
// 512 cycles to 192.  Each MFMA rounds its accumulator once, six times for 16 k against eight.
//
// What bounds it: in large products the power limit, 217 TFLOP/s of fp32 (1.3 PFLOP/s of bf16 MFMAs, what the bf16 kernels reach too)
// against 146 with fp32 MFMAs (4096 x 6144 x 2048: 475 us); in small ones how the tiles cover the compute units and, in 64x64 tiles, the
// vector instructions of the conversion (9 to an MFMA).  us, fp32 MFMAs -> here: 672x2048x512x8 98 -> 70, 1280x1280x320x6 54 -> 40,
// 672x512x1000x8 50 -> 45, 1280x320x1280x6 61 -> 51.  Error against 64 bits, 2-norm, fp32 MFMAs / here in 128x128 / 64x64 tiles (whose two chunks
// of a stage have an accumulator each): K = 36 1.1e-7 / 8.6e-8 / 5.9e-8, 512 4.1e-7 / 3.4e-7 / 2.4e-7, 2048 8.1e-7 / 7.0e-7 / 4.9e-7, 4096 1.15e-6 /
// 1.0e-6 / -; operands of a range of 2^30: 2.4e-7 / 2.4e-7 / 1.7e-7 (K = 512).
//
// The workgroup converts as it stages: global -> registers (two stages ahead) -> three bf16 planes in LDS, each laid out as the bf16 tiles of
// gemm_dma.hpp (row-major for a K-contiguous operand, k-row by k-row for the other, which the LDS read transposes).  A value is
// converted once per workgroup, 6 vector instructions, and read by two waves.
//
// Upper end of the range.  Values whose x1 is not finite (infinities, NaN, the largest 2^-9 of the range) would turn into NaN (0 x inf in a product
// with an absent x2); their x3 is NaN.  The conversion accumulates products of two x3, and a workgroup that finds the sum not to be finite does
// its tile again with fp32 MFMAs.  The sum overflows for ordinary values too, from about 2^81 on: such a tile is done twice, its result as good.
// A sum that comes within 2^-8 of the largest fp32 value can overflow here and not there (x1 y1 is that much larger than x y).
//
// Lower end.  x3 and then x2 of a value below 2^-110 fall below the smallest bf16, 2^-133: it is held to 2^-134, whatever it is multiplied with.  Error against 64
// bits, 2-norm, K = 512, all values of one operand (normally distributed) times 2^-108 3.4e-7, 2^-112 3.7e-7, 2^-115 1.2e-6, 2^-120 3.5e-5, 2^-126 2.3e-3; fp32 MFMAs
// 4.1e-7 throughout.  A matrix of nothing but such values is no operand of a gradient (features and weights are of the order of 1, gradients
// of 1e-9); beside larger ones in its row or column they do not count.  Finding them would take two more vector instructions a value.
#pragma once
#include "gemm_core.hpp"
#include "gemm_dma.hpp"
#include "gemm_tile.hpp"

namespace adpsgd {

// Workgroup tile 64 F x 64 F on 2 x 2 waves, KT of K to a stage: 16 values of each operand's half of the threads.
template <bool AKC, bool BKC, int F> struct SplitCore {
    static constexpr int KT = F == 1 ? 32 : 16, SB = 2 * KT, BM = 64 * F, BN = BM;
    typedef typename std::conditional<AKC, KcSrc<float>, McSrc<float>>::type ASrc;
    typedef typename std::conditional<BKC, KcSrc<float>, McSrc<float>>::type BSrc;
    typedef GemmDma<bf16_t, KcSrc<bf16_t>, KcSrc<bf16_t>, 2, 2, F, F, SB, 2> Planes;       // (fragment reads, swizzles, accumulator layout)
    typedef GemmDma<float, ASrc, BSrc, 2, 2, F, F, 64, F == 1 ? 4 : 3> Plain;
    static constexpr int NC = KT / 16, NACC = NC * F * F;                                  // k-chunks of a stage; accumulators: (chunk, fm, fn)
    static constexpr int PLANE = BM * SB, STAGE = 6 * PLANE;                               // bytes: a plane of one operand, a stage
    static constexpr int LDS_BYTES = 2 * STAGE > Plain::LDS_BYTES ? 2 * STAGE : Plain::LDS_BYTES;
    static_assert(BM * KT == 128 * 16, "four float4 to a thread");

    // Four float4 of one operand's stage; unit t + 128 j of the stage's BM * KT / 4.
    template <class Src> struct Loader {
        uint32_t off[4]; int k[4]; uint32_t lds[4];
        __device__ void init(const Src& src, int t) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int u = t + 128 * j;
                if constexpr (Src::kc) {
                    const int row = u / (KT / 4), kq = u % (KT / 4);
                    k[j] = 4 * kq;
                    off[j] = (uint32_t)(src.row_offset_clamped(row) + 4 * kq) * 4u;
                    lds[j] = (uint32_t)(row * SB + (((kq >> 1) ^ swz_<SB>(row)) * 16) + (kq & 1) * 8);
                } else {
                    const int kr = u / (BM / 4), rq = u % (BM / 4);
                    k[j] = kr;
                    off[j] = (uint32_t)(src.chunk_offset_clamped(kr, rq)) * 4u;
                    lds[j] = (uint32_t)(kr * (BM * 2) + (((rq >> 1) ^ Planes::template mc_swz<BM>(kr)) * 16) + (rq & 1) * 8);
                }
            }
        }
        // (of the last stage what lies past K is read from inside it and cleared before it is converted)
        __device__ void load(const Src& src, int s, int K, float4 (&v)[4]) const {
            const int k0 = s * KT;
            const char* base = (const char*)(Src::kc ? src.base + k0 : src.base + (int64_t)k0 * src.ld);
            uint32_t o[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] = off[j];
            if (k0 + KT > K) {
                const int last = Src::kc ? (K - k0 - 1) & ~3 : K - k0 - 1;
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (k[j] > last) o[j] -= Src::kc ? (uint32_t)(k[j] - last) * 4u : (uint32_t)(k[j] - last) * (uint32_t)src.ld * 4u;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = *(const float4*)(base + o[j]);
        }
        __device__ void clear_past(int s, int K, float4 (&v)[4]) const {
            const int rem = K - s * KT;
            if (rem >= KT) return;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (k[j] >= rem) v[j] = make_float4(0.f, 0.f, 0.f, 0.f);
                if (Src::kc) {                             // (rows are padded to 16 bytes where K is not a whole number of them)
                    if (k[j] + 1 >= rem) v[j].y = 0.f;
                    if (k[j] + 2 >= rem) v[j].z = 0.f;
                    if (k[j] + 3 >= rem) v[j].w = 0.f;
                }
            }
        }
        // Piece I of the conversion of the 16 values v into the three planes of the stage: of a pair of values first x1, then x2 and
        // x3 and, after two pairs, the stores.  bad becomes infinite or NaN where a value has no finite x1 (x3 is NaN then).
        struct Work { float x, y; uint32_t p[3][2]; };
        template <int I> __device__ void piece(char* lds_op, const float4 (&v)[4], Work& w, float& bad) const {
            constexpr int j = I / 4, h = I / 2 % 2;
            if constexpr (I % 2 == 0) {
                w.x = h ? v[j].z : v[j].x; w.y = h ? v[j].w : v[j].y;
                const uint32_t q = pack_bf16(w.x, w.y);
                w.x -= __builtin_bit_cast(float, q << 16); w.y -= __builtin_bit_cast(float, q & 0xffff0000u);
                w.p[0][h] = q;
            } else {
                const uint32_t q = pack_bf16(w.x, w.y);
                w.x -= __builtin_bit_cast(float, q << 16); w.y -= __builtin_bit_cast(float, q & 0xffff0000u);
                bad = fmaf(w.x, w.y, bad);
                w.p[1][h] = q; w.p[2][h] = pack_bf16(w.x, w.y);
                if constexpr (h == 1) {
#pragma unroll
                    for (int k = 0; k < 3; ++k) *(uint2*)(lds_op + k * PLANE + lds[j]) = make_uint2(w.p[k][0], w.p[k][1]);
                }
            }
        }
        __device__ void convert(char* lds_op, const float4 (&v)[4], float& bad) const {
            Work w;
            Planes::template static_for<0, 16>([&](auto i) { piece<decltype(i)::value>(lds_op, v, w, bad); });
        }
    };

    // One stage: the products of the planes at st, and (STORE) between them, piece by piece, the conversion of the next
    // stage's values v: its vector instructions run while the matrix unit does.  The scheduling barriers keep this order.
    template <bool STORE, class Ld>
    __device__ static void stage(f32x16_t (&acc)[NACC], const char* st, int wave_m, int wave_n, int lane, const Ld& ld, char* lds_op,
                                 const float4 (&v)[4], float& bad) {
        constexpr int NM = 6 * NACC;
        constexpr int QA[6] = {0, 2, 1, 0, 1, 0}, QB[6] = {2, 0, 1, 1, 0, 0};               // (the smallest products first)
        uint4 a[3][NC * F], b[3][NC * F];
        auto read = [&](int q, bool of_a) {
#pragma unroll
            for (int j = 0; j < NC * F; ++j) {
                const int ch = 2 * (j / F) + (lane >> 5), f = j % F;
                if (of_a) a[q][j] = Planes::template frag<BM, AKC>(st + q * PLANE, (wave_m * F + f) * 32, ch, lane);
                else b[q][j] = Planes::template frag<BN, BKC>(st + (3 + q) * PLANE, (wave_n * F + f) * 32, ch, lane);
            }
        };
        read(0, true); read(2, false); read(2, true); read(0, false); read(1, true); read(1, false);
        __builtin_amdgcn_sched_barrier(0);
        typename Ld::Work w;
        Planes::template static_for<0, NM>([&](auto ii) {
            constexpr int i = decltype(ii)::value, t = i / NACC, n = i % NACC, c = n / (F * F), fm = n % (F * F) / F, fn = n % F;
            mma_chunk<bf16_t>(acc[n], a[QA[t]][c * F + fm], b[QB[t]][c * F + fn]);
            if constexpr (STORE)
                Planes::template static_for<i * 16 / NM, (i + 1) * 16 / NM>([&](auto k) { ld.template piece<decltype(k)::value>(lds_op, v, w, bad); });
            __builtin_amdgcn_sched_barrier(0);
        });
    }

    __device__ static void barrier() {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // (the loads of later stages stay in flight)
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    }

    template <class Src>
    __device__ static float run_as(f32x16_t (&acc)[NACC], const Src& src, int K, char* lds, char* lds_op, int t) {
        const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        const int wave_m = wave / 2, wave_n = wave % 2, nk = (K + KT - 1) / KT;
        Loader<Src> ld;
        ld.init(src, t);
        float bad = 0.f;
        float4 v0[4], v1[4];
        ld.load(src, 0, K, v0);
        if (nk > 1) ld.load(src, 1, K, v1);
        if (nk == 1) ld.clear_past(0, K, v0);
        ld.convert(lds_op, v0, bad);
        barrier();
        // stage s, from the buffer of its parity: what it loads goes into the registers that it has converted from
        auto step = [&](int s, float4 (&cur)[4], float4 (&nxt)[4]) {
            ld.load(src, s + 2, K, cur);
            stage<true>(acc, lds + (s & 1) * STAGE, wave_m, wave_n, lane, ld, lds_op + ((s + 1) & 1) * STAGE, nxt, bad);
            barrier();
        };
        int s = 0;
        for (; s + 3 < nk; s += 2) { step(s, v0, v1); step(s + 1, v1, v0); }
        if (s + 2 < nk) {
            step(s, v0, v1); ++s;
#pragma unroll
            for (int j = 0; j < 4; ++j) v1[j] = v0[j];
        }
        if (s + 1 < nk) {
            ld.clear_past(s + 1, K, v1);
            stage<true>(acc, lds + (s & 1) * STAGE, wave_m, wave_n, lane, ld, lds_op + ((s + 1) & 1) * STAGE, v1, bad);
            barrier();
            ++s;
        }
        stage<false>(acc, lds + (s & 1) * STAGE, wave_m, wave_n, lane, ld, lds_op, v1, bad);
        return bad;
    }

    __device__ static void run(f32x16_t (&acc)[F][F], const ASrc& a, const BSrc& b, int K, char* lds) {
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), t = threadIdx.x & 127;
        float bad;
        f32x16_t part[NACC];
#pragma unroll
        for (int n = 0; n < NACC; ++n) part[n] = acc[n % (F * F) / F][n % F];              // (zeros)
        if constexpr (AKC == BKC) {
            ASrc src = a;
            if (wave >= 2) src = b;
            bad = run_as(part, src, K, lds, lds + (wave >> 1) * (3 * PLANE), t);
        } else {
            bad = wave < 2 ? run_as(part, a, K, lds, lds, t) : run_as(part, b, K, lds, lds + 3 * PLANE, t);
        }
        if (__builtin_expect(__syncthreads_or(!(bad - bad == 0.f)), 0)) {
            Plain::run_deep(acc, a, b, K, lds);
            return;
        }
#pragma unroll
        for (int n = 0; n < F * F; ++n) {
            acc[n / F][n % F] = part[n];
            if constexpr (NC == 2) acc[n / F][n % F] += part[n + F * F];
        }
    }
};

template <bool AKC, bool BKC, int F>
__device__ __forceinline__ void split_tile(const GemmDesc& p, int bid, int total, char* lds) {
    typedef SplitCore<AKC, BKC, F> Core;
    const int tiles_m = (p.M + Core::BM - 1) / Core::BM, tiles_n = (p.N + Core::BN - 1) / Core::BN;
    int grp, tm, tn;
    map_tile(bid, total, tiles_m, tiles_n, grp, tm, tn);
    const int gi = p.lmap.idx[grp / p.groupsD], gd = grp % p.groupsD;
    const int m0 = tm * Core::BM, n0 = tn * Core::BN;
    const float* A = (const float*)p.A + gi * p.sAi + gd * p.sAd;
    const float* B = (const float*)p.B + gi * p.sBi + gd * p.sBd;
    // (a rows-contiguous operand's k-rows are readable up to a whole number of 16 bytes)
    typename Core::ASrc a; typename Core::BSrc b;
    if constexpr (AKC) { a.base = A + (int64_t)m0 * p.lda; a.R = p.M - m0; } else { a.base = A + m0; a.R = (p.M - m0 + 3) & ~3; }
    a.ld = p.lda;
    if constexpr (BKC) { b.base = B + (int64_t)n0 * p.ldb; b.R = p.N - n0; } else { b.base = B + n0; b.R = (p.N - n0 + 3) & ~3; }
    b.ld = p.ldb;
    float bias[F];
    load_bias<typename Core::Planes, F>(bias, p, n0, gi, gd);
    f32x16_t acc[F][F];
    zero_tile<F, F>(acc);
    Core::run(acc, a, b, p.K, lds);
    if (m0 + Core::BM <= p.M && n0 + Core::BN <= p.N && p.ldc < (1 << 26)) store_tile_interior<float, typename Core::Planes, F, F>(acc, bias, p, m0, n0, gi, gd);
    else store_tile<float, typename Core::Planes, F, F>(acc, bias, p, m0, n0, gi, gd);
}

}  // namespace adpsgd
