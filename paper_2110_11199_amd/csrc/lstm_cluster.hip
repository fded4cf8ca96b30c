// Recurrent LSTM kernels that keep W_h on the registers of a few compute units: all T frames of one layer in one launch, for
// hidden sizes above what one compute unit holds (lstm_resident.hip).
//
// Frame by frame such a layer costs a launch, W_h from the caches and a latency-bound product per frame: 8-20 us, of which the
// products are 1-4; here 2.9-4 where all clusters run at once (both sides at the rule below).  Iterations: fp32 8 x 2 x 256 cells 1556 -> 771 us,
// 6 x 320 2709 -> 1140, bf16 5 x 2 x 360 1316 -> 608.  What is left of a frame: the exchange (0.5-1 us), products of one wave per SIMD, the cells.
//
// Here a CLUSTER of S workgroups takes 16 batch rows of one (learner, direction) through all frames (batch rows do not depend
// on each other: as many clusters as row blocks).  Workgroup m of a cluster owns U hidden units and holds their part of W_h as
// MFMA fragments in registers (a wave per SIMD, up to 320 of its 512 registers); the cell state (dL/dc) stays in registers too.
// What a frame needs of the other workgroups goes through memory:
//   forward   h_{t'} of all units (H values per row, in the operand type) - every workgroup reads all of it into LDS;
//   backward  dh = da W_h is split over its CONTRACTION: workgroup m multiplies the da of its own units (LDS) with their rows of
//             W_h and hands every workgroup the partial sums of its units (fp32): H words read and H written a row and member.
//             Splitting over the result instead would have every workgroup read all of da: 4 H words read and 4 U written in
//             fp32; with bf16 operands, two values to a word, 2 H and 2 U, about as many in all but far fewer writes (not tried).
//
// Exchange.  A 32-bit payload and a 32-bit tag travel in one aligned 64-bit word, written and read whole (two words to a
// 16-byte access, each with its own tag): a word is there or it is not, so there are no fences, no write-backs and no counters, and a
// frame costs one store-to-load latency.  The tag counts frames over launches AND iterations (a device word that the staging
// kernel of every iteration increments, so that a replayed recording gets new tags as well), so nothing is cleared between uses;
// the buffer is zeroed when the handle is made and 0 is no tag in use.  Two slots by the parity of the frame suffice: whoever
// writes frame s has received all of frame s-1, whose senders had read frame s-2.
// The words are read past the first-level cache (device scope), which the L2 of an XCD answers.  Members that all run on one
// XCD therefore store them at workgroup scope, to that L2 and no further; others have to write through to memory.  An
// all-to-all of 256 threads x N words between 8 workgroups, us: N = 1 0.64 through memory, 0.36 in one L2; 8 1.36, 0.63 (0.54 with
// 16-byte loads); 12 1.68, 0.77 (0.71); 24 2.31, 1.35 (0.97).  Workgroup ids go round the 8 XCDs, so the members of a
// cluster take ids 8 apart; what decides is not that, but the XCD each of them reads from its hardware register.
// The backward pass exchanges the most for its size, H words of 64 bits a row written and read by every member: 5 MB an XCD
// in two slots at 640 cells in bf16, more than its L2 holds.  On one XCD it writes bare values instead, waits until they are there (the
// L2 acknowledges a store) and then writes a flag to each member, tagged as above; whoever finds the flags loads the values: half the
// bytes for one more latency.  us per frame, tagged words / flags: 4 x 512 cells, batch 16 3.6 / 3.1, 16 x 512, 32 6.1 / 4.0, 32 x 512, 64 22.0 / 15.3,
// 10 x 360, 50 4.8 / 3.2, 10 x 640, 32 7.7 / 4.8, 16 x 256, 64 3.8 / 3.1; fp32 16 x 512, 32 15.9 / 13.6, 6 x 320, 64 4.4 / 3.9.  (Values and tagged words have memory of their own: a value could
// pass for a tag.)
//
// Progress.  Every workgroup counts itself into its cluster's word when it STARTS, by XCD, and exchanges nothing before
// all members have: from there on every member runs, whatever else shares the device and in whatever order workgroups are
// dispatched.  The grid may exceed the chip.  A cluster that stays incomplete for longer than the other workgroups of the
// launch can explain - other work holds the device, or other such launches with incomplete clusters of their own - is closed (a bit
// of the same word) and left to one of those that wait, which does all of it alone (forward_alone_, backward_alone_): the
// same operations in the same order, slower by the number of members and by W_h from the caches (us per frame, forward /
// backward, one cluster, together against alone: fp32 256 cells 3.2 / 3.1 against 44 / 61, bf16 640 cells 3.7 / 3.8 against 96 / 247; all 32 of
// 16 x 640, batch 32 7.3 / 8.5 against 123 / 516).  So
// nothing waits for workgroups that may not come.  Every wait of the exchange is bounded all the same (wait_ticks of
// the 100 MHz clock, or another workgroup's expiry): the workgroup raises kStatusWaitExpired and returns.
//
// MFMA operand mapping (16x16 tiles) as in lstm_resident.hip.
#include <algorithm>
#include <type_traits>
#include "gemm_core.hpp"
#include "kernels.hpp"
#include "rec_tiles.hpp"

namespace adpsgd {
namespace {

// S workgroups of 4 waves per cluster.  bf16: a wave holds the four gates of 16 units, U = 64.  fp32, whose products are 16
// times slower: two waves share 16 units, each with half of the contraction, U = 32.
template <typename T, int S_> struct Cl {
    static constexpr int S = S_, KS = sizeof(T) == 4 ? 2 : 1, NU = 4 / KS, U = 16 * NU, KP = S * U;   // KP: padded H
    static constexpr int EL = 16 / (int)sizeof(T), KC = 4 * EL, NCH = KP / KC, CW = NCH / KS;           // k-chunks: all, of a wave
    static constexpr int RB = 16;                          // batch rows of a cluster
    static constexpr int VW = 4 / (int)sizeof(T), RW = KP / VW;                 // values per exchange word, words per row of h
    static constexpr int FWD_ROW = KP * (int)sizeof(T) + 16, BWD_ROW = 4 * U * (int)sizeof(T) + 16;     // bytes of an LDS row
    // PARTS: fp32 as three bf16 parts, up to 320 cells (more than 240 registers of W_h a lane, 360 at 384 cells, and the compiler moves them about:
    // us per frame, fp32 MFMAs / parts: 256 cells 3.8 / 3.2, 320 4.3 / 3.7, 384 4.8 / 4.5 and 3 us more a launch, 512 6.2 / 6.6).  Bytes of an LDS row of a part, of the 16 rows; chunks of 32 k of a wave
    static constexpr int FWD_PART_ROW = KP * 2 + 16, BWD_PART_ROW = 4 * U * 2 + 16, FWD_PART = RB * FWD_PART_ROW, BWD_PART = RB * BWD_PART_ROW;
    static constexpr bool PARTS = sizeof(T) == 4 && S <= 10;
    static constexpr int PCW = KP / (32 * KS), PBCH = 4 * U / 32;
    static constexpr bool SETTLE_F = sizeof(T) == 2 || (PARTS && S > 8), SETTLE_B = PARTS || (sizeof(T) == 2 && S <= 8);   // (settle_)
    static constexpr int FWD_BUF = PARTS ? 3 * FWD_PART : RB * FWD_ROW, BWD_BUF = PARTS ? 3 * BWD_PART : RB * BWD_ROW;   // one frame's operand
    static constexpr int W_ROW = KP + 4;                   // words of a row of staged W_h: rows 4 apart lie 16 banks apart
    static constexpr int BCH = 4 * U / KC, NT = KP / 64;                        // backward: k-chunks, 16-column tiles of a wave
    static constexpr int PR = RB * U / 256;                                     // backward: consecutive units of a row that a thread finishes
    static constexpr int64_t FWD_SLOT = (int64_t)RB * RW, BWD_SLOT = (int64_t)S * RB * KP;              // exchange words
    // backward on one XCD: values without tags, and flags: 32-bit words of a slot, values and then a flag per (target, sender, wave)
    static constexpr int64_t RAW_VALUES = BWD_SLOT, RAW_SLOT = RAW_VALUES + (int64_t)S * 4 * S;
    static_assert(NCH % KS == 0 && KP % 64 == 0 && RW % 64 == 0 && PR * (int)sizeof(T) == 8, "tiling");
};

// Scratch words of a workgroup that does a cluster's work alone.
typedef __attribute__((address_space(1))) uint64_t word_t;
__device__ inline void scratch_put_(word_t* at, float v) {
    __hip_atomic_store(at, (uint64_t)__builtin_bit_cast(uint32_t, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline float scratch_get_(const word_t* at) {
    return __builtin_bit_cast(float, (uint32_t)__hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}

// Scopes of the accesses to exchange words (cache policy bits of the buffer instructions): stores to the L2 of this XCD, or through
// it to memory; loads past the first-level cache.
constexpr int kToL2 = 1, kToMemory = 16, kFromL2 = 16;
template <int SCOPE> __device__ inline void put_(buf_t x, uint32_t lane_bytes, uint32_t bytes, uint32_t v, uint32_t tag) {
    const u32x2_t w = {v, tag};
    __builtin_amdgcn_raw_buffer_store_b64(w, x, (int)lane_bytes, (int)bytes, SCOPE);
}
template <int SCOPE> __device__ inline void put2_(buf_t x, uint32_t lane_bytes, uint32_t bytes, float v0, float v1, uint32_t tag) {
    const u32x4_t w = {__builtin_bit_cast(uint32_t, v0), tag, __builtin_bit_cast(uint32_t, v1), tag};
    __builtin_amdgcn_raw_buffer_store_b128(w, x, (int)lane_bytes, (int)bytes, SCOPE);
}
// Cache policy of what a backward frame reads and writes once: the exchange has to stay in the L2
// beside it (us per frame, without / with, all words tagged: bf16 8 x 2 x 256 cells, batch 64 4.2 / 3.4, 512, 32 6.9 / 5.8, 5 x 2 x 360, 50 4.8 / 4.3; of which the
// loads 0.3 to 0.5).  The forward pass, which reads the lines that it writes, is the slower for it (2.7 / 3.1).
constexpr int kPassing = 2;
// Whether a wait that has looked tries + 1 times may look again.
__device__ inline bool go_on_(const ClusterDesc& p, uint32_t tries, uint64_t& t0, bool& half) {
    if ((tries & 15) != 15 && p.wait_ticks != 0) return true;
    const uint64_t now = wall_clock64();
    if (t0 == 0) t0 = now;
    const uint32_t st = __builtin_amdgcn_readfirstlane((int)__hip_atomic_load(p.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    const bool late = now - t0 >= p.wait_ticks / 2;
    if ((late && half) || p.wait_ticks == 0 || (st & kStatusWaitExpired)) {
        raise_status_(p.status, kStatusWaitExpired);
        return false;
    }
    // the bound runs out in two halves: time in which this wave and those it waits for were off the device counts
    // as one of them at most
    if (late) { half = true; t0 = now; }
    return true;
}
// Pairs of words at lane_bytes + off(0) .. off(N-1), once all of them carry the tag; false when the wait ran out.  (Every branch
// is wave-uniform for the compiler too: a divergent one has it copy the resident fragments around the loop.)
template <int N, class Off>
__device__ inline bool get_(const ClusterDesc& p, buf_t x, uint32_t lane_bytes, Off off, uint32_t tag, uint32_t (&v)[2 * N]) {
    uint64_t t0 = 0;
    bool half = false;
#pragma unroll 1
    for (uint32_t tries = 0;; ++tries) {
        u32x4_t w[N];
        asm volatile("" ::: "memory");                     // (loaded anew in every round)
#pragma unroll
        for (int i = 0; i < N; ++i) w[i] = __builtin_amdgcn_raw_buffer_load_b128(x, (int)lane_bytes, (int)off(i), kFromL2);
        uint32_t differ = 0;
#pragma unroll
        for (int i = 0; i < N; ++i) { differ |= (w[i].y ^ tag) | (w[i].w ^ tag); v[2 * i] = w[i].x; v[2 * i + 1] = w[i].z; }
        // (a bound of 0 gives up at the first exchange, whether the words are there or not)
        if (__ballot(differ != 0) == 0 && p.wait_ticks != 0) return true;
        if (!go_on_(p, tries, t0, half)) return false;
    }
}

// Waits until the n words at lane_bytes = 4 lane carry the tag; false when the wait ran out.
__device__ inline bool wait_flags_(const ClusterDesc& p, buf_t x, uint32_t bytes, int n, int lane, uint32_t tag) {
    uint64_t t0 = 0;
    bool half = false;
#pragma unroll 1
    for (uint32_t tries = 0;; ++tries) {
        asm volatile("" ::: "memory");
        const uint32_t v = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(x, lane * 4, (int)bytes, kFromL2);
        if (__ballot(lane < n && v != tag) == 0 && p.wait_ticks != 0) return true;
        if (!go_on_(p, tries, t0, half)) return false;
    }
}

// The N values of one row that a thread finishes backward, one access.
template <int N> struct Vec;
template <> struct Vec<4> {
    typedef __attribute__((ext_vector_type(4))) float type;
    template <int POLICY = 0> __device__ static type load(buf_t x, uint32_t lane_bytes, uint32_t bytes) {
        return __builtin_bit_cast(type, __builtin_amdgcn_raw_buffer_load_b128(x, (int)lane_bytes, (int)bytes, POLICY));
    }
    template <int POLICY = 0> __device__ static void store(type v, buf_t x, uint32_t lane_bytes, uint32_t bytes) {
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, v), x, (int)lane_bytes, (int)bytes, POLICY);
    }
};
template <> struct Vec<2> {
    typedef f32x2_t type;
    template <int POLICY = 0> __device__ static type load(buf_t x, uint32_t lane_bytes, uint32_t bytes) {
        return __builtin_bit_cast(type, __builtin_amdgcn_raw_buffer_load_b64(x, (int)lane_bytes, (int)bytes, POLICY));
    }
    template <int POLICY = 0> __device__ static void store(type v, buf_t x, uint32_t lane_bytes, uint32_t bytes) {
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2_t, v), x, (int)lane_bytes, (int)bytes, POLICY);
    }
};
// The same N values in the operand type: 8 bytes, four or two of them.
template <class V> __device__ inline u32x2_t operand8_(const V& v) {
    if constexpr (sizeof(V) == 16) return u32x2_t{pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
    else return __builtin_bit_cast(u32x2_t, v);            // (whole: an element of a vector, cast by itself, is its first element)
}
template <int POLICY = 0> __device__ inline void buf_store8_(u32x2_t v, buf_t x, uint32_t lane_bytes, uint32_t bytes) {
    __builtin_amdgcn_raw_buffer_store_b64(v, x, (int)lane_bytes, (int)bytes, POLICY);
}

// Exchange through memory, backward.  A lane holds four consecutive units of a row, 32 bytes of words, two accesses of 16: as they lie, each would be
// half of every line it touches, and stores that write through to memory pay for that twice.  So two lanes whose rows differ swap one of their two pairs,
// and an access covers a row of 16 units, 128 bytes, whole, the next one the other row.  Backward pass of 21 frames, us, half lines / whole (four
// rows of one unit to a thread and whole lines before): bf16 14 x 360 cells, batch 48 193 / 126 (125), 5 x 640, 80 279 / 176 (178); fp32 5 x 320, 65 154 / 136 (135),
// 6 x 348, 48 181 / 167, 12 x 384, 40 348 / 327 (324) and, the operand not read ahead of its products there (AHEAD), 164 (166) and 320.
// rows_out_: (a, b), of units 4 g and 4 g + 2 of row r (lane r + 16 g) -> of units 4 g + 2 (r / 8) of rows r % 8 and r % 8 + 8.
__device__ inline void rows_out_(float& a, float& b) {
    const int x = __builtin_bit_cast(int, a), y = __builtin_bit_cast(int, b);
    a = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(x, y, 0x128, 0xf, 0xc, false));     // lanes 8 to 15 of 16: that of lane ^ 8
    b = __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(y, x, 0x128, 0xf, 0x3, false));     // lanes 0 to 7
}
// rows_in_: (a, b), of units 4 t + 2 (row % 2) of the even row and of the odd one (lane 16 row + t) -> of units 4 t and 4 t + 2 of the lane's row.
__device__ inline void rows_in_(float& a, float& b) {
    const auto v = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b), false, false);
    a = __builtin_bit_cast(float, (uint32_t)v[0]); b = __builtin_bit_cast(float, (uint32_t)v[1]);
}

// A cluster's word: how many of its members have started, 6 bits for each XCD; kClosed and the member it is left to.
constexpr int kXcds = 8;
constexpr uint64_t kClosed = 1ull << 63;
constexpr int kClosedMember = 6 * kXcds;

// Place of this workgroup, and the tag of the launch's frame 0.
struct Place { int li, d, b0, blk, m, cluster; uint32_t tag0; };
template <class C> __device__ inline bool place_(const ClusterDesc& p, Place& w) {
    static_assert(C::S < 64, "members of a cluster");
    const int blocks = (p.r.B + 15) / 16, id = (int)blockIdx.x;
    const int cluster = p.spread ? (id / kXcds / C::S) * kXcds + id % kXcds : id / C::S, pair = cluster / blocks;
    if (pair >= p.r.L * p.r.D) return false;
    w.m = (p.spread ? id / kXcds : id) % C::S;
    w.cluster = cluster; w.blk = cluster % blocks; w.b0 = w.blk * C::RB;
    w.li = __builtin_amdgcn_readfirstlane(p.r.lmap.idx[pair / p.r.D]); w.d = pair % p.r.D;
    w.tag0 = (*p.epoch * (uint32_t)p.launches + (uint32_t)p.launch) * (uint32_t)p.r.T + 1u;
    if (threadIdx.x == 0) {
        uint32_t xcd;
        asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(xcd));
        __hip_atomic_fetch_add(p.join + cluster, 1ull << (6 * (xcd % kXcds)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return true;
}

// Waits until every member has started - kTogether: on several XCDs, kOneXcd: on one - or the cluster is left to one of those
// that have: kAlone + that member.  Exactly one of these is decided, by the cluster's word: it is closed only while
// members are missing, and those that start later find it closed.
constexpr uint32_t kTogether = 0u, kOneXcd = 1u, kAlone = 2u;
template <class C> __device__ inline uint32_t join_(const ClusterDesc& p, const Place& w) {
    if (p.join_ticks == 0) return kAlone;                  // (a bound of 0: the first member takes every cluster)
    uint64_t* const word = p.join + w.cluster;
    uint64_t t0 = 0;
#pragma unroll 1
    for (uint32_t tries = 0;; ++tries) {
        const uint64_t x = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)x), hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(x >> 32));
        const uint64_t seen = (uint64_t)lo | ((uint64_t)hi << 32);
        if (seen & kClosed) return kAlone + (uint32_t)(seen >> kClosedMember) % 64u;
        uint32_t all = 0, most = 0;
#pragma unroll
        for (int i = 0; i < kXcds; ++i) {
            const uint32_t n = (uint32_t)(seen >> (6 * i)) % 64u;
            all += n; most = n > most ? n : most;
        }
        if (all == (uint32_t)C::S) return most == all ? kOneXcd : kTogether;
        if ((tries & 15) != 15) continue;
        const uint64_t now = wall_clock64();
        if (t0 == 0) t0 = now;
        if (now - t0 < p.join_ticks) continue;
        uint64_t expected = seen;
        if (threadIdx.x == 0)
            __hip_atomic_compare_exchange_strong(word, &expected, kClosed | ((uint64_t)w.m << kClosedMember), __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// One 16-byte fragment of a row of W_h (forward): gate q of unit u, k-chunk at k0.
template <typename T, class C> __device__ inline uint4 fwd_frag_(buf_t wh, int H, int q, int u, int k0, int g) {
    const int k = k0 + g * C::EL;                          // H is a multiple of 4
    const uint32_t vw = u < H && k < H ? (uint32_t)(u * H + g * C::EL) * (uint32_t)sizeof(T) : kOutOfRange;
    uint4 v = buf_load16_(wh, vw, (uint32_t)(q * H * H + k0) * (uint32_t)sizeof(T));
    if (k + C::EL > H) v.z = v.w = 0u;                     // bf16, H = 4 mod 8: half a fragment
    return v;
}

// ---- fp32 products on the bf16 matrix units --------------------------------------------------------------
// An fp32 value as the sum of three bf16 values, and six of the nine products of two such sums (gemm_split.hpp): the products of
// a frame at one wave per SIMD, 1.9 us of fp32 MFMAs at 256 cells, take 0.7.  A value without a finite first part makes
// check infinite or NaN (so do ordinary ones from about 2^81 on, whose third parts' products overflow); where one turns up in a member's W_h or,
// backward, in its da of the frame, the member multiplies in fp32, W_h from memory.  The decision is the member's, over its whole workgroup, and a
// workgroup that does a cluster's work alone takes the same one for each member.
__device__ inline void parts2_(float x, float y, uint32_t (&p)[3], float& check) {
    p[0] = pack_bf16(x, y);
    x -= __builtin_bit_cast(float, p[0] << 16); y -= __builtin_bit_cast(float, p[0] & 0xffff0000u);
    p[1] = pack_bf16(x, y);
    x -= __builtin_bit_cast(float, p[1] << 16); y -= __builtin_bit_cast(float, p[1] & 0xffff0000u);
    p[2] = pack_bf16(x, y);
    check = fmaf(x, y, check);
}
__device__ inline void parts8_(const uint4& lo, const uint4& hi, uint4 (&p)[3], float& check) {
    uint32_t w[4][3];
    parts2_(__builtin_bit_cast(float, lo.x), __builtin_bit_cast(float, lo.y), w[0], check);
    parts2_(__builtin_bit_cast(float, lo.z), __builtin_bit_cast(float, lo.w), w[1], check);
    parts2_(__builtin_bit_cast(float, hi.x), __builtin_bit_cast(float, hi.y), w[2], check);
    parts2_(__builtin_bit_cast(float, hi.z), __builtin_bit_cast(float, hi.w), w[3], check);
#pragma unroll
    for (int i = 0; i < 3; ++i) p[i] = make_uint4(w[0][i], w[1][i], w[2][i], w[3][i]);
}
__device__ inline bool not_finite_(float check) { return !(check - check == 0.f); }
// Ends the wave if the flag (in LDS, the same for all waves behind a barrier) is set.  Not a branch for the compiler, which has every exit from a loop
// join the way back into it, and waits at the top of the loop for all that may be outstanding on either.
__device__ inline void end_if_(const int& flag) {
    const int f = __builtin_amdgcn_readfirstlane(flag);
    asm volatile("s_cmp_eq_u32 %0, 0\n\ts_cbranch_scc1 .Lgo_on%=\n\ts_endpgm\n.Lgo_on%=:" ::"s"(f) : "scc");
}
// Fragment i of a member's W_h, when ordinary code has done with it: the first 60 of a lane go to its accumulation registers, which matrix instructions
// read as they are (16 registers are left for sums).  Left to itself the compiler spreads W_h over both halves of the register file and copies
// fragments between them in every frame, 112 copies at 512 cells in bf16, and has no registers to read a frame's operand from the LDS ahead of its products:
// 8 to 16 reads and waits one after the other.  us of a pass of 21 frames, before / with both: forward bf16 16 x 2 x 512 cells, batch 64 297 / 270, 8 x 2 x 640, 96
// 333 / 296, fp32 6 x 320, 64 84 / 80; backward 317 / 312, -, 82 / 79.  SETTLE_F, SETTLE_B: the passes that are the faster for it; not
// forward at 256 cells in fp32, whose registers suffice and whose launch begins 2.4 us later (8 x 256, batch 32, 5 frames 22.1 / 24.8, 21 frames 63.6 / 66.1), nor
// backward at 640 cells in bf16 (415 / 426; there the operand is read three chunks ahead, 404), nor with W_h in fp32 (16 x 2 x 512, 16 313 / 328 and 303 / 313).
__device__ inline void settle_(uint4& w, int i) {
    if (i >= 60) return;
    u32x4_t x = __builtin_bit_cast(u32x4_t, w);
    asm volatile("" : "+a"(x));
    w = __builtin_bit_cast(uint4, x);
}
// acc[0..N) += a b[0..N), smallest products first
template <bool W_FIRST, int N, class B> __device__ inline void mma_parts_(f32x4_t (&acc)[N], const uint4 (&a)[3], B b) {
    constexpr int QA[6] = {0, 2, 1, 0, 1, 0}, QB[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
    for (int t = 0; t < 6; ++t)
#pragma unroll
        for (int j = 0; j < N; ++j) {
            if constexpr (W_FIRST) mma16_<bf16_t>(acc[j], b(j)[QB[t]], a[QA[t]]);
            else mma16_<bf16_t>(acc[j], a[QA[t]], b(j)[QB[t]]);
        }
}
// Eight fp32 values k .. k + 7 of a row of W_h (forward): gate q of unit u.
__device__ inline void fwd_row8_(buf_t wh, int H, int q, int u, int k0, int g, uint4& lo, uint4& hi) {
    const int k = k0 + 8 * g;                              // H is a multiple of 4
    const uint32_t at = (uint32_t)(u * H + 8 * g) * 4u, base = (uint32_t)(q * H * H + k0) * 4u;
    lo = buf_load16_(wh, u < H && k < H ? at : kOutOfRange, base);
    hi = buf_load16_(wh, u < H && k + 4 < H ? at : kOutOfRange, base + 16u);
}

// Gates from pre-activations, in place, and the new cell state; returns h.
__device__ inline float fwd_cell_(f32x4_t (&acc)[4], int i, float& c) {
    acc[0][i] = sigmoidf_(acc[0][i]); acc[1][i] = sigmoidf_(acc[1][i]);
    acc[2][i] = tanhf_(acc[2][i]); acc[3][i] = sigmoidf_(acc[3][i]);
    c = acc[1][i] * c + acc[0][i] * acc[2][i];
    return acc[3][i] * tanhf_(c);
}

// The da of cell i of a thread from dh, dc, the gates, c_t and c_{t'}; dc becomes that of the next frame.
// (rows past the batch and units past H: all gates were read as 0, so all four results are 0)
template <class V> __device__ inline void bwd_cell_(V (&a)[4], int i, float dh, float& dc, const V (&gate)[4], float c, float c_prev) {
    const float ig = gate[0][i], fg = gate[1][i], gg = gate[2][i], og = gate[3][i];
    const float tc = tanhf_(c);
    const float dov = dh * tc;
    const float dcv = dc + dh * og * (1.f - tc * tc);
    const float di = dcv * gg, dg = dcv * ig, df = dcv * c_prev;
    dc = dcv * fg;
    a[0][i] = di * ig * (1.f - ig); a[1][i] = df * fg * (1.f - fg);
    a[2][i] = dg * (1.f - gg * gg); a[3][i] = dov * og * (1.f - og);
}

// fp32: the two waves of a unit hold halves of the contraction; each finishes two of the four rows of a lane.
template <class C> __device__ inline void swap_halves_(f32x4_t (&acc)[4], float* red, int kh, int wave, int lane) {
    float* mine = red + (wave * 8) * 64 + lane;
    const float* other = red + ((wave ^ C::NU) * 8) * 64 + lane;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        mine[(2 * q) * 64] = kh == 0 ? acc[q][2] : acc[q][0];
        mine[(2 * q + 1) * 64] = kh == 0 ? acc[q][3] : acc[q][1];
    }
    lds_barrier_();
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        acc[q][0] = (kh == 0 ? acc[q][0] : acc[q][2]) + other[(2 * q) * 64];
        acc[q][1] = (kh == 0 ? acc[q][1] : acc[q][3]) + other[(2 * q + 1) * 64];
    }
}

// Four bytes of h: a value, or (bf16) two units of one row, swapped with the neighbouring unit's lane: row 2 i + r % 2.
template <typename T, int PR> __device__ inline uint32_t h_word_(const float (&h)[PR], int i, int r) {
    if constexpr (sizeof(T) == 2) {
        const uint32_t own = pack_bf16(h[2 * i], h[2 * i + 1]);
        const uint32_t nb = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)own, 0xB1, 0xf, 0xf, true);   // lane ^ 1
        return (r & 1) ? (nb >> 16) | (own & 0xffff0000u) : (own & 0xffffu) | (nb << 16);
    } else {
        return __builtin_bit_cast(uint32_t, h[i]);
    }
}

// The 16 bytes of consecutive rows k.. of column n of gate q of W_h (backward).
template <typename T> __device__ inline uint4 bwd_frag_(buf_t wh, int H, int q, int k, int n) {
    uint32_t v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        constexpr int EPW = 4 / (int)sizeof(T);
        const int k0 = k + i * EPW;                        // (H: a multiple of 4)
        const uint32_t at = k0 < H && n < H ? (uint32_t)((q * H + k0) * H + n) * (uint32_t)sizeof(T) : kOutOfRange;
        if constexpr (EPW == 1) v[i] = __builtin_bit_cast(uint32_t, buf_load_(wh, at, 0u));
        else v[i] = buf_load2_(wh, at, 0u) | (buf_load2_(wh, at, (uint32_t)H * 2u) << 16);
    }
    return make_uint4(v[0], v[1], v[2], v[3]);
}

// Column sums of da of member mm over the rows of its cluster, in order; bs: a thread's sums over the frames.
template <class C> __device__ inline void bias_sums_(const ClusterDesc& cd, const Place& w, float (&bred)[4][C::RB * C::U], const typename Vec<C::PR>::type (&bs)[4], int mm) {
    constexpr int U = C::U;
    const RecDesc& p = cd.r;
    const int tid = threadIdx.x, H = p.H, cu = mm * U + tid % U;
#pragma unroll
    for (int q = 0; q < 4; ++q) *(typename Vec<C::PR>::type*)&bred[q][tid * C::PR] = bs[q];
    __syncthreads();
    if (tid < 4 * U && cu < H) {
        const int q = tid / U;
        float v = bred[q][tid % U];
#pragma unroll
        for (int k = 1; k < C::RB; ++k) v += bred[q][k * U + tid % U];
        p.dbp[w.li * p.sDBi + (int64_t)w.blk * ((int64_t)p.D * H * 4) + (int64_t)w.d * 4 * H + (int64_t)q * H + cu] = v;
    }
}

// The products of a frame with W_h from memory, operand rows in the operand type in LDS.
template <typename T, class C> __device__ inline void fwd_plain_(f32x4_t (&acc)[4], const char* hl, buf_t wh, int H, int u, int kh, int r, int g) {
    const char* hrow = hl + r * C::FWD_ROW + kh * (C::CW * 64) + g * 16;
#pragma unroll 1
    for (int c = 0; c < C::CW; ++c) {
        const uint4 a = *(const uint4*)(hrow + c * 64);
#pragma unroll
        for (int q = 0; q < 4; ++q) mma16_<T>(acc[q], a, fwd_frag_<T, C>(wh, H, q, u, (kh * C::CW + c) * C::KC, g));
    }
}
template <typename T, class C> __device__ inline void bwd_plain_(f32x4_t (&acc)[C::NT], const char* al, buf_t wh, int H, int m, int wave, int r, int g) {
    const char* arow = al + r * C::BWD_ROW + g * 16;
#pragma unroll 1
    for (int c = 0; c < C::BCH; ++c) {
        const uint4 a = *(const uint4*)(arow + c * 64);
        const int q = c * C::KC / C::U, k = m * C::U + c * C::KC % C::U + g * C::EL;           // a chunk lies in one gate
#pragma unroll
        for (int j = 0; j < C::NT; ++j) {
            const int n = (wave + 4 * j) * 16 + r;
            mma16_<T>(acc[j], bwd_frag_<T>(wh, H, q, k, n), a);
        }
    }
}

// ---- a cluster left to one workgroup --------------------------------------------------------------
// What the members do, member after member in every frame, with the operations of the two kernels above on the same operands in
// the same order (the results have the same bits); the fragments of W_h come from memory for every use, and what the
// members keep in registers from frame to frame lies in memory: the cell state in its tensor (dL/dc in the buffer of the
// frame-by-frame kernels), h in LDS, dh and the sums for the bias gradients in the exchange words, tagged 0, which is no tag in use.
template <typename T, int S>
__device__ inline void forward_alone_(const ClusterDesc& cd, const Place& w, char* lds, float* red) {
    typedef Cl<T, S> C;
    constexpr int KS = C::KS, PR = 4 / KS;
    constexpr bool PARTS = C::PARTS;
    const RecDesc& p = cd.r;
    const int D = p.D, H = p.H, B = p.B, Tn = p.T, d = w.d;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), r = lane & 15, g = lane >> 4;
    const int kh = wave / C::NU, row0 = 4 * g + (KS == 2 ? 2 * kh : 0);
    const uint32_t DH = (uint32_t)(D * H), G4 = DH * 4;
    const buf_t gates = make_buf_(p.gates + w.li * p.sGi, (int64_t)Tn * B * G4 * 4);
    const buf_t cbuf = make_buf_(p.c + w.li * p.sCi + (int64_t)d * Tn * B * H, (int64_t)Tn * B * H * 4);
    const buf_t y = make_buf_((const T*)p.y + w.li * p.sYi, (int64_t)Tn * B * DH * sizeof(T));
    const buf_t wh = make_buf_((const T*)p.wh + w.li * p.sWi + d * p.sWd, (int64_t)4 * H * H * sizeof(T));
#pragma unroll 1
    for (int s = 0; s < Tn; ++s) {
        const uint32_t m = (uint32_t)(d == 0 ? s : Tn - 1 - s) * B, m_prev = (uint32_t)(d == 0 ? s - 1 : Tn - s) * B;
        const char* const hl = lds + (s & 1) * (C::RB * C::FWD_ROW);
        char* const ho = lds + ((s + 1) & 1) * (C::RB * C::FWD_ROW);
#pragma unroll 1
        for (int mm = 0; mm < S; ++mm) {
            const int u = mm * C::U + (wave % C::NU) * 16 + r;
            float pre[4][PR], cs[PR], h[PR];
            uint32_t vg[PR], vc[PR];
#pragma unroll
            for (int i = 0; i < PR; ++i) {
                const uint32_t row = w.b0 + row0 + i;
                const bool ok = u < H && (int)row < B;
                vg[i] = ok ? (row * G4 + d * 4 * H + u) * 4u : kOutOfRange;
                vc[i] = ok ? (row * H + u) * 4u : kOutOfRange;
                cs[i] = s > 0 ? buf_load_(cbuf, vc[i], m_prev * H * 4u) : 0.f;
#pragma unroll
                for (int q = 0; q < 4; ++q) pre[q][i] = buf_load_(gates, vg[i], (m * G4 + q * H) * 4u);
            }
            f32x4_t acc[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if constexpr (KS == 1) acc[q] = f32x4_t{pre[q][0], pre[q][1], pre[q][2], pre[q][3]};
                else acc[q] = kh == 0 || s == 0 ? f32x4_t{pre[q][0], pre[q][1], 0.f, 0.f} : f32x4_t{0.f, 0.f, pre[q][0], pre[q][1]};
            }
            if (s > 0) {
                bool plain = true;
                if constexpr (PARTS) {
                    const char* hrow = hl + r * C::FWD_ROW + kh * (C::PCW * 128) + g * 32;
                    f32x4_t sum[4] = {acc[0], acc[1], acc[2], acc[3]};
                    float check = 0.f, unused = 0.f;
#pragma unroll 1
                    for (int c = 0; c < C::PCW; ++c) {
                        uint4 a[3], b[4][3];
                        parts8_(*(const uint4*)(hrow + c * 128), *(const uint4*)(hrow + c * 128 + 16), a, unused);
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            uint4 lo, hi;
                            fwd_row8_(wh, H, q, u, (kh * C::PCW + c) * 32, g, lo, hi);
                            parts8_(lo, hi, b[q], check);
                        }
                        mma_parts_<false, 4>(sum, a, [&](int q) -> const uint4 (&)[3] { return b[q]; });
                    }
                    plain = __syncthreads_or(not_finite_(check));
                    if (!plain) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) acc[q] = sum[q];
                    }
                }
                if (plain) fwd_plain_<T, C>(acc, hl, wh, H, u, kh, r, g);
                if constexpr (KS == 2) swap_halves_<C>(acc, red, kh, wave, lane);
            }
#pragma unroll
            for (int i = 0; i < PR; ++i) h[i] = fwd_cell_(acc, i, cs[i]);
#pragma unroll
            for (int i = 0; i < PR / C::VW; ++i) {
                const int row = row0 + i * C::VW + (C::VW == 2 ? r & 1 : 0);
                const uint32_t hw = h_word_<T>(h, i, r);
                *(uint32_t*)(ho + row * C::FWD_ROW + u / C::VW * 4) = hw;
                const uint32_t vy = u < H && w.b0 + row < B ? ((uint32_t)(w.b0 + row) * DH + d * H + (u & ~(C::VW - 1))) * (uint32_t)sizeof(T) : kOutOfRange;
                buf_store_(__builtin_bit_cast(float, hw), y, vy, m * DH * (uint32_t)sizeof(T));
            }
#pragma unroll
            for (int i = 0; i < PR; ++i) {
#pragma unroll
                for (int q = 0; q < 4; ++q) buf_store_(acc[q][i], gates, vg[i], (m * G4 + q * H) * 4u);
                buf_store_(cs[i], cbuf, vc[i], m * H * 4u);
            }
            __syncthreads();
        }
    }
}

template <typename T, int S>
__device__ inline void backward_alone_(const ClusterDesc& cd, const Place& w, char* lds, float (&bred)[4][Cl<T, S>::RB * Cl<T, S>::U]) {
    typedef Cl<T, S> C;
    constexpr int U = C::U, PR = C::PR;
    typedef typename Vec<PR>::type V;
    const RecDesc& p = cd.r;
    const int D = p.D, H = p.H, B = p.B, Tn = p.T, d = w.d;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), r = lane & 15, g = lane >> 4;
    const uint32_t DH = (uint32_t)(D * H), G4 = DH * 4;
    const buf_t gates = make_buf_(p.gates + w.li * p.sGi, (int64_t)Tn * B * G4 * 4);
    const buf_t cbuf = make_buf_(p.c + w.li * p.sCi + (int64_t)d * Tn * B * H, (int64_t)Tn * B * H * 4);
    const buf_t dy = make_buf_(p.dy + w.li * p.sDYi, (int64_t)Tn * B * DH * 4);
    const buf_t da = make_buf_((const T*)p.da + w.li * p.sDAi, (int64_t)Tn * B * G4 * sizeof(T));
    const buf_t dcb = make_buf_(p.dc + w.li * p.sDCi + (int64_t)d * B * H, (int64_t)B * H * 4);
    const buf_t wh = make_buf_((const T*)p.wh + w.li * p.sWi + d * p.sWd, (int64_t)4 * H * H * sizeof(T));
    // scratch: dh [16 rows][KP] in the first slot of the cluster, sums of da [member][gate][unit of a thread][thread] in the second
    word_t* const dh_buf = (word_t*)cd.exchange + (int64_t)w.cluster * 2 * C::BWD_SLOT;
    word_t* const bs_buf = dh_buf + C::BWD_SLOT;
    static_assert(S * 4 * PR * 256 <= C::BWD_SLOT && S <= 16, "the sums of da fit a slot, the members a half of in_fp32");
    const int crow = tid / 16, uu = tid % 16 * PR;           // this thread's row, and the first of its units
    uint32_t in_fp32 = 0;                                  // members that multiply in fp32, by the parity of the frame (not_finite of the kernel below)
#pragma unroll 1
    for (int s = 0; s < Tn; ++s) {
        const uint32_t m = (uint32_t)(d == 0 ? Tn - 1 - s : s) * B, m_next = (uint32_t)(d == 0 ? Tn - 2 - s : s + 1) * B;
        f32x4_t sum[C::NT];                                // over the members, in order
#pragma unroll
        for (int j = 0; j < C::NT; ++j) sum[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int mm = 0; mm < S; ++mm) {
            const int cu = mm * U + uu;
            const uint32_t row = w.b0 + crow;
            const bool ok = cu < H && (int)row < B;
            const uint32_t vg = ok ? (row * G4 + d * 4 * H + cu) * 4u : kOutOfRange, vc = ok ? (row * H + cu) * 4u : kOutOfRange;
            const uint32_t vy = ok ? (row * DH + d * H + cu) * 4u : kOutOfRange;
            float check = 0.f;
            V gate[4], a4[4], dcv = s > 0 ? Vec<PR>::load(dcb, vc, 0u) : V{};
#pragma unroll
            for (int q = 0; q < 4; ++q) gate[q] = Vec<PR>::load(gates, vg, (m * G4 + q * H) * 4u);
            const V in_dy = Vec<PR>::load(dy, vy, m * DH * 4u), in_c = Vec<PR>::load(cbuf, vc, m * H * 4u);
            const V c_prev = Vec<PR>::load(cbuf, s + 1 < Tn ? vc : kOutOfRange, s + 1 < Tn ? m_next * H * 4u : 0u);
#pragma unroll
            for (int i = 0; i < PR; ++i) {
                const float dh = s > 0 ? scratch_get_(dh_buf + crow * C::KP + cu + i) : 0.f;
                float dc = dcv[i];
                bwd_cell_(a4, i, in_dy[i] + dh, dc, gate, in_c[i], c_prev[i]);
                dcv[i] = dc;
            }
            Vec<PR>::store(dcv, dcb, vc, 0u);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
#pragma unroll
                for (int i = 0; i < PR; ++i) {
                    word_t* const at = bs_buf + ((mm * 4 + q) * PR + i) * 256 + tid;
                    scratch_put_(at, (s > 0 ? scratch_get_(at) : 0.f) + a4[q][i]);
                }
                const u32x2_t v = operand8_(a4[q]);
                *(u32x2_t*)(lds + crow * C::BWD_ROW + (uu + q * U) * (int)sizeof(T)) = v;
                buf_store8_(v, da, ok ? vg / (4u / (uint32_t)sizeof(T)) : kOutOfRange, (m * G4 + q * H) * (uint32_t)sizeof(T));
                if constexpr (C::PARTS) {
                    uint32_t a3[3];
                    parts2_(a4[q][0], a4[q][1], a3, check);
                }
            }
            __syncthreads();
            if (s + 1 < Tn) {
                f32x4_t acc[C::NT];
#pragma unroll
                for (int j = 0; j < C::NT; ++j) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
                bool plain = true;
                if constexpr (C::PARTS) {
                    const char* arow = lds + r * C::BWD_ROW + g * 16;
                    float check_w = 0.f, unused = 0.f;
#pragma unroll 1
                    for (int c = 0; c < C::PBCH; ++c) {
                        uint4 a[3], b[C::NT][3];
                        parts8_(*(const uint4*)(arow + c * 128), *(const uint4*)(arow + c * 128 + 64), a, unused);
                        const int k = mm * U + 4 * g;      // rows 4 g .. and 16 + 4 g .. of gate c
#pragma unroll
                        for (int j = 0; j < C::NT; ++j) {
                            const int n = (wave + 4 * j) * 16 + r;
                            parts8_(bwd_frag_<T>(wh, H, c, k, n), bwd_frag_<T>(wh, H, c, k + 16, n), b[j], check_w);
                        }
                        mma_parts_<true, C::NT>(acc, a, [&](int j) -> const uint4 (&)[3] { return b[j]; });
                    }
                    const uint32_t bit = 1u << (mm + 16 * (s & 1));
                    if (__syncthreads_or(not_finite_(check) || not_finite_(check_w))) in_fp32 |= bit;
                    plain = (in_fp32 & bit) != 0;
                    if (plain) {
#pragma unroll
                        for (int j = 0; j < C::NT; ++j) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
                    }
                }
                if (plain) bwd_plain_<T, C>(acc, lds, wh, H, mm, wave, r, g);
#pragma unroll
                for (int j = 0; j < C::NT; ++j) sum[j] += acc[j];
            }
            __syncthreads();                               // the operand is read
        }
        if (s + 1 < Tn) {
#pragma unroll
            for (int j = 0; j < C::NT; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    scratch_put_(dh_buf + r * C::KP + (wave + 4 * j) * 16 + 4 * g + i, sum[j][i]);
            __threadfence();
            __syncthreads();
        }
    }
#pragma unroll 1
    for (int mm = 0; mm < S; ++mm) {
        V bs[4];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < PR; ++i) bs[q][i] = scratch_get_(bs_buf + ((mm * 4 + q) * PR + i) * 256 + tid);
        bias_sums_<C>(cd, w, bred, bs, mm);
        __syncthreads();
    }
}

}  // namespace

// ---- forward ------------------------------------------------------------------------------------
//   a = W_x x_t + b + W_h h_{t'}     i,f,o = sigmoid(a), g = tanh(a)     c_t = f c_{t'} + i g     h_t = o tanh(c_t)
template <typename T, int S>
__global__ __launch_bounds__(256, 1) void rec_forward_cluster_kernel(ClusterDesc cd) {
    typedef Cl<T, S> C;
    constexpr int KS = C::KS, PR = 4 / KS;                 // rows of a 16-row tile that a lane finishes
    constexpr bool PARTS = C::PARTS;
    __shared__ __attribute__((aligned(16))) char lds[2 * C::FWD_BUF];
    __shared__ float red[KS == 2 ? 4 * 8 * 64 : 1];
    __shared__ int expired;
    const RecDesc& p = cd.r;
    Place w;
    if (!place_<C>(cd, w)) return;
    if (threadIdx.x == 0) expired = 0;
    __syncthreads();
    const int D = p.D, H = p.H, B = p.B, Tn = p.T, d = w.d;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), r = lane & 15, g = lane >> 4;
    const int kh = wave / C::NU;                           // which part of the contraction
    const int u = w.m * C::U + (wave % C::NU) * 16 + r;
    const bool ok_u = u < H;
    const uint32_t DH = (uint32_t)(D * H), G4 = DH * 4;
    const buf_t gates = make_buf_(p.gates + w.li * p.sGi, (int64_t)Tn * B * G4 * 4);
    const buf_t cbuf = make_buf_(p.c + w.li * p.sCi + (int64_t)d * Tn * B * H, (int64_t)Tn * B * H * 4);
    const buf_t y = make_buf_((const T*)p.y + w.li * p.sYi, (int64_t)Tn * B * DH * sizeof(T));
    const buf_t xch = make_buf_(cd.exchange + (int64_t)w.cluster * 2 * C::FWD_SLOT, 2 * C::FWD_SLOT * 8);

    constexpr int NW = PARTS ? C::PCW : C::CW;               // k-chunks of a wave
    uint4 wf[4][NW][PARTS ? 3 : 1];
    bool plain = false;                                    // W_h has values that the parts cannot hold
    {
        const buf_t wh = make_buf_((const T*)p.wh + w.li * p.sWi + d * p.sWd, (int64_t)4 * H * H * sizeof(T));
        float check = 0.f;
#pragma unroll
        for (int c = 0; c < NW; ++c)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if constexpr (PARTS) {
                    uint4 lo, hi;
                    fwd_row8_(wh, H, q, u, (kh * NW + c) * 32, g, lo, hi);
                    parts8_(lo, hi, wf[q][c], check);
                } else {
                    wf[q][c][0] = fwd_frag_<T, C>(wh, H, q, u, (kh * NW + c) * C::KC, g);
                }
            }
        if constexpr (PARTS) plain = __syncthreads_or(not_finite_(check));
        if constexpr (C::SETTLE_F) {
#pragma unroll
            for (int c = 0; c < NW; ++c)
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int k = 0; k < (PARTS ? 3 : 1); ++k) settle_(wf[q][c][k], (c * 4 + q) * (PARTS ? 3 : 1) + k);
        }
    }
    // rows this lane finishes: row0 + i, i < PR
    const int row0 = 4 * g + (KS == 2 ? 2 * kh : 0);
    uint32_t vg[PR], vc[PR], vy[PR / C::VW];
#pragma unroll
    for (int i = 0; i < PR; ++i) {
        const uint32_t row = w.b0 + row0 + i;
        const bool ok = ok_u && (int)row < B;
        vg[i] = ok ? (row * G4 + d * 4 * H + u) * 4u : kOutOfRange;
        vc[i] = ok ? (row * H + u) * 4u : kOutOfRange;
    }
    // 4 bytes of h: one value, or (bf16) the values of two units, the even lane of the pair for the first of two rows
#pragma unroll
    for (int i = 0; i < PR / C::VW; ++i) {
        const uint32_t row = w.b0 + row0 + i * C::VW + (C::VW == 2 ? (r & 1) : 0);
        vy[i] = ok_u && (int)row < B ? (row * DH + d * H + (u & ~(C::VW - 1))) * (uint32_t)sizeof(T) : kOutOfRange;
    }
    float pre[4][PR];
    auto load_pre = [&](int s) {
        const uint32_t m = (uint32_t)(d == 0 ? s : Tn - 1 - s) * B;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int i = 0; i < PR; ++i) pre[q][i] = buf_load_(gates, vg[i], (m * G4 + q * H) * 4u);
    };
    float cs[PR];
#pragma unroll
    for (int i = 0; i < PR; ++i) cs[i] = 0.f;
    load_pre(0);
    const uint32_t how = join_<C>(cd, w);
    if (__builtin_expect(how >= kAlone, 0)) {
        if (how == kAlone + (uint32_t)w.m) forward_alone_<T, S>(cd, w, lds, red);
        return;
    }
    auto frame = [&](int s, auto later) -> bool {
        const uint32_t m = (uint32_t)(d == 0 ? s : Tn - 1 - s) * B;
        f32x4_t acc[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if constexpr (KS == 1) acc[q] = f32x4_t{pre[q][0], pre[q][1], pre[q][2], pre[q][3]};
            else acc[q] = kh == 0 ? f32x4_t{pre[q][0], pre[q][1], 0.f, 0.f} : f32x4_t{0.f, 0.f, pre[q][0], pre[q][1]};
        }
        if constexpr (decltype(later)::value) {
            // h of the frame before, all units, into LDS: 32 threads to a row, words 2 (tid % 32) + 64 i and the next
            constexpr int N = C::RW / 64;
            char* const hl = lds + (s & 1) * C::FWD_BUF;
            const uint32_t slot = (uint32_t)(s & 1) * (uint32_t)(C::FWD_SLOT * 8);
            uint32_t v[4 * N];
            const bool ok = get_<2 * N>(cd, xch, (uint32_t)((tid >> 5) * C::RW + 2 * (tid & 31)) * 8u,
                                        [&](int i) { return slot + (uint32_t)(i / N * 8 * C::RW + i % N * 64) * 8u; }, w.tag0 + s, v);
#pragma unroll
            for (int i = 0; i < 2 * N; ++i) {
                const int row = (tid >> 5) + i / N * 8;
                if (!PARTS || plain) {
                    *(uint2*)(hl + row * C::FWD_ROW + (tid & 31) * 8 + i % N * 256) = make_uint2(v[2 * i], v[2 * i + 1]);
                } else {
                    uint32_t h3[3];
                    float check = 0.f;                     // (h is finite, or NaN and so are its parts)
                    parts2_(__builtin_bit_cast(float, v[2 * i]), __builtin_bit_cast(float, v[2 * i + 1]), h3, check);
#pragma unroll
                    for (int k = 0; k < 3; ++k) *(uint32_t*)(hl + k * C::FWD_PART + row * C::FWD_PART_ROW + (tid & 31) * 4 + i % N * 128) = h3[k];
                }
            }
            if (!ok) expired = 1;
            load_pre(s + 1 < Tn ? s + 1 : s);              // (after the exchange: its loads return in order behind these)
            lds_barrier_();
            if (__builtin_amdgcn_readfirstlane(expired)) return false;
            if constexpr (PARTS) {
                if (__builtin_expect(plain, 0)) {
                    fwd_plain_<T, C>(acc, hl, make_buf_((const T*)p.wh + w.li * p.sWi + d * p.sWd, (int64_t)4 * H * H * sizeof(T)), H, u, kh, r, g);
                } else {
                    const char* hrow = hl + r * C::FWD_PART_ROW + kh * (NW * 64) + g * 16;
                    uint4 a[NW][3];
#pragma unroll
                    for (int c = 0; c < NW; ++c)
#pragma unroll
                        for (int k = 0; k < 3; ++k) a[c][k] = *(const uint4*)(hrow + c * 64 + k * C::FWD_PART);
                    if constexpr (C::SETTLE_F) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int c = 0; c < NW; ++c) mma_parts_<false, 4>(acc, a[c], [&](int q) -> const uint4 (&)[3] { return wf[q][c]; });
                }
            } else {
                const char* hrow = hl + r * C::FWD_ROW + kh * (NW * 64) + g * 16;
                uint4 a[NW];
#pragma unroll
                for (int c = 0; c < NW; ++c) a[c] = *(const uint4*)(hrow + c * 64);
                if constexpr (C::SETTLE_F) __builtin_amdgcn_sched_barrier(0);      // (all reads ahead of the products)
#pragma unroll
                for (int c = 0; c < NW; ++c)
#pragma unroll
                    for (int q = 0; q < 4; ++q) mma16_<T>(acc[q], a[c], wf[q][c][0]);
            }
            if constexpr (KS == 2) swap_halves_<C>(acc, red, kh, wave, lane);
        } else {
            if constexpr (KS == 2) {
#pragma unroll
                for (int q = 0; q < 4; ++q) { acc[q][0] = pre[q][0]; acc[q][1] = pre[q][1]; }
            }
            load_pre(Tn > 1 ? 1 : 0);
        }
        float h[PR];
#pragma unroll
        for (int i = 0; i < PR; ++i) h[i] = fwd_cell_(acc, i, cs[i]);              // (the gates replace the pre-activations)
        // h first: the other workgroups wait for it (rows past the batch and units past H too: they are read, as zeros or unused)
        const uint32_t out = (uint32_t)((s + 1) & 1) * (uint32_t)(C::FWD_SLOT * 8);
        const uint32_t out_lane = (uint32_t)((row0 + (C::VW == 2 ? r & 1 : 0)) * C::RW + u / C::VW) * 8u;
        uint32_t hw[PR / C::VW];
#pragma unroll
        for (int i = 0; i < PR / C::VW; ++i) hw[i] = h_word_<T>(h, i, r);
        if (s + 1 < Tn) {
            if (how == kOneXcd) {
#pragma unroll
                for (int i = 0; i < PR / C::VW; ++i) put_<kToL2>(xch, out_lane, out + (uint32_t)(i * C::VW * C::RW) * 8u, hw[i], w.tag0 + s + 1);
            } else {
#pragma unroll
                for (int i = 0; i < PR / C::VW; ++i) put_<kToMemory>(xch, out_lane, out + (uint32_t)(i * C::VW * C::RW) * 8u, hw[i], w.tag0 + s + 1);
            }
        }
#pragma unroll
        for (int i = 0; i < PR / C::VW; ++i) buf_store_(__builtin_bit_cast(float, hw[i]), y, vy[i], m * DH * (uint32_t)sizeof(T));
#pragma unroll
        for (int i = 0; i < PR; ++i) {
#pragma unroll
            for (int q = 0; q < 4; ++q) buf_store_(acc[q][i], gates, vg[i], (m * G4 + q * H) * 4u);
            buf_store_(cs[i], cbuf, vc[i], m * H * 4u);
        }
        return true;
    };
    frame(0, std::false_type{});                           // (outside the loop, so that the loop is entered with its stores in flight)
#pragma unroll 1
    for (int s = 1; s < Tn; ++s)
        if (!frame(s, std::true_type{})) return;
}

// ---- backward -----------------------------------------------------------------------------------
//   dh_t = dY_t + da_{t''} W_h  (t'' = the frame handled before)
//   do = dh tanh(c_t)            dc = dc_rec + dh o (1 - tanh^2 c_t)
//   di = dc g, dg = dc i, df = dc c_{t'}, dc_rec <- dc f
//   da = (di i(1-i), df f(1-f), dg (1-g^2), do o(1-o))
// A thread finishes PR consecutive units of one row, in accesses of 16 bytes (8 of the operand type): W_h is the first operand of the products, so that a
// lane's four results are consecutive units of a row too, and partial sums lie [16 units][16 rows][unit], whole lines to a wave's store (rows of 64 units,
// half lines of 16 rows to a store: 48 cycles a store instead of 15).  With four rows of one unit to a thread a frame's inputs and da are 40 accesses of 2 and
// 4 bytes instead of 10 (us of a pass, before / after: bf16 16 x 2 x 512, batch 64 308 / 299, 32 x 2 x 256, 64 246 / 235, 8 x 2 x 640, 96 399 / 405; fp32 16 x 2 x 256, 32
// 76 / 72).  It adds
// the partial sums of its positions in the order of the members.  The sums of da over the frames (bias gradients) stay in registers: one row per row
// block.
template <typename T, int S>
__global__ __launch_bounds__(256, 1) void rec_backward_cluster_kernel(ClusterDesc cd) {
    typedef Cl<T, S> C;
    constexpr int U = C::U, PR = C::PR;
    typedef typename Vec<PR>::type V;
    constexpr bool PARTS = C::PARTS;
    constexpr int OP_BYTES = 2 * C::BWD_BUF, W_BYTES = 2 * 16 * C::W_ROW * 4;
    __shared__ __attribute__((aligned(16))) char lds[OP_BYTES > W_BYTES ? OP_BYTES : W_BYTES];
    __shared__ __attribute__((aligned(16))) float bred[4][C::RB * U];
    __shared__ int expired, not_finite[2];                 // not_finite: by the parity of the frame, and never cleared
    const RecDesc& p = cd.r;
    Place w;
    if (!place_<C>(cd, w)) return;
    if (threadIdx.x == 0) { expired = 0; not_finite[0] = not_finite[1] = 0; }
    __syncthreads();
    const int D = p.D, H = p.H, B = p.B, Tn = p.T, d = w.d;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), r = lane & 15, g = lane >> 4;
    const uint32_t DH = (uint32_t)(D * H), G4 = DH * 4;
    const buf_t gates = make_buf_(p.gates + w.li * p.sGi, (int64_t)Tn * B * G4 * 4);
    const buf_t cbuf = make_buf_(p.c + w.li * p.sCi + (int64_t)d * Tn * B * H, (int64_t)Tn * B * H * 4);
    const buf_t dy = make_buf_(p.dy + w.li * p.sDYi, (int64_t)Tn * B * DH * 4);
    const buf_t da = make_buf_((const T*)p.da + w.li * p.sDAi, (int64_t)Tn * B * G4 * sizeof(T));
    const buf_t xch = make_buf_(cd.exchange + (int64_t)w.cluster * 2 * C::BWD_SLOT, 2 * C::BWD_SLOT * 8);
    const buf_t raw = make_buf_(cd.raw + (int64_t)w.cluster * 2 * C::RAW_SLOT, 2 * C::RAW_SLOT * 4);

    // cell part: this thread's row and units
    const int crow = tid / 16, uu = tid % 16 * PR, cu = w.m * U + uu;
    const uint32_t row = w.b0 + crow;
    const bool ok_c = cu < H && (int)row < B;              // (H: a multiple of 4)
    const uint32_t vg = ok_c ? (row * G4 + d * 4 * H + cu) * 4u : kOutOfRange, vc = ok_c ? (row * H + cu) * 4u : kOutOfRange;
    const uint32_t vy = ok_c ? (row * DH + d * H + cu) * 4u : kOutOfRange;
    const uint32_t at_values = (uint32_t)(uu / 16 * 256 + crow * 16 + uu % 16);      // of 16 rows of U partial sums
    const uint32_t at_words = PR == 2 ? at_values : (uint32_t)(uu / 16 * 256 + (crow & ~1) * 16 + uu % 16 + 2 * (crow & 1));   // (rows_in_)
    struct In { V dy, g[4], c; };                          // what a frame reads: dY, the gates, the cell state of the frame handled after it
    auto load_in = [&](int s, In& in) {
        const uint32_t m = (uint32_t)(d == 0 ? Tn - 1 - s : s) * B;                    // reverse of the forward order
        in.dy = Vec<PR>::template load<kPassing>(dy, vy, m * DH * 4u);
#pragma unroll
        for (int q = 0; q < 4; ++q) in.g[q] = Vec<PR>::template load<kPassing>(gates, vg, (m * G4 + q * H) * 4u);
        const bool end = s + 1 >= Tn;                      // the cell state before the first frame is 0
        const uint32_t mc = (uint32_t)(d == 0 ? Tn - 1 - (end ? Tn - 1 : s + 1) : (end ? Tn - 1 : s + 1)) * B;
        in.c = Vec<PR>::template load<kPassing>(cbuf, end ? kOutOfRange : vc, mc * H * 4u);
    };
    V c = Vec<PR>::template load<kPassing>(cbuf, vc, (uint32_t)(d == 0 ? Tn - 1 : 0) * B * H * 4u);
    In in;
    load_in(0, in);

    // product part: columns n of W_h (tiles wave, wave + 4, ...), rows: the four gates of this workgroup's units
    // Rows of W_h come in as they lie, a k-chunk (16 words of a column's fragments deep) at a time, two chunks ahead, and the
    // fragments are read from LDS: column by column from memory they took 384 two-byte loads a lane (bf16 x 360: 60 us).
    constexpr int NW = PARTS ? C::PBCH : C::BCH;
    uint4 wf[C::NT][NW][PARTS ? 3 : 1];
    bool plain = false;                                    // W_h has values that the parts cannot hold
    {
        uint4 half[PARTS ? C::NT : 1];                       // fp32: rows 4 g .. of a chunk of 32 k, rows 16 + 4 g .. come with the next 16
        float check = 0.f;
        constexpr int EPW = 4 / (int)sizeof(T);            // rows of W_h to a word
        const buf_t wh = make_buf_((const T*)p.wh + w.li * p.sWi + d * p.sWd, (int64_t)4 * H * H * sizeof(T));
        uint4 st[3][C::NT];                                // words tid + 256 j of the chunk's 16 x KP / 4 quadruples
        auto load = [&](int c, uint4 (&v)[C::NT]) {
            const int q = c * C::KC / U, unit0 = w.m * U + c * C::KC % U;              // a chunk lies in one gate
#pragma unroll
            for (int j = 0; j < C::NT; ++j) {
                const int x = tid + 256 * j, k = unit0 + x / (C::KP / 4) * EPW, n = x % (C::KP / 4) * 4;
                const uint32_t at = k < H && n < H ? (uint32_t)((q * H + k) * H + n) * (uint32_t)sizeof(T) : kOutOfRange;   // (H: a multiple of 4)
                if constexpr (EPW == 1) {
                    v[j] = buf_load16_(wh, at, 0u);
                } else {
                    const uint2 lo = buf_load8_(wh, at, 0u), hi = buf_load8_(wh, at, (uint32_t)H * 2u);
                    v[j] = make_uint4(__builtin_amdgcn_perm(hi.x, lo.x, 0x05040100u), __builtin_amdgcn_perm(hi.x, lo.x, 0x07060302u),
                                      __builtin_amdgcn_perm(hi.y, lo.y, 0x05040100u), __builtin_amdgcn_perm(hi.y, lo.y, 0x07060302u));
                }
            }
        };
        load(0, st[0]);
        load(1, st[1]);
#pragma unroll
        for (int c = 0; c < C::BCH; ++c) {
            uint32_t* const buf = (uint32_t*)lds + (c & 1) * (16 * C::W_ROW);
            if (c + 2 < C::BCH) load(c + 2, st[(c + 2) % 3]);
#pragma unroll
            for (int j = 0; j < C::NT; ++j) {
                const int x = tid + 256 * j;
                *(uint4*)(buf + x / (C::KP / 4) * C::W_ROW + x % (C::KP / 4) * 4) = st[c % 3][j];
            }
            lds_barrier_();
            const uint32_t* col = buf + 4 * g * C::W_ROW + wave * 16 + r;
#pragma unroll
            for (int j = 0; j < C::NT; ++j) {
                const uint4 x = make_uint4(col[64 * j], col[64 * j + C::W_ROW], col[64 * j + 2 * C::W_ROW], col[64 * j + 3 * C::W_ROW]);
                if constexpr (!PARTS) wf[j][c][0] = x;
                else if (c % 2 == 0) half[j] = x;
                else parts8_(half[j], x, wf[j][c / 2], check);
            }
        }
        if constexpr (PARTS) plain = __syncthreads_or(not_finite_(check));
        lds_barrier_();                                    // the operand of the products goes into the same LDS
        if constexpr (C::SETTLE_B) {
#pragma unroll
            for (int j = 0; j < C::NT; ++j)
#pragma unroll
                for (int c = 0; c < NW; ++c)
#pragma unroll
                    for (int k = 0; k < (PARTS ? 3 : 1); ++k) settle_(wf[j][c][k], (j * NW + c) * (PARTS ? 3 : 1) + k);
        }
    }
    const uint32_t how = join_<C>(cd, w);
    if (__builtin_expect(how >= kAlone, 0)) {
        if (how == kAlone + (uint32_t)w.m) backward_alone_<T, S>(cd, w, lds, bred);
        return;
    }
    float dcr[PR];
    V bs[4];
#pragma unroll
    for (int i = 0; i < PR; ++i) {
        dcr[i] = 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q) bs[q][i] = 0.f;
    }

    // The two ways of the exchange, the first frame and the last each have their own code: where branches meet the compiler waits for all that may be
    // outstanding on either, here inputs of the next frame on their way from memory and the flags just stored (us of a pass of 21 frames, one code for
    // all / this: bf16 16 x 2 x 512, batch 64 306 / 284, 10 x 2 x 360, 50 130 / 119, 32 x 2 x 256, 64 240 / 220, 8 x 2 x 640, 96 417 / 396; fp32 16 x 2 x 256, 32 73 / 69, 16 x 2 x
    // 512, 16 305 / 278).  At 640 cells in bf16 one fragment of W_h is in scratch.  Where it is loaded again behind a frame's barrier, the wait for it is one for the next
    // frame's inputs: through memory still; on one XCD no more (8 x 2 x 640, 96 382 / 327).  Inputs requested earlier, with the partial sums, delay those: 366, 156, 268.
    auto frame = [&](int s, auto one_xcd_, auto first_, auto last_) {
        constexpr bool one_xcd = decltype(one_xcd_)::value, first = decltype(first_)::value, last = decltype(last_)::value;
        const uint32_t m = (uint32_t)(d == 0 ? Tn - 1 - s : s) * B;
        float dh[PR];
#pragma unroll
        for (int i = 0; i < PR; ++i) dh[i] = 0.f;
        In next;
        if constexpr (!first) {
            bool ok = true;
            if constexpr (one_xcd) {                          // values [member][16 units][row][unit]
                const uint32_t slot = (uint32_t)(s & 1) * (uint32_t)(C::RAW_SLOT * 4);
                ok = wait_flags_(cd, raw, slot + (uint32_t)(C::RAW_VALUES + w.m * 4 * S) * 4u, 4 * S, lane, w.tag0 + s);
                asm volatile("" ::: "memory");             // (the values are loaded after the flags)
                V v[S];
#pragma unroll
                for (int j = 0; j < S; ++j) v[j] = Vec<PR>::template load<kFromL2>(raw, at_values * 4u, slot + (uint32_t)((w.m * S + j) * C::RB * U) * 4u);
#pragma unroll
                for (int j = 0; j < S; ++j)
#pragma unroll
                    for (int i = 0; i < PR; ++i) dh[i] += v[j][i];
            } else {
                // partial sums for this workgroup's units: words [member][16 units][row][unit], loaded as rows_in_ says
                const uint32_t slot = (uint32_t)((s & 1) * C::BWD_SLOT + (int64_t)w.m * S * C::RB * U) * 8u;
                constexpr int PB = PR * S <= 32 ? PR : 2;            // units gathered together
                static_assert(PR % PB == 0, "gather blocks");
#pragma unroll
                for (int i0 = 0; i0 < PR; i0 += PB) {
                    uint32_t v[PB * S];
                    ok &= get_<PB * S / 2>(cd, xch, at_words * 8u, [&](int j) { return slot + (uint32_t)((j % S) * C::RB * U) * 8u + (uint32_t)(i0 / 2 + j / S) * 128u; }, w.tag0 + s, v);
#pragma unroll
                    for (int i = 0; i < PB; ++i)
#pragma unroll
                        for (int j = 0; j < S; ++j) dh[i0 + i] += __builtin_bit_cast(float, v[2 * (i / 2 * S + j) + i % 2]);
                }
                if constexpr (PR == 4) { rows_in_(dh[0], dh[2]); rows_in_(dh[1], dh[3]); }
            }
            if (!ok) expired = 1;
        }
        char* const al = lds + (s & 1) * C::BWD_BUF;
        V a4[4];
        u32x2_t op[4];
        float check = 0.f;
#pragma unroll
        for (int i = 0; i < PR; ++i) bwd_cell_(a4, i, in.dy[i] + dh[i], dcr[i], in.g, c[i], in.c[i]);
        c = in.c;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            op[q] = operand8_(a4[q]);
#pragma unroll
            for (int i = 0; i < PR; ++i) bs[q][i] += a4[q][i];
            if constexpr (PARTS) {                           // 32 k of a gate: in the order in which the fragments of W_h hold them
                uint32_t a3[3];
                parts2_(a4[q][0], a4[q][1], a3, check);
#pragma unroll
                for (int k = 0; k < 3; ++k) *(uint32_t*)(al + k * C::BWD_PART + crow * C::BWD_PART_ROW + (8 * (uu % 16 / 4) + 4 * (uu / 16) + uu % 4 + q * U) * 2) = a3[k];
            } else {
                *(u32x2_t*)(al + crow * C::BWD_ROW + (uu + q * U) * (int)sizeof(T)) = op[q];
            }
        }
        // (Once set it holds for all later frames of the parity.  One word for each wave, written in every frame, or three words in turn cost about 1 us
        // of a pass of 20 frames at 256 cells.)
        if (PARTS && (plain || not_finite_(check))) not_finite[s & 1] = 1;
        if constexpr (!last) {
            load_in(s + 1, next);
            lds_barrier_();
            end_if_(expired);
            f32x4_t acc[C::NT];
#pragma unroll
            for (int j = 0; j < C::NT; ++j) acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            if constexpr (PARTS) {
                if (__builtin_expect(__builtin_amdgcn_readfirstlane(not_finite[s & 1]), 0)) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) *(V*)(al + crow * C::BWD_ROW + (uu + q * U) * 4) = a4[q];
                    lds_barrier_();
                    bwd_plain_<T, C>(acc, al, make_buf_((const T*)p.wh + w.li * p.sWi + d * p.sWd, (int64_t)4 * H * H * sizeof(T)), H, w.m, wave, r, g);
                } else {
                    const char* arow = al + r * C::BWD_PART_ROW + g * 16;
                    uint4 a[NW][3];
                    auto read = [&](int c) {
#pragma unroll
                        for (int k = 0; k < 3; ++k) a[c][k] = *(const uint4*)(arow + c * 64 + k * C::BWD_PART);
                    };
                    read(0);                               // (one chunk ahead of the products: 6 x 320 cells, batch 64 73 -> 71 us a pass)
#pragma unroll
                    for (int c = 0; c < NW; ++c) {
                        if (c + 1 < NW) read(c + 1);
                        __builtin_amdgcn_sched_barrier(0);
                        mma_parts_<true, C::NT>(acc, a[c], [&](int j) -> const uint4 (&)[3] { return wf[j][c]; });
                    }
                }
            } else {
                const char* arow = al + r * C::BWD_ROW + g * 16;
                constexpr bool AHEAD = sizeof(T) == 2 || one_xcd;      // (rows_out_)
                constexpr int A = !AHEAD ? 0 : C::SETTLE_B ? NW : 3;    // chunks that the operand is read ahead
                uint4 a[NW];
#pragma unroll
                for (int c = 0; c < NW && c < A; ++c) a[c] = *(const uint4*)(arow + c * 64);
                if (AHEAD) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int c = 0; c < NW; ++c) {
                    if (c + A < NW) a[c + A] = *(const uint4*)(arow + (c + A) * 64);
#pragma unroll
                    for (int j = 0; j < C::NT; ++j) mma16_<T>(acc[j], wf[j][c][0], a[c]);
                    if (AHEAD && A < NW) __builtin_amdgcn_sched_barrier(0);
                }
            }
            // a tile's results: [row r][units 4 g ..] of 16 x 16 (it lies in one workgroup's units: U is a multiple of 16)
            if constexpr (one_xcd) {                       // they are in the L2 when the wait ends
                const uint32_t at = (uint32_t)(r * 16 + 4 * g);
                const uint32_t to_slot = (uint32_t)((s + 1) & 1) * (uint32_t)(C::RAW_SLOT * 4);
#pragma unroll
                for (int j = 0; j < C::NT; ++j) {
                    const int n0 = (wave + 4 * j) * 16;
                    Vec<4>::store<kToL2>(acc[j], raw, at * 4u, to_slot + (uint32_t)(((n0 / U) * S + w.m) * C::RB * U + n0 % U * 16) * 4u);
                }
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __builtin_amdgcn_raw_buffer_store_b32(w.tag0 + s + 1, raw, lane < S ? (lane * 4 * S + w.m * 4 + wave) * 4 : (int)kOutOfRange,
                                                      (int)(to_slot + (uint32_t)C::RAW_VALUES * 4u), kToL2);
            } else {
                const uint32_t out = (uint32_t)(((s + 1) & 1) * C::BWD_SLOT + (int64_t)w.m * C::RB * U) * 8u, at_row = (uint32_t)(r % 8 * 16 + 4 * g + r / 8 * 2);
#pragma unroll
                for (int j = 0; j < C::NT; ++j) {
                    const int n0 = (wave + 4 * j) * 16;
                    const uint32_t to = out + (uint32_t)((n0 / U) * S * C::RB * U + n0 % U * 16) * 8u;
                    float v[4] = {acc[j][0], acc[j][1], acc[j][2], acc[j][3]};
                    rows_out_(v[0], v[2]); rows_out_(v[1], v[3]);
                    put2_<kToMemory>(xch, at_row * 8u, to, v[0], v[1], w.tag0 + s + 1);
                    put2_<kToMemory>(xch, at_row * 8u + 8u * 128u, to, v[2], v[3], w.tag0 + s + 1);
                }
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) buf_store8_<kPassing>(op[q], da, vg == kOutOfRange ? kOutOfRange : vg / (4u / (uint32_t)sizeof(T)), (m * G4 + q * H) * (uint32_t)sizeof(T));
        if constexpr (!last) in = next;
    };
    auto pass = [&](auto one_xcd) {
        frame(0, one_xcd, std::true_type{}, std::false_type{});
#pragma unroll 1
        for (int s = 1; s + 1 < Tn; ++s) frame(s, one_xcd, std::false_type{}, std::false_type{});
        frame(Tn - 1, one_xcd, std::false_type{}, std::true_type{});
    };
    if (how == kOneXcd) pass(std::true_type{});
    else pass(std::false_type{});
    bias_sums_<C>(cd, w, bred, bs, w.m);
}

// ---- rule and launchers -----------------------------------------------------------------------------
namespace {

// Members of a cluster: enough to hold W_h, in the sizes that are built; U units each.
int cluster_members(const RecDesc& d) {
    const int U = d.precision ? 64 : 32, need = (d.H + U - 1) / U;
    if (d.precision) return need <= 4 ? 4 : need <= 6 ? 6 : need <= 8 ? 8 : need <= 10 ? 10 : 0;
    return need <= 8 ? 8 : need <= 10 ? 10 : need <= 12 ? 12 : need <= 16 ? 16 : 0;
}
int cluster_blocks(const RecDesc& d) { return (d.B + 15) / 16; }

// Clusters that run at once with their members on one XCD each, and anywhere (a workgroup takes a compute unit: a SIMD's register
// file per wave).  One XCD unless the compute units that are left of each then cost a round of the chip.
struct Rounds { bool spread; int64_t at_once; };
Rounds cluster_rounds(int64_t clusters, int S, int cu_count) {
    const int64_t spread = (int64_t)(cu_count / kXcds / S) * kXcds, anywhere = cu_count / S;
    const bool one_xcd = spread > 0 && (clusters + spread - 1) / spread <= (clusters + anywhere - 1) / anywhere;
    return {one_xcd, one_xcd ? spread : anywhere};
}

template <typename T, int S> void launch_cluster_t(ClusterDesc& p, bool backward, int cu_count, hipStream_t s) {
    const int64_t clusters = rec_cluster_count(p.r);
    p.spread = cluster_rounds(clusters, S, cu_count).spread;
    const unsigned grid = (unsigned)((p.spread ? round_up(clusters, kXcds) : clusters) * S);
    if (backward) hipLaunchKernelGGL((rec_backward_cluster_kernel<T, S>), dim3(grid), dim3(256), 0, s, p);
    else hipLaunchKernelGGL((rec_forward_cluster_kernel<T, S>), dim3(grid), dim3(256), 0, s, p);
}

}  // namespace

// Where the clusters run: estimates of a pass both ways decide.  A round of the chip begins with W_h and takes a frame's latencies (first,
// frame), more the fuller the chip (full: gate and exchange traffic).  us for a pass of 20 frames, frame by frame / clusters (workgroups):
//   fp32 forward  16 x 256 cells, batch 32 (256) 235 / 74; 32 x 256, 64 (1024) 505 / 271, 128 (2048) 548 / 533; 32 x 320, 128 (2560) 970 / 870;
//                 16 x 384, 64 (768) 644 / 406; 24 x 512, 64 (1536) 858 / 797, 32 x 512, 64 (2048) 905 / 1065
//   fp32 backward 16 x 256, 32 254 / 73; 32 x 256, 128 641 / 501; 32 x 384, 64 (1536) 793 / 1037; 24 x 512, 64 977 / 923
//   bf16 forward  10 x 360, 50 (240) 166 / 61; 32 x 256, 128 (1024) 276 / 172; 32 x 512, 64 (1024) 417 / 260, 128 (2048) 562 / 513; 16 x 640, 64 (640)
//                 340 / 226, 96 (960) 399 / 301; 32 x 640, 128 (2560) 820 / 841
//   bf16 backward 10 x 360, 50 230 / 64; 16 x 512, 64 (512) 364 / 157; 32 x 512, 64 453 / 297, 128 726 / 575; 16 x 640, 32 (320)
//                 402 / 169, 96 (960) 453 / 381; 32 x 640, 128 1017 / 1027
// and of 5 frames: bf16 forward 32 x 512, 64 94 / 107, backward 121 / 103; fp32 forward 32 x 512, 64 200 / 331.
// Of 388 such pairs the estimates picked the longer way by more than 3 us and 5 per cent for 5, and lost 0.2 ms in all; clusters throughout
// lose 2.8, frames throughout 34.  The bf16 rows were fitted again when backward partial sums went bare, the fp32 rows and the fp32 figures above
// were not (16 x 512, batch 32 backward 313 us by the estimate, 275 measured): some fp32 passes whose two ways are close still run frame by frame;
// nor were any when backward frames became 5 to 12 per cent shorter (16-byte accesses) and forward ones up to 10 (settle_).  More rows to a cluster (two and four tiles one after the other) shorten nothing: 32 x 512, 64: 16 -> 15 and 18.
namespace {

double frames_time(const RecDesc& d, bool backward) {
    const int64_t pairs = (int64_t)d.L * d.D, split_wgs = pairs * ((d.H + 31) / 32) * ((d.B + 31) / 32);
    const double H = d.H, mb = pairs * 4.0 * H * H * (d.precision ? 2e-6 : 4e-6);          // W_h of all pairs
    // a step: latency of its contraction, W_h from the caches, more for every further 32 rows, a launch at least; the first has no
    // product.  Where the rows of W_h are not aligned the register-staged kernels take two to three times as long.
    double step;
    if (d.precision) {
        step = std::max(((backward ? 4.0 + 0.014 * H : 4.5 + 0.0085 * H) + 0.12 * mb) * (1.0 + 0.25 * ((d.B + 31) / 32 - 1)), 6.0);
    } else if (split_wgs <= 512) {                         // one round or two of the split-contraction kernels
        step = std::max(1.5 + 0.035 * H + 0.14 * mb + (backward && mb > 60.0 ? 0.1 * (mb - 60.0) : 0.0), 7.5);
        if (split_wgs > 256) step *= d.B > 32 ? 1.8 : 1.25;
    } else {
        step = 1.5 + 0.075 * H + 0.05 * mb;
        if (d.B > 64) step *= std::max(1.0, (double)(pairs * ((d.H + 31) / 32) * ((d.B + 127) / 128)) / 200.0);
    }
    if (!rec_aligned(d)) step *= backward ? 2.7 : 1.8;
    // (backward, one row block: no launch of its own for the column sums of da)
    return 7.0 + (d.T - 1) * step + (backward && cluster_blocks(d) == 1 ? 4.0 : 0.0);
}

double cluster_time(const RecDesc& d, bool backward, int cu_count) {
    struct Fit { double first, frame, full; };
    // 4, 6, 8, 10 members (bf16), 8, 10, 12, 16 (fp32)
    static const Fit fit[2][2][4] = {{{{13.2, 3.05, 0.0}, {14.9, 3.6, 0.0}, {14.2, 4.54, 0.64}, {17.8, 6.34, 0.0}},
                                      {{13.8, 2.43, 0.36}, {15.2, 2.91, 0.46}, {12.0, 3.81, 2.71}, {17.4, 5.58, 1.74}}},
                                     {{{10.4, 1.93, 0.0}, {13.7, 2.08, 0.02}, {16.8, 2.44, 0.2}, {19.2, 2.8, 0.24}},
                                      {{11.7, 1.95, 0.39}, {13.9, 2.17, 0.26}, {18.0, 2.2, 0.86}, {20.4, 2.6, 1.44}}}};
    const int S = cluster_members(d), size = d.precision ? (S - 4) / 2 : S == 16 ? 3 : (S - 8) / 2;
    const Fit& f = fit[d.precision ? 1 : 0][backward ? 1 : 0][size];
    const int64_t clusters = rec_cluster_count(d), at_once = cluster_rounds(clusters, S, cu_count).at_once;
    auto round = [&](int64_t n) { return f.first + (d.T - 1) * (f.frame + f.full * std::min(1.0, (double)(n * S) / 256.0)); };
    return (double)(clusters / at_once) * round(at_once) + (clusters % at_once ? round(clusters % at_once) : 0.0);
}

}  // namespace

bool rec_cluster_supported(const RecDesc& d, bool backward, int cu_count) {
    if (!d.direct || d.T < 2 || d.H <= 128 || !rec_quad_aligned(d) || d.L < 1 || d.L > 128 || d.D < 1 || d.D > 2 || d.B < 1) return false;
    if ((int64_t)d.T * d.B * d.D * d.H * 16 >= (int64_t)kOutOfRange) return false;     // buffer offsets
    const int S = cluster_members(d);
    if (S == 0 || cu_count < 4 * S) return false;
    if (rec_cluster_count(d) * S > 4096) return false;     // measured up to 3200
    return cluster_time(d, backward, cu_count) <= frames_time(d, backward);
}

int64_t rec_cluster_count(const RecDesc& d) { return (int64_t)d.L * d.D * cluster_blocks(d); }
int rec_cluster_batch_tiles(const RecDesc& d) { return cluster_blocks(d); }

int64_t rec_cluster_exchange_words(const RecDesc& d, bool backward) {
    const int64_t S = cluster_members(d), KP = S * (d.precision ? 64 : 32), row = backward ? S * KP : d.precision ? KP / 2 : KP;
    return rec_cluster_count(d) * 2 * 16 * row;
}

int64_t rec_cluster_raw_words(const RecDesc& d) {
    const int64_t S = cluster_members(d);
    return rec_cluster_count(d) * 2 * (16 * S * S * (d.precision ? 64 : 32) + 4 * S * S);
}

hipError_t launch_rec_cluster(const ClusterDesc& desc, bool backward, int cu_count, hipStream_t s) {
    ClusterDesc p = desc;
    if (!rec_cluster_supported(p.r, backward, cu_count) || !p.exchange || (backward && !p.raw) || !p.join || !p.epoch || !p.status || (backward && !p.r.dc)) return hipErrorInvalidValue;
    const int S = cluster_members(p.r);
    if (p.r.precision) {
        switch (S) {
            case 4: launch_cluster_t<bf16_t, 4>(p, backward, cu_count, s); break;
            case 6: launch_cluster_t<bf16_t, 6>(p, backward, cu_count, s); break;
            case 8: launch_cluster_t<bf16_t, 8>(p, backward, cu_count, s); break;
            default: launch_cluster_t<bf16_t, 10>(p, backward, cu_count, s); break;
        }
    } else {
        switch (S) {
            case 8: launch_cluster_t<float, 8>(p, backward, cu_count, s); break;
            case 10: launch_cluster_t<float, 10>(p, backward, cu_count, s); break;
            case 12: launch_cluster_t<float, 12>(p, backward, cu_count, s); break;
            default: launch_cluster_t<float, 16>(p, backward, cu_count, s); break;
        }
    }
    return hipGetLastError();
}

}  // namespace adpsgd
