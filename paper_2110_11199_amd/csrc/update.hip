// Fused mixing + SGD update over the learners' flat fp32 vectors (Algorithm 1:
// model averaging followed by the local update; Eq. 2 in matrix form).
//
// One streaming pass: every element of every active learner is read once (model
// and gradient) and written once, 12 bytes per (active learner, element).
// Pairwise mixing handles both members of a matched pair in the same thread, so
// the update is safe in place.  Arithmetic order (each operation rounded once,
// no fused multiply-add):
//     pair: m = (x_i + x_j) * 0.5      all: m = (((x_0 + x_1) + ...) ) * (1/L)
//     ring neighbours: m = ((x_left + x_i) + x_right) * (1/3)
//     x_i <- m - (lr * g_i)
// Synchronous baseline (Section III-A, Algorithm 2), the same operations in the other order:
//     u_j = x_j - (lr * g_j);   x_i <- (((u_0 + u_1) + ...)) * (1/L) for every i
#include <mutex>
#include "kernels.hpp"

namespace adpsgd {

struct PairArgs {
    const float* src; float* dst; int64_t stride; int64_t P; float lr;
    bf16_t* shadow; int emit_input;   // bf16 copy of the next gradient point: the inputs (tau = 1) or the outputs
    int nwork;
    const float* g[128];
    int16_t a[128], b[128];     // work item w mixes learners a[w], b[w] (a == b: no partner)
};

__device__ inline float sgd_(float m, float lr, float g) { return __fsub_rn(m, __fmul_rn(lr, g)); }

__device__ inline float4 pair_new_(const float4& m, float lr, const float4& g) {
    return make_float4(sgd_(m.x, lr, g.x), sgd_(m.y, lr, g.y), sgd_(m.z, lr, g.z), sgd_(m.w, lr, g.w));
}
__device__ inline float4 half_sum_(const float4& p, const float4& q) {
    return make_float4(__fmul_rn(__fadd_rn(p.x, q.x), 0.5f), __fmul_rn(__fadd_rn(p.y, q.y), 0.5f),
                       __fmul_rn(__fadd_rn(p.z, q.z), 0.5f), __fmul_rn(__fadd_rn(p.w, q.w), 0.5f));
}

// float4 positions per thread and stream.  One is best: on the 64-learner random-ring workload 5.88 TB/s
// against 5.63 (2), 5.60 (4) and 5.47 (8): smaller workgroups spread more evenly over the CUs.
constexpr int kUnroll = 1;

// one element of one work item (scalar path and tails)
__device__ inline void pair_scalar_(const float* xa, const float* xb, const float* ga, const float* gb, float* oa, float* ob,
                                    bf16_t* sha, bf16_t* shb, bool solo, int emit_input, float lr, int64_t e) {
    const float x = xa[e], y = xb[e];
    if (solo) {
        const float r = sgd_(x, lr, ga[e]);
        oa[e] = r;
        if (sha) sha[e] = f32_to_bf16(emit_input ? x : r);
    } else {
        const float m = __fmul_rn(__fadd_rn(x, y), 0.5f);
        const float va = sgd_(m, lr, ga[e]), vb = sgd_(m, lr, gb[e]);
        oa[e] = va; ob[e] = vb;
        if (sha) { sha[e] = f32_to_bf16(emit_input ? x : va); shb[e] = f32_to_bf16(emit_input ? y : vb); }
    }
}

// The models and gradients are streamed once per iteration: non-temporal loads and stores keep them
// from displacing each other in L2 (measured +11% on the 2-reads-1-write pattern).
typedef float vf4_t __attribute__((ext_vector_type(4)));
__device__ inline float4 ldnt_(const float* p, int64_t e4) {
    const vf4_t v = __builtin_nontemporal_load((const vf4_t*)p + e4);
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ inline void emit4_(bf16_t* sh, int64_t e4, const float4& v) {
    uint2 o;
    o.x = pack_bf16(v.x, v.y);
    o.y = pack_bf16(v.z, v.w);
    ((uint2*)sh)[e4] = o;
}
__device__ inline void stnt_(float* p, int64_t e4, const float4& v) {
    vf4_t w; w.x = v.x; w.y = v.y; w.z = v.z; w.w = v.w;
    __builtin_nontemporal_store(w, (vf4_t*)p + e4);
}

template <bool VEC>
__global__ __launch_bounds__(256) void pair_update_kernel(PairArgs p) {
    const int w = blockIdx.y;
    const int a = p.a[w], b = p.b[w];
    const float* xa = p.src + a * p.stride;
    const float* xb = p.src + b * p.stride;
    float* oa = p.dst + a * p.stride;
    float* ob = p.dst + b * p.stride;
    const float* ga = p.g[a];
    const float* gb = p.g[b];
    const float lr = p.lr;
    bf16_t* sha = p.shadow ? p.shadow + a * p.stride : nullptr;
    bf16_t* shb = p.shadow ? p.shadow + b * p.stride : nullptr;
    if constexpr (VEC) {
        const int64_t n4 = p.P >> 2;
        const int64_t base = (int64_t)blockIdx.x * (blockDim.x * kUnroll) + threadIdx.x;
        if (a == b) {
            float4 x[kUnroll], g[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const int64_t e = base + u * blockDim.x;
                if (e < n4) { x[u] = ldnt_(xa, e); g[u] = ldnt_(ga, e); }
            }
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const int64_t e = base + u * blockDim.x;
                if (e < n4) {
                    const float4 r = pair_new_(x[u], lr, g[u]);
                    stnt_(oa, e, r);
                    if (sha) emit4_(sha, e, p.emit_input ? x[u] : r);
                }
            }
        } else {
            float4 x[kUnroll], y[kUnroll], g[kUnroll], h[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const int64_t e = base + u * blockDim.x;
                if (e < n4) {
                    x[u] = ldnt_(xa, e); y[u] = ldnt_(xb, e);
                    g[u] = ldnt_(ga, e); h[u] = ldnt_(gb, e);
                }
            }
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const int64_t e = base + u * blockDim.x;
                if (e < n4) {
                    const float4 m = half_sum_(x[u], y[u]);
                    const float4 ra = pair_new_(m, lr, g[u]), rb = pair_new_(m, lr, h[u]);
                    stnt_(oa, e, ra);
                    stnt_(ob, e, rb);
                    if (sha) { emit4_(sha, e, p.emit_input ? x[u] : ra); emit4_(shb, e, p.emit_input ? y[u] : rb); }
                }
            }
        }
        // tail (P % 4 elements), handled by the first block
        if (blockIdx.x == 0 && threadIdx.x < (p.P & 3)) {
            const int64_t e = (n4 << 2) + threadIdx.x;
            pair_scalar_(xa, xb, ga, gb, oa, ob, sha, shb, a == b, p.emit_input, lr, e);
        }
    } else {
        const int64_t base = (int64_t)blockIdx.x * (blockDim.x * kUnroll) + threadIdx.x;
#pragma unroll
        for (int u = 0; u < kUnroll; ++u) {
            const int64_t e = base + u * blockDim.x;
            if (e >= p.P) continue;
            pair_scalar_(xa, xb, ga, gb, oa, ob, sha, shb, a == b, p.emit_input, lr, e);
        }
    }
}

// The same pairwise update with ONE member of a pair per thread: a workgroup of NX positions x 2 members; a thread
// reads its member's model and gradient (two streams, 1 KB contiguous per wave and stream), hands the model to its
// partner thread through LDS, and writes its member's result after the workgroup's barrier, i.e. after both models
// of these positions have been read: safe in place like the two-member form, same operations (the pair sum is
// commutative), bit-identical results.  For a work item without a partner (a == b) the two halves of the workgroup
// take adjacent positions of the one learner (and the workgroups past its end have nothing to do).
template <int NX>
__global__ __launch_bounds__(2 * NX) void pair_split_update_kernel(PairArgs p) {
    __shared__ float4 other[2 * NX];
    const int w = blockIdx.y, member = threadIdx.y, tx = threadIdx.x;
    const int a = p.a[w], b = p.b[w];
    const bool solo = a == b;
    const int i = member ? b : a;
    const int64_t n4 = p.P >> 2;
    // a pair: both halves of the workgroup at the same NX positions; no partner: the halves at adjacent ones
    const int64_t e = solo ? (int64_t)blockIdx.x * (2 * NX) + member * NX + tx : (int64_t)blockIdx.x * NX + tx;
    const bool ok = e < n4;
    float4 x = make_float4(0.f, 0.f, 0.f, 0.f), g = x;
    if (ok) { x = ldnt_(p.src + i * p.stride, e); g = ldnt_(p.g[i], e); }
    other[member * NX + tx] = x;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (ok) {
        const float4 m = solo ? x : half_sum_(x, other[(1 - member) * NX + tx]);
        const float4 r = pair_new_(m, p.lr, g);
        stnt_(p.dst + i * p.stride, e, r);
        if (p.shadow) emit4_(p.shadow + i * p.stride, e, p.emit_input ? x : r);
    }
    // tail (P % 4 elements): one thread handles both members of an element
    if (blockIdx.x == 0 && member == 0 && tx < (p.P & 3))
        pair_scalar_(p.src + a * p.stride, p.src + b * p.stride, p.g[a], p.g[b], p.dst + a * p.stride, p.dst + b * p.stride,
                     p.shadow ? p.shadow + a * p.stride : nullptr, p.shadow ? p.shadow + b * p.stride : nullptr, solo,
                     p.emit_input, p.lr, (n4 << 2) + tx);
}

struct AllArgs {
    const float* src; float* dst; int64_t stride; int64_t P; float lr; float inv_L; int L;
    bf16_t* shadow; int emit_input;
    const float* g[128];
};

// synchronous baseline: one element of all learners
__device__ inline void sync_scalar_(const AllArgs& p, int64_t t) {
    float s = sgd_(p.src[t], p.lr, p.g[0][t]);
    for (int j = 1; j < p.L; ++j) s = __fadd_rn(s, sgd_(p.src[j * p.stride + t], p.lr, p.g[j][t]));
    const float m = __fmul_rn(s, p.inv_L);
    for (int i = 0; i < p.L; ++i) {
        p.dst[i * p.stride + t] = m;
        if (p.shadow) p.shadow[i * p.stride + t] = f32_to_bf16(m);
    }
}

// Synchronous baseline: one thread owns an element index of all learners, reads L models and L
// gradients, and writes the mean of the updated models to all L learners (12 bytes per learner and
// element, as the other updates).  The bf16 copy, if any, is of the output (tau = 0).
template <bool VEC>
__global__ __launch_bounds__(256) void sync_update_kernel(AllArgs p) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if constexpr (VEC) {
        const int64_t n4 = p.P >> 2;
        if (e < n4) {
            float4 s = pair_new_(ldnt_(p.src, e), p.lr, ldnt_(p.g[0], e));
#pragma unroll 8
            for (int j = 1; j < p.L; ++j) {
                const float4 u = pair_new_(ldnt_(p.src + j * p.stride, e), p.lr, ldnt_(p.g[j], e));
                s.x = __fadd_rn(s.x, u.x); s.y = __fadd_rn(s.y, u.y); s.z = __fadd_rn(s.z, u.z); s.w = __fadd_rn(s.w, u.w);
            }
            const float4 m = make_float4(__fmul_rn(s.x, p.inv_L), __fmul_rn(s.y, p.inv_L), __fmul_rn(s.z, p.inv_L), __fmul_rn(s.w, p.inv_L));
#pragma unroll 8
            for (int i = 0; i < p.L; ++i) {
                stnt_(p.dst + i * p.stride, e, m);
                if (p.shadow) emit4_(p.shadow + i * p.stride, e, m);
            }
        }
        if (blockIdx.x == 0 && threadIdx.x < (p.P & 3)) sync_scalar_(p, (n4 << 2) + threadIdx.x);
    } else {
        if (e < p.P) sync_scalar_(p, e);
    }
}

__device__ inline void all_scalar_(const AllArgs& p, int64_t t) {
    float s = p.src[t];
    if (p.shadow && p.emit_input) p.shadow[t] = f32_to_bf16(s);
    for (int j = 1; j < p.L; ++j) {
        const float v = p.src[j * p.stride + t];
        if (p.shadow && p.emit_input) p.shadow[j * p.stride + t] = f32_to_bf16(v);
        s = __fadd_rn(s, v);
    }
    const float m = __fmul_rn(s, p.inv_L);
    for (int i = 0; i < p.L; ++i) {
        const float r = sgd_(m, p.lr, p.g[i][t]);
        p.dst[i * p.stride + t] = r;
        if (p.shadow && !p.emit_input) p.shadow[i * p.stride + t] = f32_to_bf16(r);
    }
}

// The mean of all learners with the learners cut into segments of SEG: a workgroup of blockDim.x positions x blockDim.y segments;
// a thread reads the SEG models and gradients of its segment (2 SEG streams instead of 2 L), and the sum of the models (FIRST:
// of the updated models, the synchronous baseline) runs through the segments in learner order, one segment per barrier,
// through LDS: the same additions in the same order as the single walk, bit-identical results.  Every model of the workgroup's
// positions has been read before the first result is written (the writes follow the last barrier), so it stays safe in place.
// The P % 4 last elements take a thread each that walks all learners: in front of the first workgroup's segments (kWithin), or in a workgroup of its own, the
// first (kOwn), for small updates, to which the walk would add its whole length.
enum Tail { kNone, kWithin, kOwn };
template <int SEG, bool FIRST, Tail TAIL>
__global__ __launch_bounds__(1024) void mean_seg_update_kernel(AllArgs p) {
    __shared__ float4 chain[64];
    const int tx = threadIdx.x, sy = threadIdx.y, nx = blockDim.x, ns = blockDim.y;
    const int64_t e = ((int64_t)blockIdx.x - (TAIL == kOwn)) * nx + tx;
    const bool ok = (TAIL != kOwn || e >= 0) && e < (p.P >> 2);
    const int j0 = sy * SEG;
    if (TAIL != kNone && blockIdx.x == 0 && sy == 0 && tx < (p.P & 3)) {
        if constexpr (FIRST) sync_scalar_(p, ((p.P >> 2) << 2) + tx);
        else all_scalar_(p, ((p.P >> 2) << 2) + tx);
    }
    float4 u[SEG], g[SEG];
#pragma unroll
    for (int j = 0; j < SEG; ++j) {
        if (!ok || j0 + j >= p.L) continue;
        u[j] = ldnt_(p.src + (j0 + j) * p.stride, e);
        g[j] = ldnt_(p.g[j0 + j], e);
        if constexpr (FIRST) u[j] = pair_new_(u[j], p.lr, g[j]);
    }
    for (int step = 0; step < ns; ++step) {
        if (sy == step && ok) {
            float4 s = u[0];
            if (step > 0) { const float4 c = chain[tx]; s = make_float4(__fadd_rn(c.x, s.x), __fadd_rn(c.y, s.y), __fadd_rn(c.z, s.z), __fadd_rn(c.w, s.w)); }
#pragma unroll
            for (int j = 1; j < SEG; ++j)
                if (j0 + j < p.L) { s.x = __fadd_rn(s.x, u[j].x); s.y = __fadd_rn(s.y, u[j].y); s.z = __fadd_rn(s.z, u[j].z); s.w = __fadd_rn(s.w, u[j].w); }
            chain[tx] = s;
        }
        __syncthreads();
    }
    if (!ok) return;
    const float4 t = chain[tx];
    const float4 m = make_float4(__fmul_rn(t.x, p.inv_L), __fmul_rn(t.y, p.inv_L), __fmul_rn(t.z, p.inv_L), __fmul_rn(t.w, p.inv_L));
#pragma unroll
    for (int j = 0; j < SEG; ++j) {
        if (j0 + j >= p.L) break;
        const float4 r = FIRST ? m : pair_new_(m, p.lr, g[j]);
        stnt_(p.dst + (j0 + j) * p.stride, e, r);
        if (p.shadow) emit4_(p.shadow + (j0 + j) * p.stride, e, !FIRST && p.emit_input ? u[j] : r);
    }
}

template <int SEG, bool FIRST>
static void launch_mean_seg_t(const AllArgs& a, hipStream_t s) {
    const int ns = (a.L + SEG - 1) / SEG;
    int nx = 64;
    while (nx * ns > 512 && nx > 8) nx >>= 1;
    const int64_t n4 = a.P >> 2;
    const unsigned blocks = (unsigned)((n4 + nx - 1) / nx);
    // (us, within / own: 64 x 262141 59.3 / 40.5, 64 x 4200001 585 / 592)
    if (a.P % 4 == 0) hipLaunchKernelGGL((mean_seg_update_kernel<SEG, FIRST, kNone>), dim3(blocks), dim3((unsigned)nx, (unsigned)ns), 0, s, a);
    else if (a.P < (1 << 20)) hipLaunchKernelGGL((mean_seg_update_kernel<SEG, FIRST, kOwn>), dim3(blocks + 1), dim3((unsigned)nx, (unsigned)ns), 0, s, a);
    else hipLaunchKernelGGL((mean_seg_update_kernel<SEG, FIRST, kWithin>), dim3(blocks), dim3((unsigned)nx, (unsigned)ns), 0, s, a);
}
template <bool FIRST>
static void launch_mean_seg(const AllArgs& a, int seg, hipStream_t s) {
    if (seg >= 8) launch_mean_seg_t<8, FIRST>(a, s);
    else if (seg >= 4) launch_mean_seg_t<4, FIRST>(a, s);
    else launch_mean_seg_t<2, FIRST>(a, s);
}

// One thread owns an element index of all learners: reads L models, forms the
// mean once, reads L gradients, writes L models.
template <bool VEC>
__global__ __launch_bounds__(256) void all_update_kernel(AllArgs p) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if constexpr (VEC) {
        const int64_t n4 = p.P >> 2;
        if (e < n4) {
            float4 s = ldnt_(p.src, e);
            const bool emit_in = p.shadow && p.emit_input, emit_out = p.shadow && !p.emit_input;
            if (emit_in) emit4_(p.shadow, e, s);
#pragma unroll 8
            for (int j = 1; j < p.L; ++j) {
                const float4 v = ldnt_(p.src + j * p.stride, e);
                if (emit_in) emit4_(p.shadow + j * p.stride, e, v);
                s.x = __fadd_rn(s.x, v.x); s.y = __fadd_rn(s.y, v.y); s.z = __fadd_rn(s.z, v.z); s.w = __fadd_rn(s.w, v.w);
            }
            const float4 m = make_float4(__fmul_rn(s.x, p.inv_L), __fmul_rn(s.y, p.inv_L), __fmul_rn(s.z, p.inv_L), __fmul_rn(s.w, p.inv_L));
#pragma unroll 8
            for (int i = 0; i < p.L; ++i) {
                const float4 g = ldnt_(p.g[i], e);
                const float4 r = pair_new_(m, p.lr, g);
                stnt_(p.dst + i * p.stride, e, r);
                if (emit_out) emit4_(p.shadow + i * p.stride, e, r);
            }
        }
        if (blockIdx.x == 0 && threadIdx.x < (p.P & 3)) {
            const int64_t t = (n4 << 2) + threadIdx.x;
            all_scalar_(p, t);
        }
    } else {
        if (e < p.P) all_scalar_(p, e);
    }
}

// ---- global mean in two kernels per chunk of the parameter index --------------------------------------
// The rate of a streaming kernel on this device falls with the number of streams one thread walks at once (measured
// with the stream probe: 6.5 TB/s with 3 streams per thread, 5.3 with 64).  The single-kernel global mean owns
// 4 streams per learner and thread.  Split: `all_mean_kernel` reads the L models of a chunk of the index and
// writes their mean to a small buffer (and the bf16 copies of the models read, when asked for); `all_apply_kernel`
// then runs once per learner (grid y) with three streams per thread: the mean (from the buffer, which a chunk
// at a time stays in the caches), the learner's gradient, the learner's new model.  Same operations in the same
// order per element as all_update_kernel, so the results are bit-identical.
struct AllSplitArgs {
    AllArgs a;
    float* mean;            // [chunk] fp32
    int64_t e0, n4c;        // chunk start and length in float4 positions
    int tail;               // last chunk: the P % 4 last elements too
};

__global__ __launch_bounds__(256) void all_mean_kernel(AllSplitArgs q) {
    const AllArgs& p = q.a;
    // the P % 4 last elements of every learner, whole, on a workgroup beside the others (a launch of their own took 15 us)
    if (blockIdx.x == 0 && q.tail && threadIdx.x < (p.P & 3)) all_scalar_(p, ((p.P >> 2) << 2) + threadIdx.x);
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= q.n4c) return;
    const int64_t e = q.e0 + c;
    float4 s = ldnt_(p.src, e);
    const bool emit_in = p.shadow && p.emit_input;
    if (emit_in) emit4_(p.shadow, e, s);
#pragma unroll 8
    for (int j = 1; j < p.L; ++j) {
        const float4 v = ldnt_(p.src + j * p.stride, e);
        if (emit_in) emit4_(p.shadow + j * p.stride, e, v);
        s.x = __fadd_rn(s.x, v.x); s.y = __fadd_rn(s.y, v.y); s.z = __fadd_rn(s.z, v.z); s.w = __fadd_rn(s.w, v.w);
    }
    ((float4*)q.mean)[c] = make_float4(__fmul_rn(s.x, p.inv_L), __fmul_rn(s.y, p.inv_L), __fmul_rn(s.z, p.inv_L), __fmul_rn(s.w, p.inv_L));
}

__global__ __launch_bounds__(256) void all_apply_kernel(AllSplitArgs q) {
    const AllArgs& p = q.a;
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= q.n4c) return;
    const int64_t e = q.e0 + c;
    const int i = blockIdx.y;
    const float4 m = ((const float4*)q.mean)[c];
    const float4 r = pair_new_(m, p.lr, ldnt_(p.g[i], e));
    stnt_(p.dst + i * p.stride, e, r);
    if (p.shadow && !p.emit_input) emit4_(p.shadow + i * p.stride, e, r);
}

// ---- ring-neighbour mixing with weights 1/3 (the circulant operator T^f of Eq. 9, and T^r = P' T^f P) -------
// One thread owns an element index of all learners and walks the ring order with the previous, current and
// next model value in registers: every model is read once (the last one of the order twice), so the update
// is safe in place and moves the same 12 bytes per learner and element as the pairwise one.
struct TriArgs {
    const float* src; float* dst; int64_t stride; int64_t P; float lr; float third; int L;
    bf16_t* shadow; int emit_input;
    const float* g[128];        // gradients in ring order
    int32_t order[128];         // learners in ring order (whole words: a scalar load each)
    int16_t order16[128];       // the same in 16 bits (vector loads)
};

__device__ inline float tri_mean_(float l, float c, float r, float third) { return __fmul_rn(__fadd_rn(__fadd_rn(l, c), r), third); }

__device__ inline void tri_scalar_(const TriArgs& p, int64_t t) {
    const float first = p.src[p.order[0] * p.stride + t];
    float prev = p.src[p.order[p.L - 1] * p.stride + t], cur = first;
    for (int q = 0; q < p.L; ++q) {
        const int i = p.order[q];
        const float next = q + 1 < p.L ? p.src[p.order[q + 1] * p.stride + t] : first;
        const float r = sgd_(tri_mean_(prev, cur, next, p.third), p.lr, p.g[q][t]);
        p.dst[i * p.stride + t] = r;
        if (p.shadow) p.shadow[i * p.stride + t] = f32_to_bf16(p.emit_input ? cur : r);
        prev = cur; cur = next;
    }
}

// BLOCK: ring positions whose loads go out together (no load passes a store, since the result may replace a model, so that a walk
// position by position waits once for each).  The walk one by one reads the order from 16-bit entries, by vector loads, which
// keep its waves from running apart: with scalar loads 16 x 3.5M takes 122 us instead of 112, 64 x 1.5M 213 instead of 192.
template <bool VEC, int BLOCK>
__global__ __launch_bounds__(256) void tri_update_kernel(TriArgs p) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if constexpr (VEC) {
        const int64_t n4 = p.P >> 2;
        if (e < n4) {
            const float4 first = ldnt_(p.src + p.order[0] * p.stride, e);
            float4 prev = ldnt_(p.src + p.order[p.L - 1] * p.stride, e), cur = first;
            for (int q0 = 0; q0 < p.L; q0 += BLOCK) {
                float4 next[BLOCK], g[BLOCK];
#pragma unroll
                for (int j = 0; j < BLOCK; ++j) {
                    if (q0 + j >= p.L) break;
                    g[j] = ldnt_(p.g[q0 + j], e);
                    next[j] = first;
                    if (q0 + j + 1 < p.L) next[j] = ldnt_(p.src + (BLOCK == 1 ? (int)p.order16[q0 + j + 1] : p.order[q0 + j + 1]) * p.stride, e);
                }
#pragma unroll
                for (int j = 0; j < BLOCK; ++j) {
                    if (q0 + j >= p.L) break;
                    const int i = BLOCK == 1 ? (int)p.order16[q0 + j] : p.order[q0 + j];
                    const float4 m = make_float4(tri_mean_(prev.x, cur.x, next[j].x, p.third), tri_mean_(prev.y, cur.y, next[j].y, p.third),
                                                 tri_mean_(prev.z, cur.z, next[j].z, p.third), tri_mean_(prev.w, cur.w, next[j].w, p.third));
                    const float4 r = pair_new_(m, p.lr, g[j]);
                    stnt_(p.dst + i * p.stride, e, r);
                    if (p.shadow) emit4_(p.shadow + i * p.stride, e, p.emit_input ? cur : r);
                    prev = cur; cur = next[j];
                }
            }
        }
        if (blockIdx.x == 0 && threadIdx.x < (p.P & 3)) tri_scalar_(p, (n4 << 2) + threadIdx.x);
    } else {
        if (e < p.P) tri_scalar_(p, e);
    }
}

// The same operator with the ring cut into segments of SEG positions.  A workgroup of blockDim.x element positions
// x blockDim.y segments covers all L learners of its element positions; a thread owns one segment at one position:
// it reads its SEG models and gradients (2 SEG streams instead of 2 L: the rate of a streaming kernel on this
// device falls with the number of streams a thread walks at once), hands the first and last model of its segment to
// the neighbouring segments through LDS, and writes its SEG results after the workgroup's barrier, i.e. after every
// model of these positions has been read: safe in place like the single walk, the same 12 bytes per learner and
// element (no model is read twice), the same operations per element, bit-identical results.
template <int SEG>
__global__ __launch_bounds__(1024) void tri_seg_update_kernel(TriArgs p) {
    __shared__ float4 edge[2 * 1024];                            // [first | last][segment][position]
    const int tx = threadIdx.x, sy = threadIdx.y, nx = blockDim.x, ns = blockDim.y;
    const int64_t e = (int64_t)blockIdx.x * nx + tx;
    const bool ok = e < (p.P >> 2);
    const int q0 = sy * SEG;
    // the P % 4 last elements of every learner: one thread each walks the whole ring
    if (blockIdx.x == 0 && sy == 0 && tx < (p.P & 3)) tri_scalar_(p, ((p.P >> 2) << 2) + tx);
    float4 x[SEG], g[SEG];
    float4 lastv = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int j = 0; j < SEG; ++j) {
        if (ok && q0 + j < p.L) {
            const int i = p.order[q0 + j];
            x[j] = ldnt_(p.src + i * p.stride, e);
            g[j] = ldnt_(p.g[q0 + j], e);
            lastv = x[j];
        }
    }
    if (ok) { edge[sy * nx + tx] = x[0]; edge[(ns + sy) * nx + tx] = lastv; }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");             // every model of this thread is in registers ...
    __syncthreads();                                             // ... and so is every other thread's: writing may begin
    if (!ok) return;
    float4 prev = edge[(ns + (sy + ns - 1) % ns) * nx + tx];
    const float4 after = edge[((sy + 1) % ns) * nx + tx];
#pragma unroll
    for (int j = 0; j < SEG; ++j) {
        if (q0 + j >= p.L) break;
        const int i = p.order[q0 + j];
        float4 next = after;
        if (j + 1 < SEG && q0 + j + 1 < p.L) next = x[j + 1 < SEG ? j + 1 : j];
        const float4 m = make_float4(tri_mean_(prev.x, x[j].x, next.x, p.third), tri_mean_(prev.y, x[j].y, next.y, p.third),
                                     tri_mean_(prev.z, x[j].z, next.z, p.third), tri_mean_(prev.w, x[j].w, next.w, p.third));
        const float4 r = pair_new_(m, p.lr, g[j]);
        stnt_(p.dst + i * p.stride, e, r);
        if (p.shadow) emit4_(p.shadow + i * p.stride, e, p.emit_input ? x[j] : r);
        prev = x[j];
    }
}

template <int SEG>
static void launch_tri_seg(const TriArgs& a, hipStream_t s) {
    const int ns = (a.L + SEG - 1) / SEG;                        // at most 128 segments (L <= 128)
    int nx = 64;
    while (nx * ns > 512 && nx > 8) nx >>= 1;
    const int64_t n4 = a.P >> 2;
    hipLaunchKernelGGL(tri_seg_update_kernel<SEG>, dim3((unsigned)((n4 + nx - 1) / nx)), dim3((unsigned)nx, (unsigned)ns), 0, s, a);
}

// ---- hybrid mixing (Section V: synchronous super-learners joined by the asynchronous ring) -----------
// Consecutive blocks of S learners form super-learners.  The mean of every super-learner first,
//     m_a = (((x_{aS} + x_{aS+1}) + ...) + x_{aS+S-1}) * (1/S),
// then the ring operator on the means (pair: (m_a + m_b) * 0.5; neighbours: ((m_left + m_a) + m_right) * (1/3)),
// then x_i <- m - (lr * g_i) for every learner i of super-learner a.  One thread owns an element index (a float4,
// or one float on the unaligned path and the tail) of all the learners it touches and reads every model once
// before it writes any of them, so the update is safe in place at 12 bytes per learner and element.
struct HybridArgs {
    const float* src; float* dst; int64_t stride; int64_t P; float lr;
    bf16_t* shadow; int emit_input;
    int S, G; float inv_S, third;
    const float* g[128];
    int16_t order[128];            // neighbours: ring order of the super-learners
    int16_t a[64], b[64];          // pair: work item w mixes super-learners a[w], b[w] (a == b: unmatched)
};

// the same code for a float4 position and for a single float
struct V4 { typedef float4 type; };
struct V1 { typedef float type; };
__device__ inline float4 hy_ld_(V4, const float* p, int64_t e) { return ldnt_(p, e); }
__device__ inline float hy_ld_(V1, const float* p, int64_t e) { return p[e]; }
__device__ inline void hy_st_(float* p, int64_t e, const float4& v) { stnt_(p, e, v); }
__device__ inline void hy_st_(float* p, int64_t e, float v) { p[e] = v; }
__device__ inline void hy_emit_(bf16_t* sh, int64_t e, const float4& v) { emit4_(sh, e, v); }
__device__ inline void hy_emit_(bf16_t* sh, int64_t e, float v) { sh[e] = f32_to_bf16(v); }
__device__ inline float4 hy_add_(const float4& p, const float4& q) {
    return make_float4(__fadd_rn(p.x, q.x), __fadd_rn(p.y, q.y), __fadd_rn(p.z, q.z), __fadd_rn(p.w, q.w));
}
__device__ inline float hy_add_(float p, float q) { return __fadd_rn(p, q); }
__device__ inline float4 hy_mul_(const float4& p, float c) {
    return make_float4(__fmul_rn(p.x, c), __fmul_rn(p.y, c), __fmul_rn(p.z, c), __fmul_rn(p.w, c));
}
__device__ inline float hy_mul_(float p, float c) { return __fmul_rn(p, c); }
__device__ inline float4 hy_sgd_(const float4& m, float lr, const float4& g) { return pair_new_(m, lr, g); }
__device__ inline float hy_sgd_(float m, float lr, float g) { return sgd_(m, lr, g); }

// mean of super-learner a at position e; emit: also write the bf16 copy of the models read (tau = 1)
template <class V>
__device__ inline typename V::type hy_mean_(const HybridArgs& p, int a, int64_t e, bool emit) {
    const int i0 = a * p.S;
    typename V::type s = hy_ld_(V(), p.src + i0 * p.stride, e);
    if (emit) hy_emit_(p.shadow + i0 * p.stride, e, s);
    for (int j = 1; j < p.S; ++j) {
        const typename V::type v = hy_ld_(V(), p.src + (i0 + j) * p.stride, e);
        if (emit) hy_emit_(p.shadow + (i0 + j) * p.stride, e, v);
        s = hy_add_(s, v);
    }
    return hy_mul_(s, p.inv_S);
}
template <class V>
__device__ inline void hy_write_(const HybridArgs& p, int a, int64_t e, const typename V::type& m, bool emit_out) {
    for (int i = a * p.S; i < (a + 1) * p.S; ++i) {
        const typename V::type r = hy_sgd_(m, p.lr, hy_ld_(V(), p.g[i], e));
        hy_st_(p.dst + i * p.stride, e, r);
        if (emit_out) hy_emit_(p.shadow + i * p.stride, e, r);
    }
}

template <class V>
__device__ inline void hy_pair_one_(const HybridArgs& p, int a, int b, int64_t e) {
    const bool emit_in = p.shadow && p.emit_input, emit_out = p.shadow && !p.emit_input;
    const typename V::type ma = hy_mean_<V>(p, a, e, emit_in);
    if (a == b) { hy_write_<V>(p, a, e, ma, emit_out); return; }
    const typename V::type mb = hy_mean_<V>(p, b, e, emit_in);
    const typename V::type m = hy_mul_(hy_add_(ma, mb), 0.5f);
    hy_write_<V>(p, a, e, m, emit_out);
    hy_write_<V>(p, b, e, m, emit_out);
}

template <class V>
__device__ inline void hy_tri_one_(const HybridArgs& p, int64_t e) {
    const bool emit_in = p.shadow && p.emit_input, emit_out = p.shadow && !p.emit_input;
    const typename V::type first = hy_mean_<V>(p, p.order[0], e, emit_in);
    if (p.G == 1) { hy_write_<V>(p, p.order[0], e, first, emit_out); return; }
    typename V::type prev = hy_mean_<V>(p, p.order[p.G - 1], e, false), cur = first;     // read again (and copied) as "next" below
    for (int q = 0; q < p.G; ++q) {
        const typename V::type next = q + 1 < p.G ? hy_mean_<V>(p, p.order[q + 1], e, emit_in) : first;
        const typename V::type m = hy_mul_(hy_add_(hy_add_(prev, cur), next), p.third);
        hy_write_<V>(p, p.order[q], e, m, emit_out);
        prev = cur; cur = next;
    }
}

template <bool VEC, bool TRI>
__global__ __launch_bounds__(256) void hybrid_update_kernel(HybridArgs p) {
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int a = TRI ? 0 : p.a[blockIdx.y], b = TRI ? 0 : p.b[blockIdx.y];
    if constexpr (VEC) {
        const int64_t n4 = p.P >> 2;
        if (e < n4) { if constexpr (TRI) hy_tri_one_<V4>(p, e); else hy_pair_one_<V4>(p, a, b, e); }
        if (blockIdx.x == 0 && threadIdx.x < (p.P & 3)) {
            const int64_t t = (n4 << 2) + threadIdx.x;
            if constexpr (TRI) hy_tri_one_<V1>(p, t); else hy_pair_one_<V1>(p, a, b, t);
        }
    } else {
        if (e < p.P) { if constexpr (TRI) hy_tri_one_<V1>(p, e); else hy_pair_one_<V1>(p, a, b, e); }
    }
}

static hipError_t launch_hybrid(const UpdateDesc& d, bool vec, hipStream_t s) {
    const int S = d.group_size, L = d.L;
    if (S < 1 || L % S != 0) return hipErrorInvalidValue;
    const int G = L / S;
    const bool tri = d.mix == 4;
    if (tri && G == 2) return hipErrorInvalidValue;
    for (int i = 0; i < L; ++i)
        if (!d.active[i]) return hipErrorInvalidValue;          // super-learners average synchronously: everybody takes part
    HybridArgs a;
    a.src = d.src; a.dst = d.dst; a.stride = d.stride; a.P = d.P; a.lr = d.lr;
    a.shadow = d.shadow; a.emit_input = d.emit_input;
    a.S = S; a.G = G; a.inv_S = 1.0f / (float)S; a.third = 1.0f / 3.0f;
    for (int i = 0; i < 128; ++i) { a.g[i] = i < L ? d.g[i] : nullptr; a.order[i] = 0; }
    for (int i = 0; i < 64; ++i) a.a[i] = a.b[i] = 0;
    bool seen[128] = {false};
    for (int q = 0; q < G; ++q) {      // the ring order must be a permutation of the super-learners, the matching an involution
        const int o = d.order[q], pq = d.partner[q];
        if (o < 0 || o >= G || seen[o] || pq < 0 || pq >= G || d.partner[pq] != q) return hipErrorInvalidValue;
        seen[o] = true; a.order[q] = (int16_t)o;
    }
    const int64_t n = vec ? ((d.P >> 2) > 0 ? (d.P >> 2) : 1) : d.P;
    const unsigned blocks = (unsigned)((n + 255) / 256);
    if (tri) {
        if (vec) hipLaunchKernelGGL((hybrid_update_kernel<true, true>), dim3(blocks), dim3(256), 0, s, a);
        else hipLaunchKernelGGL((hybrid_update_kernel<false, true>), dim3(blocks), dim3(256), 0, s, a);
        return hipGetLastError();
    }
    int nw = 0;
    for (int q = 0; q < G; ++q) {
        const int j = d.partner[q];
        if (j == q || q < j) {
            if (nw >= 64) return hipErrorInvalidValue;
            a.a[nw] = (int16_t)q; a.b[nw] = (int16_t)j; ++nw;
        }
    }
    if (vec) hipLaunchKernelGGL((hybrid_update_kernel<true, false>), dim3(blocks, (unsigned)nw), dim3(256), 0, s, a);
    else hipLaunchKernelGGL((hybrid_update_kernel<false, false>), dim3(blocks, (unsigned)nw), dim3(256), 0, s, a);
    return hipGetLastError();
}

// Learner average, the sum in learner order.  A streaming read of L vectors: a float4 of every learner per thread, eight loads
// in flight (16 x 36M: 612 us, 4.0 TB/s, with one float per thread; with the consensus distance behind it 1668 -> 820 us).
// Learners 1 .. L-1 of a position, eight loads at a time, added to s in order (a remainder one load after the other cost 16 x 300k 3 us).
// NT: the models are read past the caches.
template <bool NT, class V, class Add> __device__ inline void add_learners_(const V* x, int64_t step, int L, V& s, Add add) {
    auto load = [](const V* p) { if constexpr (NT) return (V)__builtin_nontemporal_load(p); else return *p; };
    int j0 = 1;
    for (; j0 + 8 <= L; j0 += 8) {
        V v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = load(x + (j0 + j) * step);
#pragma unroll
        for (int j = 0; j < 8; ++j) add(s, v[j]);
    }
    V v[7];
#pragma unroll
    for (int j = 0; j < 7; ++j) {
        if (j0 + j >= L) break;
        v[j] = load(x + (j0 + j) * step);
    }
#pragma unroll
    for (int j = 0; j < 7; ++j) {
        if (j0 + j >= L) break;
        add(s, v[j]);
    }
}

__global__ __launch_bounds__(256) void average_kernel(const float* x, int64_t stride, int L, int64_t P,
                                                      float inv_L, float* out, int vec) {
    typedef __attribute__((ext_vector_type(4))) float f4_t;
    const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x, n4 = vec ? P >> 2 : 0;
    if (e < n4) {
        const f4_t* p = (const f4_t*)x + e;
        f4_t s = __builtin_nontemporal_load(p);
        add_learners_<true>(p, stride >> 2, L, s, [](f4_t& a, const f4_t& b) {
            a.x = __fadd_rn(a.x, b.x); a.y = __fadd_rn(a.y, b.y); a.z = __fadd_rn(a.z, b.z); a.w = __fadd_rn(a.w, b.w);
        });
        stnt_(out, e, make_float4(__fmul_rn(s.x, inv_L), __fmul_rn(s.y, inv_L), __fmul_rn(s.z, inv_L), __fmul_rn(s.w, inv_L)));
        return;
    }
    const int64_t t = 4 * n4 + (e - n4);                   // the last P % 4 elements, or every element
    if (t >= P) return;
    float s = x[t];
    add_learners_<false>(x + t, stride, L, s, [](float& a, const float& b) { a = __fadd_rn(a, b); });
    out[t] = __fmul_rn(s, inv_L);
}

// Learners that a thread of the mean's single-kernel form owns, 0: all of a position.
int mean_learners_a_thread(int L, int64_t P, bool update_first, bool shadow) {
    // Two learners per thread are the measured best on large models (64 x 135M: 5.16 -> 5.48 TB/s, 16 x 145M:
    // 5.49 -> 5.99; four 5.40 / 5.75, eight 5.34 / 5.67) and on small ones, where few threads walk all learners one
    // after another and the models of all learners still fit caches (us, one walk -> two learners: 16 x 100k 10.4 -> 6.3,
    // x 400k 15.8 -> 14.8, x 520k 16.7 -> 18.0; 8 x 400k 8.7 -> 7.4; 5 x 400k 5.8 -> 6.3; 32 x 250k 24.6 -> 19.0, x 400k
    // 29.1 -> 31.0; 64 x 250k 46.6 -> 40.9, x 400k 57 -> 64; 128 x 100k 78 -> 47, x 250k 90 -> 100).
    if (update_first) return (P >= (4 << 20) && L >= 4) || (P >= (1 << 16) && P < (7 << 16) && L >= 8 && L * P <= (P < (1 << 18) ? 1 << 24 : 1 << 23)) ? 2 : 0;
    // The delayed mean: segments on small models (us, one walk / two learners / four / two kernels: 12 x 20k 7.6 / 4.5 /
    // 4.7 / 7.3, 16 x 100k 12.3 / 5.6 / 6.1 / 10.5, 64 x 100k 45 / 17.6 / 14.5 / 22, 64 x 250k 55 / 36.7 / 35.2 / 36.9;
    // 128 x 250k 106 / 90 / 72 / 66) and on large ones of 4 to 11 learners (4 x 12M 93.9 / 92.1, 8 x 12M 196 / 189, 11 x 12M 284 / 257, 8 x 25M 446 / 403; 8 x 60M
    // 1025 / 931, two kernels 1014; 12 and more of that size: two kernels).
    if (P < (1 << 18) && L >= 12 && L * P <= (1 << 24)) return L >= 32 ? 4 : 2;
    if (P >= (1 << 23) && L >= 4) return 2;
    // Between them, up to 32 learners: two as long as few threads are in flight (flat vectors, one walk / two: 4 x 350k 6.2 / 5.0, 6 x 500k 8.9 / 6.8, 8 x 270k 10.0 /
    // 5.8, x 500k 11.3 / 9.5, 12 x 500k 15.2 / 14.0, 16 x 270k 17.5 / 11.4, 32 x 500k 37.3 / 34.5), then one walk, which is the faster while all models fit the
    // memory-side cache (10 x 700k 15.1 / 17.2, 16 x 700k 24.4 / 25.7, 24 x 600k 33.8 / 36.1, 32 x 600k 44.3 / 49.0, 8 x 1M 16.6 / 18.6; four learners a thread lie between).
    // The line is later for few learners (4 x 700k 7.4 / 6.6, 6 x 700k 10.5 / 10.6, 8 x 600k 12.8 / 11.7, x 800k 14.7 / 14.6, x 900k 15.7 / 16.7) and where the bf16 copies are
    // written too (iterations of a model, difference: 8 x 737k -2.2, 16 x 737k -2.6, x 818k -2.2, 24 x 818k -2.9, 32 x 737k -3.8, x 992k +0.5, 5 x 958k -3.2, 8 x 992k -0.3; in fp32 8 x 737k -3.3, 16 x 737k
    // +0.1, 32 x 587k +3.2, x 737k +4.2).  Up to 8M one walk: flat vectors 8 x 1.5M 23.2 / 26.1, 8 x 3M 47.5 /
    // 50.6; in iterations 8 x 2.5M 54.5 / 49.4, 8 x 3.8M 71.4 / 69.4.
    if (L < 4 || L > 32) return 0;
    return P < (L <= 8 && shadow ? 1 << 20 : L <= 8 || shadow ? 13 << 16 : 1 << 19) ? 2 : 0;
}

hipError_t launch_update(const UpdateDesc& d, hipStream_t s) {
    if (d.L < 1 || d.L > 128 || d.P < 1) return hipErrorInvalidValue;
    bool vec = ((uintptr_t)d.src % 16 == 0) && ((uintptr_t)d.dst % 16 == 0) && (d.stride % 4 == 0);
    for (int i = 0; i < d.L; ++i)
        if ((uintptr_t)d.g[i] % 16 != 0) vec = false;
    if (d.update_first && d.mix != 2) return hipErrorInvalidValue;
    if (d.mix == 3 || d.mix == 4) return launch_hybrid(d, vec, s);
    if (d.mix == 2) {
        AllArgs a;
        a.src = d.src; a.dst = d.dst; a.stride = d.stride; a.P = d.P; a.lr = d.lr; a.L = d.L;
        a.inv_L = 1.0f / (float)d.L;
        a.shadow = d.shadow; a.emit_input = d.emit_input;
        for (int i = 0; i < 128; ++i) a.g[i] = i < d.L ? d.g[i] : nullptr;
        if (d.update_first) {
            for (int i = 0; i < d.L; ++i)
                if (!d.active[i]) return hipErrorInvalidValue;     // the baseline waits for every learner
            if (d.emit_input) return hipErrorInvalidValue;         // and has no staleness
        }
        if (vec && !d.update_first && d.mean_buf && d.mean_elems >= 1024 && d.L >= 4 && (d.P >> 2) > 0 &&
            (uintptr_t)d.mean_buf % 16 == 0) {
            // Equal chunks (a short last one leaves the chip idle at its end), and a grid of whole rounds of the 8 XCDs: the
            // workgroups of one position then run on one XCD for every learner and find its mean in that L2.
            const int64_t n4 = d.P >> 2, chunks = (n4 + (d.mean_elems >> 2) - 1) / (d.mean_elems >> 2);
            const int64_t chunk4 = round_up((n4 + chunks - 1) / chunks, 256);     // whole workgroups: every chunk starts on a line
            AllSplitArgs q;
            q.a = a; q.mean = d.mean_buf;
            for (int64_t e0 = 0; e0 < n4; e0 += chunk4) {
                q.e0 = e0; q.n4c = n4 - e0 < chunk4 ? n4 - e0 : chunk4;
                q.tail = e0 + chunk4 >= n4;
                // (workgroups of 64 or 128 threads instead of 256 change nothing here: 5.8 - 6.0 TB/s in all nine combinations;
                // a mean kernel with one (position, learner) per thread and the sum through LDS is slower: 5.1 - 5.8)
                const unsigned blocks = (unsigned)(((q.n4c + 255) / 256 + 7) / 8 * 8);
                hipLaunchKernelGGL(all_mean_kernel, dim3(blocks), dim3(256), 0, s, q);
                hipLaunchKernelGGL(all_apply_kernel, dim3(blocks, (unsigned)d.L), dim3(256), 0, s, q);
            }
        } else if (vec) {
            const int64_t n4 = d.P >> 2;
            const unsigned blocks = (unsigned)((n4 > 0 ? n4 : 1) + 255) / 256;
            const int seg = d.sync_segment >= 0 ? d.sync_segment : mean_learners_a_thread(d.L, d.P, d.update_first, d.shadow != nullptr);
            if (n4 > 0 && seg >= 2 && d.L > seg) {
                if (d.update_first) launch_mean_seg<true>(a, seg, s);
                else launch_mean_seg<false>(a, seg, s);
            } else if (d.update_first) hipLaunchKernelGGL(sync_update_kernel<true>, dim3(blocks), dim3(256), 0, s, a);
            else hipLaunchKernelGGL(all_update_kernel<true>, dim3(blocks), dim3(256), 0, s, a);
        } else {
            const unsigned blocks = (unsigned)((d.P + 255) / 256);
            if (d.update_first) hipLaunchKernelGGL(sync_update_kernel<false>, dim3(blocks), dim3(256), 0, s, a);
            else hipLaunchKernelGGL(all_update_kernel<false>, dim3(blocks), dim3(256), 0, s, a);
        }
        return hipGetLastError();
    }
    if (d.mix == 1) {
        TriArgs a;
        a.src = d.src; a.dst = d.dst; a.stride = d.stride; a.P = d.P; a.lr = d.lr; a.L = d.L;
        a.third = 1.0f / 3.0f;
        a.shadow = d.shadow; a.emit_input = d.emit_input;
        // the order must be a permutation of 0..L-1 (an index out of range would address another learner's memory)
        bool seen[128] = {false};
        for (int i = 0; i < d.L; ++i) {
            if (d.order[i] < 0 || d.order[i] >= d.L || seen[d.order[i]]) return hipErrorInvalidValue;
            seen[d.order[i]] = true;
        }
        for (int q = 0; q < 128; ++q) { a.order[q] = q < d.L ? d.order[q] : 0; a.order16[q] = (int16_t)a.order[q]; a.g[q] = q < d.L ? d.g[d.order[q]] : nullptr; }
        // Segments against the single walk: the walk has the fewest loads, but a thread walks 2 L streams (long rings of large
        // models) and takes all learners' time (small models, a few workgroups per compute unit).  us, walk / segments of one / two:
        // L = 5 7.7M 81 / 86 / 117, 145M 1636 / 1622 / 2232; L = 6 4.3M 55 / 54 / 70, 145M 1972 / 1804 / 2408; L = 8 7.7M 132 / 125 / 141,
        // 145M 2641 / 2344 / 2666; L = 9 4.3M 84 / 94 / 84, 30M 602 / 646 / 579; L = 11 7.7M 183 / 185 / 173; L = 16 7.7M 276 / 258 / 244,
        // 145M 5.5 / 5.8 / 6.1 TB/s (four positions 5.0); and L = 16 100k 8.8 / 6.6 / 6.6, 400k 15.2 / 13.4 / 15.0, 900k 30 / 33 / 33; L = 8 400k
        // 8.7 / 7.5 / 9.0, 900k 14.1 / 16.3 / 18.0.
        const int seg = d.tri_segment >= 0 ? d.tri_segment
                        : d.P >= (4 << 20) ? (d.L >= 9 ? 2 : d.L >= 6 ? 1 : 0)
                        : (d.P < (1 << 19) && d.L >= 8 ? 1 : 0);
        // The walk: four positions at a time where the last round of the grid (2^21 elements fill the chip) is short, one by one where
        // long rings fill it.  us, one by one / four: 12 x 600k 23.6 / 16.1, x 1.25M 37 / 34, 16 x 2.1M 78 / 72, 64 x 900k 138 / 131; and 16 x
        // 1.5M 48 / 51, x 3.5M 112 / 123, 64 x 1.2M 167 / 177, x 1.5M 192 / 222, x 3.5M 481 / 533, 12 x 3.5M 84 / 91, 8 x 3.5M 56 / 59.
        const bool one = d.P < (4 << 20) && (d.P < (1 << 21) ? d.P >= (d.L >= 64 ? 1100000 : 1500000) && d.L >= 12
                                                             : d.L >= 12 ? d.P >= 2800000 : d.L >= 8 && d.P >= 3300000);
        if (vec && (d.P >> 2) > 0 && seg >= 1 && d.L > seg) {
            if (seg == 1) launch_tri_seg<1>(a, s);
            else if (seg >= 8) launch_tri_seg<8>(a, s);
            else if (seg >= 4) launch_tri_seg<4>(a, s);
            else launch_tri_seg<2>(a, s);
        } else if (vec) {
            const int64_t n4 = d.P >> 2;
            if (one) hipLaunchKernelGGL((tri_update_kernel<true, 1>), dim3((unsigned)(((n4 > 0 ? n4 : 1) + 255) / 256)), dim3(256), 0, s, a);
            else hipLaunchKernelGGL((tri_update_kernel<true, 4>), dim3((unsigned)(((n4 > 0 ? n4 : 1) + 255) / 256)), dim3(256), 0, s, a);
        } else {
            hipLaunchKernelGGL((tri_update_kernel<false, 1>), dim3((unsigned)((d.P + 255) / 256)), dim3(256), 0, s, a);
        }
        return hipGetLastError();
    }
    PairArgs a;
    a.src = d.src; a.dst = d.dst; a.stride = d.stride; a.P = d.P; a.lr = d.lr;
    a.shadow = d.shadow; a.emit_input = d.emit_input;
    for (int i = 0; i < 128; ++i) { a.g[i] = i < d.L ? d.g[i] : nullptr; a.a[i] = a.b[i] = 0; }
    int n = 0;
    for (int i = 0; i < d.L; ++i) {
        if (!d.active[i]) continue;
        const int j = d.partner[i];
        if (j == i) { a.a[n] = a.b[n] = (int16_t)i; ++n; }
        else if (i < j) { a.a[n] = (int16_t)i; a.b[n] = (int16_t)j; ++n; }
    }
    a.nwork = n;
    if (n == 0) return hipSuccess;
    // One member per thread in workgroups of 64 positions x 2 members is the measured best on large models (64 x 135M,
    // random ring, 10 % stragglers: 5.9 -> 6.3 TB/s; 16 x 145M: 5.9 -> 6.6; 128 positions 6.15 / 6.3, 32: 6.1 / 6.45,
    // 256: 6.0 / 6.25; the two-member kernel in workgroups of 64 threads 6.1 / 6.3).
    const int split = d.pair_split < 0 ? (d.P >= (1 << 20) ? 64 : 0) : d.pair_split;
    if (vec && split > 0 && (d.P >> 2) > 0) {
        const int64_t n4 = d.P >> 2;
        if (split == 128)
            hipLaunchKernelGGL(pair_split_update_kernel<128>, dim3((unsigned)((n4 + 127) / 128), (unsigned)n), dim3(128, 2), 0, s, a);
        else
            hipLaunchKernelGGL(pair_split_update_kernel<64>, dim3((unsigned)((n4 + 63) / 64), (unsigned)n), dim3(64, 2), 0, s, a);
        return hipGetLastError();
    }
    if (vec) {
        const int64_t n4 = d.P >> 2;
        const int64_t per = 256 * kUnroll;
        const unsigned blocks = (unsigned)(((n4 > 0 ? n4 : 1) + per - 1) / per);
        hipLaunchKernelGGL(pair_update_kernel<true>, dim3(blocks, (unsigned)n), dim3(256), 0, s, a);
    } else {
        const int64_t per = 256 * kUnroll;
        hipLaunchKernelGGL(pair_update_kernel<false>, dim3((unsigned)((d.P + per - 1) / per), (unsigned)n), dim3(256), 0, s, a);
    }
    return hipGetLastError();
}

// Consensus distance: the squared deviations of the L models from their mean, summed in fp64.  Bound by one read of the models,
// which a thread holds in registers between the mean and the deviations: those of its position of four elements, up to
// 8 learners all (SPLIT 1); more are split over two (up to 16) or four waves, wave w the learners w, w + SPLIT, ..., whose sums
// meet in LDS.  us, one thread walking all learners of an element twice / four waves / SPLIT: 2 x 8M 27 / 37 / 15, 5 x
// 1M 9.2 / 11.5 / 7.3, 8 x 8M 79 / 54 / 43; shared by two waves 12 x 450k 8.7 / 9.7 / 8.3, 16 x 8M
// 227 / 90 / 83.  The order of the sums does not depend on the alignment (VEC:
// every vector 16-byte aligned).  Block sums through LDS, then one block adds the partial sums in index order (a fixed
// order: the result is reproducible).
template <int NL, bool VEC, int SPLIT>    // learners per wave; waves that share the learners of a position
__global__ __launch_bounds__(256) void consensus_partial_kernel(const float* x, int64_t stride, int L, int64_t P, double* partial) {
    constexpr int W = 4, GROUPS = 4 / SPLIT;
    __shared__ double sums[SPLIT > 1 ? 2 : 1][SPLIT > 1 ? 4 : 1][W][64];
    __shared__ double sh[256];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, part = wave % SPLIT;
    const int64_t n = (P + W - 1) / W, nv = P / W;         // positions, whole positions
    double acc = 0.0;
    int buf = 0;
    for (int64_t p0 = ((int64_t)blockIdx.x * GROUPS + wave / SPLIT) * 64; p0 < n; p0 += (int64_t)gridDim.x * GROUPS * 64, buf ^= 1) {
        const int64_t e = p0 + lane;
        float v[NL][W];
        const float* q = x + part * stride;                // of learner part + SPLIT j
        if (e < nv) {
#pragma unroll
            for (int j = 0; j < NL; ++j) {
                if (part + SPLIT * j >= L) break;
                if constexpr (VEC) {
                    const float4 f = ldnt_(q + SPLIT * j * stride, e);
                    v[j][0] = f.x; v[j][1] = f.y; v[j][2] = f.z; v[j][3] = f.w;
                } else {
#pragma unroll
                    for (int c = 0; c < W; ++c) v[j][c] = q[SPLIT * j * stride + e * W + c];
                }
            }
        } else {                                           // the last P % W elements; 0 past the end and past it no deviation
#pragma unroll
            for (int j = 0; j < NL; ++j) {
                if (part + SPLIT * j >= L) break;
#pragma unroll
                for (int c = 0; c < W; ++c) v[j][c] = e * W + c < P ? q[SPLIT * j * stride + e * W + c] : 0.f;
            }
        }
        double s[W];
#pragma unroll
        for (int c = 0; c < W; ++c) s[c] = 0.0;
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            if (part + SPLIT * j >= L) break;
#pragma unroll
            for (int c = 0; c < W; ++c) s[c] += (double)v[j][c];
        }
        double mean[W];
        if constexpr (SPLIT > 1) {
#pragma unroll
            for (int c = 0; c < W; ++c) sums[buf][wave][c][lane] = s[c];
            __syncthreads();                               // (one barrier a round: the next round writes the other buffer)
#pragma unroll
            for (int c = 0; c < W; ++c)
            {
                const int w0 = wave - part;
                double t = sums[buf][w0][c][lane] + sums[buf][w0 + 1][c][lane];
                if constexpr (SPLIT == 4) t = (t + sums[buf][w0 + 2][c][lane]) + sums[buf][w0 + 3][c][lane];
                mean[c] = t / (double)L;
            }
        } else {
#pragma unroll
            for (int c = 0; c < W; ++c) mean[c] = s[c] / (double)L;
        }
#pragma unroll
        for (int j = 0; j < NL; ++j) {
            if (part + SPLIT * j >= L) break;
#pragma unroll
            for (int c = 0; c < W; ++c) { const double d = (double)v[j][c] - mean[c]; acc += d * d; }
        }
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) sh[threadIdx.x] += sh[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = sh[0];
}
__global__ __launch_bounds__(256) void consensus_final_kernel(const double* partial, int n, double* out) {
    __shared__ double sh[256];
    double acc = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) acc += partial[i];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) sh[threadIdx.x] += sh[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[0] = sh[0];
}

template <bool VEC>
static void consensus_partial_t(const float* x, int64_t stride, int L, int64_t P, double* partial, unsigned blocks, hipStream_t s) {
    if (L <= 8) hipLaunchKernelGGL((consensus_partial_kernel<8, VEC, 1>), dim3(blocks), dim3(256), 0, s, x, stride, L, P, partial);
    else if (L <= 16) hipLaunchKernelGGL((consensus_partial_kernel<8, VEC, 2>), dim3(blocks), dim3(256), 0, s, x, stride, L, P, partial);
    else if (L <= 32) hipLaunchKernelGGL((consensus_partial_kernel<8, VEC, 4>), dim3(blocks), dim3(256), 0, s, x, stride, L, P, partial);
    else hipLaunchKernelGGL((consensus_partial_kernel<32, VEC, 4>), dim3(blocks), dim3(256), 0, s, x, stride, L, P, partial);
}

hipError_t launch_consensus(const float* x, int64_t stride, int L, int64_t P, double* partial, double* out, hipStream_t s) {
    if (L < 1 || L > 128 || P < 1) return hipErrorInvalidValue;
    const bool vec = (uintptr_t)x % 16 == 0 && stride % 4 == 0;
    const int64_t per_block = L <= 8 ? 256 : L <= 16 ? 128 : 64;          // positions of four elements
    int64_t blocks = ((P + 3) / 4 + per_block - 1) / per_block;
    if (blocks > kConsensusBlocks) blocks = kConsensusBlocks;
    if (vec) consensus_partial_t<true>(x, stride, L, P, partial, (unsigned)blocks, s);
    else consensus_partial_t<false>(x, stride, L, P, partial, (unsigned)blocks, s);
    hipLaunchKernelGGL(consensus_final_kernel, dim3(1), dim3(256), 0, s, (const double*)partial, (int)blocks, out);
    return hipGetLastError();
}

// ---- the same reduction for callers that cannot allocate ----------------------------------------
// The per-workgroup partial sums live in a file-scope device array instead of caller-provided memory.
// Every GPU holds its own copy of the array at its own address: the address is looked up once per device,
// with that device current, and only that address (never the array's name, which is a host-side stand-in
// in host code) is handed to kernels.  All calls on one GPU share the array: calls that overlap on one GPU
// race.  Nothing in it has to start at zero (a call writes every partial sum it later reads).
static __device__ __align__(256) double scratch[kConsensusBlocks];

static std::mutex g_scratch_mutex;
static double* g_scratch_ptr[kMaxDevices] = {nullptr};

hipError_t launch_consensus_static(const float* x, int64_t stride, int L, int64_t P, double* out, hipStream_t s) {
    if (L < 1 || P < 1) return hipErrorInvalidValue;
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    double* ptr = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        if (!g_scratch_ptr[dev]) {
            void* p = nullptr;
            e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
            if (e != hipSuccess) return e;
            if (!p) return hipErrorInvalidSymbol;
            g_scratch_ptr[dev] = (double*)p;
        }
        ptr = g_scratch_ptr[dev];
    }
    return launch_consensus(x, stride, L, P, ptr, out, s);
}

hipError_t launch_average(const float* x, int64_t stride, int L, int64_t P, float* out, hipStream_t s) {
    // One element to a thread while there are too few for float4 threads to fill the chip (us, float / float4: 8 x 1M 5.8 / 6.5, 12 x
    // 450k 4.2 / 5.2, 16 x 300k 4.0 / 4.8, 24 x 300k 5.2 / 6.4; and 9 x 1M 7.7 / 6.8, 64 x 100k 13.6 / 7.8).
    const bool few = L * P <= (L <= 32 ? 1 << 23 : 1 << 22);
    const int vec = !few && (uintptr_t)x % 16 == 0 && stride % 4 == 0 && (uintptr_t)out % 16 == 0;
    const int64_t work = vec ? (P >> 2) + (P & 3) : P;
    hipLaunchKernelGGL(average_kernel, dim3((unsigned)((work + 255) / 256)), dim3(256), 0, s, x, stride, L, P,
                       1.0f / (float)L, out, vec);
    return hipGetLastError();
}

}  // namespace adpsgd
