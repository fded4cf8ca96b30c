// Host-side launch interface of the HIP kernels (internal to the library).
#pragma once
#include "common.hpp"

namespace adpsgd {

// Compacted list of the learners a launch works on: entry j of the launch is learner idx[j].
// Stragglers (Section IV-D: a learner that sits an iteration out) are left out of every launch
// of the gradient phase this way; without stragglers it is the identity.
struct LearnerMap {
    uint8_t idx[128];
    void identity() { for (int i = 0; i < 128; ++i) idx[i] = (uint8_t)i; }
};

// ---- grouped GEMM  C[z] = A[z] * B[z]' (+ bias) ------------------------------
// Group z = j*groupsD + d works on learner i = lmap.idx[j]; operand X of it starts at
// X + i*sXi + d*sXd (strides in elements).
struct GemmDesc {
    int precision;            // 0 fp32 operands, 1 bf16 operands
    int a_kc, b_kc;           // operand stored K-contiguous ([rows][K]) or not ([K][rows])
    int c_elem;               // C stored in the operand type instead of fp32
    int M, N, K;
    const void* A; int64_t lda, sAi, sAd;
    const void* B; int64_t ldb, sBi, sBd;
    void* C; int64_t ldc, sCi, sCd;
    const float* bias; int64_t sBiasI, sBiasD;
    int groupsI, groupsD;
    int k_padded;             // rows of K-contiguous operands are readable up to the next multiple of 16 bytes past K
    int tile;                 // tile configuration (see gemm.hip): -1 automatic, or 0, 5, 11 .. 15
    LearnerMap lmap;
};
// Returns hipSuccess, or hipErrorInvalidValue when the operands do not meet the
// alignment rules (rows and strides multiples of 4 elements).
hipError_t launch_gemm(const GemmDesc& d, hipStream_t s);
// ---- fused mixing + SGD update ------------------------------------------------
struct UpdateDesc {
    int L;
    int mix;                   // 0 pair, 1 ring neighbours (thirds), 2 all, 3 / 4 hybrid: mean inside super-learners of
                               // group_size consecutive learners, pair / ring-neighbour operator across them (partner and
                               // order are then over the L / group_size super-learners)
    int group_size;
    int64_t P;                 // elements per learner
    const float* src;          // x^k, learner i at src + i*stride
    float* dst;                // x^{k+1}, learner i at dst + i*stride (may equal src)
    int64_t stride;
    const float* g[128];       // gradient of learner i
    int16_t partner[128];
    int16_t order[128];        // ring order (mix 1): order[p] = learner at ring position p
    int16_t active[128];
    float lr;
    bf16_t* shadow;            // optional [L][stride] bf16 copy of the next gradient point, or NULL
    int emit_input;            // shadow = bf16(x^k) (tau = 1) instead of bf16(x^{k+1})
    int update_first;          // mix 2 only: average the updated models x_j - lr*g_j (synchronous baseline)
    int pair_split;            // mix 0: 64 / 128 = one member of a pair per thread in workgroups of that many positions (models
                               // exchanged through LDS), 0 = both members per thread, -1 = default
    int sync_segment;          // synchronous baseline, global mean in one kernel: learners per thread (2, 4 or 8), 0: one thread owns all learners of a position, -1: default
    int tri_segment;           // mix 1: ring positions per thread (2, 4 or 8), 0: one thread walks the whole ring, -1: default
    float* mean_buf;           // mix 2: optional buffer of mean_elems floats; when given the global mean runs chunk by
    int64_t mean_elems;        //   chunk of that many elements in two kernels (fewer streams per thread); NULL: one kernel
};
hipError_t launch_update(const UpdateDesc& d, hipStream_t s);
int mean_learners_a_thread(int L, int64_t P, bool update_first, bool shadow);
hipError_t launch_average(const float* x, int64_t stride, int L, int64_t P, float* out, hipStream_t s);
// out[0] = sum_i sum_e (x_i[e] - mean_i x_i[e])^2 in fp64; partial: kConsensusBlocks doubles of scratch
constexpr int kConsensusBlocks = 2048;
hipError_t launch_consensus(const float* x, int64_t stride, int L, int64_t P, double* partial, double* out, hipStream_t s);
// the same with the partial sums in a device array owned by the library (one per GPU, shared by all calls on it)
constexpr int kMaxDevices = 64;
hipError_t launch_consensus_static(const float* x, int64_t stride, int L, int64_t P, double* out, hipStream_t s);

// ---- LSTM gradient pieces -------------------------------------------------------
struct StageDesc {             // copy / cast the minibatches into the workspace
    int L, precision;          // L: learners of this launch (entries of lmap)
    LearnerMap lmap;
    int64_t rows;              // T*B
    int I, ldx;                // feature dim and padded row stride of the staged copy
    const float* feats[128];
    const int32_t* labels[128];
    void* x0; int64_t sX0;     // [L][rows][ldx] operand type
    int32_t* y; int64_t sY;    // [L][rows]
    uint32_t* epoch;           // incremented once (may be NULL), and
    uint64_t* join; int64_t joins;       // these words are cleared
    // optional (bf16): W_x of layer 0, pad_rows rows of I floats, learner stride pad_sS, into bf16 rows of ldx, zero-padded, as the inputs
    const float* pad_src; int64_t pad_sS; bf16_t* pad_dst; int64_t pad_sD, pad_rows;
};
hipError_t launch_stage(const StageDesc& d, hipStream_t s);
hipError_t launch_cast_bf16(const float* src, bf16_t* dst, int64_t n, hipStream_t s);
struct RecDesc {               // one time step of one layer, all learners and directions
    int precision;
    int L, D, B, H, T;         // L: learners of this launch (entries of lmap)
    LearnerMap lmap;
    int direct;                // 0: register-staged kernels only (tuning)
    int step;                  // processing step 0..T-1 (frame = step, or T-1-step for d = 1)
    // forward: gates buffer holds W_x x + b on entry, the activated gates on exit
    float* gates; int64_t sGi;           // [L][T*B][D*4H] fp32
    float* c; int64_t sCi;               // [L][D][T*B][H] fp32
    void* y; int64_t sYi;                // [L][T*B][D*H] operand type (layer output)
    const void* wh; int64_t sWi, sWd;    // W_h [D][4H][H] operand type, learner stride
    // backward only
    const float* dy; int64_t sDYi;       // [L][T*B][D*H] fp32, gradient w.r.t. the layer output
    void* da; int64_t sDAi;              // [L][T*B][D*4H] operand type, gate pre-activation grads
    float* dc; int64_t sDCi;             // [L][D][B][H] fp32 running dL/dc
    // column sums of da over the batch rows of every tile (partial bias gradients), summed over the
    // frames and batch tiles afterwards: [L][T * batch tiles][D*4H] fp32
    float* dbp; int64_t sDBi;
};
// Rows of dbp per frame that launch_rec_backward writes for this layer (its batch tiles); at most ceil(B / 32).
int rec_backward_batch_tiles(const RecDesc& d);
// Which kernels the steps of a layer whose tensors meet rec_aligned run on (pairs: learners x directions): 0 register-staged,
// 1 direct-to-LDS, 2 contraction split over the waves.
int rec_step_kind(int precision, bool backward, int pairs, int H, int B);
hipError_t launch_rec_forward(const RecDesc& d, hipStream_t s);
hipError_t launch_rec_backward(const RecDesc& d, hipStream_t s);
// The same step with the contraction split over the waves of a workgroup and the operands read straight into registers
// (lstm_small.hip); needs 16-byte aligned operand rows and H a multiple of 16 bytes.
hipError_t launch_rec_split(const RecDesc& d, bool backward, hipStream_t s);

// Whether every operand row that is loaded in 16-byte pieces is 16-byte aligned and a whole number of them.
bool rec_aligned(const RecDesc& d);
// Whether the rows of W_h are whole, aligned groups of four values: what the buffer loads of the kernels that hold W_h in
// registers need (a 16-byte buffer load asks for 4-byte alignment only).
bool rec_quad_aligned(const RecDesc& d);

// All T frames of one layer in one launch, W_h held in registers, a workgroup per (learner, direction) and 16 batch rows
// (lstm_resident.hip; hidden sizes up to 128).  d.step is not used; the backward pass writes rec_resident_batch_tiles(d)
// rows of dbp for all frames together.
bool rec_resident_supported(const RecDesc& d);
int rec_resident_batch_tiles(const RecDesc& d);
hipError_t launch_rec_resident(const RecDesc& d, bool backward, hipStream_t s);

// Bits of the device-side status word of a handle (0 = fine).  Words 2 and 3 behind it hold the address of pinned host memory,
// a word per bit, where a kernel that raises a bit leaves a 1: no copy in the stream while all is well.
constexpr uint32_t kStatusBadLabel = 1u;       // a label outside [0, classes) was met (and clamped)
constexpr uint32_t kStatusWaitExpired = 2u;    // a bounded wait between workgroups ran out
__device__ inline void raise_status_(uint32_t* status, uint32_t bit) {
    __hip_atomic_fetch_or(status, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    uint32_t* host = *(uint32_t**)(status + 2);
    __hip_atomic_store(host + (bit >> 1), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// All T frames of one layer in one launch, W_h spread over clusters of workgroups that exchange h (partial sums of dh) through
// `exchange` (lstm_cluster.hip).  r.step is not used; the backward pass writes rec_cluster_batch_tiles(r) rows of dbp for all
// frames together.
struct ClusterDesc {
    RecDesc r;
    uint64_t* exchange;                  // rec_cluster_exchange_words(r, backward) words, zero before the handle's first launch
    uint32_t* raw;                       // backward: rec_cluster_raw_words(r) words, zero before the handle's first launch
    const uint32_t* epoch;               // differs from iteration to iteration, 0 in none
    int launch, launches;                // this launch among those of an iteration
    uint64_t* join;                      // rec_cluster_count(r) words, zero before the launch
    int spread;                          // set by launch_rec_cluster: the ids of a cluster's workgroups lie 8 apart
    uint32_t* status;                    // kStatusWaitExpired is or-ed in
    unsigned long long wait_ticks;       // bound of one wait of the exchange
    unsigned long long join_ticks;       // after which a cluster whose workgroups have not all started is left to one of them
};
bool rec_cluster_supported(const RecDesc& d, bool backward, int cu_count);
int rec_cluster_batch_tiles(const RecDesc& d);
int64_t rec_cluster_count(const RecDesc& d);
int64_t rec_cluster_exchange_words(const RecDesc& d, bool backward);
int64_t rec_cluster_raw_words(const RecDesc& d);
hipError_t launch_rec_cluster(const ClusterDesc& p, bool backward, int cu_count, hipStream_t s);

// All T frames of one layer for ngl (learner, direction) pairs in one launch, W_h held in registers
// (lstm_persist.hip).  r: the tensors of the layer (r.L, r.lmap, r.step and r.direct are not used);
// pair j of the launch is learner gl_learner[j], direction gl_dir[j].
struct PersistDesc {
    RecDesc r;
    int ngl;                             // pairs of this launch, 1..64; ngl * H/32 workgroups, at most one per compute unit
    uint8_t gl_learner[64], gl_dir[64];
    uint32_t* counters;                  // [ngl] device words, zero before the launch: workgroups that have finished a frame
    uint32_t* status;                    // the handle's status word (kStatusWaitExpired is or-ed in)
    unsigned long long wait_ticks;       // bound of one wait between workgroups, in ticks of the 100 MHz wall clock
};
bool rec_persist_supported(const RecDesc& d, int cu_count);
hipError_t launch_rec_persist(const PersistDesc& p, bool backward, int cu_count, hipStream_t s);

// one wave that idles for `ticks` of the 100 MHz wall clock (the wall-clock model of the slow-learner experiment)
hipError_t launch_delay(unsigned long long ticks, hipStream_t s);

// ---- measurement probes (probe.hip) ----------------------------------------------------------------
hipError_t launch_mfma_peak(float* out, int blocks, int iters, hipStream_t s);       // out: [blocks * 256] floats
// reads : writes_f32 : writes_bf16 one of 1:0:0, 1:1:0, 2:1:0, 2:1:1, 4:2:0, 4:2:2, 8:4:4, 16:8:8, 32:16:16; the streams
// are `pitch` bytes apart in buf
hipError_t launch_stream_probe(int reads, int writes_f32, int writes_bf16, void* buf, int64_t pitch, int64_t elems, hipStream_t s);

struct SoftmaxDesc {
    int precision, L;          // L: learners of this launch (entries of lmap)
    LearnerMap lmap;
    uint32_t* status;          // device status word: kStatusBadLabel is or-ed in
    int64_t rows; int C;
    const float* logits; int64_t ldl, sLi;    // [L][rows][C], rows ldl apart
    const int32_t* y; int64_t sYi;
    void* dlogits; int64_t ldd, sDi;     // [L][rows][C] operand type, rows ldd apart: (softmax - onehot)/rows
    float* row_loss;                     // [L][rows]
};
hipError_t launch_softmax_ce(const SoftmaxDesc& d, hipStream_t s);
// The product that gives the logits and launch_softmax_ce in one launch (output_small.hip); the logits are not stored.
bool output_small_supported(const GemmDesc& g, const SoftmaxDesc& p);
hipError_t launch_output_small(const GemmDesc& g, const SoftmaxDesc& p, hipStream_t s);

// out[z][n] = sum_m in[z][m][n]   (bias gradients), z = lmap.idx[0..L)
struct ColsumDesc {
    int precision, L;
    LearnerMap lmap;
    const void* in; int64_t ld, sIi;     // operand type
    int64_t rows; int N;
    float* out; int64_t sOi;
    // with loss != NULL also loss[i] = mean of row_loss[i][0..rows) for the learners whose bit is set, 0 for the other L_all
    float* loss; const float* row_loss; int L_all; uint32_t active_bits[4];
};
hipError_t launch_colsum(const ColsumDesc& d, hipStream_t s);
bool colsum_ok(const ColsumDesc& d);

// What follows from one gradient matrix dA: dX = dA W, weight gradients dW = dA' X, column sums.  They are independent, and share a
// launch as far as their tiles allow (gemm_multi.hip).
struct GradProducts {
    bool has_dx, has_cs;
    GemmDesc dx;                         // a_kc = 1, b_kc = 0
    int ndw; GemmDesc dw[2];             // a_kc = b_kc = 0
    ColsumDesc cs;
};
// Launches that the weight gradients take part in (dX has one of its own or shares theirs), and whether the column sums are apart.
int grad_product_launches(const GradProducts& g, bool& colsum_apart);
hipError_t launch_grad_products(const GradProducts& g, hipStream_t s);
// dst[z][0..n) = 0 for z = lmap.idx[0..L)  (a fill kernel, not a memset node: safe under stream capture)
hipError_t launch_zero(float* dst, int64_t sDi, int64_t n, int L, const LearnerMap& lmap, hipStream_t s);

}  // namespace adpsgd
