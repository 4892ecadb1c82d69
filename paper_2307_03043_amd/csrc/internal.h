// Internal declarations of libchamfer: device helpers, the per-call device
// parameter block, the workspace layout and the kernel launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "chamfer.h"

namespace chamfer {

constexpr uint32_t kPurposeGrid = 1;    // shifts z' and key multipliers M
constexpr uint32_t kPurposeEmbed = 2;   // Gaussian embedding matrix
constexpr uint32_t kPurposeSample = 3;  // importance-sampling draws
constexpr uint32_t kPurposeSketch = 4;  // p-stable direction of the reduction
constexpr uint32_t kPurposePart = 5;    // shifts and multipliers of the partition grid
constexpr uint32_t kPurposePad = 6;     // signs of the padding coordinates
constexpr uint64_t kEmptyKey = ~0ull;   // bucket keys are < 2^63
constexpr int kMaxScales = 64;
// The per-coordinate min/max is accumulated in kLohiReps copies, half of them
// for A and half for B (workgroup id mod kLohiReps / 2 picks one), so that the
// global atomics of many workgroups do not queue on the same 2d words; the
// calibration folds the copies into the first, [lo(d) | hi(d)], which every
// later kernel reads, and keeps the centre of the l2 exact pass in the words
// after it (half_centre).
constexpr int kLohiReps = 8;
inline size_t lohi_bytes(int d) { return (size_t)kLohiReps * 2 * (size_t)d * sizeof(uint32_t); }
constexpr int kMaxWindow = 32;          // W of the multi-probe CrudeNN
constexpr int kMaxReps = 64;            // k of the multi-probe CrudeNN
// flags of the probe launches of the multi-probe CrudeNN
constexpr int kProbeMerge = 1;  // keep the better of this and the previous structure's result
constexpr int kProbeLast = 2;   // last structure: also reduce max D_a

constexpr int kMaxRepl = 64;     // replicas of the per-workgroup maxima (one per lane)
constexpr int kReplStride = 32;  // uint32 words between replicas: one 128-byte line each

// Device-resident parameters of one call; written by the kernels, read by
// later kernels of the same call (no host round trip).
struct DevParams {
    int32_t status;      // CHAMFER_OK / CHAMFER_ENONFINITE
    int32_t e_top;       // top grid scale exponent
    int32_t s;           // fixed-point exponent of the weights
    int32_t all_zero;    // every D_a == 0
    uint32_t nonfinite;  // an input coordinate is NaN or Inf
    uint64_t W;          // fixed-point total
    double S;            // sum_k (hi_k - lo_k)
    uint32_t fallbacks;  // 32-row blocks the l2 exact pass evaluated in full
    int32_t he;          // l2 exact pass: the operands' scale is 2^he
    float half_box;      // l2 exact pass: upper bound of |(b - centre) 2^he| over B (d <= 10)
    float sad_inv;       // l1 exact pass: byte steps per unit (0: the bytes tell nothing)
    int32_t sad_in;      // l1 exact pass: every row of B lies in the bytes' box
    uint32_t pad32[1];
    // The maxima of D_a and (l2 exact pass) of |y|^2 and |y - y~|^2 (words 0
    // and 1 of a replica) reduced over thousands of workgroups: each
    // workgroup's atomicMax goes to replica (id mod kMaxRepl), one 128-byte
    // line each, since atomics queued on one address serialise at its cache
    // channel; readers take the max over the replicas (rep_fold).
    uint32_t max_d_rep[kMaxRepl * kReplStride];
    uint32_t half_rep[kMaxRepl * kReplStride];
};

__device__ __forceinline__ void rep_max(uint32_t *rep, int64_t id, uint32_t m) {
    atomicMax(&rep[(id % kMaxRepl) * kReplStride], m);
}

// Max over the replicas (unsigned: the bits of non-negative floats order as
// the floats); a whole wavefront calls it, lane r reading replica r.
__device__ __forceinline__ uint32_t rep_fold(const uint32_t *rep) {
    uint32_t m = rep[(threadIdx.x & 63) * kReplStride];
    for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off));
    return m;
}

// Lane l's 64-bit value in every lane (l wave-uniform; a scalar register
// read, no LDS round trip).
__device__ __forceinline__ unsigned long long lane_u64(unsigned long long v, int l) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l);
    return ((unsigned long long)hi << 32) | lo;
}

// One bucket of a scale's open-addressing table: key -> lowest b index.
struct alignas(16) Bucket {
    unsigned long long key;
    int32_t val;
    int32_t pad;
};

// ---------------------------------------------------------------- helpers

__device__ __forceinline__ uint32_t float_to_ordered(float f) {
    uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float ordered_to_float(uint32_t o) {
    uint32_t u = (o & 0x80000000u) ? (o & 0x7fffffffu) : ~o;
    return __uint_as_float(u);
}

// Philox4x64-10 (Salmon, Moraes, Dror, Shaw, SC 2011): key (k0, k1),
// counter c[0..3]; returns the four output words in c.
__device__ __forceinline__ void philox4x64_10(uint64_t c[4], uint64_t k0, uint64_t k1) {
    constexpr uint64_t kMul0 = 0xD2E7470EE14C6C93ull, kMul1 = 0xCA5A826395121157ull;
    constexpr uint64_t kBump0 = 0x9E3779B97F4A7C15ull, kBump1 = 0xBB67AE8584CAA73Bull;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t h0 = __umul64hi(kMul0, c[0]), l0 = kMul0 * c[0];
        const uint64_t h1 = __umul64hi(kMul1, c[2]), l1 = kMul1 * c[2];
        const uint64_t x0 = h1 ^ c[1] ^ k0, x2 = h0 ^ c[3] ^ k1;
        c[0] = x0;
        c[1] = l1;
        c[2] = x2;
        c[3] = l0;
        k0 += kBump0;
        k1 += kBump1;
    }
}

// smallest e with 2^e >= x (x > 0)
__device__ __forceinline__ int ceil_log2_pos(double x) {
    int e;
    const double m = frexp(x, &e);
    return m == 0.5 ? e - 1 : e;
}

// ------------------------------------------------------------ workspace

struct Plan {
    // problem
    int64_t nA, nB, T;
    int32_t d, metric, L, ke, kh, q, precision, window, reps, sampling;
    int32_t thr_copies;  // of the exact pass's thresholds (0: it keeps none)
    uint64_t seed;
    int log2cap;  // per-scale table capacity is 2^log2cap
    bool part;    // B's tables come from the partitioned build (W = 1)
    // byte offsets into the workspace
    size_t off_params, off_lohi, off_zfrac, off_mult, off_embed, off_tables, off_D,
        off_nn, off_scale, off_blocksums, off_P, off_idx, off_best, off_partial, off_nbh, off_bhalf,
        off_xhalf, off_xstat, off_gthr, off_part,
        off_bq, off_xq, off_lpf, total;
};

// Row block of the fixed-point scan: 256 threads x 4 items.
constexpr int kScanItems = 4;
constexpr int kScanThreads = 256;
constexpr int kScanBlock = kScanItems * kScanThreads;

// ------------------------------------------------------- block coordinates
// Every stage kernel is a device body over workgroup coordinates (id, n): a
// direct launch runs it with (blockIdx.x, gridDim.x); a batched launch runs
// the blocks of every request of a batch with request-local coordinates.
struct Blk {
    int64_t id, n;
};
__device__ __forceinline__ Blk grid_blk() { return Blk{(int64_t)blockIdx.x, (int64_t)gridDim.x}; }

// Work order of the exact passes (nq query blocks x nchunk chunks of B):
// workgroup ids are dealt to the 8 XCDs round-robin, so id runs on XCD
// id % 8 as its (id / 8)-th workgroup.  With nchunk a multiple of 8, XCD x
// takes the chunks cb = 8c + x in turn and, for each, all its query blocks
// one after the other: the workgroups of one chunk run on one XCD at about
// the same time and read the chunk through that XCD's L2 once.  Otherwise
// the chunk varies fastest.
__device__ __forceinline__ void chunk_major(int64_t id, int64_t nq, int nchunk, int &cb,
                                            int64_t &qb) {
    if ((nchunk & 7) == 0) {
        const int64_t s = id >> 3;
        cb = (int)((s / nq) * 8 + (id & 7));
        qb = s % nq;
    } else {
        cb = (int)(id % nchunk);
        qb = id / nchunk;
    }
}

// ---------------------------------------------------------------- batches
// One request of a batched estimate: its inputs, workspace regions, output
// slots and the block counts of each of its launches (the same counts its
// direct launch would use).
struct Job {
    const float *A, *B;
    int64_t nA, nB, T;
    uint64_t seed;
    int32_t d, metric, L, ke, kh, q, log2cap, precision;
    DevParams *p;
    uint32_t *lohi;
    float *zfrac;
    uint64_t *mult;
    const int8_t *embed;
    Bucket *tables;
    int64_t table_count;
    float *D;
    int32_t *nn;
    unsigned long long *blocksums, *P;  // block totals (then offsets); in-block prefixes
    int32_t *idx;
    unsigned long long *best;
    uint8_t *bq, *xq;  // low precision: cast B and draws
    float *lpf;
    uint16_t *bhalf, *xhalf;  // float32 l2: the FP16 tables of B and of the draws,
    float *nbh;               // -|y|^2 / 2 per row of B and the draws' norms
    float4 *xstat;
    uint32_t *gthr;  // float32 l2: thresholds of the exact pass
    int32_t thr_copies;
    int32_t nn_qw;  // l1: wavefronts of a workgroup with queries of their own
    int32_t nn_vector;  // the exact pass takes this job in the vector form (batch_vector)
    double *eta;
    chamfer_aux aux;
    // geometry
    int32_t nb_init, nb_grid, nb_fill;
    int32_t nb_mmA, nb_mmB, mm_wide;
    int64_t mm_strideA, mm_strideB;
    int32_t nb_hashB, nb_hashA, nb_scan, nb_sample;
    int32_t nb_castB, nb_castX, nn_nchunk, nb_nn;
    int64_t nn_chunk;
};

// Stages of a batched estimate, one launch each.
enum BatchStage {
    kBsSetup,   // parameter block, shifts and multipliers, empty tables
    kBsMinmax,  // per-coordinate min/max of A and of B
    kBsCalib,   // S and e_top
    kBsInsert,  // B into the tables
    kBsProbe,   // CrudeNN of A
    kBsWsum,    // fixed-point weights: block sums
    kBsWscan,   // scan of the block sums, W and s
    kBsSample,  // T draws
    kBsCast,    // low-precision copies, or the FP16 tables, of B and of the sampled rows
    kBsNN,      // exact nearest neighbours of the samples
    kBsFinal,   // eta and the per-request outputs
    kBsCount
};

constexpr int kBatchMax = 256;

struct alignas(16) Batch {
    int32_t njobs;
    int32_t pad[3];
    int32_t start[kBsCount][kBatchMax + 1];  // prefix of the jobs' block counts
    Job job[kBatchMax];
};

// Pointers read from a batch descriptor are generic to the compiler (flat
// loads and stores).  glb() states that one points to global memory, so the
// accesses compile as they do from a kernel argument; ro() also states that
// the memory is not written while the kernel runs, so loads at wave-uniform
// addresses go through the scalar cache (which every dispatch invalidates
// at its start).
template <class T>
__device__ __forceinline__ T *glb(T *p) {
    return (T *)(__attribute__((address_space(1))) T *)p;
}
#define CH_RO __attribute__((address_space(4)))
template <class T>
__device__ __forceinline__ const CH_RO T *ro(const T *p) {
    return (const CH_RO T *)p;
}
// 16-byte loads through such a pointer (HIP's vector classes cannot be
// copied out of another address space).
__device__ __forceinline__ float4 ld(const CH_RO float4 *p) {
    typedef float v4 __attribute__((ext_vector_type(4)));
    const v4 v = *reinterpret_cast<const CH_RO v4 *>(p);
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ uint4 ld(const CH_RO uint4 *p) {
    typedef unsigned v4 __attribute__((ext_vector_type(4)));
    const v4 v = *reinterpret_cast<const CH_RO v4 *>(p);
    return make_uint4(v.x, v.y, v.z, v.w);
}

// The centre of the l2 exact pass (d floats), in the words after the folded
// min/max.
__device__ __forceinline__ const CH_RO float *half_centre(const uint32_t *lohi, int d) {
    return ro(reinterpret_cast<const float *>(lohi + 2 * d));
}

// FP16 of v for the l2 exact pass, with subnormals replaced by zero (whatever
// the matrix cores do with them); a value beyond FP16's range returns its
// largest.  half_rest: the rounding error, infinite outside FP16's range.
__device__ __forceinline__ _Float16 half_of(float v) {
    const _Float16 h = (_Float16)fmaxf(fminf(v, 65504.0f), -65504.0f);
    return fabsf(v) < 6.103515625e-05f ? (_Float16)0.0f : h;
}
__device__ __forceinline__ float half_rest(float v, _Float16 h) {
    return fabsf(v) <= 65504.0f ? v - (float)h : INFINITY;
}
__device__ __forceinline__ uint32_t half_bits(_Float16 h) {
    return (uint32_t)__builtin_bit_cast(uint16_t, h);
}

// The l2 exact pass's score of a query z against a row y is within
// half_err_query(z) + half_err_row(y) of z.y - |y|^2 / 2.  Every term is a
// product of a query's and a row's magnitude or a square, and a product is split
// by 2 a b <= l a^2 + b^2 / l, so that a row far out costs itself a wide margin
// and no other row anything; for a query far out the products with the largest
// of the rows (by >= |y|, be >= |y - y~|) are less.  With zt >= |z~|, ze >= |z - z~| (half_stat), s2
// the computed |y|^2 and e2 the computed |y - y~|^2, u = 2^-24:
//   operands      zt |y - y~| + ze |y|, split with l near the
//                 ratio of an operand's rounding error to its size;
//   three products (d <= kHalfRawDim; slots 16 or 32): the dropped m m, and
//                 |y - y~| <= 1.1 2^-22 |y| + sqrt(d) 2^-14 in place of e2;
//   accumulation  of exact products into float32, from -|y|^2 / 2 on, every step
//                 with an error of at most 2 u of the partial sum;
//   |y|^2 / 2     (d + 8) u, and x - c, b - c u of their own.
struct HalfErr {
    float q2, e2q, q1;  // query: q2 zt^2 + e2q ze^2 + q1 zt,
    float p1;           // or zt (be + p1 by) + ze by + q1 zt, whichever is less
    float s2, e2;       // row: s2 |y|^2 + e2 |y - y~|^2
};
constexpr int kHalfRawDim = 10;
__host__ __device__ inline HalfErr half_err(int d, int slots) {
    constexpr float kU = 1.0f / 16777216.0f;
    const bool raw = d <= kHalfRawDim;
    const float split = raw ? 1.0f / 8388608.0f : 1.0f / 4096.0f;
    const float three = raw ? 2.12f / 4194304.0f : 0.0f;
    const float acc = (float)(slots + 8) * (kU * 2.2f), nrm = (float)(d + 9) * (kU * 1.1f);
    HalfErr h;  // (the factors also cover the roundings of these expressions)
    h.q2 = 0.50002f * (split + three + 1.02f * acc);
    h.e2q = 0.50002f / split;
    h.p1 = 1.00001f * (three + 1.02f * acc);
    h.q1 = raw ? sqrtf((float)d) * (1.01f / 16384.0f) : 0.0f;
    h.s2 = 0.51f * (split + three + 2.02f * acc + nrm) + 1e-9f;
    h.e2 = raw ? 0.0f : 0.51f / split;
    return h;
}
// -|y|^2 / 2 raised by the row's part of the bound: the score's first term.  A
// row outside FP16's range (half_scale; d <= kHalfRawDim: |y| above kHalfRawReach) has
// kHalfAlways, above any threshold; the maxima over B, and so every query's margin,
// are infinite then: thresholds come from canonical distances alone.
constexpr float kHalfAlways = 3e38f;
constexpr float kHalfRawReach = 63300.0f;
__device__ __forceinline__ float half_norm(float s2, float e2, float es2, float ee2) {
    return fmaf(e2, ee2, fmaf(s2, es2, -0.5f * s2));
}

// (|z|^2, |z| rounded up, |z - z~| rounded up, 0) from the float32 sums of
// squares of a row's coordinates and of their rounding errors (at most 256
// terms: relative error below 1.8e-5), the difference x - c included.
__device__ __forceinline__ float4 half_stat(float s2, float e2) {
    const float zn = sqrtf(s2 * 1.00004f) * 1.000001f + 1e-18f;
    return make_float4(s2, zn, sqrtf(e2 * 1.00004f) * 1.000001f + zn * 1.3e-7f, 0.0f);
}

// Canonical float32 accumulators of M pairs of rows x and b, each with LPH
// consecutive lanes: lane s holds coordinates [s S, (s + 1) S), S <= 16, of both
// rows (one batch of loads for all pairs) and continues the sum of lane s - 1, so
// the terms are added in coordinate order.  The results are in the last lane.
// All lanes must call it.
template <int METRIC, int LPH, int MAXD, int M>
__device__ __forceinline__ void hit_acc(const float *const *x, const float *const *b, int d,
                                        float *out) {
    constexpr int N = LPH == 1 ? MAXD : 16;  // coordinates per lane, at most
    // opaque: what follows from them is rare work whose lane masks must not be
    // hoisted into (and spilled around) the caller's tile loop
    int s = (threadIdx.x & 63) % LPH;
    asm volatile("" : "+v"(s), "+s"(d));
    const int S = LPH == 1 ? d : (d + 4 * LPH - 1) / (4 * LPH) * 4;
    const int k0 = s * S, k1 = min(d, k0 + S);
    float t[M][N];  // zero past the lane's coordinates: adds nothing
    uintptr_t low = 0;
#pragma unroll
    for (int m = 0; m < M; ++m)
        low |= reinterpret_cast<uintptr_t>(x[m]) | reinterpret_cast<uintptr_t>(b[m]);
    if (LPH > 1 && (d & 3) == 0 && (low & 15) == 0) {
        float4 u[M][N / 4 > 0 ? N / 4 : 1], v[M][N / 4 > 0 ? N / 4 : 1];
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
            for (int i = 0; i < N / 4; ++i) {
                const int k = max(min(k0 + 4 * i, d - 4), 0);
                u[m][i] = ld(reinterpret_cast<const CH_RO float4 *>(ro(x[m]) + k));
                v[m][i] = ld(reinterpret_cast<const CH_RO float4 *>(ro(b[m]) + k));
            }
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
            for (int i = 0; i < N / 4; ++i) {  // d, S multiples of 4: whole quads
                const bool in = k0 + 4 * i < k1;
                t[m][4 * i] = in ? u[m][i].x - v[m][i].x : 0.0f;
                t[m][4 * i + 1] = in ? u[m][i].y - v[m][i].y : 0.0f;
                t[m][4 * i + 2] = in ? u[m][i].z - v[m][i].z : 0.0f;
                t[m][4 * i + 3] = in ? u[m][i].w - v[m][i].w : 0.0f;
            }
    } else {
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const int k = min(k0 + i, d - 1);
                const float u = ro(x[m])[k] - ro(b[m])[k];
                t[m][i] = k0 + i < k1 ? u : 0.0f;
            }
    }
    // a loop, not unrolled: this code runs once or twice per workgroup and its
    // time is that of fetching its instructions
#pragma unroll
    for (int m = 0; m < M; ++m) out[m] = 0.0f;
#pragma unroll 1
    for (int q = 0; q < LPH; ++q) {
#pragma unroll
        for (int m = 0; m < M; ++m) {
            // the lane below's sum (row shift right by one: LPH <= 16 lanes of a row)
            float sum = LPH > 1 ? __uint_as_float(__builtin_amdgcn_update_dpp(
                                      0u, __float_as_uint(out[m]), 0x111, 0xf, 0xf, true))
                                : 0.0f;
            if (q == 0) sum = 0.0f;
#pragma unroll
            for (int i = 0; i < N; ++i)
                sum = METRIC == CHAMFER_L1 ? sum + fabsf(t[m][i]) : fmaf(t[m][i], t[m][i], sum);
            out[m] = s == q ? sum : out[m];
        }
    }
}

// Canonical float32 distance accumulator between rows a and b: k ascending,
// one rounding per operation; l1: acc + |a_k - b_k|, l2: fma(t, t, acc) with
// t = a_k - b_k (the caller takes the square root for l2).  Loads are issued
// in batches of BATCH x 16 bytes ahead of the (sequential) arithmetic, so a
// row costs a few memory round trips instead of one per 16 bytes (kernels
// with registers to spare take BATCH = 16: two round trips at d = 128).
// Both rows must be read-only for the kernel that calls it (they are read
// through the constant address space).
template <int METRIC, int BATCH = 8>
__device__ __forceinline__ float canon_acc(const float *__restrict__ a,
                                           const float *__restrict__ b, int d) {
    float acc = 0.0f;
    auto step = [&](float x, float y) {
        const float t = x - y;
        acc = METRIC == CHAMFER_L1 ? acc + fabsf(t) : fmaf(t, t, acc);
    };
    if ((d & 3) == 0 &&
        ((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b)) & 15) == 0) {
        const auto *a4 = reinterpret_cast<const CH_RO float4 *>(ro(a));
        const auto *b4 = reinterpret_cast<const CH_RO float4 *>(ro(b));
        const int d4 = d >> 2;
        constexpr int kBatch = BATCH;
        int k0 = 0;
        for (; k0 + kBatch <= d4; k0 += kBatch) {  // whole batches: no guards
            float4 u[kBatch], v[kBatch];
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
                u[i] = ld(a4 + k0 + i);
                v[i] = ld(b4 + k0 + i);
            }
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
                step(u[i].x, v[i].x);
                step(u[i].y, v[i].y);
                step(u[i].z, v[i].z);
                step(u[i].w, v[i].w);
            }
        }
        if (k0 < d4) {  // the last, partial batch: loads clamped in bounds
            float4 u[kBatch], v[kBatch];
#pragma unroll
            for (int i = 0; i < kBatch; ++i) {
                u[i] = ld(a4 + min(k0 + i, d4 - 1));
                v[i] = ld(b4 + min(k0 + i, d4 - 1));
            }
#pragma unroll
            for (int i = 0; i < kBatch; ++i)
                if (k0 + i < d4) {
                    step(u[i].x, v[i].x);
                    step(u[i].y, v[i].y);
                    step(u[i].z, v[i].z);
                    step(u[i].w, v[i].w);
                }
        }
        return acc;
    }
    constexpr int kBatch = 16;
    for (int k0 = 0; k0 < d; k0 += kBatch) {
        float u[kBatch], v[kBatch];
#pragma unroll
        for (int i = 0; i < kBatch; ++i)
            if (k0 + i < d) {
                u[i] = ro(a)[k0 + i];
                v[i] = ro(b)[k0 + i];
            }
#pragma unroll
        for (int i = 0; i < kBatch; ++i)
            if (k0 + i < d) step(u[i], v[i]);
    }
    return acc;
}

// Persistent loop of a batched stage: workgroup g takes the batch's blocks
// g, g + gridDim.x, ... of the stage (jobs in order, each job's blocks
// consecutive) and runs body(job, request-local coordinates).  The bodies
// have no barrier after a wave-dependent return, so the barrier that closes
// each iteration is reached by every wavefront.
template <class Body>
__device__ __forceinline__ void batch_loop(const Batch *__restrict__ bt, int stage, Body &&body) {
    __shared__ int32_t st[kBatchMax + 1];
    const int nj = bt->njobs;
    for (int i = threadIdx.x; i <= nj; i += blockDim.x) st[i] = bt->start[stage][i];
    __syncthreads();
    const int total = st[nj];
    int j = 0;
    for (int v = blockIdx.x; v < total; v += gridDim.x) {
        while (st[j + 1] <= v) ++j;
        j = __builtin_amdgcn_readfirstlane(j);
        body(bt->job[j], Blk{(int64_t)(v - st[j]), (int64_t)(st[j + 1] - st[j])});
        __syncthreads();
    }
}

// --------------------------------------------------------------- launchers
// All launchers enqueue on `st` and return hipGetLastError().

hipError_t launch_init_params(DevParams *p, uint32_t *lohi, int d, hipStream_t st);
// init_params, the rep-0 grid tables and (tables non-null) the empty W = 1
// tables of `count` buckets, in one launch
hipError_t launch_setup(DevParams *p, uint32_t *lohi, int d, uint64_t seed, int L, int kh,
                        float *zfrac, uint64_t *mult, Bucket *tables, size_t count,
                        hipStream_t st);
// rep: index of the independent LSH structure (0 for the single one)
hipError_t launch_grid_tables(uint64_t seed, int L, int kh, float *zfrac, uint64_t *mult,
                              int rep, hipStream_t st);
hipError_t launch_minmax(const float *X, int64_t n, int d, bool isB, uint32_t *lohi, DevParams *p,
                         hipStream_t st);
// The same over A and B in one launch (two when d > 2048).
hipError_t launch_minmax_pair(const float *A, int64_t nA, const float *B, int64_t nB, int d,
                              uint32_t *lohi, DevParams *p, hipStream_t st);
// B (may be null): also the centre and scale of the l2 exact pass
// (half_supported) or the corner and step of the l1 exact pass (sad_supported);
// X (may be null; rows[i], i < nx, of it if given): points that the queries are
// or are drawn from.  check: a non-finite coordinate sets the status, and the
// min/max holds X's points.
hipError_t launch_calib_final(uint32_t *lohi, int d, DevParams *p, const float *B, int64_t nB,
                              int metric, const float *X, const int32_t *rows, int64_t nx,
                              bool check, hipStream_t st);
hipError_t launch_table_fill(Bucket *tables, size_t count, hipStream_t st);
// mode 0: insert B into the tables; 1: probe A (CrudeNN); 2: write keys;
// 5: write B's keys for launch_part_build (duplicates within a wavefront
// dropped), of whose tables 1 takes the keys and, as half_dp, part_probe_bits; 3 / 4: insert / probe with a window of W points per bucket (the
// tables are then keys [L][cap] followed by members [L][cap][W]).  Modes 0, 3
// and 5 also write B's FP16 table of the l2 exact pass when half_out is set
// (with nbh_out and the maxima in p).  flags: kProbe*.
hipError_t launch_hash(int mode, const float *X, int64_t n, const float *Bpts, int64_t nB,
                       int d, int metric, int L, int ke, const uint32_t *lohi,
                       const int8_t *embed, const float *zfrac, const uint64_t *mult,
                       Bucket *tables, int log2cap, uint64_t *keys_out, float *D_out,
                       int32_t *nn_out, int32_t *scale_out, float *nbh_out, DevParams *p,
                       int W, int flags, hipStream_t st, uint16_t *half_out = nullptr,
                       int half_dp = 0);
// Bytes of the tables of L scales of 2^log2cap buckets with window W.
size_t table_bytes(int L, int log2cap, int W);
// The partitioned build of the W = 1 tables (no global atomics): keys of B
// from launch_hash mode 5 into w.keys, then launch_part_build.  Usable when
// part_build_ok(log2cap) (at most 1024 regions of 2^11 slots per scale;
// up to 20480 keys regions have up to 2^13).
struct PartWork {
    uint64_t *keys;    // [L][nB] (the empty key for a dropped duplicate)
    uint32_t *offs;    // [L][blocks][regions]
    uint32_t *bins;    // [L][regions][2]: first entry, count
    uint3 *entries;    // [L][nB] (key lo, key hi, b) grouped by region
};
bool part_build_ok(int log2cap);
// log2 of the slots that a probe of these tables goes round in.
int part_probe_bits(int64_t nB, int log2cap);
// Workspace bytes of the build; with w, also lays the regions out from base.
size_t part_work_bytes(int L, int64_t nB, int log2cap, PartWork *w = nullptr,
                       char *base = nullptr);
hipError_t launch_part_build(const PartWork &w, int64_t nB, int L, int log2cap, Bucket *tables,
                             hipStream_t st);
// Empty tables (window W).
hipError_t launch_tables_empty(Bucket *tables, int L, int log2cap, int W, hipStream_t st);
// Weights: per-block totals into blocksums (scanned in place to the blocks'
// offsets) and each point's in-block inclusive prefix into Ploc [n_A].
hipError_t launch_weights(const float *D, int64_t nA, int q, uint64_t *blocksums, uint64_t *Ploc,
                          DevParams *p, hipStream_t st);
// Draws from P_a = offs[a / kScanBlock] + Ploc_a (launch_weights' outputs;
// q as for launch_weights); best[l] and gthr[c T + l], c < copies, are reset.
hipError_t launch_sample(uint64_t seed, const uint64_t *Ploc, const uint64_t *offs, int64_t nA,
                         int64_t T, int q, int32_t *idx, unsigned long long *best, uint32_t *gthr,
                         int copies, DevParams *p, hipStream_t st);
hipError_t launch_estimate_final(const unsigned long long *best, const int32_t *idx,
                                 const float *D, int64_t T, int metric, DevParams *p,
                                 double *eta_out, chamfer_aux aux, hipStream_t st);
hipError_t launch_fill_u64(unsigned long long *p, int64_t n, unsigned long long v,
                           hipStream_t st);
// Exact nearest neighbours on the vector ALU (l1, and l2 outside the
// matrix-core dimensions).
hipError_t launch_nnmin(const float *X, const int32_t *rows, int64_t nx, const float *B,
                        int64_t nB, int d, int metric, unsigned long long *best, DevParams *p,
                        hipStream_t st);
// The l2 exact pass on the FP16 matrix cores (d <= 10 and 12 <= d <= 256),
// after launch_calib_final with B: for d >= 12 (half_tabled) launch_half_rows
// writes the tables (half_table_bytes) of B (unless the hash of B did: nbh,
// bs) and of the queries (rows X[rows[i]], i < nx, or X[i]; xs, stat), then
// launch_nnmin_half returns the canonical float32 minima.  seed (may be
// null): seed[row of X] bounds the query's distance from above.  best [nx] and
// gthr [copies][nx] (the thresholds known so far; may be null) start as all ones;
// copies is 8 (one per XCD) or 1.
// Copies for an estimate's draws (gthr lies in table space that is dead by then; the
// passes over all points take 8 up to 1024 points: 100 x 100000 x 20 87 us with one,
// 70 with 8, 4000 x 100000 x 20 150 and 175).  A few thousand queries are in use by
// all XCDs at once, and their thresholds lie on few cache lines: each XCD gets a
// copy, used through its own L2, unless B is large and the queries many, where a
// threshold known to all XCDs is worth more than the contention costs (exact pass
// of 2000 draws over 10^6 x 128 points: 605 us with 8 copies, 547 with 1; whole
// call with 300 draws over 3 10^5 x 128: 466 and 480).  With many queries the XCDs
// work on different ones at a time.
__host__ __device__ inline int half_copies(int64_t nx, int64_t nB) {
    return nx < 16384 && (nB < 262144 || nx < 1024) ? 8 : 1;
}
bool half_supported(int d, int metric);
bool half_pays(int64_t nx, int64_t nB, int d, bool seeded);  // against launch_nnmin
bool half_tabled(int d);
size_t half_table_bytes(int64_t n, int d);
int64_t half_row_blocks(int64_t n, int d, bool isB);
hipError_t launch_half_rows(const float *B, int64_t nB, uint16_t *bs, float *nbh, const float *X,
                            const int32_t *rows, int64_t nx, uint16_t *xs, float4 *stat, int d,
                            const uint32_t *lohi, DevParams *p, hipStream_t st);
hipError_t launch_nnmin_half(const float *X, const int32_t *rows, int64_t nx, const uint16_t *Xs,
                             const float4 *stat, const float *seed, const float *B,
                             const uint16_t *Bs, int64_t nB, int d, const float *nbh,
                             const uint32_t *lohi, unsigned long long *best, uint32_t *gthr,
                             int copies, DevParams *p, hipStream_t st);
// The l1 exact pass on byte differences (9 <= d <= 256), after launch_calib_final
// with B: returns the canonical float32 minima.  seed (may be null): seed[row of X]
// bounds the query's distance from above.  best [nx] and gthr [nx] (may be null)
// start as all ones.
constexpr int kSadMinDim = 8;
bool sad_supported(int d, int metric);
bool sad_pays(int64_t nx, int64_t nB, int d, bool seeded);  // against launch_nnmin
hipError_t launch_nnmin_sad(const float *X, const int32_t *rows, int64_t nx, const float *seed,
                            const float *B, int64_t nB, int d, const uint32_t *lohi,
                            unsigned long long *best, uint32_t *gthr, DevParams *p,
                            hipStream_t st);
// Low-precision (BF16 / FP8-E4M3) l2 nearest neighbours with float32 re-rank.
int lowp_dpad(int d, int precision);
bool lowp_supported(int d, int metric, int precision);
size_t lowp_row_bytes(int d, int precision);
hipError_t launch_cast_rows(int precision, const float *X, const int32_t *rows, int64_t n, int d,
                            uint8_t *out, float *scale, float *n2, const DevParams *p,
                            hipStream_t st);
hipError_t launch_nnmin_lowp(int precision, const uint8_t *Xq, const float *xsc, int64_t nx,
                             const float *X, const int32_t *rows, const uint8_t *Bq,
                             const float *bsc, const float *bn2, const float *B, int64_t nB,
                             int d, unsigned long long *best, const DevParams *p,
                             hipStream_t st);
hipError_t launch_nn_finalize(const unsigned long long *best, int64_t nx, int metric,
                              float *min_out, int32_t *arg_out, double *partial,
                              const DevParams *p, hipStream_t st);
hipError_t launch_sum_final(const double *partial, int64_t nparts, const DevParams *p,
                            double *out, hipStream_t st);
hipError_t launch_copy_status(const DevParams *p, int32_t *status_out, hipStream_t st);
// Uniform sampling: D_a = 1 for every a (nn, scale = -1 when given) and
// max D_a = 1.
hipError_t launch_unit_weights(float *D, int32_t *nn, int32_t *scale, int64_t nA, DevParams *p,
                               hipStream_t st);
int nn_finalize_blocks(int64_t nx);

// ------------------------------------------------------------ geometry
// Block counts of the direct launches, shared with the batched ones.
int64_t init_blocks(int d);
int64_t grid_table_blocks(int L, int kh);
int64_t table_fill_blocks(size_t count);
// minmax over n rows: the 16-byte form when wide (d <= 2048), stride in float4;
// else in elements.  batch: one of many jobs
void minmax_geom(int64_t n, int d, bool wide, int64_t *blocks, int64_t *stride,
                 bool batch = false);
bool minmax_wide(int d);
int64_t hash_blocks(int64_t n);
int64_t scan_blocks(int64_t nA);
int64_t sample_blocks(int64_t T);
int64_t cast_blocks(int64_t n);
struct NNGeom {
    int64_t blocks, chunk;
    int32_t nchunk;
};
// target: workgroups the split of B aims for (0: the direct-launch target)
NNGeom valu_geom(int64_t nx, int64_t nB, int d, int64_t target = 0);
// A launch has fewer than 2^32 threads: with chunks of B no longer than 65536 rows,
// 2 10^7 x 2 10^7 points are 2.4 10^7 workgroups of 256.  The launchers of the half
// and sad passes take their queries in parts of at most *_launch_queries.
constexpr int64_t kMaxLaunchWGs = 1 << 23;
int64_t half_launch_queries(int64_t nx, int64_t nB, int d);
int64_t sad_launch_queries(int64_t nx, int64_t nB, int d);
NNGeom half_geom(int64_t nx, int64_t nB, int d, int64_t target = 0);
NNGeom half_batch_geom(int64_t nx, int64_t nB, int d, int64_t target = 0);
NNGeom sad_geom(int64_t nx, int64_t nB, int d, int64_t target, int32_t &qw);
int64_t half_target_wgs(int d);  // the direct-launch target of half_geom
// Whether a job of a batch takes the vector form; batches of the dimensions where
// there is another one too (batch_both) launch both.
bool batch_both(int d, int metric);
bool batch_vector(int64_t T, int64_t nB, int d, int metric);
constexpr int64_t kValuTargetWGs = 4096;
NNGeom lowp_geom(int64_t nx, int64_t nB, int d, int precision);
constexpr int kMaxLdsL1Dim = 240;  // widest l1 tile staged in LDS by the hash

// --------------------------------------------------------- batched launches
// Each launches one persistent grid over every job of *bt (device memory);
// d, metric, ke and precision are the same for every job of the batch.
hipError_t launch_batch_setup(const Batch *bt, hipStream_t st);
hipError_t launch_batch_minmax(const Batch *bt, int d, hipStream_t st);
hipError_t launch_batch_calib(const Batch *bt, int d, hipStream_t st);
hipError_t launch_batch_hash(int mode, const Batch *bt, int d, int metric, int ke,
                             hipStream_t st);
hipError_t launch_batch_weights(const Batch *bt, hipStream_t st);
hipError_t launch_batch_sample(const Batch *bt, hipStream_t st);
hipError_t launch_batch_cast(const Batch *bt, int d, int precision, hipStream_t st);
hipError_t launch_batch_nn(const Batch *bt, int d, int metric, int precision, hipStream_t st);
hipError_t launch_batch_sad(const Batch *bt, int d, hipStream_t st);
hipError_t launch_batch_half_rows(const Batch *bt, hipStream_t st);
hipError_t launch_batch_half(const Batch *bt, int d, hipStream_t st);
hipError_t launch_batch_lowp(const Batch *bt, int d, int precision, hipStream_t st);
hipError_t launch_batch_final(const Batch *bt, int metric, hipStream_t st);

// Host side of batching (api.hip): validate a request and fill its job with
// the layout of chamfer_estimate in workspace ws; for l2, embed_host
// receives the packed embedding (embedding_packed, embed_bytes(d, ke)) that
// the caller must place at embed_dev before the batch runs.
int job_prepare(const float *A, const float *B, int64_t nA, int64_t nB, int32_t d,
                int32_t metric, double eps, int64_t T, uint64_t seed, const chamfer_opts *opts,
                void *ws, size_t ws_bytes, double *eta, chamfer_aux aux, const int8_t *embed_dev,
                int8_t *embed_host, Job *job);
// Block counts of every stage of a job.
void job_stage_blocks(const Job &job, int64_t out[kBsCount]);

// Host Philox4x64-10 (counter c, key (k0, k1); output in c), the quantised
// l2 -> l1 embedding matrix ([ke][d] int8) and its packed operand layout for
// the hash kernels (embed_bytes(d, ke) bytes).
void philox_host(uint64_t c[4], uint64_t k0, uint64_t k1);
void embedding_host(uint64_t seed, int d, int ke, int8_t *Z);
size_t embed_bytes(int d, int ke);
void embedding_packed(uint64_t seed, int d, int ke, int8_t *out);

// chamfer_estimate / chamfer_workspace_bytes with opts->reduction set.
size_t reduced_workspace_bytes(int64_t n_A, int64_t n_B, int32_t d, int32_t metric, double eps,
                               int64_t T, const chamfer_opts *opts);
int estimate_reduced(const float *A, const float *B, int64_t n_A, int64_t n_B, int32_t d,
                     int32_t metric, double eps, int64_t T, uint64_t seed, double *eta_out,
                     chamfer_aux *aux, const chamfer_opts *opts, void *ws, size_t ws_bytes,
                     void *stream);
// Re-split B for the exact pass of a job in a batch: the exact float32
// passes give the exact nearest neighbour for any split, so a batch shares
// one workgroup target among its jobs in proportion to their work instead
// of every job splitting B finely enough to fill the device alone.  The
// low-precision pass keeps the direct split (its candidates depend on it).
void job_share_nn(Job *jobs, int n);
// The launch sequence of a batched estimate (what a captured graph holds).
int launch_estimate_batch(const Batch *bt, int d, int metric, int ke, int precision,
                          hipStream_t st);

}  // namespace chamfer
