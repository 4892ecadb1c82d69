// CrudeNN on the GPU (the CrudeNN figure and the appendix lemma on the grid
// hash at every scale): scale calibration, per-scale shifts and key
// multipliers, the open-addressing bucket tables of B, and the probe of A
// that yields the first colliding scale, the candidate b and D_a.
//
// Layout: one workgroup of four wavefronts per tile of 64 consecutive
// points, one point per lane; the wavefronts split the scales.  The tile's
// hashed coordinates are staged in LDS with an odd row stride, so the
// per-lane reads of row p, coordinate k hit 64 distinct banks.  Shifts and
// multipliers are indexed only by the (wave-uniform) scale and coordinate,
// so they are read through the scalar cache.  B's keys are written once,
// [L][n_B], and its tables built from them region by region in LDS (the
// partitioned build below; the serving path and the window tables insert
// directly); A's keys are never written: they are recomputed scale by
// scale until the first hit.
#include <climits>

#include "internal.h"

namespace chamfer {

// ------------------------------------------------------------- parameters

__device__ __forceinline__ void init_params(DevParams *p, uint32_t *lohi, int d, Blk b) {
    const int64_t t = b.id * blockDim.x + threadIdx.x;
    if (t == 0) {
        p->status = CHAMFER_OK;
        p->e_top = 0;
        p->s = 0;
        p->all_zero = 0;
        p->nonfinite = 0;
        p->W = 0;
        p->S = 0.0;
        p->fallbacks = 0;
        p->he = 0;
        p->half_box = 0.0f;
        p->sad_inv = 0.0f;
        p->sad_in = 0;
    }
    for (int64_t k = t; k < kMaxRepl; k += b.n * blockDim.x) {
        p->max_d_rep[k * kReplStride] = 0u;
        p->half_rep[k * kReplStride] = 0u;
        p->half_rep[k * kReplStride + 1] = 0u;
    }
    if (lohi != nullptr)
        for (int64_t k = t; k < (int64_t)kLohiReps * 2 * d; k += b.n * blockDim.x)
            lohi[k] = (k % (2 * d)) < d ? 0xffffffffu : 0u;  // running min / max (ordered)
}

__global__ void k_init_params(DevParams *p, uint32_t *lohi, int d) {
    init_params(p, lohi, d, grid_blk());
}

int64_t init_blocks(int d) { return ((int64_t)kLohiReps * 2 * d + 255) / 256; }

hipError_t launch_init_params(DevParams *p, uint32_t *lohi, int d, hipStream_t st) {
    const int blocks = lohi ? (int)init_blocks(d) : 1;
    k_init_params<<<blocks, 256, 0, st>>>(p, lohi, d);
    return hipGetLastError();
}

// Key multipliers from the second Philox word: two odd 24-bit values.
__host__ __device__ inline uint64_t key_multipliers(uint64_t w1) {
    return ((w1 & 0xffffffull) | 1ull) | ((((w1 >> 32) & 0xffffffull) | 1ull) << 32);
}

// Shifts z'_ik (cell units, 24-bit lattice in [0,1)) and key multipliers
// M_ik from Philox4x64-10, counter (k, i, GRID, rep), key (seed, 0).
__device__ __forceinline__ void grid_tables(uint64_t seed, int L, int kh, float *zfrac,
                                            uint64_t *mult, int rep, Blk b) {
    const int t = (int)(b.id * blockDim.x + threadIdx.x);
    if (t >= L * kh) return;
    const int i = t / kh, k = t - i * kh;
    uint64_t c[4] = {(uint64_t)k, (uint64_t)i, (uint64_t)kPurposeGrid, (uint64_t)rep};
    philox4x64_10(c, seed, 0);
    zfrac[t] = ldexpf((float)(uint32_t)(c[0] >> 40), -24);
    mult[t] = key_multipliers(c[1]);
}

__global__ void k_grid_tables(uint64_t seed, int L, int kh, float *zfrac, uint64_t *mult,
                              int rep) {
    grid_tables(seed, L, kh, zfrac, mult, rep, grid_blk());
}

int64_t grid_table_blocks(int L, int kh) { return ((int64_t)L * kh + 255) / 256; }

hipError_t launch_grid_tables(uint64_t seed, int L, int kh, float *zfrac, uint64_t *mult,
                              int rep, hipStream_t st) {
    k_grid_tables<<<(unsigned)grid_table_blocks(L, kh), 256, 0, st>>>(seed, L, kh, zfrac, mult,
                                                                      rep);
    return hipGetLastError();
}

// Per-coordinate min and max over a point set, and a non-finite flag.  The
// flat element e has coordinate e mod d; the grid stride is a multiple of d,
// so every thread keeps one coordinate.  Min/max use integer atomics on an
// order-preserving encoding, whose result does not depend on their order.
// This form (4-byte loads) serves d > 2048 only.
__device__ __forceinline__ uint32_t *lohi_copy(uint32_t *lohi, int d, bool isB, int64_t id) {
    constexpr int kHalf = kLohiReps / 2;
    return lohi + ((isB ? kHalf : 0) + (int)(id % kHalf)) * 2 * (int64_t)d;
}

__global__ __launch_bounds__(256) void k_minmax(const float *__restrict__ X, int64_t total,
                                                int d, int64_t stride, bool isB, uint32_t *lohi,
                                                DevParams *p) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= stride) return;
    uint32_t lo = 0xffffffffu, hi = 0u;
    int bad = 0;
    for (int64_t e = g; e < total; e += stride) {
        const float v = ro(X)[e];
        bad |= !isfinite(v);
        const uint32_t o = float_to_ordered(v);
        lo = min(lo, o);
        hi = max(hi, o);
    }
    uint32_t *rep = lohi_copy(lohi, d, isB, blockIdx.x);
    const int k = (int)(g % d);
    atomicMin(&rep[k], lo);
    atomicMax(&rep[d + k], hi);
    if (bad) atomicOr(&p->nonfinite, 1u);
}

// Same with 16-byte loads, any d <= 2048 and any 4-byte aligned X: the
// elements before the first 16-byte boundary and after the last are taken by
// block 0, and thread g keeps the four coordinates (4 g + i + head) mod d of
// float4 g (the stride, in float4, is a multiple of d / gcd(d, 4)).  Small d
// would send a wavefront's LDS atomics to a few words, so the block's min/max
// is kept in C copies that lanes pick by id (minmax_copies) and folds them at
// the end.  d = 3, 2 10^5 rows: 19.2 us with 4-byte loads, see minmax_geom.
__host__ __device__ inline int minmax_copies(int d) {
    return d <= 16 ? 16 : d <= 32 ? 4 : d <= 64 ? 2 : 1;
}
inline size_t minmax_lds(int d) { return (size_t)minmax_copies(d) * 2 * d * sizeof(uint32_t); }

__device__ __forceinline__ void minmax4(const float *__restrict__ X, int64_t total, int d,
                                        int64_t stride4, bool isB, uint32_t *lohi, DevParams *p,
                                        Blk b) {
    extern __shared__ uint32_t sm[];
    const int C = minmax_copies(d);
    for (int i = threadIdx.x; i < C * 2 * d; i += blockDim.x) sm[i] = i < C * d ? 0xffffffffu : 0u;
    __syncthreads();
    uint32_t *mine_lo = sm + (threadIdx.x & (C - 1)) * d, *mine_hi = mine_lo + C * d;
    const int64_t head =
        min(total, (int64_t)(((16 - (reinterpret_cast<uintptr_t>(X) & 15)) & 15) >> 2));
    const int64_t total4 = (total - head) / 4;
    const auto *Xr = reinterpret_cast<const CH_RO float4 *>(ro(X) + head);
    const int64_t g = b.id * blockDim.x + threadIdx.x;
    uint32_t lo[4] = {0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu};
    uint32_t hi[4] = {0u, 0u, 0u, 0u};
    int bad = 0;
    auto take = [&](const float4 v) {
        const float c[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            bad |= !isfinite(c[i]);
            const uint32_t o = float_to_ordered(c[i]);
            lo[i] = min(lo[i], o);
            hi[i] = max(hi[i], o);
        }
    };
    if (g < stride4 && g < total4) {
        int64_t e = g;
        // up to 16 loads per thread (10^5 x 128 points: exactly 16) eight go
        // out together; on longer runs eight at a time was slower (10^6:
        // 0.21 -> 0.23 ms), so those keep four
        if (total4 <= 16 * stride4)
            for (; e + 7 * stride4 < total4; e += 8 * stride4) {
                float4 v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = ld(Xr + e + u * stride4);
#pragma unroll
                for (int u = 0; u < 8; ++u) take(v[u]);
            }
        for (; e + 3 * stride4 < total4; e += 4 * stride4) {
            const float4 v0 = ld(Xr + e), v1 = ld(Xr + e + stride4),
                         v2 = ld(Xr + e + 2 * stride4), v3 = ld(Xr + e + 3 * stride4);
            take(v0);
            take(v1);
            take(v2);
            take(v3);
        }
        for (; e < total4; e += stride4) take(ld(Xr + e));
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int k = (int)((4 * g + i + head) % d);
            atomicMin(&mine_lo[k], lo[i]);
            atomicMax(&mine_hi[k], hi[i]);
        }
    }
    // the ends: elements [0, head) and [head + 4 total4, total)
    if (b.id == 0 && (int64_t)threadIdx.x < total - 4 * total4) {
        const int64_t e =
            (int64_t)threadIdx.x < head ? (int64_t)threadIdx.x : 4 * total4 + threadIdx.x;
        const float v = ro(X)[e];
        bad |= !isfinite(v);
        const int k = (int)(e % d);
        atomicMin(&mine_lo[k], float_to_ordered(v));
        atomicMax(&mine_hi[k], float_to_ordered(v));
    }
    if (bad) atomicOr(&p->nonfinite, 1u);
    __syncthreads();
    uint32_t *rep = lohi_copy(lohi, d, isB, b.id);
    for (int i = threadIdx.x; i < 2 * d; i += blockDim.x) {
        const bool low = i < d;
        const uint32_t *s = low ? sm + i : sm + (C - 1) * d + i;
        uint32_t v = s[0];
        for (int c = 1; c < C; ++c) v = low ? min(v, s[c * d]) : max(v, s[c * d]);
        if (low) {
            if (v != 0xffffffffu) atomicMin(&rep[i], v);
        } else if (v != 0u) {
            atomicMax(&rep[i], v);
        }
    }
}

// Blocks [0, nbA) take A, the rest B.
__global__ __launch_bounds__(256) void k_minmax4(const float *__restrict__ A, int64_t totalA,
                                                 int64_t strideA, int64_t nbA,
                                                 const float *__restrict__ B, int64_t totalB,
                                                 int64_t strideB, int d, uint32_t *lohi,
                                                 DevParams *p) {
    const int64_t b = blockIdx.x;
    if (b < nbA)
        minmax4(A, totalA, d, strideA, false, lohi, p, Blk{b, nbA});
    else
        minmax4(B, totalB, d, strideB, true, lohi, p, Blk{b - nbA, (int64_t)gridDim.x - nbA});
}

bool minmax_wide(int d) { return d <= 2048; }

void minmax_geom(int64_t n, int d, bool wide, int64_t *blocks_out, int64_t *stride_out,
                 bool batch) {
    const int64_t total = n * (int64_t)d;
    int64_t blocks;
    if (wide) {
        // float4 per thread: 16 where a block ends with many global atomics
        // (2 d of them; 50000 x 64 points: 11.5 us with 4, 7.6 with 16), 4 for
        // small d, whose clouds are a few MB and would otherwise leave most of
        // the chip idle (the jobs of a batch fill it: 48 of 8000 x 16 15 us with 4, 9
        // with 16)
        const int64_t per = d >= 64 || batch ? 16 : d > 16 ? 8 : 4;
        const int64_t total4 = total / 4, p4 = (d & 3) == 0 ? d / 4 : (d & 1) == 0 ? d / 2 : d;
        blocks = (total4 + 256 * per - 1) / (256 * per);
        if (blocks > 1024) blocks = 1024;
        const int64_t min_blocks = (p4 + 255) / 256;
        if (blocks < min_blocks) blocks = min_blocks;
        *stride_out = (blocks * 256 / p4) * p4;
    } else {
        blocks = (total + 16383) / 16384;
        if (blocks > 2048) blocks = 2048;
        const int64_t min_blocks = (d + 255) / 256;
        if (blocks < min_blocks) blocks = min_blocks;
        *stride_out = (blocks * 256 / d) * d;
    }
    *blocks_out = blocks;
}

hipError_t launch_minmax(const float *X, int64_t n, int d, bool isB, uint32_t *lohi, DevParams *p,
                         hipStream_t st) {
    if (minmax_wide(d))
        return isB ? launch_minmax_pair(nullptr, 0, X, n, d, lohi, p, st)
                   : launch_minmax_pair(X, n, nullptr, 0, d, lohi, p, st);
    int64_t blocks, stride;
    minmax_geom(n, d, false, &blocks, &stride);
    k_minmax<<<(unsigned)blocks, 256, 0, st>>>(X, n * (int64_t)d, d, stride, isB, lohi, p);
    return hipGetLastError();
}

hipError_t launch_minmax_pair(const float *A, int64_t nA, const float *B, int64_t nB, int d,
                              uint32_t *lohi, DevParams *p, hipStream_t st) {
    if (!minmax_wide(d)) {
        hipError_t e = nA > 0 ? launch_minmax(A, nA, d, false, lohi, p, st) : hipSuccess;
        return e != hipSuccess || nB <= 0 ? e : launch_minmax(B, nB, d, true, lohi, p, st);
    }
    int64_t nbA = 0, sA = 0, nbB = 0, sB = 0;
    if (nA > 0) minmax_geom(nA, d, true, &nbA, &sA);
    if (nB > 0) minmax_geom(nB, d, true, &nbB, &sB);
    if (nbA + nbB == 0) return hipSuccess;
    k_minmax4<<<(unsigned)(nbA + nbB), 256, minmax_lds(d), st>>>(
        A, nA * (int64_t)d, sA, nbA, B, nB * (int64_t)d, sB, d, lohi, p);
    return hipGetLastError();
}

// Mean and ends of 16 values without a few that lie far from the others: where one
// half's range is more than 16 times the other's, of that other half.  (This code
// runs in one workgroup, once: its time is that of fetching its instructions.)
struct Sample {
    float mean, lo, hi;
};
__device__ __forceinline__ Sample sample16(const float (&v)[16]) {
    Sample h[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        h[j] = Sample{0.0f, INFINITY, -INFINITY};
#pragma unroll
        for (int i = 8 * j; i < 8 * j + 8; ++i) {
            h[j].mean += v[i] * 0.125f;
            h[j].lo = fminf(h[j].lo, v[i]);
            h[j].hi = fmaxf(h[j].hi, v[i]);
        }
    }
    const float r0 = (h[0].hi - h[0].lo) * 0.0625f, r1 = (h[1].hi - h[1].lo) * 0.0625f;
    if (r0 > 16.0f * r1 || !(r0 < INFINITY)) return h[1];
    if (r1 > 16.0f * r0 || !(r1 < INFINITY)) return h[0];
    return Sample{0.5f * h[0].mean + 0.5f * h[1].mean, fminf(h[0].lo, h[1].lo),
                  fmaxf(h[0].hi, h[1].hi)};
}

// The scale 2^he takes B's largest coordinate to [2^10, 2^11) (rows that were not
// in the min/max may be 2^5 times larger), less where A's largest would leave
// [0, 2^15).  reach: the bits it may give up before the others' operands (FP16 ends
// at 2^-14) lose what rules rows out.  Points further out than that are few or a
// cloud of their own, as samples tell (16 times theirs is kept in range): few are
// left outside FP16's range, each evaluated on its own (one row of B at 10^9 times
// the extent, exact 40000^2 x 3: 5.2 ms with all of them in range, 0.3 without it).
// Largest |x - c| of A and B (all), B (rows) and B's sample (typical).
struct HalfScale {
    int he;
    bool query;  // the queries' sample has to be looked at
};
__device__ __forceinline__ HalfScale half_scale(float all, float rows, float typical, int d,
                                                bool known) {
    const int reach = d <= kHalfRawDim ? 10 : 14;
    if (typical > 0.0f && !(rows <= ldexpf(typical, reach))) rows = ldexpf(typical, 4);
    const bool span = all > 0.0f && isfinite(all);
    if (!(rows > 0.0f && isfinite(rows)))  // B is one point, or not finite
        return HalfScale{span ? 14 - ilogbf(all) : 0, false};
    const int he = 10 - ilogbf(rows), least = span ? 14 - ilogbf(all) : INT_MIN;
    const bool query = !known || least < he - reach;
    return HalfScale{query ? he : min(he, least), query};
}

// Fold the kLohiReps copies of the running min/max into the first.  With B
// (d <= 256), also the centre and the scale of the l2 exact pass, or for l1 the
// corner and the step of the byte differences.  Both look at 16 rows spread over B.
// l2: c_k the mean of those (any c is valid; near the mean it keeps the operands, and
// so their rounding errors, small), and half_scale of what is found around c.  X (nx
// rows, or rows[i] of them): the queries, of which the min/max knows all (known) or
// none.  d <= kHalfRawDim: the corner distance of B's box from c bounds |y|
// (infinite where rows lie outside FP16's range).
__device__ __forceinline__ void fold_lohi(uint32_t *lohi, int d, DevParams *p,
                                          const float *__restrict__ B, int64_t nB, int metric,
                                          const float *__restrict__ X,
                                          const int32_t *__restrict__ rows, int64_t nx,
                                          bool known) {
    __shared__ uint32_t most[4];  // l2: half_scale's three, the queries' sample; l1: all, sample
    __shared__ float box[kHalfRawDim];
    if (threadIdx.x < 4) most[threadIdx.x] = 0u;
    __syncthreads();
    uint32_t mine[3] = {0u, 0u, 0u};
    float corner = 0.0f, low = 0.0f;  // l1: of coordinate threadIdx.x (d <= blockDim.x)
    for (int k = threadIdx.x; k < d; k += blockDim.x) {
        float c = 0.0f;
        float v[16];
        Sample e{};
        if (B) {
            // 16 rows in one batch of loads (the first row 16 times when nB < 16)
#pragma unroll
            for (int i = 0; i < 16; ++i) v[i] = ro(B)[(nB / 16) * i * d + k];
            e = sample16(v);
            c = isfinite(e.mean) ? e.mean : 0.0f;
        }
        uint32_t lo[2], hi[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            lo[h] = 0xffffffffu;
            hi[h] = 0u;
#pragma unroll
            for (int r = 0; r < kLohiReps / 2; ++r) {  // one batch of loads, with B's
                const uint32_t *rep = lohi + (size_t)(h * (kLohiReps / 2) + r) * 2 * d;
                lo[h] = min(lo[h], rep[k]);
                hi[h] = max(hi[h], rep[d + k]);
            }
        }
        lohi[k] = min(lo[0], lo[1]);
        lohi[d + k] = max(hi[0], hi[1]);
        if (B) {
            const float hb = ordered_to_float(hi[1]), lb = ordered_to_float(lo[1]);
            float m[3] = {0.0f, 0.0f, 0.0f};
            if (metric == CHAMFER_L1) {
                low = lb;
                corner = e.lo;
                m[0] = hb - lb;
                m[1] = e.hi - e.lo;
            } else {
                lohi[2 * d + k] = __float_as_uint(c);
                m[0] = fmaxf(ordered_to_float(max(hi[0], hi[1])) - c,
                             c - ordered_to_float(min(lo[0], lo[1])));
                m[1] = isfinite(hb) && isfinite(lb) ? fmaxf(hb - c, c - lb) : INFINITY;
                m[2] = fmaxf(e.hi - c, c - e.lo);
                if (k < kHalfRawDim) box[k] = m[1];
            }
#pragma unroll
            for (int i = 0; i < 3; ++i) mine[i] = max(mine[i], __float_as_uint(fabsf(m[i])));
        }
    }
    if (B) {
        for (int off = 32; off > 0; off >>= 1)
#pragma unroll
            for (int i = 0; i < 3; ++i)
                mine[i] = max(mine[i], (uint32_t)__shfl_xor((int)mine[i], off));
        if ((threadIdx.x & 63) == 0)
#pragma unroll
            for (int i = 0; i < 3; ++i)
                if (mine[i] != 0u) atomicMax(&most[i], mine[i]);
    }
    __syncthreads();
    if (B == nullptr) return;
    const float all = __uint_as_float(most[0]), some = __uint_as_float(most[1]);
    if (metric == CHAMFER_L1) {
        // MB: the widest of the sampled rows, M: of all.  Rows far out would make
        // the steps too wide for all others: beyond 8 to 1 the box is that of the
        // samples and half their width around it, and rows outside are clamped
        const float M = all, MB = some;
        const bool every = !(M > 8.0f * MB) || MB == 0.0f;
        if ((int)threadIdx.x < d)
            lohi[2 * d + threadIdx.x] =
                __float_as_uint(every ? low : fmaxf(low, corner - 0.5f * MB));
        if (threadIdx.x == 0) {
            const float inv = 254.9997f / (every ? M : 2.0f * MB);
            p->sad_inv = inv > 0.0f && inv < 1e30f ? inv : 0.0f;
            p->sad_in = every;
        }
        return;
    }
    HalfScale sc = half_scale(all, some, __uint_as_float(most[2]), d, known);
    if (sc.query && X && nx > 0) {  // (uniform)
        for (int k = threadIdx.x; k < d; k += blockDim.x) {
            const float c = __uint_as_float(lohi[2 * d + k]);  // (this thread's store)
            float q[2] = {0.0f, 0.0f};  // of the nearer half
#pragma unroll 1
            for (int i = 0; i < 16; i += 8) {
                float w[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int64_t r = (nx / 16) * (i + j);
                    w[j] = ro(X)[(rows ? (int64_t)ro(rows)[r] : r) * d + k];
                }
#pragma unroll
                for (int j = 0; j < 8; ++j) q[1] = fmaxf(q[1], fabsf(w[j] - c));
                if (i == 0) q[0] = q[1], q[1] = 0.0f;
            }
            atomicMax(&most[3], __float_as_uint(fminf(q[0], q[1])));
        }
        __syncthreads();
        const float far = __uint_as_float(most[3]);
        if (far > 0.0f && isfinite(far)) sc.he = min(sc.he, (known ? 10 : 12) - ilogbf(far));
    }
    if (threadIdx.x == blockDim.x - 1) {
        const int he = sc.he;
        p->he = he;
        if (d <= kHalfRawDim) {
            float s = 0.0f;
            for (int k = 0; k < d; ++k) {
                const float y = ldexpf(box[k], he);
                s = fmaf(y, y, s);
            }
            const float by = sqrtf(s) * 1.00001f;
            p->half_box = by < kHalfRawReach ? by : INFINITY;
        }
    }
}

__global__ void k_calib_final_wide(uint32_t *lohi, int d, DevParams *p, bool check) {
    fold_lohi(lohi, d, p, nullptr, 0, 0, nullptr, nullptr, 0, false);
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    double S = 0.0;
    for (int k = 0; k < d; ++k)
        S = S + ((double)ordered_to_float(lohi[d + k]) - (double)ordered_to_float(lohi[k]));
    p->S = S;
    p->e_top = S > 0.0 ? ceil_log2_pos(S) : 0;
    if (check && p->nonfinite) p->status = CHAMFER_ENONFINITE;
}

// S = sum_k (hi_k - lo_k) in double, k ascending; e_top = ceil(log2 S).
// The per-coordinate spans are gathered in parallel; one thread sums them
// in order.
__device__ __forceinline__ void calib_final(uint32_t *lohi, int d, DevParams *p,
                                            const float *__restrict__ B, int64_t nB, int metric,
                                            const float *__restrict__ X,
                                            const int32_t *__restrict__ rows, int64_t nx,
                                            bool check) {
    extern __shared__ double span[];
    fold_lohi(lohi, d, p, B, nB, metric, X, rows, nx, check);
    __syncthreads();
    for (int k = threadIdx.x; k < d; k += blockDim.x)
        span[k] = (double)ordered_to_float(lohi[d + k]) - (double)ordered_to_float(lohi[k]);
    __syncthreads();
    if (threadIdx.x != 0) return;
    double S = 0.0;
    for (int k = 0; k < d; k += 8) {  // in order; the reads of eight go out together
        double v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = span[min(k + i, d - 1)];
#pragma unroll
        for (int i = 0; i < 8; ++i) S = S + (k + i < d ? v[i] : 0.0);
    }
    p->S = S;
    p->e_top = S > 0.0 ? ceil_log2_pos(S) : 0;
    if (check && p->nonfinite) p->status = CHAMFER_ENONFINITE;
}

__global__ __launch_bounds__(256) void k_calib_final(uint32_t *lohi, int d, DevParams *p,
                                                     const float *__restrict__ B, int64_t nB,
                                                     int metric, const float *__restrict__ X,
                                                     const int32_t *__restrict__ rows, int64_t nx,
                                                     bool check) {
    calib_final(lohi, d, p, B, nB, metric, X, rows, nx, check);
}

hipError_t launch_calib_final(uint32_t *lohi, int d, DevParams *p, const float *B, int64_t nB,
                              int metric, const float *X, const int32_t *rows, int64_t nx,
                              bool check, hipStream_t st) {
    if ((size_t)d * sizeof(double) > 60000) {
        // very wide points: spans recomputed by the summing thread
        if (B != nullptr) return hipErrorInvalidValue;
        k_calib_final_wide<<<1, 64, 0, st>>>(lohi, d, p, check);
        return hipGetLastError();
    }
    if (B != nullptr && nB < 1) return hipErrorInvalidValue;
    k_calib_final<<<1, 256, (size_t)d * sizeof(double), st>>>(lohi, d, p, B, nB, metric, X, rows, nx,
                                                              check);
    return hipGetLastError();
}

// Empty W = 1 tables: `count` buckets (key EMPTY, value INT_MAX), then the
// count fingerprint bytes that follow them (0 = empty slot).
__device__ __forceinline__ void table_fill(Bucket *t, size_t count, Blk b) {
    const size_t stride = (size_t)b.n * blockDim.x;
    for (size_t i = (size_t)b.id * blockDim.x + threadIdx.x; i < count; i += stride) {
        Bucket b;
        b.key = kEmptyKey;
        b.val = INT_MAX;
        b.pad = 0;
        t[i] = b;
    }
    uint4 *fp = reinterpret_cast<uint4 *>(t + count);
    for (size_t i = (size_t)b.id * blockDim.x + threadIdx.x; i < count / 16; i += stride)
        fp[i] = make_uint4(0u, 0u, 0u, 0u);
}

__global__ void k_table_fill(Bucket *t, size_t count) { table_fill(t, count, grid_blk()); }

int64_t table_fill_blocks(size_t count) {
    size_t blocks = (count + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    return (int64_t)blocks;
}

// Parameter block, lo/hi, shifts and multipliers of structure 0 and (tables
// non-null) the empty W = 1 tables in one launch: the three independent
// bodies over consecutive block ranges.
__global__ __launch_bounds__(256) void k_setup(DevParams *p, uint32_t *lohi, int d, uint64_t seed,
                                               int L, int kh, float *zfrac, uint64_t *mult,
                                               Bucket *tables, size_t count, int nb_init,
                                               int nb_grid, int nb_fill) {
    const int64_t b = blockIdx.x;
    if (b < nb_init) {
        init_params(p, lohi, d, Blk{b, nb_init});
    } else if (b < nb_init + nb_grid) {
        grid_tables(seed, L, kh, zfrac, mult, 0, Blk{b - nb_init, nb_grid});
    } else {
        table_fill(tables, count, Blk{b - nb_init - nb_grid, nb_fill});
    }
}

hipError_t launch_setup(DevParams *p, uint32_t *lohi, int d, uint64_t seed, int L, int kh,
                        float *zfrac, uint64_t *mult, Bucket *tables, size_t count,
                        hipStream_t st) {
    const int nb_init = (int)init_blocks(d), nb_grid = (int)grid_table_blocks(L, kh);
    const int nb_fill = tables ? (int)table_fill_blocks(count) : 0;
    k_setup<<<(unsigned)(nb_init + nb_grid + nb_fill), 256, 0, st>>>(
        p, lohi, d, seed, L, kh, zfrac, mult, tables, count, nb_init, nb_grid, nb_fill);
    return hipGetLastError();
}

hipError_t launch_table_fill(Bucket *tables, size_t count, hipStream_t st) {
    k_table_fill<<<(unsigned)table_fill_blocks(count), 256, 0, st>>>(tables, count);
    return hipGetLastError();
}

// ------------------------------------------------------------------ keys

// Key of hashed coordinates y (stride 1) at the scale of side 2^e:
// cell_k = floor(fma(y_k, 2^-e, z'_k)) as an int32 (y_k 2^-e is exact, so one
// rounding, of the sum), K1 = sum_k (cell_k mod 2^24) M1_k mod 2^32, K2 the
// same with M2_k, key = (K1 2^32 + K2) >> 1; M_k = M1_k | M2_k << 32 (odd
// 24-bit multipliers).  Four VALU operations per coordinate: one fma, the
// floor conversion and two 24-bit multiply-adds.  CLAMP: saturate the
// shifted coordinate at the int32 range first (NaN to the upper bound);
// needed only when a cell index can leave that range: more than 30 scales,
// or sides below 2^-126 (2^-e not finite).  Sums are mod 2^32 and split
// over two accumulator pairs to shorten the dependent chains.
template <bool CLAMP>
__device__ __forceinline__ uint32_t cell24(float q) {
    if (CLAMP) q = fmaxf(fminf(q, 2147483520.0f), -2147483648.0f);
    return (uint32_t)(int32_t)floorf(q);
}

template <bool CLAMP, class PZ, class PM>
__device__ __forceinline__ unsigned long long bucket_key(const float *y, int kh, int e, PZ zf,
                                                         PM M) {
    const float p = ldexpf(1.0f, -e);
    uint32_t a1 = 0, a2 = 0, b1 = 0, b2 = 0;
    int k = 0;
    for (; k + 2 <= kh; k += 2) {
        const uint32_t c0 = cell24<CLAMP>(fmaf(y[k], p, zf[k]));
        const uint32_t c1 = cell24<CLAMP>(fmaf(y[k + 1], p, zf[k + 1]));
        const unsigned long long m0 = M[k], m1 = M[k + 1];
        a1 += __umul24(c0, (uint32_t)m0);
        a2 += __umul24(c0, (uint32_t)(m0 >> 32));
        b1 += __umul24(c1, (uint32_t)m1);
        b2 += __umul24(c1, (uint32_t)(m1 >> 32));
    }
    if (k < kh) {
        const uint32_t c0 = cell24<CLAMP>(fmaf(y[k], p, zf[k]));
        const unsigned long long m0 = M[k];
        a1 += __umul24(c0, (uint32_t)m0);
        a2 += __umul24(c0, (uint32_t)(m0 >> 32));
    }
    return (((unsigned long long)(a1 + b1) << 32) | (unsigned long long)(a2 + b2)) >> 1;
}

// Same, with y_k = x_k - lo_k read from HBM (l1 with d too large for LDS).
template <bool CLAMP, class PX, class PL, class PZ, class PM>
__device__ __forceinline__ unsigned long long bucket_key_global(PX x, PL lohi, int kh, int e,
                                                                PZ zf, PM M) {
    const float p = ldexpf(1.0f, -e);
    uint32_t a1 = 0, a2 = 0;
    for (int k = 0; k < kh; ++k) {
        const float y = x[k] - ordered_to_float(lohi[k]);
        const uint32_t c = cell24<CLAMP>(fmaf(y, p, zf[k]));
        const unsigned long long m = M[k];
        a1 += __umul24(c, (uint32_t)m);
        a2 += __umul24(c, (uint32_t)(m >> 32));
    }
    return (((unsigned long long)a1 << 32) | (unsigned long long)a2) >> 1;
}

// Home slot: the top bits of the key times an odd 64-bit constant (the
// golden-ratio multiplier), which carries the well-mixed low bits of the two
// 32-bit sums into the top (the top bits of a sum of small cells times
// 24-bit multipliers are not uniform by themselves).  The fingerprint of a
// key is the next 8 bits of the same product, 0 mapped to 1 (0 marks an
// empty slot in the fingerprint bytes that follow a W = 1 table).
__device__ __forceinline__ uint64_t home_slot(unsigned long long key, int log2cap) {
    return (uint64_t)((key * 0x9E3779B97F4A7C15ull) >> (64 - log2cap));
}

__device__ __forceinline__ uint32_t key_fp(unsigned long long key, int log2cap) {
    const uint32_t f = (uint32_t)((key * 0x9E3779B97F4A7C15ull) >> (56 - log2cap)) & 0xffu;
    return f ? f : 1u;
}

// Fingerprint bytes of scale i of W = 1 tables of 2^log2cap buckets per scale.
__device__ __forceinline__ uint8_t *table_fps(Bucket *tables, int L, int log2cap, int i) {
    return reinterpret_cast<uint8_t *>(tables + ((size_t)L << log2cap)) + ((size_t)i << log2cap);
}

// Insert (key -> b) keeping the lowest b per key.  Linear probing; a slot's
// key changes only from EMPTY, by CAS, so each key owns exactly one slot,
// and the lane that claims it writes the key's fingerprint byte.  The slot
// is read first, so a key already present costs a load (and an atomicMin
// only when b is lower than the stored value).
__device__ void table_insert(Bucket *tab, uint8_t *fps, int log2cap, unsigned long long key,
                             int b) {
    const uint64_t mask = (1ull << log2cap) - 1;
    uint64_t slot = home_slot(key, log2cap);
    for (;;) {
        Bucket *e = tab + slot;
        unsigned long long cur =
            __hip_atomic_load(&e->key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (cur == kEmptyKey) {
            const unsigned long long prev = atomicCAS(&e->key, kEmptyKey, key);
            if (prev == kEmptyKey || prev == key) {
                if (prev == kEmptyKey) fps[slot] = (uint8_t)key_fp(key, log2cap);
                atomicMin(&e->val, b);
                return;
            }
            cur = prev;
        }
        if (cur == key) {
            if (__hip_atomic_load(&e->val, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > b)
                atomicMin(&e->val, b);
            return;
        }
        slot = (slot + 1) & mask;
    }
}

// Lowest b stored under key, or -1.  Runs in a later kernel than every
// insert.  The probe walks the fingerprint bytes, 16 per load, and reads a
// bucket only where the fingerprint matches: a missing key (most probes
// below a point's first colliding scale) touches only the fingerprints,
// 1/16 of the table's bytes.  It goes round within the 2^rbits slots around
// the home slot (the whole table, or a region of launch_part_build).  A region
// that holds no empty slot may have had no room for a key: the scale's keys
// (nB of them, ascending b) are searched instead.
__device__ __forceinline__ int table_probe(const CH_RO Bucket *tab, const CH_RO uint8_t *fps,
                                           int log2cap, int rbits, unsigned long long key,
                                           const CH_RO unsigned long long *keys, int64_t nB) {
    const uint64_t mask = (1ull << rbits) - 1;
    const uint32_t f = key_fp(key, log2cap);
    uint64_t slot = home_slot(key, log2cap);
    const uint64_t region = slot & ~mask, first = slot & ~15ull;
    do {
        const uint64_t base = slot & ~15ull;
        const uint4 w = ld(reinterpret_cast<const CH_RO uint4 *>(fps + base));
        for (int q = (int)(slot - base); q < 16; ++q) {
            const uint32_t word = q < 4 ? w.x : q < 8 ? w.y : q < 12 ? w.z : w.w;
            const uint32_t byte = (word >> (8 * (q & 3))) & 0xffu;
            if (byte == 0) return -1;
            if (byte == f) {
                const uint4 bk = ld(reinterpret_cast<const CH_RO uint4 *>(tab + base + q));
                const unsigned long long k =
                    (unsigned long long)bk.x | ((unsigned long long)bk.y << 32);
                if (k == key) return (int)bk.z;
            }
        }
        slot = region | ((base + 16) & mask);
    } while (slot != first);
    if (keys != nullptr)
        for (int64_t b = 0; b < nB; ++b)
            if (keys[b] == key) return (int)b;
    return -1;
}

// Window tables (multi-probe CrudeNN): a bucket holds its key and the W
// smallest b inserted under it, ascending, INT_MAX for empty positions.
// W smallest suffice: a probe that has seen s < W points at finer scales
// needs W - s unseen points of the bucket, and at most s of its W smallest
// are seen, so the W - s smallest unseen ones are among them.
// The insert runs b through the W positions as a chain of atomicMin: each
// position keeps the smaller of its value and the incoming one and passes
// the larger on, so position j ends with the (j+1)-th smallest b inserted,
// whatever the interleaving.  A position already below b is skipped (values
// only decrease), and an empty position ends the chain.
__device__ void wide_insert(unsigned long long *keys, int *mem, int log2cap,
                            unsigned long long key, int b, int W) {
    const uint64_t mask = (1ull << log2cap) - 1;
    uint64_t slot = home_slot(key, log2cap);
    for (;;) {
        unsigned long long cur =
            __hip_atomic_load(&keys[slot], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (cur == kEmptyKey) {
            const unsigned long long prev = atomicCAS(&keys[slot], kEmptyKey, key);
            if (prev == kEmptyKey || prev == key) break;
            cur = prev;
        }
        if (cur == key) break;
        slot = (slot + 1) & mask;
    }
    int *m = mem + slot * (uint64_t)W;
    int x = b;
    for (int j = 0; j < W; ++j) {
        if (__hip_atomic_load(&m[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < x) continue;
        const int old = atomicMin(&m[j], x);
        if (old == INT_MAX) return;  // x took an empty position
        x = max(old, x);             // the larger one moves on
    }
}

// Bucket index of key in a window table, or -1.
__device__ __forceinline__ int64_t wide_find(const CH_RO unsigned long long *keys, int log2cap,
                                             unsigned long long key) {
    const uint64_t mask = (1ull << log2cap) - 1;
    uint64_t slot = home_slot(key, log2cap);
    for (;;) {
        const unsigned long long k = keys[slot];
        if (k == key) return (int64_t)slot;
        if (k == kEmptyKey) return -1;
        slot = (slot + 1) & mask;
    }
}

// Canonical float32 distance (square root of the accumulator for l2).
template <int METRIC>
__device__ __forceinline__ float dist32(const float *__restrict__ a, const float *__restrict__ b,
                                        int d) {
    const float acc = canon_acc<METRIC, 4>(a, b, d);
    return METRIC == CHAMFER_L1 ? acc : sqrtf(acc);
}

constexpr int kTile = 64;        // points per workgroup
constexpr int kWaves = 4;        // wavefronts per workgroup; they split the scales
constexpr int kThreads = 64 * kWaves;
constexpr int kEmbedChunk = 64;  // coordinates of x - lo staged per pass (l2), by default

// Copy rows [np][kc] of the tile (row stride d, from column k0) into LDS
// rows of stride ldr, less lo_k (the ordered-int lower corner) when lo is
// given: each thread issues a batch of loads before it stores any of them,
// so a tile costs a few memory round trips instead of one per element.  The
// loads are in bounds and unconditional (rows past np and elements past the
// tile read its last element, and are not stored), so the batch is in flight
// at once; in the float4 form a thread always takes the same quad of
// columns, whose lo it loads once, first.
template <int BATCH>
__device__ __forceinline__ void stage_rows(const float *__restrict__ X, int64_t p0, int np, int d,
                                           int k0, int kc, float *dst, int ldr,
                                           const uint32_t *__restrict__ lo) {
    const auto *Xr = ro(X);
    if (kc == 64 && (d & 3) == 0 && (k0 & 3) == 0 &&
        (reinterpret_cast<uintptr_t>(X) & 15) == 0) {
        // 64 coordinates per row as 16 float4 loads (row r, quad c of
        // element e: r = e / 16, c = e % 16 = thread % 16), four per thread
        // in one batch
        const auto *X4 = reinterpret_cast<const CH_RO float4 *>(Xr);
        constexpr int kRowsPerPass = kThreads / 16;
        const int c = (int)threadIdx.x & 15, r0 = (int)threadIdx.x >> 4;
        // without lo the quad is read from X itself and not used
        const bool sub = lo != nullptr;
        const auto *lr = sub ? ro(lo) + k0 + 4 * c : ro(reinterpret_cast<const uint32_t *>(X));
        const uint32_t l0 = lr[0], l1 = lr[1], l2 = lr[2], l3 = lr[3];
        float4 v[kTile * 16 / kThreads];
#pragma unroll
        for (int i = 0; i < kTile * 16 / kThreads; ++i) {
            const int r = min(i * kRowsPerPass + r0, np - 1);
            v[i] = ld(X4 + (((p0 + r) * d + k0) >> 2) + c);
        }
        const float4 off = sub ? make_float4(ordered_to_float(l0), ordered_to_float(l1),
                                             ordered_to_float(l2), ordered_to_float(l3))
                               : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
        for (int i = 0; i < kTile * 16 / kThreads; ++i) {
            const int r = i * kRowsPerPass + r0;
            if (r < np) {
                float *o = dst + r * ldr + 4 * c;
                o[0] = v[i].x - off.x;
                o[1] = v[i].y - off.y;
                o[2] = v[i].z - off.z;
                o[3] = v[i].w - off.w;
            }
        }
        return;
    }
    const int total = np * kc;
    const bool sub = lo != nullptr;
    const auto *lr = sub ? ro(lo) + k0 : ro(reinterpret_cast<const uint32_t *>(X));
    for (int base = 0; base < total; base += BATCH * kThreads) {
        float v[BATCH];
        uint32_t o[BATCH];
#pragma unroll
        for (int i = 0; i < BATCH; ++i) {
            const int e = min(base + i * kThreads + (int)threadIdx.x, total - 1);
            const int r = e / kc, k = e - r * kc;
            v[i] = Xr[(p0 + r) * d + k0 + k];
            o[i] = lr[sub ? k : 0];
        }
#pragma unroll
        for (int i = 0; i < BATCH; ++i) {
            const int e = base + i * kThreads + (int)threadIdx.x;
            if (e < total) {
                const int r = e / kc, k = e - r * kc;
                dst[r * ldr + k] = v[i] - (sub ? ordered_to_float(o[i]) : 0.0f);
            }
        }
    }
}

// Probe grids of at least this many tiles compute the candidate distances
// with all four wavefronts (l2, d = 128, tile_dist against the gather by
// wavefront 0: gather faster by 10% at 1563 tiles and 4% at 3907, tile_dist
// faster by 1% at 6250 tiles and 4% at 15625; quad_dist 2% faster again at
// 15625, and 8% for l1 at d = 64).
constexpr int64_t kCoopDistTiles = 5000;

// Canonical float32 distance of each point of the tile to its candidate row
// cand[p] of B (an LDS list; rows past np are never used): the workgroup
// stages t = x_k - b_k for 64 coordinates of all points at a time into LDS
// (rows read whole by consecutive lanes, both rows of a point in one batch
// of loads; when d is a multiple of 64 the next chunk's loads are in flight
// while the current one is summed), and lane p of wavefront 0 adds point p's
// terms in coordinate order, so the result is the one dist32 computes.  tb:
// LDS of kTile rows of (min(d, 64) | 1) floats.  Every thread of the
// workgroup must call it; the distance is returned in wavefront 0's lanes.
template <int METRIC>
__device__ __forceinline__ float tile_dist(const float *__restrict__ X, int64_t p0, int np, int d,
                                           const float *__restrict__ Bpts, const int *cand,
                                           float *tb) {
    const auto *Xr = ro(X);
    const auto *Br = ro(Bpts);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ldt = min(d, 64) | 1;
    float acc = 0.0f;
    auto term = [&](float t) { acc = METRIC == CHAMFER_L1 ? acc + fabsf(t) : fmaf(t, t, acc); };
    if ((d & 63) == 0) {
        // element (row 4 i + wave, coordinate lane): rows are wave-uniform
        constexpr int kPer = kTile * 64 / kThreads;
        float a[kPer], b[kPer];
        auto load = [&](int k0) {
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                const int r = min(kThreads / 64 * i + wave, np - 1);
                const int c = __builtin_amdgcn_readfirstlane(cand[r]);
                a[i] = Xr[(p0 + r) * d + k0 + lane];
                b[i] = Br[(int64_t)c * d + k0 + lane];
            }
        };
        load(0);
        for (int k0 = 0; k0 < d; k0 += 64) {
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                const int r = kThreads / 64 * i + wave;
                if (r < np) tb[r * ldt + lane] = a[i] - b[i];
            }
            __syncthreads();
            if (k0 + 64 < d) load(k0 + 64);
            if (wave == 0 && lane < np) {
                const float *t = tb + lane * ldt;
#pragma unroll
                for (int k = 0; k < 64; k += 16) {
                    float v[16];
#pragma unroll
                    for (int j = 0; j < 16; ++j) v[j] = t[k + j];
#pragma unroll
                    for (int j = 0; j < 16; ++j) term(v[j]);
                }
            }
            __syncthreads();
        }
    } else {
        constexpr int kPer = 8;  // elements per thread per batch
        float a[kPer], b[kPer];
        for (int k0 = 0; k0 < d; k0 += 64) {
            const int kc = min(64, d - k0);
            const int total = np * kc;
            for (int base = 0; base < total; base += kPer * kThreads) {
#pragma unroll
                for (int i = 0; i < kPer; ++i) {
                    const int e = min(base + i * kThreads + (int)threadIdx.x, total - 1);
                    const int r = e / kc, k = e - r * kc;
                    a[i] = Xr[(p0 + r) * d + k0 + k];
                    b[i] = Br[(int64_t)cand[r] * d + k0 + k];
                }
#pragma unroll
                for (int i = 0; i < kPer; ++i) {
                    const int e = base + i * kThreads + (int)threadIdx.x;
                    if (e < total) {
                        const int r = e / kc, k = e - r * kc;
                        tb[r * ldt + k] = a[i] - b[i];
                    }
                }
            }
            __syncthreads();
            if (wave == 0 && lane < np)
                for (int k = 0; k < kc; ++k) term(tb[lane * ldt + k]);
            __syncthreads();
        }
    }
    return METRIC == CHAMFER_L1 ? acc : sqrtf(acc);
}

// Canonical float32 distance of the tile's point pp to B's row c with four
// lanes: lane 4 j + s holds quarter s of both rows (coordinates
// [s S, (s + 1) S), S = ceil(d / 4) <= kQuadCols, all loaded in one batch)
// and continues the sum of quarter s - 1, which moves one lane up between
// quarters, so the terms are added in coordinate order as dist32 adds them.
// The distance is returned in lane 4 j + 3.  All 64 lanes must call it.
constexpr int kQuadCols = 32;
template <int METRIC>
__device__ __forceinline__ float quad_dist(const float *__restrict__ X, int64_t p0, int pp, int d,
                                           const float *__restrict__ Bpts, int c) {
    const int lane = threadIdx.x & 63, s = lane & 3;
    const int S = (d + 3) >> 2;
    const int k0 = s * S, k1 = min(d, k0 + S);
    const auto *xr = ro(X) + (p0 + pp) * d;
    const auto *br = ro(Bpts) + (int64_t)c * d;
    float t[kQuadCols];
    if ((S & 3) == 0 && (d & 3) == 0 &&
        ((reinterpret_cast<uintptr_t>(X) | reinterpret_cast<uintptr_t>(Bpts)) & 15) == 0) {
        // quarters of whole 16-byte quads (d a multiple of 16)
        float4 xv[kQuadCols / 4], bv[kQuadCols / 4];
#pragma unroll
        for (int i = 0; i < kQuadCols / 4; ++i) {
            const int k = min(k0 + 4 * i, d - 4);
            xv[i] = ld(reinterpret_cast<const CH_RO float4 *>(xr + k));
            bv[i] = ld(reinterpret_cast<const CH_RO float4 *>(br + k));
        }
#pragma unroll
        for (int i = 0; i < kQuadCols / 4; ++i) {
            t[4 * i] = xv[i].x - bv[i].x;
            t[4 * i + 1] = xv[i].y - bv[i].y;
            t[4 * i + 2] = xv[i].z - bv[i].z;
            t[4 * i + 3] = xv[i].w - bv[i].w;
        }
    } else {
        float xv[kQuadCols], bv[kQuadCols];
#pragma unroll
        for (int i = 0; i < kQuadCols; ++i) {
            const int k = min(k0 + i, d - 1);
            xv[i] = xr[k];
            bv[i] = br[k];
        }
#pragma unroll
        for (int i = 0; i < kQuadCols; ++i) t[i] = xv[i] - bv[i];
    }
    float acc = 0.0f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float prev = __shfl_up(acc, 1, 4);  // quarter q - 1's sum, in the lane below
        if (s == q) {
            acc = q == 0 ? 0.0f : prev;
#pragma unroll
            for (int i = 0; i < kQuadCols; ++i)
                if (k0 + i < k1) acc = METRIC == CHAMFER_L1 ? acc + fabsf(t[i]) : fmaf(t[i], t[i], acc);
        }
    }
    return METRIC == CHAMFER_L1 ? acc : sqrtf(acc);
}

// MODE 0: insert the tile's points (B) into the L tables.
// MODE 1: probe (A): first scale with a hit, candidate, D_a; max D_a.
// MODE 2: write keys[L][n].
// MODE 5: write keys[L][n] of B for the partitioned table build: a lane
//         whose key a lower lane of its wavefront also holds writes the
//         empty key instead (it cannot be the lowest index of its bucket),
//         and the l2 row norms are computed as in MODE 0.
// MODE 3: insert into window tables (W smallest b per bucket).
// MODE 4: probe window tables: the first W distinct b over the scales, finest
//         first (wavefront 0 walks the scales of its lane's point; the
//         retrieved b are kept in LDS), candidate = the closest of them.
// With kProbeMerge a probe keeps the better of its candidate and the one
// already stored for the point (an earlier LSH structure), by (D_a, b); the
// max of D_a is reduced only with kProbeLast.
// KE: embedding dimension for l2 (0 for l1).  YG: l1 coordinates from HBM.
// Lane p of every wavefront works on point p of the tile; wavefront w takes
// scales w, w + 4, w + 8, ...  For the probe each wavefront stops at its own
// first hit (or once another wavefront has hit at a finer scale); the first
// colliding scale is the smallest over the four.
// EC: coordinates of x staged per pass of the l2 embedding.
// B's FP16 table for the l2 exact pass (half_of of (x_k - c_k) 2^he for
// k < half_dp, zero past d), written from the staged rows while B is hashed (B
// is read once), with the same values as k_half_rows.  Coordinates
// [k0, k0 + kc) of the tile's np points are staged at xs[point * ld + k - k0],
// the centre's at cen; the last chunk also writes the padding
// [k0 + kc, half_dp).  Thread t takes 16 consecutive coordinates of point
// t / 4 per 64-coordinate step and adds their squares and those of their
// rounding errors to s2 and e2.
__device__ __forceinline__ void half_staged(const float *xs, int ld, const float *cen, int he,
                                            int64_t p0, int np, int k0, int kc, bool last,
                                            int half_dp, uint16_t *out, float &s2, float &e2) {
    const int pp = threadIdx.x >> 2;
    if (pp >= np) return;
    uint16_t *row = out + (size_t)(p0 + pp) * half_dp;
    const int kend = last ? half_dp : k0 + kc;
    for (int c = k0 + (threadIdx.x & 3) * 16; c < kend; c += 64) {
        uint32_t w[8];
#pragma unroll
        for (int e = 0; e < 16; e += 2) {
            uint32_t hb[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int a = c + e + q - k0;
                const float v = a < kc ? ldexpf(xs[pp * ld + a] - cen[a], he) : 0.0f;
                const _Float16 h = half_of(v);
                const float r = half_rest(v, h);
                s2 = fmaf(v, v, s2);
                e2 = fmaf(r, r, e2);
                hb[q] = half_bits(h);
            }
            w[e / 2] = hb[0] | (hb[1] << 16);
        }
        uint4 *hd = reinterpret_cast<uint4 *>(row + c);
        hd[0] = make_uint4(w[0], w[1], w[2], w[3]);
        hd[1] = make_uint4(w[4], w[5], w[6], w[7]);
    }
}

template <int METRIC, int MODE, int KE, bool YG, int EC = kEmbedChunk>
__device__ __forceinline__ void hash_tile(
    const float *__restrict__ X, int64_t n, const float *__restrict__ Bpts, int d, int L,
    const uint32_t *__restrict__ lohi, const int8_t *__restrict__ embed,
    const float *__restrict__ zfrac, const uint64_t *__restrict__ mult, Bucket *tables,
    int log2cap, unsigned long long *keys_out, float *D_out, int32_t *nn_out,
    int32_t *scale_out, float *nbh_out, DevParams *p, int64_t nB, int W, int flags, Blk blk,
    uint16_t *half_out = nullptr, int half_dp = 0) {
    extern __shared__ float smem[];
    __shared__ float los[EC > kEmbedChunk ? EC : kEmbedChunk];
    __shared__ int hit_scale[kTile];
    __shared__ int hit_cand[kWaves][kTile];
    __shared__ int wave_scale[kWaves][kTile];
    const int tid = threadIdx.x;
    // wave-uniform by construction; readfirstlane lets the compiler know, so
    // the per-scale tables and the embedding columns go through scalar loads
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t p0 = blk.id * kTile;
    const int np = (int)min<int64_t>(kTile, n - p0);
    const int64_t pt = p0 + lane;
    const bool active = lane < np;

    if (p->status != CHAMFER_OK) {
        if ((MODE == 1 || MODE == 4) && wave == 0 && active) {
            D_out[pt] = __builtin_nanf("");
            nn_out[pt] = -1;
            if (scale_out) scale_out[pt] = -1;
        }
        return;
    }
    const int kh = METRIC == CHAMFER_L1 ? d : KE;
    const int khp = kh | 1;  // odd row stride: lanes read distinct banks
    float *ys = smem;        // [kTile][khp]
    const int e_top = p->e_top;

    if (METRIC == CHAMFER_L1) {
        if (!YG) {
            stage_rows<16>(X, p0, np, d, 0, d, ys, khp, lohi);
        }
    } else {
        // The quantised embedding: u_k = floor(min((x_k - lo_k) 2^(24 - e_top),
        // 2^24 - 1)), Y_j = sum_k Zq_jk u_k exactly, on the int8 matrix cores:
        // wavefront w takes points 16 w + i of the tile (A rows: the three
        // bytes of u offset by -128, 16 coordinates per lane), B is Zq^T from
        // the packed table (16-column tiles of j, 64-coordinate steps), one
        // int32 accumulator per byte; then Y_j = sum_a 2^(8a) (acc_a + 128 R_j)
        // with R_j = sum_k Zq_jk, and y_j = (float)((Y_j 2^(e_top - 24)) inv),
        // inv = 1 / (beta KE 32).  The raw rows are staged 64 coordinates at a
        // time; B's FP16 table of the l2 exact pass is written from them too.
        constexpr int NT = (KE + 15) / 16;
        constexpr int ECM = kEmbedChunk;  // one 64-coordinate MFMA step per staged chunk
        const int nks = (d + ECM - 1) / ECM;
        const int i16 = lane & 15, g4 = lane >> 4;
        float *xs = smem + kTile * khp;  // [kTile][ECM + 1]
        typedef int v4i __attribute__((ext_vector_type(4)));
        v4i acc[3][NT];
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[a][t] = v4i{0, 0, 0, 0};
        const auto *zpk = reinterpret_cast<const CH_RO uint4 *>(ro(embed));
        constexpr bool kHalfMode = MODE == 0 || MODE == 3 || MODE == 5;
        __shared__ float cens[ECM];
        __shared__ uint32_t hmx[2];
        const bool want_half = kHalfMode && half_out != nullptr;
        float s2 = 0.0f, e2 = 0.0f;
        if (kHalfMode && tid < 2) hmx[tid] = 0u;
        for (int ks = 0; ks < nks; ++ks) {
            const int k0 = ks * ECM;
            const int kc = min(ECM, d - k0);
            __syncthreads();
            stage_rows<16>(X, p0, np, d, k0, kc, xs, ECM + 1, nullptr);
            if (tid < kc) los[tid] = ordered_to_float(ro(lohi)[k0 + tid]);
            if (want_half && tid < kc) cens[tid] = half_centre(lohi, d)[k0 + tid];
            __syncthreads();
            if (want_half)
                half_staged(xs, ECM + 1, cens, p->he, p0, np, k0, kc, ks == nks - 1, half_dp,
                            half_out, s2, e2);
            // A: 16 coordinates k0 + 16 g4 + e of point 16 wave + i16, as the
            // three bytes of u, each offset by -128 (xor 0x80); four
            // coordinates at a time give one dword of each byte's operand
            v4i ab[3];
            const float *xr = xs + (16 * wave + i16) * (ECM + 1) + 16 * g4;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                uint32_t u[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int k = 16 * g4 + 4 * q + e;
                    const float v = ldexpf(xr[4 * q + e] - los[k < kc ? k : 0], 24 - e_top);
                    u[e] = k < kc ? (uint32_t)(int32_t)floorf(fminf(v, 16777215.0f)) : 0u;
                }
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const uint32_t sel = (uint32_t)a | ((uint32_t)(4 + a) << 8);
                    const uint32_t lo2 = __builtin_amdgcn_perm(u[1], u[0], sel);
                    const uint32_t hi2 = __builtin_amdgcn_perm(u[3], u[2], sel);
                    ab[a][q] = (int)(__builtin_amdgcn_perm(hi2, lo2, 0x05040100u) ^ 0x80808080u);
                }
            }
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                const uint4 bz = ld(zpk + ((size_t)(t * nks + ks) * 64 + lane));
                const v4i bv = v4i{(int)bz.x, (int)bz.y, (int)bz.z, (int)bz.w};
#pragma unroll
                for (int a = 0; a < 3; ++a)
                    acc[a][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ab[a], bv, acc[a][t], 0, 0, 0);
            }
        }
        // lane (g4, i16) holds points 16 wave + 4 g4 + r of column j = 16 t + i16
        const auto *rsum = reinterpret_cast<const CH_RO int32_t *>(ro(embed) + (size_t)NT * nks * 1024);
        const double inv = 1.0 / (sqrt(2.0 / 3.14159265358979323846) * (double)KE * 32.0);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int j = 16 * t + i16;
            const int32_t r128 = 128 * rsum[j];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t Y = (int64_t)(acc[0][t][r] + r128) +
                                  ((int64_t)(acc[1][t][r] + r128) << 8) +
                                  ((int64_t)(acc[2][t][r] + r128) << 16);
                if (j < KE)
                    ys[(16 * wave + 4 * g4 + r) * khp + j] =
                        (float)(ldexp((double)Y, e_top - 24) * inv);
            }
        }
        if (want_half) {
            // four lanes per point; one atomic per maximum and tile
#pragma unroll
            for (int off = 1; off < 4; off <<= 1) {
                s2 += __shfl_xor(s2, off);
                e2 += __shfl_xor(e2, off);
            }
            const HalfErr he_ = half_err(d, half_dp);
            // (a row outside FP16's range keeps its clamped operands: nothing
            // beside kHalfAlways)
            if ((tid & 3) == 0 && (tid >> 2) < np)
                nbh_out[p0 + (tid >> 2)] =
                    isfinite(s2 + e2) ? half_norm(s2, e2, he_.s2, he_.e2) : kHalfAlways;
            uint32_t my = __float_as_uint(s2), me = __float_as_uint(e2);
            for (int off = 32; off > 2; off >>= 1) {
                my = max(my, (uint32_t)__shfl_xor((int)my, off));
                me = max(me, (uint32_t)__shfl_xor((int)me, off));
            }
            if (lane == 0) {
                atomicMax(&hmx[0], my);
                atomicMax(&hmx[1], me);
            }
            __syncthreads();
            if (tid < 2) rep_max(p->half_rep + tid, blk.id, hmx[tid]);
        }
    }
    if (MODE == 1 && wave == 0) hit_scale[lane] = L;
    __syncthreads();

    const float *yrow = ys + lane * khp;
    const float *xrow = X + pt * d;
    // cell indices can leave the int32 range only with more than 30 scales
    // or sides below 2^-126
    const bool clamp = L > 30 || e_top - (L - 1) <= -127;
    auto key_at = [&](int i) -> unsigned long long {
        const int e = e_top - (L - 1 - i);
        const auto zi = ro(zfrac) + (size_t)i * kh;
        const auto mi = ro(mult) + (size_t)i * kh;
        if (METRIC == CHAMFER_L1 && YG)
            return clamp ? bucket_key_global<true>(ro(xrow), ro(lohi), kh, e, zi, mi)
                         : bucket_key_global<false>(ro(xrow), ro(lohi), kh, e, zi, mi);
        return clamp ? bucket_key<true>(yrow, kh, e, zi, mi) : bucket_key<false>(yrow, kh, e, zi, mi);
    };

    if (MODE == 0) {
        // At coarse scales most lanes share a bucket.  A lane skips its
        // insert when a lower lane holds the same key (it has a lower index),
        // so the lowest index per bucket is unchanged and the hot buckets see
        // one access per wavefront instead of one per point.
        // Up to kLeaders distinct keys of the wavefront are deduplicated by
        // leader election (the leader is the lowest lane holding the key);
        // all remaining inserts then run in parallel.
        constexpr int kLeaders = 4;
        for (int i = wave; i < L; i += kWaves) {
            const unsigned long long key = active ? key_at(i) : kEmptyKey;
            unsigned long long rest = __ballot(active);
            bool mine = false;
            for (int it = 0; it < kLeaders && rest != 0; ++it) {
                const int leader = __ffsll((long long)rest) - 1;
                const unsigned long long lk = lane_u64(key, leader);
                rest &= ~__ballot(active && key == lk);
                mine |= lane == leader;
            }
            mine |= ((rest >> lane) & 1ull) != 0;
            if (mine)
                table_insert(tables + ((size_t)i << log2cap), table_fps(tables, L, log2cap, i),
                             log2cap, key, (int)pt);
        }
        return;
    }
    if (MODE == 5) {
        constexpr int kLeaders = 4;
        for (int i = wave; i < L; i += kWaves) {
            const unsigned long long key = active ? key_at(i) : kEmptyKey;
            unsigned long long rest = __ballot(active);
            bool mine = false;
            for (int it = 0; it < kLeaders && rest != 0; ++it) {
                const int leader = __ffsll((long long)rest) - 1;
                const unsigned long long lk = lane_u64(key, leader);
                rest &= ~__ballot(active && key == lk);
                mine |= lane == leader;
            }
            mine |= ((rest >> lane) & 1ull) != 0;
            if (active) keys_out[(size_t)i * n + pt] = mine ? key : kEmptyKey;
        }
        return;
    }
    if (MODE == 2) {
        if (active)
            for (int i = wave; i < L; i += kWaves) keys_out[(size_t)i * n + pt] = key_at(i);
        return;
    }
    // keep the better of (D, c, s) and the stored result of an earlier
    // structure; then store, and reduce max D on the last structure
    // store (D, c, s) for point ptx of the tile's points when act; with
    // wave_max, the wavefront's max of the stored D goes to p->max_d_rep
    // (kProbeLast).  Returns the stored D.
    auto finish_at = [&](int64_t ptx, bool act, float D, int c, int s, bool wave_max) {
        if (act) {
            if (flags & kProbeMerge) {
                const float Dp = D_out[ptx];
                const int cp = nn_out[ptx];
                if (Dp < D || (Dp == D && cp < c)) {
                    D = Dp;
                    c = cp;
                }
                if (scale_out) s = min(s, scale_out[ptx]);
            }
            D_out[ptx] = D;
            nn_out[ptx] = c;
            if (scale_out) scale_out[ptx] = s;
        }
        if (wave_max && (flags & kProbeLast)) {
            // wavefront max of D (D >= 0, so its bits order as floats)
            uint32_t m = act ? __float_as_uint(D) : 0u;
            for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off));
            if (lane == 0) rep_max(p->max_d_rep, blk.id, m);
        }
        return D;
    };
    auto finish = [&](float D, int c, int s) { finish_at(pt, active, D, c, s, true); };
    if (MODE == 3) {
        unsigned long long *wkeys = reinterpret_cast<unsigned long long *>(tables);
        int *wmem = reinterpret_cast<int *>(wkeys + ((size_t)L << log2cap));
        // lanes sharing a key: only the W lowest (smallest b) can be among
        // the bucket's W smallest; the rest skip, as in MODE 0
        constexpr int kLeaders = 4;
        for (int i = wave; i < L; i += kWaves) {
            const unsigned long long key = active ? key_at(i) : kEmptyKey;
            unsigned long long rest = __ballot(active);
            bool mine = false;
            for (int it = 0; it < kLeaders && rest != 0; ++it) {
                const int leader = __ffsll((long long)rest) - 1;
                const unsigned long long lk = lane_u64(key, leader);
                const unsigned long long same = __ballot(active && key == lk);
                if ((same >> lane) & 1ull) mine = __popcll(same & ((1ull << lane) - 1)) < W;
                rest &= ~same;
            }
            mine |= ((rest >> lane) & 1ull) != 0;
            if (mine)
                wide_insert(wkeys + ((size_t)i << log2cap), wmem + ((size_t)i << log2cap) * W,
                            log2cap, key, (int)pt, W);
        }
        return;
    }
    if (MODE == 4) {
        if (wave != 0) return;  // no barrier follows
        const auto *wk = reinterpret_cast<const unsigned long long *>(tables);
        const auto *wkeys = ro(wk);
        const auto *wmem = ro(reinterpret_cast<const int *>(wk + ((size_t)L << log2cap)));
        const int lds_floats = METRIC == CHAMFER_L1 ? (YG ? 0 : kTile * khp)
                                                    : kTile * (khp + EC + 1);
        int *got = reinterpret_cast<int *>(smem + lds_floats) + lane * W;
        int ng = 0, first = L;
        float D = 0.0f;
        int c = 0;
        if (active) {
            for (int i = 0; i < L && ng < W; ++i) {
                const int64_t s = wide_find(wkeys + ((size_t)i << log2cap), log2cap, key_at(i));
                if (s < 0) continue;
                const auto *m = wmem + (((size_t)i << log2cap) + (size_t)s) * W;
                for (int j = 0; j < W && ng < W; ++j) {
                    const int b = m[j];
                    if (b == INT_MAX) break;
                    bool seen = false;
                    for (int t = 0; t < ng; ++t) seen |= got[t] == b;
                    if (!seen) {
                        if (ng == 0) first = i;
                        got[ng++] = b;
                    }
                }
            }
            if (ng == 0)  // no collision at any scale: the window is b = 0 .. W - 1
                for (int b = 0; b < W && b < nB; ++b) got[ng++] = b;
            c = -1;
            for (int t = 0; t < ng; ++t) {
                const int b = got[t];
                const float v = dist32<METRIC>(xrow, Bpts + (size_t)b * d, d);
                if (c < 0 || v < D || (v == D && b < c)) {
                    D = v;
                    c = b;
                }
            }
        }
        finish(D, c, first);
        return;
    }
    // MODE 1: probe.
    int found = L, cand = 0;
    if (active) {
        for (int i = wave; i < L; i += kWaves) {
            if (i > __hip_atomic_load(&hit_scale[lane], __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_WORKGROUP))
                break;  // a finer scale already collided
            // (keys_out, half_dp: launch_part_build's keys and region)
            const int v = table_probe(
                ro((const Bucket *)tables) + ((size_t)i << log2cap),
                ro((const uint8_t *)table_fps(tables, L, log2cap, i)), log2cap,
                half_dp > 0 ? half_dp : log2cap, key_at(i),
                keys_out ? ro((const unsigned long long *)keys_out) + (size_t)i * nB : nullptr,
                nB);
            if (v >= 0) {
                found = i;
                cand = v;
                atomicMin(&hit_scale[lane], i);
                break;
            }
        }
    }
    wave_scale[wave][lane] = found;
    hit_cand[wave][lane] = cand;
    __syncthreads();
    // Small grids (about one round of resident workgroups) finish sooner when
    // wavefront 0 gathers both rows itself and the other three leave at once;
    // large ones are faster with all four wavefronts on the distances: four
    // lanes per point (quad_dist, d <= 128) or coalesced chunks (tile_dist).
    const bool coop = !(METRIC == CHAMFER_L1 && YG) && (n + kTile - 1) / kTile >= kCoopDistTiles;
    if (coop && d <= 4 * kQuadCols) {
        // wavefront w: points 16 w + j, four lanes each
        const int pq = 16 * wave + (lane >> 2);
        int sq = L, cq = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w)
            if (wave_scale[w][pq] < sq) {
                sq = wave_scale[w][pq];
                cq = hit_cand[w][pq];
            }
        const bool aq = (lane & 3) == 3 && pq < np;
        const float Dq = finish_at(p0 + pq, aq,
                                   quad_dist<METRIC>(X, p0, min(pq, np - 1), d, Bpts, cq), cq, sq,
                                   false);
        if (flags & kProbeLast) {  // one atomic per tile: the wavefronts' maxima meet in LDS
            uint32_t m = aq ? __float_as_uint(Dq) : 0u;
            for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor((int)m, off));
            if (lane == 0) hit_scale[wave] = (int)m;
            __syncthreads();
            if (tid == 0)
                rep_max(p->max_d_rep, blk.id,
                        max(max((uint32_t)hit_scale[0], (uint32_t)hit_scale[1]),
                            max((uint32_t)hit_scale[2], (uint32_t)hit_scale[3])));
        }
        return;
    }
    // the finest colliding scale over the four wavefronts (every wavefront
    // computes it for its lane's point; wavefront 0 keeps it)
    int best_s = L, best_c = 0;
    if (active) {
#pragma unroll
        for (int w = 0; w < kWaves; ++w)
            if (wave_scale[w][lane] < best_s) {
                best_s = wave_scale[w][lane];
                best_c = hit_cand[w][lane];
            }
    }
    if (!coop) {
        if (wave != 0) return;
        finish(active ? dist32<METRIC>(xrow, Bpts + (size_t)best_c * d, d) : 0.0f, best_c,
               best_s);
        return;
    }
    if (wave == 0) hit_scale[lane] = best_c;  // the scale walk is over: reuse as the row list
    __syncthreads();
    const float D = tile_dist<METRIC>(X, p0, np, d, Bpts, hit_scale, smem);
    if (wave != 0) return;
    finish(active ? D : 0.0f, best_c, best_s);
}

int64_t hash_blocks(int64_t n) { return (n + kTile - 1) / kTile; }

// WAVES: wavefronts per SIMD the register allocation must allow.
template <int METRIC, int MODE, int KE, bool YG, int EC, int WAVES>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(WAVES))) void k_hash(
    const float *__restrict__ X, int64_t n, const float *__restrict__ Bpts, int d, int L,
    const uint32_t *__restrict__ lohi, const int8_t *__restrict__ embed,
    const float *__restrict__ zfrac, const uint64_t *__restrict__ mult, Bucket *tables,
    int log2cap, unsigned long long *keys_out, float *D_out, int32_t *nn_out,
    int32_t *scale_out, float *nbh_out, DevParams *p, int64_t nB, int W, int flags,
    uint16_t *half_out, int half_dp) {
    hash_tile<METRIC, MODE, KE, YG, EC>(X, n, Bpts, d, L, lohi, embed, zfrac, mult, tables,
                                        log2cap, keys_out, D_out, nn_out, scale_out, nbh_out, p,
                                        nB, W, flags, grid_blk(), half_out, half_dp);
}


template <int METRIC, int KE, bool YG, int EC = kEmbedChunk>
static size_t hash_lds(int d) {
    const int kh = METRIC == CHAMFER_L1 ? d : KE;
    if (METRIC == CHAMFER_L1) return YG ? 0 : (size_t)kTile * (kh | 1) * sizeof(float);
    return (size_t)kTile * ((kh | 1) + EC + 1) * sizeof(float);
}

template <int METRIC, int KE, bool YG>
static hipError_t launch_hash_t(int mode, const float *X, int64_t n, const float *Bpts,
                                int64_t nB, int d, int L, const uint32_t *lohi,
                                const int8_t *embed, const float *zfrac, const uint64_t *mult,
                                Bucket *tables, int log2cap, uint64_t *keys_out, float *D_out,
                                int32_t *nn_out, int32_t *scale_out, float *nbh_out,
                                DevParams *p, int W, int flags, hipStream_t st,
                                uint16_t *half_out, int half_dp) {
    const unsigned blocks = (unsigned)hash_blocks(n);
    auto *ko = reinterpret_cast<unsigned long long *>(keys_out);
#define CH_KARGS X, n, Bpts, d, L, lohi, embed, zfrac, mult, tables, log2cap, ko, D_out, nn_out, \
                 scale_out, nbh_out, p, nB, W, flags, half_out, half_dp
    // Four wavefronts per SIMD for every mode: measured against six and
    // eight (l2, 10^5 points: probe 90, 117 and 141 us; keys and insert
    // within noise or slower).
    const size_t lds = hash_lds<METRIC, KE, YG>(d);
    switch (mode) {
        case 0: k_hash<METRIC, 0, KE, YG, kEmbedChunk, 4><<<blocks, kThreads, lds, st>>>(CH_KARGS); break;
        case 1: k_hash<METRIC, 1, KE, YG, kEmbedChunk, 4><<<blocks, kThreads, lds, st>>>(CH_KARGS); break;
        case 2: k_hash<METRIC, 2, KE, YG, kEmbedChunk, 4><<<blocks, kThreads, lds, st>>>(CH_KARGS); break;
        case 3: k_hash<METRIC, 3, KE, YG, kEmbedChunk, 4><<<blocks, kThreads, lds, st>>>(CH_KARGS); break;
        case 4:  // retrieved b per lane after the tile
            k_hash<METRIC, 4, KE, YG, kEmbedChunk, 4>
                <<<blocks, kThreads, lds + (size_t)kTile * W * sizeof(int), st>>>(CH_KARGS);
            break;
        case 5: k_hash<METRIC, 5, KE, YG, kEmbedChunk, 4><<<blocks, kThreads, lds, st>>>(CH_KARGS); break;
        default: return hipErrorInvalidValue;
    }
#undef CH_KARGS
    return hipGetLastError();
}

size_t table_bytes(int L, int log2cap, int W) {
    const size_t buckets = (size_t)L << log2cap;
    // W = 1: buckets, then a fingerprint byte per bucket
    return W <= 1 ? buckets * (sizeof(Bucket) + 1) : buckets * (sizeof(uint64_t) + (size_t)W * 4);
}

hipError_t launch_tables_empty(Bucket *tables, int L, int log2cap, int W, hipStream_t st) {
    const size_t buckets = (size_t)L << log2cap;
    if (W <= 1) return launch_table_fill(tables, buckets, st);
    auto *keys = reinterpret_cast<unsigned long long *>(tables);
    hipError_t e = launch_fill_u64(keys, (int64_t)buckets, ~0ull, st);
    if (e != hipSuccess) return e;
    // members: INT_MAX in both halves of each 64-bit word (W * buckets is even)
    return launch_fill_u64(keys + buckets, (int64_t)(buckets * W / 2), 0x7fffffff7fffffffull, st);
}

// kMaxLdsL1Dim: largest l1 dimension whose tile (64 x (d|1) floats) plus the
// static LDS fits the default 64 KiB.

hipError_t launch_hash(int mode, const float *X, int64_t n, const float *Bpts, int64_t nB,
                       int d, int metric, int L, int ke, const uint32_t *lohi,
                       const int8_t *embed, const float *zfrac, const uint64_t *mult,
                       Bucket *tables, int log2cap, uint64_t *keys_out, float *D_out,
                       int32_t *nn_out, int32_t *scale_out, float *nbh_out, DevParams *p,
                       int W, int flags, hipStream_t st, uint16_t *half_out, int half_dp) {
    if (n <= 0) return hipSuccess;
    if (W < 1 || W > kMaxWindow) return hipErrorInvalidValue;
    // the FP16 table is written from the l2 embedding's staged rows (B's
    // hashing modes only; half_dp a multiple of 64 at or above d, or 32)
    if (half_out != nullptr &&
        (metric != CHAMFER_L2 || !(mode == 0 || mode == 3 || mode == 5) || half_dp < d ||
         (half_dp % 64 != 0 && half_dp != 32)))
        return hipErrorInvalidValue;
#define CH_ARGS mode, X, n, Bpts, nB, d, L, lohi, embed, zfrac, mult, tables, log2cap, keys_out, \
                D_out, nn_out, scale_out, nbh_out, p, W, flags, st, half_out, half_dp
    if (metric == CHAMFER_L1) {
        // the window probe also keeps W ints per lane in LDS
        const int room = mode == 4 ? kMaxLdsL1Dim - W : kMaxLdsL1Dim;
        if (d <= room) return launch_hash_t<CHAMFER_L1, 0, false>(CH_ARGS);
        return launch_hash_t<CHAMFER_L1, 0, true>(CH_ARGS);
    }
    switch (ke) {
        case 8: return launch_hash_t<CHAMFER_L2, 8, false>(CH_ARGS);
        case 16: return launch_hash_t<CHAMFER_L2, 16, false>(CH_ARGS);
        case 32: return launch_hash_t<CHAMFER_L2, 32, false>(CH_ARGS);
        case 64: return launch_hash_t<CHAMFER_L2, 64, false>(CH_ARGS);
        default: return hipErrorInvalidValue;
    }
#undef CH_ARGS
}

// ------------------------------------------------------ partitioned build
// The W = 1 tables of the direct path, built without global atomics from B's
// keys (hash mode 5, a wavefront's duplicate keys dropped).  A table of 2^c
// slots is cut into regions, and a key's region is the top bits of its home
// slot.  One workgroup per (scale, region) inserts the region's keys into a
// table in LDS -- linear probing from the home slot that goes round within the
// region, lowest b per key, LDS atomics only -- and writes it out: every
// fingerprint byte, and the buckets in use (the probe reads no other).
//
// Up to kDirectKeys keys the workgroups (regions of up to 2^13 slots) read all
// keys of their scale and pick theirs (k_direct_build).  Beyond, each block of
// kPartBlock keys counts its keys per region of up to 2^11 slots (k_part_hist),
// the counts become offsets (small partitions: inside k_part_scatter, each
// workgroup from its scale's counts; large ones: k_part_scan_rows and
// k_part_base), the blocks write their (key, b) pairs grouped by region
// (k_part_scatter, runs of a region contiguous) and k_region_build inserts them.
//
// A region of S slots holds about S / 2 keys (tables are at most half full).
// Where it gets more than S distinct ones, those without a slot are left out,
// and a probe that finds neither its key nor an empty slot searches the keys.

constexpr int kRegionBits = 11;
constexpr int kDirectBits = 13;
constexpr int64_t kDirectKeys = 20480;
constexpr int kPartBlock = 4096;   // keys per histogram / scatter workgroup
constexpr int kMaxRegions = 1024;  // regions per scale the scan and scatter hold in LDS

__host__ __device__ inline int region_bits(int log2cap) {
    return log2cap < kRegionBits ? log2cap : kRegionBits;
}

// log2 of the slots that a probe of launch_part_build's tables goes round in.
int part_probe_bits(int64_t nB, int log2cap) {
    if (nB > kDirectKeys) return region_bits(log2cap);
    return log2cap < kDirectBits ? log2cap : kDirectBits;
}

__host__ __device__ inline int64_t part_regions(int log2cap) {
    return (int64_t)1 << (log2cap - region_bits(log2cap));
}
int64_t part_blocks(int64_t nB) { return (nB + kPartBlock - 1) / kPartBlock; }
bool part_build_ok(int log2cap) { return part_regions(log2cap) <= kMaxRegions; }

static_assert(sizeof(uint3) == 12, "a (key, b) pair is three words");

size_t part_work_bytes(int L, int64_t nB, int log2cap, PartWork *w, char *base) {
    const int64_t R = part_regions(log2cap), nblk = part_blocks(nB);
    auto al = [](size_t x) { return (x + 255) / 256 * 256; };
    const size_t b_keys = al((size_t)L * nB * sizeof(uint64_t));
    const size_t b_offs = al((size_t)L * nblk * R * sizeof(uint32_t));
    const size_t b_bins = al((size_t)L * R * 2 * sizeof(uint32_t));
    const size_t b_ent = al((size_t)L * nB * sizeof(uint3));
    if (w) {
        w->keys = reinterpret_cast<uint64_t *>(base);
        w->offs = reinterpret_cast<uint32_t *>(base + b_keys);
        w->bins = reinterpret_cast<uint32_t *>(base + b_keys + b_offs);
        w->entries = reinterpret_cast<uint3 *>(base + b_keys + b_offs + b_bins);
    }
    return b_keys + b_offs + b_bins + b_ent;
}

__device__ __forceinline__ uint32_t key_region(unsigned long long key, int log2cap) {
    return (uint32_t)(home_slot(key, log2cap) >> region_bits(log2cap));
}

// In-place exclusive prefix sum of v[0..R) (R <= 1024) by a workgroup of
// 256 threads; returns the total.  Each thread sums up to four consecutive
// values, the 256 partial sums are scanned by wavefront shuffles (tmp: the
// four wavefronts' totals), then written back.
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t *v, int R, uint32_t *tmp) {
    const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
    const int per = (R + 255) / 256;
    uint32_t loc[4] = {0, 0, 0, 0};
    uint32_t sum = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (q < per && t * per + q < R) {
            loc[q] = v[t * per + q];
            sum += loc[q];
        }
    // inclusive scan of the groups' sums: shuffles in each wavefront, then
    // the totals of the wavefronts before
    uint32_t x = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)x, off);
        if (lane >= off) x += y;
    }
    if (lane == 63) tmp[wv] = x;
    __syncthreads();
    uint32_t before = 0;
    for (int w = 0; w < wv; ++w) before += tmp[w];
    const uint32_t total = tmp[0] + tmp[1] + tmp[2] + tmp[3];
    uint32_t run = before + x - sum;  // exclusive prefix of this thread's group
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (q < per && t * per + q < R) {
            v[t * per + q] = run;
            run += loc[q];
        }
    __syncthreads();
    return total;
}

// Counts per (scale i, block j, region): offs[(i nblk + j) R + g].
__global__ __launch_bounds__(256) void k_part_hist(const uint64_t *__restrict__ keys, int64_t nB,
                                                   int log2cap, int64_t nblk, uint32_t *offs) {
    extern __shared__ uint32_t cnt[];
    const int R = (int)part_regions(log2cap);
    const int64_t i = blockIdx.x / nblk, j = blockIdx.x - i * nblk;
    for (int g = threadIdx.x; g < R; g += 256) cnt[g] = 0;
    __syncthreads();
    const CH_RO uint64_t *kr = ro(keys) + i * nB;
    // all of the thread's keys are loaded (in bounds, unconditionally, so
    // the loads are in flight together) before any is counted
    constexpr int kPer = kPartBlock / 256;
    unsigned long long k[kPer];
#pragma unroll
    for (int t = 0; t < kPer; ++t) k[t] = kr[min(j * kPartBlock + t * 256 + threadIdx.x, nB - 1)];
#pragma unroll
    for (int t = 0; t < kPer; ++t)
        if (j * kPartBlock + t * 256 + threadIdx.x < nB && k[t] != kEmptyKey)
            atomicAdd(&cnt[key_region(k[t], log2cap)], 1u);
    __syncthreads();
    uint32_t *o = offs + (size_t)(i * nblk + j) * R;
    for (int g = threadIdx.x; g < R; g += 256) o[g] = cnt[g];
}

// Large partitions (many blocks and regions): the counts become offsets in
// two launches (offs: the exclusive prefix over blocks of each region's
// counts; bins[(i R + g) 2 + {0, 1}] = the region's first entry in the scale's
// [nB] span of entries and its count):
// k_part_scan_rows takes 64 regions of one scale per workgroup, each
// wavefront a contiguous quarter of the blocks (loads coalesced over the
// regions, eight in flight per lane), and writes the regions' totals;
// k_part_base scans the totals of each scale into the regions' first
// entries.
__global__ __launch_bounds__(256) void k_part_scan_rows(int log2cap, int64_t nblk,
                                                        uint32_t *offs, uint32_t *bins) {
    __shared__ uint32_t part[4][64];
    const int R = (int)part_regions(log2cap);
    const int gpb = (R + 63) / 64;  // workgroups per scale
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t i = blockIdx.x / gpb;
    const int g = (int)(blockIdx.x % gpb) * 64 + lane;
    const bool live = g < R;
    const int64_t q = (nblk + 3) / 4;
    const int64_t j0 = min(nblk, w * q), j1 = min(nblk, j0 + q);
    uint32_t *o = offs + (size_t)i * nblk * R + g;
    uint32_t sum = 0;
    if (live) {
        int64_t j = j0;
        for (; j + 8 <= j1; j += 8) {
            uint32_t c[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) c[e] = o[(j + e) * R];
#pragma unroll
            for (int e = 0; e < 8; ++e) sum += c[e];
        }
        for (; j < j1; ++j) sum += o[j * R];
    }
    part[w][lane] = sum;
    __syncthreads();
    uint32_t run = 0, tot = 0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const uint32_t x = part[v][lane];
        run += v < w ? x : 0u;
        tot += x;
    }
    if (!live) return;
    int64_t j = j0;
    for (; j + 8 <= j1; j += 8) {
        uint32_t c[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) c[e] = o[(j + e) * R];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            o[(j + e) * R] = run;
            run += c[e];
        }
    }
    for (; j < j1; ++j) {
        const uint32_t c = o[j * R];
        o[j * R] = run;
        run += c;
    }
    if (w == 0) {
        bins[((size_t)i * R + g) * 2 + 1] = tot;
    }
}

__global__ __launch_bounds__(256) void k_part_base(int log2cap, uint32_t *bins) {
    __shared__ uint32_t tot[kMaxRegions + 256];
    const int R = (int)part_regions(log2cap);
    const int64_t i = blockIdx.x;
    for (int g = threadIdx.x; g < R; g += 256) tot[g] = bins[((size_t)i * R + g) * 2 + 1];
    __syncthreads();
    block_exclusive_scan(tot, R, tot + R);
    for (int g = threadIdx.x; g < R; g += 256) bins[((size_t)i * R + g) * 2] = tot[g];
}

// The block's (key, b) pairs grouped by region: counted in LDS, placed in
// LDS in region order, then written so that consecutive threads write
// consecutive entries of a region's run.
// fused (small partitions, nblk x R <= kPartScanOneGroup): offs holds the
// raw counts of k_part_hist; the workgroup derives its offsets in every
// region and the regions' first entries from its scale's counts itself,
// and workgroup j = 0 of each scale writes the scale's bins (what
// k_part_scan_rows and k_part_base do for large partitions).
__global__ __launch_bounds__(256) void k_part_scatter(const uint64_t *__restrict__ keys,
                                                      int64_t nB, int log2cap, int64_t nblk,
                                                      const uint32_t *__restrict__ offs,
                                                      uint32_t *bins, uint3 *entries, int fused) {
    extern __shared__ uint32_t sm[];
    const int R = (int)part_regions(log2cap);
    uint32_t *cnt = sm;               // [R] counts, then the block's region starts
    uint32_t *fill = sm + R;          // [R + 256] scan scratch, then positions per region
    auto *sk = reinterpret_cast<unsigned long long *>(sm + 2 * R + 256);  // [kPartBlock]
    int32_t *sb = reinterpret_cast<int32_t *>(sk + kPartBlock);                      // [kPartBlock]
    uint32_t *gbase = reinterpret_cast<uint32_t *>(sb + kPartBlock);  // [R] fused: first entry
    uint32_t *gtot = gbase + R;                                        // [R] fused: region totals
    __shared__ uint32_t total;
    const int64_t i = blockIdx.x / nblk, j = blockIdx.x - i * nblk;
    if (fused) {
        for (int g = threadIdx.x; g < R; g += 256) {
            const CH_RO uint32_t *o = ro(offs) + (size_t)i * nblk * R + g;
            uint32_t before = 0, all = 0;
#pragma unroll 8
            for (int64_t b = 0; b < nblk; ++b) {
                const uint32_t c = o[b * R];
                before += b < j ? c : 0u;
                all += c;
            }
            gbase[g] = before;
            gtot[g] = all;
            if (j == 0) bins[((size_t)i * R + g) * 2 + 1] = all;
        }
        __syncthreads();
        block_exclusive_scan(gtot, R, fill);
        for (int g = threadIdx.x; g < R; g += 256) {
            gbase[g] += gtot[g];
            if (j == 0) bins[((size_t)i * R + g) * 2] = gtot[g];
        }
    }
    for (int g = threadIdx.x; g < R; g += 256) cnt[g] = 0;
    __syncthreads();
    constexpr int kPer = kPartBlock / 256;
    unsigned long long k[kPer];
    const CH_RO uint64_t *kr = ro(keys) + i * nB;
    // loads first (in bounds, unconditional: in flight together), then the
    // counts; keys past n_B become the empty key
#pragma unroll
    for (int t = 0; t < kPer; ++t) k[t] = kr[min(j * kPartBlock + t * 256 + threadIdx.x, nB - 1)];
#pragma unroll
    for (int t = 0; t < kPer; ++t) {
        if (j * kPartBlock + t * 256 + threadIdx.x >= nB) k[t] = kEmptyKey;
        if (k[t] != kEmptyKey) atomicAdd(&cnt[key_region(k[t], log2cap)], 1u);
    }
    __syncthreads();
    const uint32_t tsum = block_exclusive_scan(cnt, R, fill);  // fill: scan scratch
    for (int g = threadIdx.x; g < R; g += 256) fill[g] = cnt[g];
    if (threadIdx.x == 0) total = tsum;
    __syncthreads();
#pragma unroll
    for (int t = 0; t < kPer; ++t) {
        if (k[t] == kEmptyKey) continue;
        const uint32_t pos = atomicAdd(&fill[key_region(k[t], log2cap)], 1u);
        sk[pos] = k[t];
        sb[pos] = (int32_t)(j * kPartBlock + t * 256 + threadIdx.x);
    }
    __syncthreads();
    const uint32_t n = total;
    const uint32_t *o = offs + (size_t)(i * nblk + j) * R;
    const uint32_t *bn = bins + (size_t)i * R * 2;
    for (uint32_t pos = threadIdx.x; pos < n; pos += 256) {
        const unsigned long long key = sk[pos];
        const uint32_t g = key_region(key, log2cap);
        const uint32_t first = fused ? gbase[g] : bn[g * 2] + o[g];
        const size_t dst = (size_t)i * nB + first + (pos - cnt[g]);
        entries[dst] = make_uint3((uint32_t)key, (uint32_t)(key >> 32), (uint32_t)sb[pos]);
    }
}

// (key, b) into the S slots of a region in LDS (lowest b per key); no effect when
// it is full.
__device__ __forceinline__ void region_insert(unsigned long long *tk, int32_t *tv, int S,
                                              unsigned long long key, int b, int log2cap) {
    const int home = (int)(home_slot(key, log2cap) & (uint64_t)(S - 1));
    int s = home;
    for (;;) {
        unsigned long long cur = tk[s];
        if (cur == kEmptyKey) cur = atomicCAS(&tk[s], kEmptyKey, key);
        if (cur == kEmptyKey || cur == key) break;
        s = (s + 1) & (S - 1);
        if (s == home) return;
    }
    atomicMin(&tv[s], b);
}

// All fingerprints and the buckets in use (all: every bucket) of the S slots from
// `first` of scale i.
template <int NT>
__device__ __forceinline__ void region_write(const unsigned long long *tk, const int32_t *tv,
                                             int S, int64_t first, int64_t i, int L, int log2cap,
                                             Bucket *tables, bool all) {
    Bucket *out = tables + ((size_t)i << log2cap) + first;
    uint8_t *ofp = table_fps(tables, L, log2cap, (int)i) + first;
    for (int s = threadIdx.x; s < S; s += NT) {
        const unsigned long long k = tk[s];
        if (!all && k == kEmptyKey) continue;
        Bucket bk;
        bk.key = k;
        bk.val = tv[s];
        bk.pad = 0;
        out[s] = bk;
    }
    for (int s4 = threadIdx.x; s4 < S / 4; s4 += NT) {
        uint32_t w = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const unsigned long long k = tk[4 * s4 + q];
            w |= (k == kEmptyKey ? 0u : key_fp(k, log2cap)) << (8 * q);
        }
        reinterpret_cast<uint32_t *>(ofp)[s4] = w;
    }
}

// Few keys: one workgroup per (scale, region of 2^rb slots) reads all of the
// scale's keys.  Bound by latencies: one launch in place of the partition's
// three (4096 keys, 16 scales: 28 and 11 us).  The line at kDirectKeys: whole l1
// calls, partition and direct, 16300 keys 101 and 95 us, 32000 117 and 121, 65000 146
// and 158.
__global__ __launch_bounds__(1024) void k_direct_build(const uint64_t *__restrict__ keys,
                                                       int64_t nB, int L, int log2cap, int rb,
                                                       Bucket *tables) {
    __shared__ unsigned long long tk[1 << kDirectBits];
    __shared__ int32_t tv[1 << kDirectBits];
    const int S = 1 << rb;
    const int64_t R = (int64_t)1 << (log2cap - rb);
    const int64_t i = blockIdx.x / R, g = blockIdx.x - i * R;
    const CH_RO uint64_t *kr = ro(keys) + i * nB;
    constexpr int kPer = 8;
    unsigned long long k[kPer];
    auto load = [&](int64_t b0) {  // in bounds, in flight together
#pragma unroll
        for (int t = 0; t < kPer; ++t) k[t] = kr[min(b0 + t * 1024 + threadIdx.x, nB - 1)];
    };
    load(0);
    for (int s = threadIdx.x; s < S; s += 1024) {
        tk[s] = kEmptyKey;
        tv[s] = INT_MAX;
    }
    __syncthreads();
    for (int64_t b0 = 0; b0 < nB; b0 += 1024 * kPer) {
#pragma unroll
        for (int t = 0; t < kPer; ++t) {
            const int64_t b = b0 + t * 1024 + threadIdx.x;
            if (b < nB && k[t] != kEmptyKey &&
                (int64_t)(home_slot(k[t], log2cap) >> rb) == g)
                region_insert(tk, tv, S, k[t], (int)b, log2cap);
        }
        if (b0 + 1024 * kPer < nB) load(b0 + 1024 * kPer);
    }
    __syncthreads();
    region_write<1024>(tk, tv, S, g << rb, i, L, log2cap, tables, false);
}

// One workgroup per (scale, region): the region's pairs into an LDS table of
// S slots, written to the table.  Up to kRegionPrefetch pairs per thread are
// read before any is inserted (one round of loads).
constexpr int kRegionPrefetch = 8;

__global__ __launch_bounds__(256) void k_region_build(const uint3 *__restrict__ entries,
                                                      int64_t nB, int L, int log2cap,
                                                      Bucket *tables,
                                                      const uint32_t *__restrict__ bins) {
    extern __shared__ unsigned long long tk[];  // [S] keys, then [S] values
    const int qb = region_bits(log2cap);
    const int S = 1 << qb;
    int32_t *tv = reinterpret_cast<int32_t *>(tk + S);
    const int64_t R = part_regions(log2cap);
    const int64_t i = blockIdx.x / R, g = blockIdx.x - i * R;
    const uint32_t start = bins[(i * R + g) * 2], count = bins[(i * R + g) * 2 + 1];
    for (int s = threadIdx.x; s < S; s += 256) {
        tk[s] = kEmptyKey;
        tv[s] = INT_MAX;
    }
    const uint3 *run = entries + (size_t)i * nB + start;
    const int lane = threadIdx.x & 63;
    for (uint32_t base = 0; base < count; base += 256 * kRegionPrefetch) {
        uint3 e[kRegionPrefetch];
#pragma unroll
        for (int q = 0; q < kRegionPrefetch; ++q) {
            // in bounds and unconditional (predicated, each load was waited for
            // before the next: 316 against 240 us at 10^6 points)
            e[q] = run[min(base + q * 256 + threadIdx.x, count - 1)];
        }
        if (base == 0) __syncthreads();  // the table is initialised
#pragma unroll
        for (int q = 0; q < kRegionPrefetch; ++q) {
            const unsigned long long key = (unsigned long long)e[q].x |
                                           ((unsigned long long)e[q].y << 32);
            const bool valid = base + q * 256 + threadIdx.x < count;
            int b = (int)e[q].z;
            // the lowest lane's key: its lanes fold their b into it (a key
            // repeated across wavefronts at coarse scales goes in once per
            // wavefront); the others insert on their own
            const unsigned long long vm = __ballot(valid);
            const int first = vm ? __ffsll((long long)vm) - 1 : 0;  // wave-uniform
            const unsigned long long lk = lane_u64(key, first);
            const bool same = valid && key == lk;
            // the lowest b among the lanes holding the first valid lane's key
            const int mb = __ockl_wfred_min_i32(same ? b : INT_MAX);
            const bool leader = same && lane == first;
            if (leader) b = mb;
            if (!valid || (same && !leader)) continue;
            region_insert(tk, tv, S, key, b, log2cap);
        }
    }
    __syncthreads();
    region_write<256>(tk, tv, S, g << qb, i, L, log2cap, tables, count > (uint32_t)S / 4);
}

// Largest count table (blocks x regions) of one scale that each scatter
// workgroup reads and scans itself (10^5 points: 25 x 128); above it the
// two-launch scan (10^6 points, 245 x 1024: 88 us in one workgroup per
// scale, about 15 us in two launches).
constexpr int64_t kPartScanOneGroup = 16384;

hipError_t launch_part_build(const PartWork &w, int64_t nB, int L, int log2cap, Bucket *tables,
                             hipStream_t st) {
    if (nB <= 0 || L <= 0) return hipSuccess;
    if (!part_build_ok(log2cap)) return hipErrorInvalidValue;
    if (nB <= kDirectKeys) {
        const int rb = part_probe_bits(nB, log2cap);
        k_direct_build<<<(unsigned)((int64_t)L << (log2cap - rb)), 1024, 0, st>>>(
            w.keys, nB, L, log2cap, rb, tables);
        return hipGetLastError();
    }
    const int64_t R = part_regions(log2cap), nblk = part_blocks(nB);
    const int S = 1 << region_bits(log2cap);
    k_part_hist<<<(unsigned)(L * nblk), 256, (size_t)R * sizeof(uint32_t), st>>>(
        w.keys, nB, log2cap, nblk, w.offs);
    const bool fused = nblk * R <= kPartScanOneGroup;  // the scatter scans the counts itself
    if (!fused) {
        k_part_scan_rows<<<(unsigned)(L * ((R + 63) / 64)), 256, 0, st>>>(log2cap, nblk, w.offs,
                                                                         w.bins);
        k_part_base<<<(unsigned)L, 256, 0, st>>>(log2cap, w.bins);
    }
    const size_t lds_sc = (2 * (size_t)R + 256) * sizeof(uint32_t) + (size_t)kPartBlock * 12 +
                          (fused ? 2 * (size_t)R * sizeof(uint32_t) : 0);
    k_part_scatter<<<(unsigned)(L * nblk), 256, lds_sc, st>>>(
        w.keys, nB, log2cap, nblk, w.offs, w.bins, w.entries, fused ? 1 : 0);
    k_region_build<<<(unsigned)(L * R), 256, (size_t)S * 12, st>>>(w.entries, nB, L, log2cap,
                                                                   tables, w.bins);
    return hipGetLastError();
}

// ---------------------------------------------------------------- batched
// Persistent grids over all jobs of a batch (see batch_loop).  A job's
// blocks are the blocks of its direct launches, so every job computes what
// chamfer_estimate computes for it alone.

constexpr unsigned kGridSetup = 512, kGridMinmax = 1024, kGridCalib = kBatchMax,
                   kGridHash = 2048;

__global__ __launch_bounds__(256) void kb_setup(const Batch *__restrict__ bt) {
    batch_loop(bt, kBsSetup, [&](const Job &J, Blk b) {
        if (b.id < J.nb_init) {
            init_params(J.p, J.lohi, J.d, Blk{b.id, J.nb_init});
            return;
        }
        int64_t r = b.id - J.nb_init;
        if (r < J.nb_grid) {
            grid_tables(J.seed, J.L, J.kh, J.zfrac, J.mult, 0, Blk{r, J.nb_grid});
            return;
        }
        r -= J.nb_grid;
        table_fill(J.tables, (size_t)J.table_count, Blk{r, J.nb_fill});
    });
}

__global__ __launch_bounds__(256) void kb_minmax(const Batch *__restrict__ bt) {
    batch_loop(bt, kBsMinmax, [&](const Job &J, Blk b) {
        const bool isA = b.id < J.nb_mmA;
        minmax4(isA ? J.A : J.B, (isA ? J.nA : J.nB) * (int64_t)J.d, J.d,
                isA ? J.mm_strideA : J.mm_strideB, !isA, J.lohi, J.p,
                isA ? Blk{b.id, J.nb_mmA} : Blk{b.id - J.nb_mmA, J.nb_mmB});
    });
}

__global__ __launch_bounds__(256) void kb_calib(const Batch *__restrict__ bt) {
    batch_loop(bt, kBsCalib, [&](const Job &J, Blk) {
        calib_final(J.lohi, J.d, J.p, J.d <= 256 ? J.B : nullptr, J.nB, J.metric, J.A, nullptr, J.nA,
                    true);
    });
}

template <int METRIC, int MODE, int KE, bool YG>
__global__ __launch_bounds__(kThreads) void kb_hash(const Batch *__restrict__ bt) {
    batch_loop(bt, MODE == 0 ? kBsInsert : kBsProbe, [&](const Job &J, Blk b) {
        if (MODE == 0)
            hash_tile<METRIC, 0, KE, YG>(J.B, J.nB, J.B, J.d, J.L, J.lohi, J.embed, J.zfrac,
                                         J.mult, J.tables, J.log2cap, nullptr, nullptr, nullptr,
                                         nullptr, nullptr, J.p, J.nB, 1, 0, b);
        else
            hash_tile<METRIC, 1, KE, YG>(J.A, J.nA, J.B, J.d, J.L, J.lohi, J.embed, J.zfrac,
                                         J.mult, J.tables, J.log2cap, nullptr, J.D, J.nn,
                                         nullptr, nullptr, J.p, J.nB, 1, kProbeLast, b);
    });
}

hipError_t launch_batch_setup(const Batch *bt, hipStream_t st) {
    kb_setup<<<kGridSetup, 256, 0, st>>>(bt);
    return hipGetLastError();
}

hipError_t launch_batch_minmax(const Batch *bt, int d, hipStream_t st) {
    if (d > 2048) return hipErrorInvalidValue;
    kb_minmax<<<kGridMinmax, 256, minmax_lds(d), st>>>(bt);
    return hipGetLastError();
}

hipError_t launch_batch_calib(const Batch *bt, int d, hipStream_t st) {
    if (d > 2048) return hipErrorInvalidValue;
    kb_calib<<<kGridCalib, 256, (size_t)d * sizeof(double), st>>>(bt);
    return hipGetLastError();
}

template <int METRIC, int KE, bool YG>
static hipError_t launch_batch_hash_t(int mode, const Batch *bt, int d, hipStream_t st) {
    const size_t lds = hash_lds<METRIC, KE, YG>(d);
    if (mode == 0)
        kb_hash<METRIC, 0, KE, YG><<<kGridHash, kThreads, lds, st>>>(bt);
    else
        kb_hash<METRIC, 1, KE, YG><<<kGridHash, kThreads, lds, st>>>(bt);
    return hipGetLastError();
}

hipError_t launch_batch_hash(int mode, const Batch *bt, int d, int metric, int ke,
                             hipStream_t st) {
    if (mode != 0 && mode != 1) return hipErrorInvalidValue;
    if (metric == CHAMFER_L1) {
        if (d <= kMaxLdsL1Dim) return launch_batch_hash_t<CHAMFER_L1, 0, false>(mode, bt, d, st);
        return launch_batch_hash_t<CHAMFER_L1, 0, true>(mode, bt, d, st);
    }
    switch (ke) {
        case 8: return launch_batch_hash_t<CHAMFER_L2, 8, false>(mode, bt, d, st);
        case 16: return launch_batch_hash_t<CHAMFER_L2, 16, false>(mode, bt, d, st);
        case 32: return launch_batch_hash_t<CHAMFER_L2, 32, false>(mode, bt, d, st);
        case 64: return launch_batch_hash_t<CHAMFER_L2, 64, false>(mode, bt, d, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace chamfer
