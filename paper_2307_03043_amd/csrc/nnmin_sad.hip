// Exact l1 nearest neighbours for 9 <= d <= 256, returning the same canonical
// float32 result as the VALU form (the minimum over b of the sum of |x_k - b_k|
// in ascending k, ties to the lower b) from byte sums of absolute differences.
//
// v_sad_u8 adds four byte differences per instruction where the VALU form takes
// eight (a subtract and an add per coordinate), but only rules rows out.  With lo
// a corner and 1 / inv a step that take B's box to [0, 255]^d (calib_final),
// T(x)_k = (x_k - lo_k) inv, T_c its clamp to [0, 255] and i its rounding,
//   |x - b| inv >= sum |T_c(x) - T_c(b)| + excess(x)
//               >= SAD(i(x), i(b)) - e(x) - e(b) + excess(x),
// e = sum |T_c - i|, measured, and excess(x) = sum |T(x) - T_c(x)| when every row
// of B lies in the box (else 0: both sides are clamped).  A row can only reach
// the canonical minimum if its sum reaches a threshold that follows from the best
// canonical distance known for the query; rows that do are queued in LDS and
// evaluated with the canonical distance, 64 lanes at a time, and their minimum
// lowers the threshold.  Every row whose bound does not exclude it is evaluated,
// and the per-query minima merge with 64-bit atomicMin of (bits << 32 | b).
//
// A lane holds the bytes of two queries (with four the kernel was no faster: fewer
// wavefronts in flight, more rows to evaluate at once); B's rows are rounded while
// their tile is stored to LDS (16 coordinates a thread, no table in memory) and
// read back as broadcasts, one 16-byte read for 32 byte differences per lane.
//
// Bound by v_sad_u8, which runs at 3.5e13 lanes/s here (an fma: 6.2e13).  10^6 x 64
// points, 2000 draws: 5.04 ms in the VALU form, 1.43 here (the differences alone 0.93);
// exact 30000^2 x 100, which the VALU form takes in its any-dimension kernel: 33.4
// and 1.4 ms.
#include <algorithm>
#include <cfloat>
#include <climits>
#include <cmath>

#include "internal.h"

namespace chamfer {

bool sad_supported(int d, int metric) { return metric == CHAMFER_L1 && d > kSadMinDim && d <= 256; }

// At the dimensions that the VALU form is compiled for it starts and ends faster: a
// query without a distance to start from (seeded: it has one) first meets rows that
// its threshold does not rule out.  Bytes need a product that makes up for that, and
// at d = 16, where they hardly save operations, a long B.  Calls in us, VALU and bytes:
// d = 16, 10^6 x 1000 565 and 953, 20000^2 252 and 298, 10^5 x 20000 1114 and 947; 1700
// draws of 10^5 rows 270 and 281, 2000 of 10^5 612 and 604.  d = 32, 10^5 x 2000 253 and
// 280, 2500 x 100000 301 and 237; 450 draws of 2 10^5 379 and 442, 1600 of 50000 234 and
// 211.  d = 64, 10^5 x 1000 261 and 292, 10^6 x 1000 2116 and 1879, 2500 x 20001 160 and
// 134, 1000 x 40000 126 and 140, 300 x 400000 509 and 336; 400 draws of 50000 217 and
// 241.  d = 128, 300 draws of 4096 154 and 164, 400 of 50000 372 and 318.  Other
// dimensions up to 16: d = 12, 500 x 10000 64 and 76, 3000^2 70 and 67.
bool sad_pays(int64_t nx, int64_t nB, int d, bool seeded) {
    const double pairs = (double)nx * (double)nB;
    switch (d) {
        case 16: return seeded ? nB >= 65536 && pairs >= 2e8 : nB >= 16384 && pairs >= 5e8;
        case 32: return pairs >= 2.5e8 || (seeded && nx >= 1024 && pairs >= 7e7);
        case 64:
            return pairs >= 3e7 && (seeded || ((nB >= 2048 || pairs >= 5e8) &&
                                               (nx >= 2048 || pairs >= 1e8)));
        case 128: return pairs >= 1.6e7;
        default: return d > 16 || seeded || pairs > 6e6;
    }
}

// Dwords per row: whole 16-byte units.
static int sad_words(int d) {
    return d <= 16 ? 4 : d <= 32 ? 8 : d <= 64 ? 16 : d <= 112 ? 28 : d <= 128 ? 32 : 64;
}

__device__ __forceinline__ unsigned long long sad_pack(float v, int64_t b) {
    return ((unsigned long long)__float_as_uint(v) << 32) | (unsigned long long)(uint32_t)b;
}

// Entries of a wavefront's queue; half full, it is evaluated.
constexpr int kSadQueue = 384;
constexpr int kSadRowBits = 24;  // chunk rows in an entry (8 bits of query)
// A workgroup one of whose wavefronts has queued this many entries and eight per row of
// its chunk, or holds this many queries that no bound reaches, evaluates the rest of
// the chunk in full (direct): a row costs a wavefront's 128 queries 4 d vector
// operations there, an entry about a fifth of that.  An estimate whose draws are all
// one point at 10^9 times the extent: 2 10^5 x 64 27 -> 2.1 ms, 6 10^4 x 100 15.4 ->
// 1.2; with four queries, exact 20000^2 x 64 with a hundredth of both clouds there took
// 2.0 ms instead of 0.8.
constexpr int kSadPlainFirst = 8192;
constexpr int kSadPlainQueries = 16;

// Up to 16 coordinates from k0 of a row, in registers (clamped past d).
__device__ __forceinline__ void sad_load(const float *__restrict__ x, int d, int k0, bool quads,
                                         float *v) {
    asm volatile("" : "+v"(k0));  // (or the clamped offsets stay in registers)
    if (quads) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4 u =
                ld(reinterpret_cast<const CH_RO float4 *>(ro(x) + min(k0 + 4 * i, d - 4)));
            v[4 * i] = u.x, v[4 * i + 1] = u.y, v[4 * i + 2] = u.z, v[4 * i + 3] = u.w;
        }
    } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = ro(x)[min(k0 + i, d - 1)];
    }
}

// Their bytes; err and excess in steps.  box: (lo_k, inv) per coordinate, inv = 0
// past d.
__device__ __forceinline__ uint4 sad_bytes(const float *v, const float2 *box, float &err,
                                           float &excess) {
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        w[i] = 0u;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int k = 4 * i + c;
            const float2 b = box[k];
            const float t = (v[k] - b.x) * b.y;
            const float tc = fminf(fmaxf(t, 0.0f), 255.0f);
            const float q = rintf(tc);
            err += fabsf(tc - q);
            excess += fabsf(t - tc);
            w[i] |= (uint32_t)q << (8 * c);
        }
    }
    return make_uint4(w[0], w[1], w[2], w[3]);
}

// Every row from t on (the wavefront's groups of four in tiles of TR rows) for its 128
// queries: eight rows and four coordinates at a time, a lane with queries l and l + 64,
// rows wave-uniform (scalar loads).
__device__ __forceinline__ uint4 sad_direct(const float *Xv, int32_t row0, int32_t row1,
                                            const float *Bv, int tv, int lenv, int dv, int TRv,
                                            int first, int stepv, int quadsv) {
    constexpr int NR = 8, Q = 2;
    auto u32 = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    auto ptr = [&](const float *q) {
        const uint64_t a = reinterpret_cast<uint64_t>(q);
        return reinterpret_cast<const float *>(((uint64_t)(uint32_t)u32((int)(a >> 32)) << 32) |
                                               (uint32_t)u32((int)(uint32_t)a));
    };
    const float *B = ptr(Bv);
    const int len = u32(lenv), d = u32(dv), TR = u32(TRv), step4 = u32(stepv);
    const bool quads = u32(quadsv) != 0;
    int t = u32(tv);
    const CH_RO float *xr[Q];
    uint32_t bv[Q];
    int bi[Q];
#pragma unroll
    for (int j = 0; j < Q; ++j) {
        xr[j] = ro(Xv) + (int64_t)(j == 0 ? row0 : row1) * d;
        bv[j] = 0xffffffffu;
        bi[j] = 0;
    }
    const int r0 = u32(first);
    int r = r0;
#pragma unroll 1
    for (; t < len; r = r0, t += TR)
#pragma unroll 1
        for (; r < TR && t + r < len; r += 2 * step4) {
            const CH_RO float *b[NR];
            int row[NR];
            float acc[NR][Q] = {};
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                const int g = r + (i >> 2) * step4;
                row[i] = g < TR ? t + g + (i & 3) : len;
                b[i] = ro(B) + (int64_t)min(row[i], len - 1) * d;
            }
            int k = 0;
#pragma unroll 1
            for (; k + 4 <= d; k += 4) {
                float x[Q][4];
#pragma unroll
                for (int j = 0; j < Q; ++j) {
                    if (quads) {
                        const float4 u = ld(reinterpret_cast<const CH_RO float4 *>(xr[j] + k));
                        x[j][0] = u.x, x[j][1] = u.y, x[j][2] = u.z, x[j][3] = u.w;
                    } else {
#pragma unroll
                        for (int c = 0; c < 4; ++c) x[j][c] = xr[j][k + c];
                    }
                }
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int i = 0; i < NR; ++i) {
                        const float bk = b[i][k + c];
#pragma unroll
                        for (int j = 0; j < Q; ++j) acc[i][j] += fabsf(x[j][c] - bk);
                    }
            }
#pragma unroll 1
            for (; k < d; ++k)
#pragma unroll
                for (int i = 0; i < NR; ++i)
#pragma unroll
                    for (int j = 0; j < Q; ++j) acc[i][j] += fabsf(xr[j][k] - b[i][k]);
#pragma unroll
            for (int i = 0; i < NR; ++i)
#pragma unroll
                for (int j = 0; j < Q; ++j) {  // (bits order like the values, NaN last)
                    const uint32_t a = __float_as_uint(acc[i][j]);
                    if (a < bv[j] && row[i] < len) bv[j] = a, bi[j] = row[i];
                }
        }
    return make_uint4(bv[0], (uint32_t)bi[0], bv[1], (uint32_t)bi[1]);
}

// The same as a function of its own, for the batched kernels, whose registers are
// short (inlined, its values cost the tile loop 30 spilled registers at d = 100).
__device__ __attribute__((noinline)) uint4 sad_direct_call(const float *X, int32_t row0,
                                                           int32_t row1, const float *B, int t,
                                                           int len, int d, int TR, int first,
                                                           int step, int quads) {
    return sad_direct(X, row0, row1, B, t, len, d, TR, first, step, quads);
}

// One chunk of B against the workgroup's queries.  qw (1, 2 or 4) wavefronts
// have queries of their own; 4 / qw share a tile's row groups.  seed (may be
// null): seed[row of X] bounds the query's distance from above.  gthr (may be
// null): the thresholds of all workgroups, all ones at first.
template <int W, bool BATCH>
__device__ __forceinline__ void nnmin_sad(const float *__restrict__ X,
                                          const int32_t *__restrict__ rows, int64_t nx,
                                          const float *__restrict__ seed,
                                          const float *__restrict__ B, int64_t nB, int d,
                                          const uint32_t *__restrict__ lohi, int64_t chunk,
                                          int nchunk, int qw, unsigned long long *best,
                                          uint32_t *gthr, DevParams *p, Blk blk) {
    constexpr int UPR = W / 4;          // 16-byte units per row
    constexpr int RW = 64 / UPR;        // rows a wavefront stores per tile
    constexpr int TR = 4 * RW;          // rows per tile: one unit per thread
    constexpr int Q = 2;                // queries per lane
    constexpr int WQ = 64 * Q;          // queries per wavefront
    constexpr int LPH = W <= 4 ? 1 : W <= 8 ? 2 : W <= 16 ? 4 : W <= 32 ? 8 : 16;
    constexpr int QN = kSadQueue;
    __shared__ uint4 tile_s[2][TR * UPR];
    __shared__ __attribute__((aligned(16))) uint32_t base_s[2][TR];
    __shared__ float2 box_s[4 * W];
    __shared__ uint2 queue[4][QN];
    __shared__ uint2 lead[4][WQ];
    __shared__ unsigned long long best_s[4][WQ];
    __shared__ float off_s[4][WQ];     // threshold = acc grow + off
    __shared__ uint32_t thr_s[4][WQ];
    __shared__ uint32_t top_s[4][WQ];  // settle: each query's least queued sum
    __shared__ int32_t row_s[4][WQ];
    // a word per wavefront: the workgroup is to end its tiles and go on with direct;
    // from this row; entries queued so far
    __shared__ __attribute__((aligned(16))) uint32_t plain_s[2][4];
    __shared__ int32_t rest_s[4], evals_s[4];

    if (p->status != CHAMFER_OK) return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t wgq = (int64_t)qw * WQ, nq = (nx + wgq - 1) / wgq;
    int cb;
    int64_t qb;
    chunk_major(blk.id, nq, nchunk, cb, qb);
    const int64_t b0 = (int64_t)cb * chunk, b1 = min(nB, b0 + chunk);
    if (b0 >= b1) return;  // uniform over the workgroup
    int len = (int)(b1 - b0);
    const int64_t qbase = qb * wgq + (int64_t)(wave & (qw - 1)) * WQ;
    const int phase = wave / qw, step4 = 4 / qw * 4;  // its first row group, rows to the next
    bool active = qbase < nx;
    const float inv = p->sad_inv;
    const bool inbox = p->sad_in != 0;
    const bool quads = (d & 3) == 0 && ((reinterpret_cast<uintptr_t>(X) |
                                         reinterpret_cast<uintptr_t>(B)) & 15) == 0;
    const auto *lo = ro(reinterpret_cast<const float *>(lohi + 2 * d));
    for (int k = tid; k < 4 * W; k += 256)
        box_s[k] = make_float2(lo[min(k, d - 1)], k < d ? inv : 0.0f);
    __syncthreads();

    // eps: error of a computed T (two roundings at up to 255, and the step's);
    // the row part of the bound is at most half a step per coordinate
    const float eps = 6e-5f * (float)d;
    const uint32_t E = (uint32_t)(d / 2 + 3);
    const float rho = (float)(d + 4) * (1.1f / 16777216.0f);
    const float grow = inv * (1.0f + 1.1f * rho + 1e-6f);
    auto thr_of = [&](float off, float acc) {  // NaN, inf: no bound
        const float t = fmaf(acc, grow, off) + fabsf(off) * 2e-7f;
        return t < 4.2e9f ? (uint32_t)fmaxf(t, 0.0f) : 0xffffffffu;
    };

    // ---- B's tiles: a unit of 16 coordinates per thread
    const int fr = wave * RW + lane / UPR, fu = lane % UPR;
    const bool mine = lane < RW * UPR;
    float pr[16];
    auto fetch = [&](int t) {
        sad_load(B + (b0 + min(t + fr, len - 1)) * d, d, 16 * fu, quads, pr);
    };
    auto land = [&](int slot) {
        float e = 0.0f, ex = 0.0f;
        const uint4 w = sad_bytes(pr, &box_s[16 * fu], e, ex);
        float sum = 0.0f;
#pragma unroll
        for (int i = 0; i < UPR; ++i) sum += __shfl(e, lane - fu + i);
        if (mine) {
            tile_s[slot][fr * UPR + fu] = w;
            if (fu == 0) {
                // (0, the lowest, when a coordinate is not a number: such a row answers
                // no query, and as sad_inv is 0 then it rules none out either)
                const float m = ceilf(sum * 1.0001f + eps);
                base_s[slot][fr] = m < (float)E ? E - (uint32_t)m : 0u;
            }
        }
    };
    fetch(0);

    // ---- the queries: bytes in registers, thresholds
    uint32_t x[Q][W];
    uint32_t thr[Q], marg[Q];
    int none = 0;  // queries without a bound
#pragma unroll
    for (int j = 0; j < Q; ++j) {
        const int q = 64 * j + lane;
        const int64_t qi = qbase + q;
        const int64_t row = qi < nx ? (rows ? (int64_t)ro(rows)[qi] : qi) : 0;
        float e = 0.0f, ex = 0.0f;
#pragma unroll
        for (int u = 0; u < UPR; ++u) {
            float v[16];
            sad_load(X + row * d, d, 16 * u, quads, v);
            const uint4 w = sad_bytes(v, &box_s[16 * u], e, ex);
            x[j][4 * u] = w.x, x[j][4 * u + 1] = w.y, x[j][4 * u + 2] = w.z,
            x[j][4 * u + 3] = w.w;
            // packed now, and no loads of later units before (registers)
            asm volatile("" : "+v"(x[j][4 * u]), "+v"(x[j][4 * u + 1]), "+v"(x[j][4 * u + 2]),
                         "+v"(x[j][4 * u + 3]), "+v"(e), "+v"(ex));
            __builtin_amdgcn_sched_barrier(0);
        }
        e = e * 1.0001f;
        const float out = inbox ? ex * 0.99998f : 0.0f;
        const float off = e - out + 4.0f * eps + (float)E + 1.0f;
        // a row known at s is at most s + 2 (its own part) away: excludes sums above,
        // unless its canonical sum may overflow (all rows at infinity are equal, and
        // the lowest index counts)
        const float mg = 2.0f * (e + (float)E) + 8.0f * eps + ex * 0.0002f +
                         2.4f * rho * (256.0f * (float)d + ex) + 4.0f;
        marg[j] = inbox && mg < 1e9f && 256.0f * (float)d + ex < 3e38f * inv ? (uint32_t)mg
                                                                             : 0x7fffffffu;
        uint32_t t = 0u;
        bool live = qi < nx;
        if (live) {
            const unsigned long long known =
                __hip_atomic_load(&best[qi], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            float acc = known != ~0ull ? __uint_as_float((uint32_t)(known >> 32)) : INFINITY;
            if (seed) acc = fminf(acc, ro(seed)[row] * 1.000001f);
            t = thr_of(off, acc);
            if (gthr)
                t = min(t, __hip_atomic_load(&gthr[qi], __ATOMIC_RELAXED,
                                             __HIP_MEMORY_SCOPE_AGENT));
        }
        thr[j] = t;
        const float lost = inv == 0.0f ? INFINITY : inbox ? mg : ex;
        none += __popcll(__ballot(live && !(lost < 255.0f * (float)d)));
        // lanes without a query: no sum is below E - d / 2 - 1 >= 1
        if (!live) marg[j] = 0u;
        thr_s[wave][q] = t;
        off_s[wave][q] = off;
        row_s[wave][q] = (int32_t)row;
        best_s[wave][q] = ~0ull;
    }
    land(0);
    if (TR < len) fetch(TR);
    evals_s[wave] = 0;
    rest_s[wave] = INT_MAX;
    plain_s[0][wave] = 0u;
    plain_s[1][wave] = none >= kSadPlainQueries ? 1u : 0u;

    auto sync_lds = [] {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    const unsigned long long below = (1ull << lane) - 1;
    int cnt = 0;
    // Sums of rows [r, r + 4) of the tile into acc.
    auto sums = [&](int slot, int r, uint32_t (&acc)[4][Q]) {
        const uint4 c = *reinterpret_cast<const uint4 *>(&base_s[slot][r]);
        const uint32_t cs[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < Q; ++j) acc[i][j] = cs[i];
#pragma unroll
        for (int u = 0; u < UPR; ++u)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint4 b = tile_s[slot][(r + i) * UPR + u];
                const uint32_t bw[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int j = 0; j < Q; ++j)
                        acc[i][j] = __builtin_amdgcn_sad_u8(x[j][4 * u + k], bw[k], acc[i][j]);
                if (i == 3 && (u & 1)) __builtin_amdgcn_sched_barrier(0);  // (registers)
            }
    };
    // Rows r .. r + 3 of the chunk that reach a threshold into the queue; true when
    // it is full.
    auto push = [&](const uint32_t (&acc)[4][Q], int r) {
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            uint32_t m = 0xffffffffu;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (r + i < len) m = min(m, acc[i][j]);
            if (m <= thr[j]) thr[j] = min(thr[j], m + marg[j]);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const bool hit = acc[i][j] <= thr[j] && r + i < len;
                const unsigned long long mk = __ballot(hit);
                if (mk == 0) continue;
                if (cnt > QN - 64) return true;
                if (hit)
                    queue[wave][cnt + __popcll(mk & below)] = make_uint2(
                        acc[i][j],
                        (uint32_t)(r + i) | ((uint32_t)(64 * j + lane) << kSadRowBits));
                cnt += __popcll(mk);
            }
        }
        return false;
    };
    // Thresholds after canonical distances in best_s, in thr_s.
    auto lower = [&] {
        sync_lds();
#pragma unroll 1
        for (int q = lane; q < WQ; q += 64) {
            const unsigned long long k = best_s[wave][q];
            if (k != ~0ull) {
                const uint32_t t = thr_of(off_s[wave][q], __uint_as_float((uint32_t)(k >> 32)));
                if (t < thr_s[wave][q]) {
                    thr_s[wave][q] = t;
                    if (gthr && qbase + q < nx)
                        __hip_atomic_fetch_min(&gthr[qbase + q], t, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
        sync_lds();
    };
    auto settle = [&](int t, int step) {
        const int evals = evals_s[wave] + cnt;
        evals_s[wave] = evals;
        if (__builtin_amdgcn_readfirstlane(evals) > kSadPlainFirst + 2 * qw * t) {
            active = false;
            rest_s[wave] = t;
            plain_s[(step >> 4) & 1][wave] = 1u;
        }
        // thresholds to LDS and to the other workgroups, and theirs
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            const int64_t qi = qbase + 64 * j + lane;
            if (gthr && qi < nx) {
                if (thr[j] < thr_s[wave][64 * j + lane])
                    __hip_atomic_fetch_min(&gthr[qi], thr[j], __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
                thr[j] = min(thr[j], __hip_atomic_load(&gthr[qi], __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_AGENT));
            }
            thr_s[wave][64 * j + lane] = thr[j];
            top_s[wave][64 * j + lane] = 0xffffffffu;
        }
        sync_lds();
        // the row of each query's least sum first: its canonical distance excludes
        // most of the others
        for (int i = lane; i < cnt; i += 64)
            atomicMin(&top_s[wave][queue[wave][i].y >> kSadRowBits], queue[wave][i].x);
#pragma unroll 1
        for (int turn = 0; turn < 2; ++turn) {
            sync_lds();
            int n = 0, nl = 0;
            for (int i = 0; i < cnt; i += 64) {
                const uint2 en = queue[wave][min(i + lane, cnt - 1)];
                const int q = (int)(en.y >> kSadRowBits);
                const bool keep = i + lane < cnt && en.x <= thr_s[wave][q];
                const bool first = keep && turn == 0 && en.x == top_s[wave][q];
                unsigned long long mk = __ballot(first);
                const int at = nl + __popcll(mk & below);
                const bool taken = first && at < WQ;
                if (taken) lead[wave][at] = en;
                nl = min(nl + __popcll(mk), WQ);
                mk = __ballot(keep && !taken);
                if (keep && !taken) queue[wave][n + __popcll(mk & below)] = en;
                n += __popcll(mk);
            }
            cnt = n;
            sync_lds();
            const uint2 *list = turn == 0 ? lead[wave] : queue[wave];
            const int todo = turn == 0 ? nl : n;
            constexpr int M = 1;  // passes in flight
            for (int i = 0; i < todo; i += 64 / LPH * M) {
                const float *xp[M], *bp[M];
                float acc[M];
                uint32_t ey[M];
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    ey[m] = list[min(i + m * (64 / LPH) + lane / LPH, todo - 1)].y;
                    xp[m] = X + (int64_t)row_s[wave][ey[m] >> kSadRowBits] * d;
                    bp[m] = B + (b0 + (int64_t)(ey[m] & ((1u << kSadRowBits) - 1u))) * d;
                }
                hit_acc<CHAMFER_L1, LPH, 16, M>(xp, bp, d, acc);
#pragma unroll
                for (int m = 0; m < M; ++m)
                    if (i + m * (64 / LPH) + lane / LPH < todo && lane % LPH == LPH - 1)
                        atomicMin(&best_s[wave][ey[m] >> kSadRowBits],
                                  sad_pack(acc[m], b0 + (int64_t)(ey[m] &
                                                                  ((1u << kSadRowBits) - 1u))));
            }
            lower();
            if (cnt == 0) break;
        }
        cnt = 0;
#pragma unroll
        for (int j = 0; j < Q; ++j) thr[j] = min(thr[j], thr_s[wave][64 * j + lane]);
    };
    // Rows [r, r + 4) of the chunk evaluated for all of the wavefront's queries.
    auto evaluate = [&](int r) {
#pragma unroll 1
        for (int q = lane; q < WQ; q += 64) {
            if (qbase + q >= nx) break;
            const auto *xr = ro(X) + (int64_t)row_s[wave][q] * d;
            float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
            for (int k = 0; k < d; ++k) {
                const float xk = xr[k];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    acc[i] += fabsf(xk - ro(B)[(b0 + min(r + i, len - 1)) * d + k]);
            }
            unsigned long long m = ~0ull;
#pragma unroll
            for (int i = 0; i < 4; ++i) m = min(m, sad_pack(acc[i], b0 + min(r + i, len - 1)));
            atomicMin(&best_s[wave][q], m);
        }
        lower();
#pragma unroll
        for (int j = 0; j < Q; ++j) thr[j] = min(thr[j], thr_s[wave][64 * j + lane]);
    };

    __syncthreads();
    // (16 steps write one set of words, read after the barrier of the last of them;
    // by the time that it is written again every wavefront has passed that read)
    auto any_plain = [&](int g) {
        const uint4 w = *reinterpret_cast<const uint4 *>(plain_s[g & 1]);
        return __builtin_amdgcn_readfirstlane((int)(w.x | w.y | w.z | w.w)) != 0;
    };
    if (any_plain(1)) len = 0;
    for (int t = 0, slot = 0, step = 0;; t += TR, slot ^= 1, ++step) {
        const bool more = t + TR < len;  // uniform
        if (more) land(slot ^ 1);
        if (t + 2 * TR < len) fetch(t + 2 * TR);
        if (active) {
            int tries = 0, r = 4 * phase;
            for (;;) {
                bool full = false;
                if (r < TR && t + r < len) {
                    uint32_t acc[4][Q];
                    sums(slot, r, acc);
                    bool any = false;
#pragma unroll
                    for (int j = 0; j < Q; ++j)
                        any |= min(min(acc[0][j], acc[1][j]), min(acc[2][j], acc[3][j])) <= thr[j];
                    if (__ballot(any) != 0) full = push(acc, t + r);
                }
                // no room: the rows are taken again, against the thresholds of those
                // evaluated meanwhile, and the third time (duplicates) in full
                tries = full ? tries + 1 : 0;
                const bool whole = tries == 3;
                if (!full || whole) r += step4;
                const bool end = !(r < TR && t + r < len);
                if (full || cnt >= QN / 2 || (end && !more && cnt > 0)) settle(t, step);
                if (whole) {
                    evaluate(t + r - step4);
                    tries = 0;
                }
                if (end || !active) break;
            }
        }
        if (!more) break;
        if (gthr && active && (step & 15) == 15) {
#pragma unroll
            for (int j = 0; j < Q; ++j)
                thr[j] = min(thr[j], __hip_atomic_load(&gthr[min(qbase + 64 * j + lane, nx - 1)],
                                                       __ATOMIC_RELAXED,
                                                       __HIP_MEMORY_SCOPE_AGENT));
        }
        __syncthreads();
        if ((step & 15) == 15 && any_plain(step >> 4)) len = min(len, t + 2 * TR);
    }
    if (qbase >= nx) return;
    const int rest = min(len, __builtin_amdgcn_readfirstlane(rest_s[wave]));
    len = (int)(b1 - b0);
    if (rest < len) {
        const int32_t r0 = row_s[wave][lane], r1 = row_s[wave][64 + lane];
        const uint4 f = BATCH ? sad_direct_call(X, r0, r1, B + b0 * d, rest, len, d, TR, 4 * phase,
                                                step4, quads)
                              : sad_direct(X, r0, r1, B + b0 * d, rest, len, d, TR, 4 * phase,
                                           step4, quads);
        if (f.x != 0xffffffffu)
            atomicMin(&best_s[wave][lane],
                      ((unsigned long long)f.x << 32) | (uint32_t)(b0 + f.y));
        if (f.z != 0xffffffffu)
            atomicMin(&best_s[wave][64 + lane],
                      ((unsigned long long)f.z << 32) | (uint32_t)(b0 + f.w));
    }
    sync_lds();
#pragma unroll
    for (int j = 0; j < Q; ++j) {
        const int64_t qi = qbase + 64 * j + lane;
        const unsigned long long k = best_s[wave][64 * j + lane];
        if (qi < nx && k != ~0ull) atomicMin(&best[qi], k);
    }
}

// Wavefronts per SIMD that the queries' registers allow.
template <int W>
__host__ __device__ constexpr int sad_waves() {
    return W <= 8 ? 4 : W <= 32 ? 3 : 2;
}

template <int W>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sad_waves<W>())))
void k_nnmin_sad(const float *__restrict__ X, const int32_t *__restrict__ rows, int64_t nx,
                 const float *__restrict__ seed, const float *__restrict__ B, int64_t nB, int d,
                 const uint32_t *__restrict__ lohi, int64_t chunk, int nchunk, int qw,
                 unsigned long long *best, uint32_t *gthr, DevParams *p) {
    nnmin_sad<W, false>(X, rows, nx, seed, B, nB, d, lohi, chunk, nchunk, qw, best, gthr, p, grid_blk());
}

static int sad_resident_wgs(int d) {
    const int W = sad_words(d);
    return 256 * (W <= 8 ? sad_waves<8>() : W <= 32 ? sad_waves<32>() : sad_waves<64>());
}

// Wavefronts with queries of their own (qw) and the split of B.  target 0: as many
// chunks as give the least number of rounds of resident workgroups times the rows
// of a round (a workgroup starts and ends in the time of about 128 rows); qw is
// lowered where too few workgroups would be left.  cold: the queries start without a
// distance.  Every workgroup of few such queries evaluates its first rows and writes
// to the same few (100 x 100000 x 20 in 768 chunks 385 us, in 256 130; 500 x 100000
// x 20 188 and 145, x 100 214 and 300).
static NNGeom sad_geom(int64_t nx, int64_t nB, int d, bool cold, int64_t target, int32_t &qw) {
    const int64_t slots = sad_resident_wgs(d);
    const bool few = cold && nx <= (sad_words(d) <= 8 ? 512 : 256);
    const int64_t cmin = (nB + 65535) / 65536,
                  cmax = few ? std::min((nB + 155) / 156, std::max<int64_t>(256, cmin))
                             : (nB + 63) / 64;
    NNGeom g;
    for (qw = nx > 256 ? 4 : nx > 128 ? 2 : 1;; qw /= 2) {
        const int64_t nq = (nx + 128 * qw - 1) / (128 * qw);
        auto whole = [&](int64_t nc) {  // one chunk's workgroups share an XCD
            if (nc < cmin) nc = cmin;
            if (nc > cmax) nc = cmax;
            return nc > 1 ? (nc + 7) / 8 * 8 : (int64_t)1;
        };
        int64_t nc = whole(((target > 0 ? target : slots) + nq - 1) / nq);
        if (target <= 0) {
            double least = 1e300;
            for (int64_t c = whole(1); c <= whole(4 * slots / nq + 1); c = c < 8 ? 8 : c + 8) {
                const double rounds = (double)((nq * c + slots - 1) / slots);
                const double cost = rounds * ((double)nB / (double)c + 128.0);
                if (cost < least) least = cost, nc = c;
            }
        }
        g.chunk = ((nB + nc - 1) / nc + 3) / 4 * 4;
        g.nchunk = (int32_t)nc;
        g.blocks = nq * nc;
        if (qw == 1 || g.blocks >= 256 || (target > 0 && g.blocks >= target)) return g;
    }
}

NNGeom sad_geom(int64_t nx, int64_t nB, int d, int64_t target, int32_t &qw) {
    return sad_geom(nx, nB, d, false, target, qw);
}

int64_t sad_launch_queries(int64_t nx, int64_t nB, int d) {
    int32_t qw;
    while (nx > 1 && sad_geom(nx, nB, d, false, 0, qw).blocks > kMaxLaunchWGs) nx = (nx + 1) / 2;
    return nx;
}

hipError_t launch_nnmin_sad(const float *X, const int32_t *rows, int64_t nx, const float *seed,
                            const float *B, int64_t nB, int d, const uint32_t *lohi,
                            unsigned long long *best, uint32_t *gthr, DevParams *p,
                            hipStream_t st) {
    if (nx <= 0) return hipSuccess;
    const int64_t part = sad_launch_queries(nx, nB, d);
    if (part < nx) {
        for (int64_t q = 0; q < nx; q += part) {
            const int64_t x0 = rows ? 0 : q;  // first row of X
            const hipError_t e = launch_nnmin_sad(
                X + x0 * d, rows ? rows + q : nullptr, nx - q < part ? nx - q : part,
                seed ? seed + x0 : nullptr, B, nB, d, lohi, best + q, gthr ? gthr + q : nullptr, p,
                st);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    int32_t qw;
    const NNGeom g = sad_geom(nx, nB, d, seed == nullptr, 0, qw);
#define CH_SAD(W)                                                                           \
    k_nnmin_sad<W><<<(unsigned)g.blocks, 256, 0, st>>>(X, rows, nx, seed, B, nB, d, lohi,   \
                                                       g.chunk, g.nchunk, qw, best, gthr, p)
    switch (sad_words(d)) {
        case 4: CH_SAD(4); break;
        case 8: CH_SAD(8); break;
        case 16: CH_SAD(16); break;
        case 28: CH_SAD(28); break;
        case 32: CH_SAD(32); break;
        default: CH_SAD(64); break;
    }
#undef CH_SAD
    return hipGetLastError();
}

// ---------------------------------------------------------------- batched

constexpr unsigned kGridNNSad = 1024;

template <int W>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sad_waves<W>())))
void kb_nn_sad(const Batch *__restrict__ bt) {
    batch_loop(bt, kBsNN, [&](const Job &J, Blk b) {
        if (J.nn_vector) return;
        nnmin_sad<W, true>(glb(J.A), glb(J.idx), J.T, glb(J.D), glb(J.B), J.nB, J.d, glb(J.lohi),
                     J.nn_chunk, J.nn_nchunk, J.nn_qw, glb(J.best), glb(J.gthr), glb(J.p), b);
    });
}

hipError_t launch_batch_sad(const Batch *bt, int d, hipStream_t st) {
    switch (sad_words(d)) {
        case 4: kb_nn_sad<4><<<kGridNNSad, 256, 0, st>>>(bt); break;
        case 8: kb_nn_sad<8><<<kGridNNSad, 256, 0, st>>>(bt); break;
        case 16: kb_nn_sad<16><<<kGridNNSad, 256, 0, st>>>(bt); break;
        case 28: kb_nn_sad<28><<<kGridNNSad, 256, 0, st>>>(bt); break;
        case 32: kb_nn_sad<32><<<kGridNNSad, 256, 0, st>>>(bt); break;
        default: kb_nn_sad<64><<<kGridNNSad, 256, 0, st>>>(bt); break;
    }
    return hipGetLastError();
}

}  // namespace chamfer
