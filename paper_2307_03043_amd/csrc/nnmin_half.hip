// Exact l2 nearest neighbours on the FP16 matrix cores (gfx950
// v_mfma_f32_32x32x16_f16), returning the same canonical float32 result as
// the VALU form: the minimum over b of (fma-chain accumulator of
// (x_k - b_k)^2 in ascending k, b), ties to the lower b.
//
// The matrix cores only rule rows out.  With c a centre near B's mean and 2^he
// a common scale (calib_final), y = (b - c) 2^he and z = (x - c) 2^he are held
// as h = fp16(.), which is within 2^-11 of the value, and the tile pass forms
// v = z~.y~ - |y|^2 / 2 for every (x, b): |z - y|^2 = |z|^2 - 2 v up to the
// error 2 e below, so a row can only reach the canonical minimum if its v
// reaches a threshold that follows from the best canonical distance known for
// the query.  Rows that do are queued in LDS per wavefront and evaluated with
// the canonical distance, 64 at a time; their minimum raises the threshold.
// The result is the canonical minimum whatever the order: every row whose
// bound does not exclude it is evaluated, and the per-query minima merge with
// 64-bit atomicMin of (accumulator bits << 32 | b).
//
// The error of v is bounded by a part of the query and a part of the row
// (half_err); the row's is added to -|y|^2 / 2 and the query's taken off its
// threshold, so neither a row nor a query far out loosens the bounds of others.
// The rounding errors of the operands, the largest term, are measured when the
// tables are written (about 0.4 of the worst case 2^-11 per operand).  A query
// whose error is not finite (a coordinate outside FP16's range, an overflowing
// norm) has the operand 0 and the threshold -inf: every row is evaluated.
//
// d <= 10 (point clouds): FP16 alone would leave many rows of a dense cloud to
// evaluate, and 3 d <= 32 slots of the matrix product are free, so a row holds
// [h | m | h], m = fp16(y - h), against the query's [h | h | m]: three
// products, errors of 2^-21.  B's rows are split while their tile is staged
// (no table).  12 <= d <= 256: one product, B's table written by the kernel
// that hashes B, or by k_half_rows.
//
// Why one FP16 product instead of the three (four) BF16 products of a
// two-term split: the pass is bound by the matrix cores, and the rows left to
// evaluate are few (about one in 10^4) because a threshold is carried along
// and seeded with the CrudeNN distance of a draw.
#include <algorithm>
#include <cfloat>
#include <climits>
#include <cmath>
#include <type_traits>

#include "internal.h"

namespace chamfer {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));

// Slots of a row in the matrix product.
__host__ __device__ inline int half_slots(int d) {
    return d <= 5 ? 16 : d <= 32 ? 32 : d <= 64 ? 64 : d <= 128 ? 128 : 256;
}

bool half_supported(int d, int metric) {
    return metric == CHAMFER_L2 && (d <= kHalfRawDim || (d >= 12 && d <= 256));
}
bool half_tabled(int d) { return d > kHalfRawDim; }

// Three dimensions have a compiled vector form, which starts and ends faster.  A pass
// whose queries have no distance to start from (seeded: they do) takes it while B is
// small, or the product is (exact calls in us, matrix cores and vector: 10^6 x 1000 350
// and 208, 10^5 x 10^4 198 and 184, 10^5 x 20000 297 and 342; 30000^2 181 and 172,
// 60000 x 30000 263 and 317; 10000 x 40000 97 and 92, 20000 x 40000 141 and 161;
// 400 x 10^5 58 and 55, 5000 x 10^5 117 and 120, 1500 x 150000 83 and 92).
bool half_pays(int64_t nx, int64_t nB, int d, bool seeded) {
    if (d != 3 || seeded) return true;
    const double pairs = (double)nx * (double)nB;
    return nB > 12288 && pairs > (nB <= 32768 ? 9e8 : nB <= 100000 ? 4e8 : 0.0);
}
size_t half_table_bytes(int64_t n, int d) { return (size_t)n * half_slots(d) * 2; }

// Bound of the relative error of the canonical accumulator against the exact
// squared distance.
__host__ __device__ inline float half_rho(int d) {
    return (float)(d + 4) * (1.1f / 16777216.0f);
}
// The query's part of the error bound (zt >= |z~|, ze >= |z - z~|; over B
// by >= |y|, be >= |y - y~|).
__host__ __device__ inline float half_err_query(const HalfErr &h, float zt, float ze, float by,
                                                float be) {
    const float a = h.q2 * zt * zt + h.e2q * ze * ze, b = zt * (be + h.p1 * by) + ze * by;
    return ((b < a ? b : a) + h.q1 * zt) * 1.000001f + 1e-30f;
}

__device__ __forceinline__ unsigned long long half_pack(float v, int64_t b) {
    return ((unsigned long long)__float_as_uint(v) << 32) | (unsigned long long)(uint32_t)b;
}

// ------------------------------------------------------------- row tables

// Rows per thread group.  B's maxima cost two global atomics per workgroup, so
// its workgroups take four once they fill the chip; few rows, and those of a draw, are
// spread as wide as they go (2000 x 128 draws: 6.9 us with four passes, 4.6 with one;
// 2500 queries and 20001 rows x 16: 9.3 and 5).
constexpr int64_t kHalfRowsWide = 1 << 18;
__host__ __device__ inline int half_row_passes(int64_t n, int slots, bool isB) {
    return isB && n * (slots / 8) > kHalfRowsWide ? 4 : 1;
}

// Rows of 12 <= d <= 256 coordinates: slots / 8 consecutive lanes per row, 8
// coordinates each.  For queries (rows may pick them) stat[r] = (|z|^2, |z|
// up, |z - z~| up, 0), and a row that leaves FP16's range is zero; for B nbh[r]
// = half_norm and the maxima of |y|^2 and
// |y - y~|^2 in p (one atomic each per workgroup).
__device__ __forceinline__ void half_rows(const float *__restrict__ X,
                                          const int32_t *__restrict__ rows, int64_t n, int d,
                                          int slots, const uint32_t *__restrict__ lohi,
                                          uint16_t *out, float4 *stat, float *nbh, DevParams *p,
                                          Blk blk) {
    __shared__ uint32_t mx[2];
    if (threadIdx.x < 2) mx[threadIdx.x] = 0u;
    __syncthreads();
    if (p->status != CHAMFER_OK) return;
    const int per = slots / 8;
    const int he = p->he;
    const auto *cen = half_centre(lohi, d);
    const int64_t total = n * per;
    const HalfErr he_ = half_err(d, slots);
    const int passes = half_row_passes(n, slots, nbh != nullptr);
    uint32_t my = 0u, me = 0u;
#pragma unroll 1
    for (int64_t t = blk.id * (256 * passes) + threadIdx.x, i = 0; i < passes && t < total;
         ++i, t += 256) {
        const int64_t r = t / per;
        const int k0 = (int)(t - r * per) * 8;
        const int64_t src = rows ? (int64_t)ro(rows)[r] : r;
        const auto *x = ro(X) + src * d;
        float xv[8];
        if ((d & 3) == 0 && k0 + 8 <= d && (reinterpret_cast<uintptr_t>(X) & 15) == 0) {
            const float4 u = ld(reinterpret_cast<const CH_RO float4 *>(x + k0));
            const float4 v = ld(reinterpret_cast<const CH_RO float4 *>(x + k0 + 4));
            xv[0] = u.x, xv[1] = u.y, xv[2] = u.z, xv[3] = u.w;
            xv[4] = v.x, xv[5] = v.y, xv[6] = v.z, xv[7] = v.w;
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) xv[i] = x[min(k0 + i, d - 1)];
        }
        uint32_t w[4];
        float s2 = 0.0f, e2 = 0.0f;
#pragma unroll
        for (int i = 0; i < 8; i += 2) {
            uint32_t hb[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int k = k0 + i + q;
                const float v = k < d ? ldexpf(xv[i + q] - cen[min(k, d - 1)], he) : 0.0f;
                const _Float16 h = half_of(v);
                const float e = half_rest(v, h);
                s2 = fmaf(v, v, s2);
                e2 = fmaf(e, e, e2);
                hb[q] = half_bits(h);
            }
            w[i / 2] = hb[0] | (hb[1] << 16);
        }
        for (int off = per / 2; off > 0; off >>= 1) {
            s2 += __shfl_xor(s2, off);
            e2 += __shfl_xor(e2, off);
        }
        const bool in = isfinite(s2 + e2);
        *reinterpret_cast<uint4 *>(out + (size_t)r * slots + k0) =
            in ? make_uint4(w[0], w[1], w[2], w[3]) : make_uint4(0u, 0u, 0u, 0u);
        if (k0 == 0) {
            if (stat) {
                stat[r] = half_stat(s2, e2);
            } else {
                nbh[r] = in ? half_norm(s2, e2, he_.s2, he_.e2) : kHalfAlways;
                my = max(my, __float_as_uint(s2));
                me = max(me, __float_as_uint(e2));
            }
        }
    }
    if (nbh == nullptr) return;
    for (int off = 32; off > 0; off >>= 1) {
        my = max(my, (uint32_t)__shfl_xor((int)my, off));
        me = max(me, (uint32_t)__shfl_xor((int)me, off));
    }
    if ((threadIdx.x & 63) == 0) {
        atomicMax(&mx[0], my);
        atomicMax(&mx[1], me);
    }
    __syncthreads();
    if (threadIdx.x < 2) rep_max(p->half_rep + threadIdx.x, blk.id, mx[threadIdx.x]);
}

// B's table and then the queries' in one launch (either may be absent).
__global__ __launch_bounds__(256) void k_half_rows(
    const float *__restrict__ B, int64_t nB, uint16_t *bs, float *nbh, int64_t nbB,
    const float *__restrict__ X, const int32_t *__restrict__ rows, int64_t nx, uint16_t *xs,
    float4 *stat, int d, int slots, const uint32_t *__restrict__ lohi, DevParams *p) {
    const int64_t b = blockIdx.x;
    if (b < nbB)
        half_rows(B, nullptr, nB, d, slots, lohi, bs, nullptr, nbh, p, Blk{b, nbB});
    else
        half_rows(X, rows, nx, d, slots, lohi, xs, stat, nullptr, p,
                  Blk{b - nbB, (int64_t)gridDim.x - nbB});
}

int64_t half_row_blocks(int64_t n, int d, bool isB) {
    const int64_t per_wg = 256 * half_row_passes(n, half_slots(d), isB);
    return (n * (half_slots(d) / 8) + per_wg - 1) / per_wg;
}

hipError_t launch_half_rows(const float *B, int64_t nB, uint16_t *bs, float *nbh, const float *X,
                            const int32_t *rows, int64_t nx, uint16_t *xs, float4 *stat, int d,
                            const uint32_t *lohi, DevParams *p, hipStream_t st) {
    const int64_t nbB = B ? half_row_blocks(nB, d, true) : 0,
                  nbX = X ? half_row_blocks(nx, d, false) : 0;
    if (nbB + nbX <= 0) return hipSuccess;
    if (nbB + nbX > kMaxLaunchWGs && nbX > 0) {  // the queries in halves, B with the first
        const int64_t h = nx / 2;
        const hipError_t e = launch_half_rows(B, nB, bs, nbh, X, rows, h, xs, stat, d, lohi, p, st);
        if (e != hipSuccess) return e;
        return launch_half_rows(nullptr, 0, bs, nbh, rows ? X : X + h * d, rows ? rows + h : nullptr,
                                nx - h, xs + h * half_slots(d), stat + h, d, lohi, p, st);
    }
    k_half_rows<<<(unsigned)(nbB + nbX), 256, 0, st>>>(B, nB, bs, nbh, nbB, X, rows, nx, xs, stat,
                                                       d, half_slots(d), lohi, p);
    return hipGetLastError();
}

// -------------------------------------------------------------- tile pass

// A workgroup is two wavefronts of queries times two of rows: a wavefront
// keeps NB blocks of 32 queries in registers and takes every other 32-row
// block of the tile, so a 1 KB operand read from LDS feeds NB matrix products
// (with NB = 2 the LDS reads took as long as the matrix cores).
// A small launch (half_small) is bound by latencies, most of all those of the
// rows evaluated at the end of a chunk, and takes NB = 2: half the queries per
// wavefront, longer chunks, and registers for more rows in flight.
__host__ __device__ constexpr int half_nb(int slots, bool small) {
    return slots > 128 || small ? 2 : 4;  // at 256 slots 64 queries take 128 registers
}
// Rows per LDS tile: 8 to 32 KB of operands, 512 or more cycles of matrix work
// per wavefront and barrier (RAW: a row per thread).
template <int DP, bool RAW>
__host__ __device__ constexpr int half_tile_rows() {
    return RAW ? 256 : DP <= 64 ? 128 : 64;
}
// Queue of (v, row, query) per wavefront, of what LDS leaves for two (three up
// to 32 slots) workgroups per CU; a pass over it starts when half of it is full
// (or the chunk ends).  RAW: it also holds 64 queries' operands at first.
template <int DP, bool RAW>
__host__ __device__ constexpr int half_queue() {
    return RAW ? (DP == 16 ? 320 : 512) : DP == 32 ? 224 : DP == 64 ? 256 : DP == 128 ? 320 : 128;
}
constexpr int kHalfRowBits = 25;  // chunk rows in a queue entry (7 bits of query)
// d <= kHalfRawDim: a workgroup one of whose wavefronts has queued this many entries
// and one per row of its chunk evaluates the rest of the chunk in full (direct).
// Where no bound tells rows apart (a cloud 10^5 beside B; a hundredth of both clouds at
// 10^9 times the extent), exact 40000^2 x 3 takes 0.58 and 0.44 ms, 1.54 and 1.73
// without; with 1024 here one far row of B set it off (0.30 -> 0.35 ms).
constexpr int kPlainFirst = 2048;

// Thresholds known to other workgroups, one word per query: smaller is a
// higher threshold, all ones (which decodes to NaN, dropped by fmaxf) is none.
__device__ __forceinline__ uint32_t thr_code(float t) { return ~float_to_ordered(t); }
__device__ __forceinline__ float thr_decode(uint32_t c) { return ordered_to_float(~c); }

// Loads straight to LDS: 16 (4) bytes per lane from the lane's address to LDS
// byte address `to` + 16 (4) lane (to: wave-uniform).  Written as assembly so
// that the compiler does not hold up reads of the tile in use until the loads
// of the next ones have landed; lds_wait and a barrier separate a load from its
// readers.  They have no register results, and nothing else in these kernels
// uses m0.  _sc0: past the L1, _sc1: past the XCD's L2.
__device__ __forceinline__ void lds_load16(const void *from, uint32_t to) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off"
                 :
                 : "s"(to), "v"(from)
                 : "memory");
}
__device__ __forceinline__ void lds_load4(const void *from, uint32_t to) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off"
                 :
                 : "s"(to), "v"(from)
                 : "memory");
}
__device__ __forceinline__ void lds_load4_sc0(const void *from, uint32_t to) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off sc0"
                 :
                 : "s"(to), "v"(from)
                 : "memory");
}
__device__ __forceinline__ void lds_load4_sc1(const void *from, uint32_t to) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off sc1"
                 :
                 : "s"(to), "v"(from)
                 : "memory");
}
// All but the wavefront's N newest memory operations are done, and its LDS ones.
template <int N>
__device__ __forceinline__ void lds_wait() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"(N) : "memory");
}
__device__ __forceinline__ uint32_t lds_address(const void *p) {
    return __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char *)p);
}
// A workgroup barrier that leaves loads in flight (lds_wait comes first).
__device__ __forceinline__ void bare_barrier() {
    asm volatile("s_barrier" : : : "memory");
}

// One chunk of B against the workgroup's queries.  RAW (d <= 10): rows of B
// are read as float32 and split when their tile is stored; the queries too.
// seed (may be null): seed[row of X] is an upper bound of the query's
// distance.  gthr[q] (may be null): the thresholds of all workgroups (thr_code),
// in copies gstride words apart, one per XCD, when gstride is not 0.
template <int DP, bool RAW, int NB>
__device__ __forceinline__ void nnmin_half(
    const float *__restrict__ X, const int32_t *__restrict__ rows, int64_t nx,
    const uint16_t *__restrict__ Xs, const float4 *__restrict__ stat,
    const float *__restrict__ seed, const float *__restrict__ B, const uint16_t *__restrict__ Bs,
    int64_t nB, int d, const float *__restrict__ nbh, const uint32_t *__restrict__ lohi,
    int64_t chunk, int nchunk, unsigned long long *best, uint32_t *gthr,
    int64_t gstride, DevParams *p, Blk blk) {
    constexpr int WQ = 32 * NB;             // queries per wavefront
    constexpr int NS = DP / 16;             // matrix products per 32 x 32 block
    constexpr int TR = half_tile_rows<DP, RAW>();
    constexpr int NH = TR / 32;             // 32-row blocks per tile
    constexpr int RB = 2 * DP;              // bytes per row
    constexpr int UPR = RB / 16;            // 16-byte units per row
    constexpr int PER_T = TR * UPR / 256;   // units per thread and tile
    constexpr int RPI = 256 / UPR;          // rows per load pass
    constexpr int KH = DP == 16 ? 5 : 10;   // RAW: first slot of m; 2 KH: of the second h
    constexpr int LPH = RAW ? 1 : DP / 16;  // lanes per evaluated row
    // Unit u of row r is kept at position u ^ swz(r), so the 16-byte reads of
    // 16 consecutive rows at one unit hit 64 distinct banks; the rows have no
    // padding, as the loads that go straight to LDS need.
    constexpr int RPB = RB >= 256 ? 1 : 256 / RB;  // rows per 256 bytes of banks
    auto swz = [](int r) { return (r / RPB) & (UPR < 16 ? UPR - 1 : 15); };
    // Tiles: one in use, two on their way (a load takes about as long as two
    // tiles' work), one at 256 slots (LDS); RAW: one on its way, in registers.  A
    // tile holds the rows' operands, then their -|y|^2 / 2.
    constexpr int TB = TR * RB + TR * 4;
    constexpr int NT = RAW || DP == 256 ? 2 : 3;
    __shared__ __attribute__((aligned(16))) uint8_t tiles[NT * TB];
    constexpr int QN = half_queue<DP, RAW>();
    static_assert(!RAW || QN * 8 >= 64 * RB, "64 queries' operands");
    __shared__ __attribute__((aligned(16))) uint2 queue[4][QN];
    __shared__ unsigned long long best_s[4][WQ];
    __shared__ float thr_s[4][WQ];
    __shared__ int32_t row_s[4][WQ];
    __shared__ float tlo_s[4][WQ];
    __shared__ float marg_s[4][WQ];
    __shared__ uint32_t seen_s[4][WQ];  // gthr as last read (written by look)
    __shared__ uint32_t vtop_s[4][WQ];  // settle: each query's largest queued v,
    __shared__ uint2 lead[4][WQ];       // and its row
    // d <= kHalfRawDim, a word per wavefront: the workgroup is to end its tiles and go
    // on with direct; from this row; entries queued so far (scalar registers are short)
    __shared__ __attribute__((aligned(16))) uint32_t plain_s[2][4];
    __shared__ int32_t rest_s[4], evals_s[4];

    const int32_t status = p->status;  // (looked at once the first loads are out)
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = lane >> 5, j = lane & 31;
    int cb;
    int64_t qb;
    // each XCD starts its chunk at another query block, so that a query's chunks
    // follow one another and all but the first start with a threshold
    const int64_t nq = (nx + 2 * WQ - 1) / (2 * WQ);
    chunk_major(blk.id, nq, nchunk, cb, qb);
    qb = (qb + (cb & 7) * nq / 8) % nq;
    gthr += (cb & 7) * gstride;
    const int64_t qbase = (qb * 2 + (wave >> 1)) * WQ;
    const int64_t b0 = (int64_t)cb * chunk;
    const int64_t b1 = min(nB, b0 + chunk);
    if (b0 >= b1) return;  // uniform over the workgroup
    bool wave_active = qbase < nx;
    int len = (int)(b1 - b0);
    const int he = p->he;
    const auto *cen = half_centre(lohi, d);
    const HalfErr err = half_err(d, DP);
    // Thresholds are shared through gthr: read every fourth tile and before rows
    // are evaluated, written then and after; by draws with long chunks also as soon
    // as a score raises one (exact pass of 2000 draws: 2 10^5 x 3 points 58 -> 54
    // us, 10^5 x 128 116 -> 111; all-points passes of 2500 x 20001 lose 10%).
    const bool share = gthr != nullptr && nchunk > 1, eager = gstride != 0 && len > 1024;
    // A copy per XCD is used through that XCD's L2: workgroup-scope atomics, and
    // loads past the L1 only.  Were its users on several XCDs, they would see
    // fewer of each other's thresholds; every value stored is valid.
    const bool local = gstride != 0;
    auto gthr_raise = [&](int q, float t) {
        if (local)
            __hip_atomic_fetch_min(&gthr[qbase + q], thr_code(t), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
        else
            __hip_atomic_fetch_min(&gthr[qbase + q], thr_code(t), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
    };

    // ---- B's tiles: fetch(tile, t) starts the loads of the tile at row t
    // (straight to LDS; RAW: into registers, split and stored by land).  Rows
    // past the chunk are read at its last row, so every load is in bounds;
    // push skips them.
    float pr[RAW ? KH : 1];
    const int fr0 = tid / UPR, fu = tid - (tid / UPR) * UPR;
    const uint32_t tiles_at = lds_address(tiles);
    auto fetch = [&](int slot, int t) {
        if constexpr (RAW) {
            const auto *src = ro(B) + (b0 + min(t + tid, len - 1)) * d;
#pragma unroll
            for (int k = 0; k < KH; ++k) pr[k] = src[min(k, d - 1)];
        } else {
            const uint8_t *src = reinterpret_cast<const uint8_t *>(Bs) + b0 * RB;
#pragma unroll
            for (int i = 0; i < PER_T; ++i) {
                const int r = fr0 + i * RPI;
                const uint8_t *a =
                    src + (size_t)min(t + r, len - 1) * RB + ((fu ^ swz(r)) * 16);
                lds_load16(a, tiles_at + slot * TB + i * 4096 + wave * 1024);
            }
            // wavefront w: 64 rows' norms (the same ones by several when TR < 256)
            const int nr = (wave * 64) % TR;
            lds_load4(nbh + b0 + min(t + nr + lane, len - 1),
                      tiles_at + slot * TB + TR * RB + nr * 4);
        }
    };
    auto land = [&](int slot) {
        if constexpr (RAW) {
            uint8_t *tile = tiles + slot * TB;
            uint32_t hb[KH], mb[KH];
            float s2 = 0.0f;
#pragma unroll
            for (int k = 0; k < KH; ++k) {
                const float v = k < d ? ldexpf(pr[k] - cen[min(k, d - 1)], he) : 0.0f;
                const _Float16 h = half_of(v);
                s2 = fmaf(v, v, s2);
                hb[k] = half_bits(h);
                mb[k] = half_bits(half_of(v - (float)h));
            }
            const bool in = s2 < 4e9f;  // kHalfRawReach squared: no coordinate above 2^15.98
            if (!in) {
#pragma unroll
                for (int k = 0; k < KH; ++k) hb[k] = mb[k] = 0u;
            }
#pragma unroll
            for (int u = 0; u < UPR; ++u) {
                uint32_t w[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint32_t a[2];
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        const int s = 8 * u + 2 * i + q;
                        a[q] = s < KH ? hb[s]
                                      : s < 2 * KH ? mb[s - KH] : s < 3 * KH ? hb[s - 2 * KH] : 0u;
                    }
                    w[i] = a[0] | (a[1] << 16);
                }
                *reinterpret_cast<uint4 *>(&tile[tid * RB + ((u ^ swz(tid)) * 16)]) =
                    make_uint4(w[0], w[1], w[2], w[3]);
            }
            *reinterpret_cast<float *>(&tile[TR * RB + tid * 4]) =
                in ? half_norm(s2, 0.0f, err.s2, 0.0f) : kHalfAlways;
        }
    };
    // loads of a wavefront per step: a tile and its norms; every fourth step also
    // the thresholds (look)
    constexpr int LPS = PER_T + 1, LPL = LPS + WQ / 64;
    fetch(0, 0);
    if constexpr (RAW) land(0);
    if ((RAW || NT == 3) && TR < len) fetch(1, TR);
    // the queries' operands: lane (g, j) holds coordinates
    // [g DP / 2, (g + 1) DP / 2) of queries 32 nb + j, 8 per product
    v8h xq[NB][NS];
    if constexpr (!RAW) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const int64_t qi = min(qbase + 32 * nb + j, nx - 1);
            const auto *xs =
                reinterpret_cast<const CH_RO uint4 *>(ro(Xs) + (size_t)qi * DP + g * (DP / 2));
#pragma unroll
            for (int s = 0; s < NS; ++s) xq[nb][s] = __builtin_bit_cast(v8h, ld(xs + s));
        }
    }
    if (status != CHAMFER_OK) {  // uniform
        lds_wait<0>();
        return;
    }

    // ---- the queries' thresholds, a query per lane: with e the query's part of
    // the error bound a row can reach the canonical accumulator acc only if
    // v >= (|z|^2 (1 - rho) - (acc + under) 2^2he (1 + 2 rho)) / 2 - e (thr_of), and a
    // row known at v1 excludes every v below v1 - marg (marg: the parts of both
    // rows and twice the query's; B's largest row part).  Loops that are not
    // unrolled: this code runs once, and its time is that of fetching its
    // instructions.
    // Float32 with some slack (3e-7 |z|^2 for the roundings of |z|^2 / 2).  acc is
    // within rho of the squared distance but for what its steps lose below
    // float32's normal range, at most 2^-150 each (and the seed's square twice):
    // under, which the scale makes large for clouds of extent 1e-20 and less.
    const float rho = half_rho(d), under = ldexpf((float)(d + 4), -149);
    float by, be = 0.0f, erow;
    if constexpr (RAW) {
        by = p->half_box;
        erow = err.s2 * by * by;
    } else {
        const float grow = 1.000001f + 2.0f * rho;
        const float s2 = __uint_as_float(rep_fold(p->half_rep)) * grow;
        by = sqrtf(s2) * 1.000001f;
        const float e2 = __uint_as_float(rep_fold(p->half_rep + 1)) * grow;
        be = sqrtf(e2) + by * 1.2e-7f;
        erow = err.s2 * s2 + err.e2 * e2;
    }
    const float rho2 = 2.1f * rho + 1e-6f;
    auto thr_of = [&](float tlo, float acc) {
        const float h = ldexpf(acc + under, 2 * he - 1) * (1.0f + rho2);
        return tlo - h - (fabsf(tlo) + h) * 2.4e-7f;
    };
    auto prepare = [&](int q) {
        const int64_t qi = qbase + q;
        const int64_t row = qi < nx ? (rows ? (int64_t)ro(rows)[qi] : qi) : 0;
        float t0 = INFINITY, tlo = -INFINITY, marg = 0.0f;
        float4 sq = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        if constexpr (RAW) {
            uint32_t hb[KH], mb[KH];
            float s2 = 0.0f, e2 = 0.0f;
#pragma unroll
            for (int k = 0; k < KH; ++k) {
                const float v =
                    k < d ? ldexpf(ro(X)[row * d + min(k, d - 1)] - cen[min(k, d - 1)], he) : 0.0f;
                const _Float16 h = half_of(v);
                const float r = half_rest(v, h);
                const _Float16 m = half_of(r);
                const float e = r - (float)m;
                s2 = fmaf(v, v, s2);
                e2 = fmaf(e, e, e2);
                hb[k] = half_bits(h);
                mb[k] = half_bits(m);
            }
            sq = half_stat(s2, e2);
            if (!isfinite(s2 + e2)) {
#pragma unroll
                for (int k = 0; k < KH; ++k) hb[k] = mb[k] = 0u;
            }
            // [h | h | m] for the fragments below, in the (still empty) queue
            uint4 *st = reinterpret_cast<uint4 *>(&queue[wave][0]) + lane * UPR;
#pragma unroll
            for (int u = 0; u < UPR; ++u) {
                uint32_t w[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint32_t a[2];
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const int s = 8 * u + 2 * i + c;
                        a[c] = s < KH ? hb[s]
                                      : s < 2 * KH ? hb[s - KH] : s < 3 * KH ? mb[s - 2 * KH] : 0u;
                    }
                    w[i] = a[0] | (a[1] << 16);
                }
                st[u] = make_uint4(w[0], w[1], w[2], w[3]);
            }
        }
        if (qi < nx) {
            if constexpr (!RAW) sq = ld(ro(stat) + qi);
            const unsigned long long known =
                __hip_atomic_load(&best[qi], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint32_t gt = gthr ? __hip_atomic_load(&gthr[qi], __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT)
                                     : 0xffffffffu;
            const float sd = seed ? ro(seed)[row] : INFINITY;
            const float zt = sq.y + sq.z, zn2 = sq.x;
            const float e = half_err_query(err, zt, sq.z, by, be) + 3e-7f * zn2;
            const float vmax = 0.5f * by * by + 1.02f * zt * by;
            marg = (2.0f * (e + erow) + 2.2f * rho * (0.5f * zn2 + vmax + e + erow)) * 1.00001f +
                   ldexpf(under, 2 * he);
            // a row whose canonical sum may overflow excludes nothing by its score:
            // all rows at infinity are equal, and the lowest index counts
            if (!(ldexpf((zt + by) * (zt + by), -2 * he) < 3e38f)) marg = INFINITY;
            tlo = 0.5f * zn2 * (1.0f - rho - 1e-6f) - 1.00001f * e;
            t0 = -INFINITY;
            if (tlo > -INFINITY) {  // (or NaN: no bound, every row is evaluated)
                float acc = known != ~0ull ? __uint_as_float((uint32_t)(known >> 32)) : INFINITY;
                acc = fminf(acc, sd * sd * 1.000001f);
                t0 = fmaxf(thr_of(tlo, acc), thr_decode(gt));
                if (!(t0 > -INFINITY)) t0 = -INFINITY;
            }
        }
        thr_s[wave][q] = t0;
        tlo_s[wave][q] = tlo;
        marg_s[wave][q] = marg;
        row_s[wave][q] = (int32_t)row;
        seen_s[wave][q] = 0xffffffffu;
        best_s[wave][q] = ~0ull;
    };

    float thr[NB];
    auto sync_lds = [] {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    if constexpr (RAW) {
#pragma unroll
        for (int i = 0; i < WQ / 64; ++i) {
            prepare(64 * i + lane);
            sync_lds();
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint4 *st = reinterpret_cast<const uint4 *>(&queue[wave][0]) +
                                  (32 * h + j) * UPR + g * (UPR / 2);
#pragma unroll
                for (int s = 0; s < NS; ++s) xq[2 * i + h][s] = __builtin_bit_cast(v8h, st[s]);
            }
            sync_lds();
        }
    } else {
#pragma unroll
        for (int q = 0; q < WQ; q += 64) prepare(q + lane);
        sync_lds();
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) thr[nb] = thr_s[wave][32 * nb + j];
    const unsigned long long below = (1ull << lane) - 1;
    int cnt = 0;            // queued rows (wave-uniform)
    uint32_t crowded = 0u;  // 32-row blocks of the tile to evaluate in full
    // Rows of the 32 x 32 block acc (first row `row` of the chunk) above the
    // threshold of block nb's queries into the queue, with the lane's largest v
    // (m) as their v.  m may raise the threshold.  This runs for most blocks until
    // the thresholds have settled: two instructions per register, and one round
    // of the loop unless a lane has several rows.  True when the queue is full.
    auto push = [&](int nb, const v16f &acc, float m, int row) {
        float nt = m - marg_s[wave][32 * nb + j];
        if (__ballot(thr[nb] == -INFINITY) != 0) nt = fmaxf(nt, __shfl_xor(nt, 32));
        if (nt > thr[nb]) {
            thr[nb] = nt;
            if (eager) gthr_raise(32 * nb + j, nt);
        }
        uint32_t hm = 0u;  // bit r: register r
#pragma unroll
        for (int r = 15; r >= 0; --r) hm = hm + hm + (acc[r] > thr[nb] ? 1u : 0u);
        if (row + 32 > len) {  // rows past the chunk (uniform)
            const int left = len - row - 4 * g;  // rows 8 i + (r & 3) below it are in
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (8 * (r >> 2) + (r & 3) >= left) hm &= ~(1u << r);
        }
        for (;;) {
            const unsigned long long mk = __ballot(hm != 0u);
            if (mk == 0) return false;
            if (cnt > QN - 64) return true;
            if (hm) {
                const int r = __ffs((int)hm) - 1;
                queue[wave][cnt + __builtin_amdgcn_mbcnt_hi(
                                      (uint32_t)(mk >> 32),
                                      __builtin_amdgcn_mbcnt_lo((uint32_t)mk, 0u))] =
                    make_uint2(__float_as_uint(m),
                               (uint32_t)(row + 8 * (r >> 2) + (r & 3) + 4 * g) |
                                   ((uint32_t)(32 * nb + j) << kHalfRowBits));
                hm &= hm - 1u;
            }
            cnt += __popcll(mk);
        }
    };
    // The thresholds of the other workgroups: read into seen_s while a tile is
    // computed, taken up before the next one.
    const uint32_t seen_at = lds_address(&seen_s[wave][0]);
    auto look = [&] {
#pragma unroll
        for (int i = 0; i < WQ / 64; ++i) {
            const uint32_t *from = gthr + min(qbase + 64 * i + lane, nx - 1);
            if (local) lds_load4_sc0(from, seen_at + 256 * i);
            else lds_load4_sc1(from, seen_at + 256 * i);
        }
    };
    // This wavefront's thresholds, into thr_s and to the others.
    auto publish = [&] {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            const float o = fmaxf(thr[nb], __shfl_xor(thr[nb], 32));
            if (g == 0 && o > thr_s[wave][32 * nb + j]) {
                thr_s[wave][32 * nb + j] = o;
                if (share) gthr_raise(32 * nb + j, o);
            }
        }
    };
    auto take_up = [&] {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
            thr[nb] = fmaxf(thr[nb], thr_decode(seen_s[wave][32 * nb + j]));
    };
    // Scores of the wavefront's row blocks of a tile (rows t .. of the chunk),
    // from block hh on; the block to go on with when the queue is full, else NH.
    // A block is gone on with at the query block where it stopped, against the
    // thresholds of the rows evaluated meanwhile; one that fills the queue a third
    // time (duplicates) is evaluated in full.
    int from_nb = 0, tries = 0;
    // scan: nothing is queued, the scores only raise the thresholds, the first tile,
    // before its rows are queued.  At 256 slots (280 draws of 3000 rows 114 -> 108 us),
    // and on small launches whose queries start without a distance (2000 x 10000 x 20
    // 50.6 -> 46.5, 2500 x 20001 x 16 59.3 -> 58.7); with twice the queries, or with
    // one, it cost as much as it saved.
    auto compute = [&](const uint8_t *tile, int t, int hh, bool scan) {
#pragma unroll 1
        for (; hh < NH; hh += 2) {
            if (t + 32 * hh >= len) break;
            const int nb0 = from_nb;
            from_nb = 0;
            // unit g UPR / 2 + s of the lane's row, at (.. ^ swz) 16: s flips bits
            // of the first address only; opaque, or the addresses of every s
            // would be kept in registers
            uint32_t at = (32 * hh + j) * RB + ((g * (UPR / 2)) ^ swz(32 * hh + j)) * 16;
            asm volatile("" : "+v"(at));
            const float *tnb = reinterpret_cast<const float *>(tile + TR * RB) + 32 * hh + 4 * g;
            v16f c0, a[NB];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const v4f n4 = *reinterpret_cast<const v4f *>(&tnb[8 * i]);
#pragma unroll
                for (int q = 0; q < 4; ++q) c0[4 * i + q] = n4[q];
            }
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const v8h o = __builtin_bit_cast(
                    v8h, *reinterpret_cast<const uint4 *>(tile + (at ^ (16 * s))));
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    a[nb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(o, xq[nb][s],
                                                                   s == 0 ? c0 : a[nb], 0, 0, 0);
            }
            float m[NB];
            bool any = false;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                m[nb] = a[nb][0];
#pragma unroll
                for (int r = 1; r < 15; r += 2) m[nb] = fmaxf(fmaxf(m[nb], a[nb][r]), a[nb][r + 1]);
                m[nb] = fmaxf(m[nb], a[nb][15]);
                any |= m[nb] > thr[nb];
            }
            if (scan) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    float nt = m[nb] - marg_s[wave][32 * nb + j];
                    nt = fmaxf(nt, __shfl_xor(nt, 32));
                    thr[nb] = fmaxf(thr[nb], nt);
                }
                continue;
            }
            if (__ballot(any) != 0) {
                bool full = false;
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) {
                    if (full || nb < nb0 || __ballot(m[nb] > thr[nb]) == 0) continue;
                    if (push(nb, a[nb], m[nb], t + 32 * hh)) {
                        full = true;
                        from_nb = nb;
                    }
                }
                if (full) {
                    if (++tries <= 2) return hh;
                    crowded |= 1u << hh;
                    from_nb = 0;
                }
            }
            tries = 0;
        }
        return NH;
    };
    // Thresholds after canonical distances in best_s, in thr_s; published when
    // higher.
    auto raise = [&] {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll 1
        for (int q = lane; q < WQ; q += 64) {
            const unsigned long long k = best_s[wave][q];
            const float tlo = tlo_s[wave][q];
            if (k != ~0ull && tlo > -INFINITY) {
                const float t = thr_of(tlo, __uint_as_float((uint32_t)(k >> 32)));
                if (t > thr_s[wave][q]) {
                    thr_s[wave][q] = t;
                    if (share) gthr_raise(q, t);
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    // Evaluate the queue, and every row of the crowded blocks of the tile at t.
    auto settle = [&](int t, int step) {
        if constexpr (RAW) {
            const int evals = evals_s[wave] + cnt + QN * __popc(crowded);
            evals_s[wave] = evals;
            if (__builtin_amdgcn_readfirstlane(evals) > kPlainFirst + t) {
                wave_active = false;
                rest_s[wave] = t;
                plain_s[(step >> 2) & 1][wave] = 1u;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // what the other workgroups know by now: most queued rows were queued
        // against a lower threshold
        publish();
        if (share) look();
        if (share) lds_wait<0>();
        for (int q = lane; q < WQ; q += 64) {
            vtop_s[wave][q] = 0u;
            thr_s[wave][q] = fmaxf(thr_s[wave][q], thr_decode(seen_s[wave][q]));
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        // the row of each query's largest v is evaluated first: its canonical
        // distance excludes most of the others (a margin of e instead of 2 e)
        for (int i = lane; i < cnt; i += 64) {
            const uint2 en = queue[wave][i];
            atomicMax(&vtop_s[wave][en.y >> kHalfRowBits], float_to_ordered(__uint_as_float(en.x)));
        }
#pragma unroll 1
        for (int turn = 0; turn < 2; ++turn) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            int n = 0, nl = 0;
            for (int i = 0; i < cnt; i += 64) {
                const uint2 en = queue[wave][min(i + lane, cnt - 1)];
                const float v = __uint_as_float(en.x);
                const int q = (int)(en.y >> kHalfRowBits);
                const bool keep = i + lane < cnt && v > thr_s[wave][q];
                const bool first = keep && turn == 0 && float_to_ordered(v) == vtop_s[wave][q];
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
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            const uint2 *list = turn == 0 ? lead[wave] : queue[wave];
            const int todo = turn == 0 ? nl : n;
            // passes in flight, as registers allow
            constexpr int M = RAW || NB * NS > 16 ? 1 : DP == 128 ? 3 : 2;
            for (int i = 0; i < todo; i += 64 / LPH * M) {
                const float *xp[M], *bp[M];
                float acc[M];
                uint32_t ey[M];
#pragma unroll
                for (int m = 0; m < M; ++m) {
                    ey[m] = list[min(i + m * (64 / LPH) + lane / LPH, todo - 1)].y;
                    xp[m] = X + (int64_t)row_s[wave][ey[m] >> kHalfRowBits] * d;
                    bp[m] = B + (b0 + (int64_t)(ey[m] & ((1u << kHalfRowBits) - 1u))) * d;
                }
                hit_acc<CHAMFER_L2, LPH, KH, M>(xp, bp, d, acc);
#pragma unroll
                for (int m = 0; m < M; ++m)
                    if (i + m * (64 / LPH) + lane / LPH < todo && lane % LPH == LPH - 1)
                        atomicMin(&best_s[wave][ey[m] >> kHalfRowBits],
                                  half_pack(acc[m], b0 + (int64_t)(ey[m] &
                                                                   ((1u << kHalfRowBits) - 1u))));
            }
            raise();
            if (cnt == 0) break;
        }
        cnt = 0;
        if (crowded != 0u) {
            // lane l takes queries l, l + 64 .. against every row, 8 rows and 4
            // coordinates at a time
            for (int q = lane; q < WQ; q += 64) {
                if (qbase + q >= nx) break;
                const auto *x = ro(X) + (int64_t)row_s[wave][q] * d;
                unsigned long long mine = ~0ull;
                for (int hh = 0; hh < NH; ++hh) {
                    if (((crowded >> hh) & 1u) == 0u) continue;
                    const int e = min(len, t + 32 * hh + 32);
                    for (int r = t + 32 * hh; r < e; r += 8) {
                        float acc[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
                        for (int k = 0; k < d; k += 4) {
                            float xk[4];
#pragma unroll
                            for (int c = 0; c < 4; ++c) xk[c] = x[min(k + c, d - 1)];
#pragma unroll
                            for (int i = 0; i < 8; ++i) {
                                const auto *b = ro(B) + (b0 + min(r + i, e - 1)) * d;
#pragma unroll
                                for (int c = 0; c < 4; ++c) {
                                    float u = xk[c] - b[min(k + c, d - 1)];
                                    if (k + c >= d) u = 0.0f;
                                    acc[i] = fmaf(u, u, acc[i]);
                                }
                            }
                        }
#pragma unroll
                        for (int i = 0; i < 8; ++i)
                            mine = min(mine, half_pack(acc[i], b0 + min(r + i, e - 1)));
                    }
                }
                atomicMin(&best_s[wave][q], mine);
            }
            if (lane == 0) atomicAdd(&p->fallbacks, (uint32_t)__popc(crowded));
            crowded = 0u;
            raise();
        }
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) thr[nb] = fmaxf(thr[nb], thr_s[wave][32 * nb + j]);
    };
    // Every row from t on (the wavefront's blocks) for every query, d <= kHalfRawDim: on the vector ALU (9
    // operations a pair), a lane with queries l, l + 64 .., rows wave-uniform (scalar
    // loads).  From row 0 where a query has no bound at all (2 10^5 x 3 points, 1700
    // draws of one point at 10^9 times the extent: whole call 1232 -> 256 us).
    auto direct = [&](int t) {
        constexpr int NQ = WQ / 64, NR = 8;
        float x[NQ][KH];
        uint32_t bv[NQ];
        int bi[NQ];
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const auto *xr = ro(X) + (int64_t)row_s[wave][64 * i + lane] * d;
#pragma unroll
            for (int k = 0; k < KH; ++k) x[i][k] = xr[min(k, d - 1)];
            bv[i] = 0xffffffffu;
            bi[i] = 0;
        }
        auto rows8 = [&](int r, int left, auto dim) {
            constexpr int D = decltype(dim)::value;  // 0: d
            const int dd = D ? D : d;
            const auto *b = ro(B) + (b0 + r) * dd;
            float acc[NR][NQ] = {};
#pragma unroll
            for (int k = 0; k < (D ? D : KH); ++k) {
                if (k >= dd) break;
#pragma unroll
                for (int j = 0; j < NR; ++j) {
                    const float bk = b[(D ? j : min(j, left - 1)) * dd + k];
#pragma unroll
                    for (int i = 0; i < NQ; ++i) {
                        const float u = x[i][k] - bk;
                        acc[j][i] = fmaf(u, u, acc[j][i]);
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < NR; ++j)
#pragma unroll
                for (int i = 0; i < NQ; ++i) {  // (bits order like the values, NaN last)
                    const uint32_t a = __float_as_uint(acc[j][i]);
                    if (a < bv[i] && j < left) bv[i] = a, bi[i] = r + j;
                }
        };
#pragma unroll 1
        for (int hb = t + 32 * (wave & 1); hb < len; hb += 64)
#pragma unroll 1
            for (int r = hb; r < min(len, hb + 32); r += NR) {
                if (d == 3 && r + NR <= len) rows8(r, NR, std::integral_constant<int, 3>());
                else rows8(r, min(NR, len - r), std::integral_constant<int, 0>());
            }
#pragma unroll
        for (int i = 0; i < NQ; ++i)
            if (bv[i] != 0xffffffffu)
                atomicMin(&best_s[wave][64 * i + lane],
                          ((unsigned long long)bv[i] << 32) | (uint32_t)(b0 + bi[i]));
    };
    if constexpr (RAW) {
        bool none = false;
        for (int q = lane; q < WQ; q += 64)
            none |= qbase + q < nx && !(tlo_s[wave][q] > -INFINITY);
        evals_s[wave] = 0;
        rest_s[wave] = INT_MAX;
        plain_s[0][wave] = 0u;
        plain_s[1][wave] = __ballot(none) != 0 ? 1u : 0u;
    }
    // (the builtin: the compiler then knows that the queries' loads are done too)
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
    __syncthreads();
    // (four steps write one set of words, read after the barrier of the last of them;
    // by the time that it is written again every wavefront has passed that read)
    auto any_plain = [&](int g) {
        const uint4 w = *reinterpret_cast<const uint4 *>(plain_s[g & 1]);
        return __builtin_amdgcn_readfirstlane((int)(w.x | w.y | w.z | w.w)) != 0;
    };
    if (RAW && any_plain(1)) len = 0;
    for (int t = 0, slot = 0, step = 0;; t += TR, ++step) {
        // start the loads of the tile NT - 1 ahead (its slot was read before the
        // barrier that ended the previous step; RAW: two ahead, into registers),
        // compute the tile at t, wait for the next one
        const bool more = t + TR < len, more2 = t + 2 * TR < len;  // uniform
        const int next = slot + 1 == NT ? 0 : slot + 1;
        if constexpr (RAW) {
            if (more) land(next);
            if (more2) fetch(slot, t + 2 * TR);
        } else if constexpr (NT == 3) {
            if (more2) fetch(next + 1 == NT ? 0 : next + 1, t + 2 * TR);
        } else {
            if (more) fetch(next, t + TR);
        }
        if (wave_active) {
            int hh = wave & 1;
            bool scan = step == 0 && (DP == 256 || (!RAW && DP <= 64 && NB == 2 && seed == nullptr));
            do {
                hh = compute(tiles + slot * TB, t, hh, scan);
                if (scan) {
                    scan = false;
                    hh = wave & 1;
                    continue;
                }
                if (hh < NH || crowded != 0u || cnt >= QN / 2 || (!more && cnt > 0)) settle(t, step);
            } while (hh < NH && wave_active);
        }
        const bool polls = share && more && (step & 3) == 0;
        if (polls) look();
        if (!RAW && NT == 3 && more2) {  // all but this step's loads
            if (polls) lds_wait<LPL>();
            else lds_wait<LPS>();
        } else {
            lds_wait<0>();
        }
        if (!more) break;
        bare_barrier();
        if (RAW && (step & 3) == 3 && any_plain(step >> 2)) len = min(len, t + 2 * TR);
        if (share && (step & 3) <= 1) take_up();
        slot = next;
    }
    if (qbase >= nx) return;
    if constexpr (RAW) {
        const int rest = min(len, __builtin_amdgcn_readfirstlane(rest_s[wave]));
        len = (int)(b1 - b0);
        if (rest < len) direct(rest);
    }
#pragma unroll
    for (int i = 0; i < WQ / 64; ++i) {
        const int64_t qi = qbase + 64 * i + lane;
        const unsigned long long k = best_s[wave][64 * i + lane];
        if (qi < nx && k != ~0ull) atomicMin(&best[qi], k);
    }
}

// Wavefronts per SIMD that registers and LDS allow: the queries alone take 64
// to 128 registers above 32 slots.
template <int DP, bool RAW>
__host__ __device__ constexpr int half_waves() {
    return DP == 16 || (DP == 32 && !RAW) ? 3 : 2;
}

template <int DP, bool RAW, int NB>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(half_waves<DP, RAW>())))
void k_nnmin_half(const float *__restrict__ X, const int32_t *__restrict__ rows, int64_t nx,
                  const uint16_t *__restrict__ Xs, const float4 *__restrict__ stat,
                  const float *__restrict__ seed, const float *__restrict__ B,
                  const uint16_t *__restrict__ Bs, int64_t nB, int d,
                  const float *__restrict__ nbh, const uint32_t *__restrict__ lohi, int64_t chunk,
                  int nchunk, unsigned long long *best, uint32_t *gthr, int64_t gstride,
                  DevParams *p) {
    nnmin_half<DP, RAW, NB>(X, rows, nx, Xs, stat, seed, B, Bs, nB, d, nbh, lohi, chunk, nchunk,
                            best, gthr, gstride, p, grid_blk());
}

// Workgroups a launch aims for: two per CU.
int64_t half_target_wgs(int d) {
    (void)d;
    return 512;
}

// Whether a launch is bound by latencies (half_nb).  NB = 4 against 2, whole
// calls in us: 300 draws of 3000 x 150000 x 3 (7e8 products) 211 and 206, exact
// 2500 x 20001 x 16 (1.6e9) 67 and 60, x 64 (3.2e9) 81 and 73; 1600 draws of
// 40000 x 50000 x 64 (5e9) 183 and 185, 1800 of 2 10^5 x 3 (6e9) 336 and 350, exact
// 30000^2 x 128 (1e11) 397 and 431.  Few rows of few slots are over before the larger
// workgroup has paid for its start: 10^6 x 1000 x 16 537 and 512.
static bool half_small(int64_t nx, int64_t nB, int d) {
    return (double)nx * (double)nB * half_slots(d) <= 4e9 || (nB <= 1024 && half_slots(d) <= 32);
}

// target 0: as many chunks as give the least number of rounds of resident
// workgroups times the rows of a round (a workgroup starts and ends in the time
// of about 128 rows).  1600 draws are 7 query blocks: with 80 chunks, the multiple
// of 8 above 512 / 7, a second round of 48 workgroups followed the first.
// cold: the queries start without a distance.
static NNGeom half_geom(int64_t nx, int64_t nB, int d, bool small, bool cold, int64_t target) {
    const int64_t wq = 64 * half_nb(half_slots(d), small);
    const int64_t nq = (nx + wq - 1) / wq;
    const int64_t slots = half_target_wgs(d);
    // few cold queries: every workgroup evaluates its first rows and writes to the same
    // few (100 x 20000 x 20 in 320 chunks 71 us, in 128 43; 100 x 400000 in 512 219 and 122)
    const int64_t cmin = (nB + 65535) / 65536,
                  cmax = cold && nq <= 4 ? std::min((nB + 155) / 156, std::max<int64_t>(128, cmin))
                                         : (nB + 63) / 64;
    auto whole = [&](int64_t nc) {  // one chunk's workgroups share an XCD
        if (nc < cmin) nc = cmin;
        if (nc > cmax) nc = cmax;
        return nc > 1 ? (nc + 7) / 8 * 8 : (int64_t)1;
    };
    int64_t nc = whole(((target > 0 ? target : slots) + nq - 1) / nq);
    if (target <= 0) {
        auto cost = [&](int64_t c) {
            return (double)((nq * c + slots - 1) / slots) * ((double)nB / (double)c + 128.0);
        };
        double least = 1e300;
        for (int64_t c = whole(1); c <= whole(2 * slots / nq + 1); c = c < 8 ? 8 : c + 8)
            if (cost(c) < least) least = cost(c), nc = c;
        // one round that gives some CUs two workgroups and others one takes as long as
        // a full one (10^5 x 5000 x 16: 300 us, in eight chunks 197)
        if (nc == 1 && 2 * nq > slots && nq < slots && cost(whole(8)) <= 1.3 * least) nc = whole(8);
    }
    NNGeom g;
    g.chunk = ((nB + nc - 1) / nc + 31) / 32 * 32;  // whole 32-row blocks
    g.nchunk = (int32_t)nc;
    g.blocks = nq * nc;
    return g;
}

NNGeom half_geom(int64_t nx, int64_t nB, int d, int64_t target) {
    return half_geom(nx, nB, d, false, false, target);
}
// Jobs of a batch: few draws each, so a workgroup takes 128 of them where the table is
// in memory (whole retrievals in us with 256 and 128: 48 pairs of 8000 x 128, 1600
// draws 1972 and 1696; 256 of 1000 x 20, 400 draws 896 and 763).
__host__ __device__ constexpr bool half_batch_small(bool raw) { return !raw; }
NNGeom half_batch_geom(int64_t nx, int64_t nB, int d, int64_t target) {
    return half_geom(nx, nB, d, half_batch_small(!half_tabled(d)), false, target);
}

int64_t half_launch_queries(int64_t nx, int64_t nB, int d) {
    while (nx > 1 && half_geom(nx, nB, d, half_small(nx, nB, d), false, 0).blocks > kMaxLaunchWGs)
        nx = (nx + 1) / 2;
    return nx;
}

hipError_t launch_nnmin_half(const float *X, const int32_t *rows, int64_t nx, const uint16_t *Xs,
                             const float4 *stat, const float *seed, const float *B,
                             const uint16_t *Bs, int64_t nB, int d, const float *nbh,
                             const uint32_t *lohi, unsigned long long *best, uint32_t *gthr,
                             int copies, DevParams *p, hipStream_t st) {
    if (nx <= 0) return hipSuccess;
    const int64_t part = half_launch_queries(nx, nB, d);
    if (part < nx && copies <= 1) {
        for (int64_t q = 0; q < nx; q += part) {
            const int64_t x0 = rows ? 0 : q;  // first row of X
            const hipError_t e = launch_nnmin_half(
                X + x0 * d, rows ? rows + q : nullptr, nx - q < part ? nx - q : part,
                Xs ? Xs + q * half_slots(d) : nullptr, stat ? stat + q : nullptr,
                seed ? seed + x0 : nullptr, B, Bs, nB, d, nbh, lohi, best + q,
                gthr ? gthr + q : nullptr, copies, p, st);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    const bool small = half_small(nx, nB, d);
    const NNGeom g = half_geom(nx, nB, d, small, seed == nullptr, 0);
#define CH_HALF_NB(DP, RAW, NB)                                                              \
    k_nnmin_half<DP, RAW, NB><<<(unsigned)g.blocks, 256, 0, st>>>(                           \
        X, rows, nx, Xs, stat, seed, B, Bs, nB, d, nbh, lohi, g.chunk, g.nchunk, best, gthr, \
        copies > 1 ? nx : 0, p)
#define CH_HALF(DP, RAW)                     \
    do {                                     \
        if (small) CH_HALF_NB(DP, RAW, 2);   \
        else CH_HALF_NB(DP, RAW, 4);         \
    } while (0)
    if (!half_tabled(d)) {
        if (half_slots(d) == 16) CH_HALF(16, true);
        else CH_HALF(32, true);
        return hipGetLastError();
    }
    if (Xs == nullptr || stat == nullptr || Bs == nullptr || nbh == nullptr)
        return hipErrorInvalidValue;
    switch (half_slots(d)) {
        case 32: CH_HALF(32, false); break;
        case 64: CH_HALF(64, false); break;
        case 128: CH_HALF(128, false); break;
        default: CH_HALF_NB(256, false, 2); break;
    }
#undef CH_HALF
#undef CH_HALF_NB
    return hipGetLastError();
}

// ---------------------------------------------------------------- batched
// A job's tables live at J.bhalf, J.nbh (B) and J.xhalf, J.xstat (the draws);
// its cast stage fills them (12 <= d <= 256).

constexpr unsigned kGridHalfRows = 1024, kGridNNHalf = 1024;

__global__ __launch_bounds__(256) void kb_half_rows(const Batch *__restrict__ bt) {
    batch_loop(bt, kBsCast, [&](const Job &J, Blk b) {
        if (b.id < J.nb_castB)
            half_rows(J.B, nullptr, J.nB, J.d, half_slots(J.d), J.lohi,
                      J.bhalf, nullptr, J.nbh, J.p, Blk{b.id, J.nb_castB});
        else
            half_rows(J.A, J.idx, J.T, J.d, half_slots(J.d), J.lohi, J.xhalf, J.xstat, nullptr,
                      J.p, Blk{b.id - J.nb_castB, J.nb_castX});
    });
}

template <int DP, bool RAW>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(DP == 16 ? 3 : 2)))
void kb_nn_half(const Batch *__restrict__ bt) {
    batch_loop(bt, kBsNN, [&](const Job &J, Blk b) {
        if (J.nn_vector) return;
        nnmin_half<DP, RAW, half_nb(DP, half_batch_small(RAW))>(glb(J.A), glb(J.idx), J.T, glb(J.xhalf), glb(J.xstat), glb(J.D),
                            glb(J.B), glb(J.bhalf), J.nB, J.d, glb(J.nbh), glb(J.lohi),
                            J.nn_chunk, J.nn_nchunk, glb(J.best), glb(J.gthr),
                            J.thr_copies > 1 ? J.T : 0, glb(J.p), b);
    });
}

hipError_t launch_batch_half_rows(const Batch *bt, hipStream_t st) {
    kb_half_rows<<<kGridHalfRows, 256, 0, st>>>(bt);
    return hipGetLastError();
}

hipError_t launch_batch_half(const Batch *bt, int d, hipStream_t st) {
    if (!half_tabled(d)) {
        if (half_slots(d) == 16)
            kb_nn_half<16, true><<<kGridNNHalf, 256, 0, st>>>(bt);
        else
            kb_nn_half<32, true><<<kGridNNHalf, 256, 0, st>>>(bt);
        return hipGetLastError();
    }
    switch (half_slots(d)) {
        case 32: kb_nn_half<32, false><<<kGridNNHalf, 256, 0, st>>>(bt); break;
        case 64: kb_nn_half<64, false><<<kGridNNHalf, 256, 0, st>>>(bt); break;
        case 128: kb_nn_half<128, false><<<kGridNNHalf, 256, 0, st>>>(bt); break;
        default: kb_nn_half<256, false><<<kGridNNHalf, 256, 0, st>>>(bt); break;
    }
    return hipGetLastError();
}

}  // namespace chamfer

extern "C" double chamfer_half_score_bound(int32_t d, double zt, double ze, double by, double be) {
    using namespace chamfer;
    if (d < 1 || !half_supported(d, CHAMFER_L2)) return -1.0;
    const HalfErr h = half_err(d, half_slots(d));
    const float q = half_err_query(h, (float)zt, (float)ze, (float)by, (float)be);
    return (double)q * 1.000001 + (double)h.s2 * by * by + (double)h.e2 * be * be;
}
