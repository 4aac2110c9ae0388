// Matrix-core filter of the exact fp32 search.
//
// The exact search sums (q - x)^2 (or q x) directly in fp32, one multiply-add per value on the vector
// units.  Almost all of that work rejects items that are nowhere near: this file does the rejecting on
// the matrix cores and leaves the direct sums to the few items that may be among the k nearest (f32_finish_kernel
// narrows them down once more).  The
// results are the ones of the direct kernel bit for bit, because the final distances are formed by the
// same operations in the same order (search_f32.hip) and the filter never loses an item that belongs:
//
//   score       s = q.x - |x|^2 / 2 (L2; larger = nearer) or q.x (inner product)
//   split       q = qh + ql, x = xh + xl in bf16 (round to nearest), and
//               acc = qh.xh + qh.xl + ql.xh accumulated in fp32
//   error       |acc - q.x| <= 2^-15 sum |q x|  (what the split drops.  bf16 keeps 8 bits, so |ql| <= 2^-8 |q| and the
//                              remainder of q is at most 2^-17 |q|: ql.xl 2^-16, the two remainders 2^-17 each;
//                              1.00391388 squared, just below a tie, is off by 0.994 2^-15)
//                            + 3 d 2^-23 sum |q x|  (3 d accumulations, each off by an ulp)
//               |x|^2 is off by d 2^-24 of itself, the directly summed distance by (d / 8 + 8) 2^-24 of
//               itself, at most (d / 4 + 16) 2^-24 (|q|^2 + |x|^2) on the score's scale, and the few operations
//               that form a bound by an ulp of it each; sum |q x| <= (|q|^2 + |x|^2) / 2 = M, so all of it
//               together is less than  (2^-15 + 2^-18 + d 2^-21) M, and stays below
//               C (|q|^2 + |x|^2) / 2   with   C = 2^-14 + d 2^-20   (f32_filter_constant)
//
// so  acc - |x|^2 / 2 -+ C (|q|^2 + |x|^2) / 2  bounds an item's score from both sides, split into a part
// per item and a part per query.  A seeding pass over a sample takes, per query, the k-th largest
// group maximum of the lower bounds (at least k items reach it); the scan collects every item whose
// upper bound does.  (An absolute 2^-110 covers products that underflow.)  Queries that collect too many
// (data whose distances are tiny next to its norms), vectors beyond 1e30 in square and anything not finite go
// through the direct kernel instead; the scan collects nothing more for a query whose region has overflowed,
// and a workgroup ends when none of its queries is left.
//
// Two scans follow the seeding pass.  The first forms ONE product, of operands rounded to fp16: a third of the matrix
// work, half the LDS and half the vector work of the split, and a tile of 256 queries instead of 128.
//
//   error       |acc - q.x| <= 2 (2^-11 + 2^-23) sum |q x| + d 2^-23 sum |q x|, everything else as above, so
//               C = 2^-10 + 2^-15 + d 2^-21   (f32_half_filter_constant)
//   range       a query is scaled by a power of two to a norm of 1 to 2, the rows of a tile by the mean of its queries'
//               scales (not at all where that lies near one), so that fp16 holds both; what is too small for its
//               normal range is off by 2^-25, sqrt(d) 2^-25 (|q| + |x|) in all: the first part is in the threshold
//               (sqrt(d) 2^-22: f32_half_filter_small), the second in C's slack.  Rows beyond 2^15 after scaling are set
//               aside, up to 16 of a wave, and summed in fp32 at the workgroup's end; where there are more, and queries
//               2^24 away from the others, go to the second scan.
//
// On ordinary data the wider bound lets through a tenth more (1M x 128, k = 10: 281 items instead of 261 a query).
// The second scan, with C and the split, takes query tiles where the seeding pass has more than twice k groups within
// the first one's error (hard), and queries that overflowed in the first.  1M x 128 shifted by 30 or 100 (inner
// product, all hard) 0.90 / 1.00 -> 0.86 / 0.92 ms.
//
// Measured (whole search, k = 10, L2): 1M x 128, 1000 queries 0.91 -> 0.43 ms (with the split alone; 8.3 with the direct
// kernel alone), 64 queries 0.156 -> 0.139, 256 0.29 -> 0.18; 1M x 96, 1000 0.75 -> 0.42; 300 000 x 771, 1000
// 2.53 -> 0.89; 200 000 x 128, 10 000 2.03 -> 1.04; 2M x 24, 2000 1.81 -> 1.00.
//
// Layout: workgroups of eight waves on tiles of 256 items x 64 WQ queries, as in search_mfma_stream.hip;
// a stage is 32 features.  Items come from HBM in fp32 through registers (two stages ahead), are rounded or split
// and written to LDS as one fp16 or two bf16 planes, their squared norms summed on the way; the queries, rounded or
// split once per search, are copied asynchronously.  Bound by the vector work that the two waves of a SIMD do in step
// (rounding and norms between the matrix instructions of a stage's first half, the epilogue of a tile behind its last:
// 34 % of the first scan's cycles, next to 33 % with the matrix pipe busy) and by the barrier of each stage.
#include <cmath>
#include <type_traits>

#include "mfma_common.h"
#include "wave_ops.h"

namespace lpq {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f_any __attribute__((ext_vector_type(4), aligned(4)));
typedef __bf16 v4b __attribute__((ext_vector_type(4)));
typedef __bf16 v8b __attribute__((ext_vector_type(8)));
typedef _Float16 v4h __attribute__((ext_vector_type(4)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));

constexpr int FW = 8;                 // waves per workgroup
constexpr int TILE_ROWS = 256;
constexpr int KF = 32;                // features per stage
constexpr int PB = KF * 2;            // bytes of a row in one plane of a stage
constexpr int RUN = 16;               // a tile is 16 runs of 16 rows
constexpr float HUGE_NORM = 1e30f;
constexpr float HALF_NORM = 0x1p30f;  // squared norm of a scaled row up to which its values are far from overflowing in fp16
constexpr int HALF_RANGE = 24;        // powers of two by which a query's norm may differ from those of its tile
constexpr int NO_SCALE = INT32_MIN;   // in FilterIo::qe: the query counts as zero (or is a padding row)
constexpr int ZERO_SCALE = 12;        // ... which holds up to this scale of its tile
constexpr int NEAR_ONE_LO = -10, NEAR_ONE_HI = 6;   // scales of a tile that rows do without: fp16 holds norms of 2^-6 to 2^10 well
constexpr float NEAR_ONE_ROWS = 0x1p21f;   // ... where their mean squared norm is at most this: one row in 512 beyond HALF_NORM
constexpr int ASIDE = 16;             // rows beyond HALF_NORM that a wave of the first scan sets aside
constexpr float LONG_NORM = 0x1p90f;  // ... up to this squared norm: what is formed of it stays finite
enum { AGAIN = 1, DIRECT = 2 };       // bits of FilterIo::again

struct FilterIo {
    const float *x;
    int64_t n, ldx;
    int d, dp;                // dp: d rounded up to pairs of stages
    int kst;                  // stages to a tile: what holds d, an even number of them in fp16
    const __bf16 *qh, *ql;    // [nq_pad][dp] the queries' two planes
    const float *qn;          // [nq_pad] squared norms
    int64_t nq;
    int qtiles, S;
    int tiles;                // as in search_mfma_stream.hip: split s takes tiles s, s + S, ...
    int64_t tile_stride, run_gap;
    float h;                  // an item's bound is acc - h |x|^2
    float c;                  // C above
    int32_t *gmax;            // seeding pass: [nq_pad][G] group maxima (order-preserving images), G = S * SEG * 2 * (8 / WQ)
    int SEG;
    float *nxsum;             // seeding pass: the sampled rows' squared norms together, eight times over for each query tile
    float nxper;              // ... times this is their mean
    const _Float16 *qf;       // first scan: [nq_pad][dp] the queries in fp16, each scaled to a norm of 1 to 2
    const int32_t *qe;        // ... by two to this power
    float ch;                 // ... and the constant of its error
    int32_t *qx;              // [nq_pad] ... which leaves here what its scores are scaled by, two to this power
    const int32_t *hard;      // scans: [nq_pad / 128] set where only the second scan can resolve the queries
    int32_t *again;           // [nq_pad] AGAIN: the first scan could not; DIRECT: neither can the second
    const int32_t *kth;       // scan: [nq] k-th largest group maximum
    cand_t *cbuf;             // [nq][S][Cs] rows that may belong: (~ image of acc - h |x|^2, row)
    int32_t *ccnt;            // [nq][S]
    int Cs;
};

#define LPQF_INLINE __attribute__((always_inline))
constexpr int FDUMPS = 32;
// Control words of a workgroup of the scan, in LDS: queries that are done (their region has overflowed, or the slot holds
// none), what wave 0 has said of them, whether a row is lost to both scans, the sum and number of the queries' scales,
// whether rows were set aside, the number of hard tiles, and how many rows each wave of the first scan has set aside, and which.
enum { CTL_DONE = 0, CTL_SAID = 1 /* [2] */, CTL_HUGE = 3, CTL_SCALES = 4, CTL_SCALED = 5, CTL_ANY = 6, CTL_HARD = 7, CTL_ASIDE = 8 /* [FW] */,
       CTL_ROWS = CTL_ASIDE + FW /* [FW][ASIDE] */, CTL_WORDS = CTL_ROWS + FW * ASIDE };
constexpr int ALL_LOST = 1 << 20;     // in CTL_DONE: a row was seen that the bounds do not hold for
constexpr size_t filter_lds_bytes(int wq, bool seed, bool fp16)
{
    return (size_t)2 * (TILE_ROWS + 64 * wq) * (fp16 ? 1 : 2) * PB + 4 * TILE_ROWS * 4 + (size_t)64 * wq * 12 + CTL_WORDS * 4 +
           (seed ? 0 : (size_t)FW * FDUMPS * 80);
}

__device__ __forceinline__ void split4(v4f v, v4b &hi, v4b &lo)
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        hi[e] = (__bf16)v[e];
        lo[e] = (__bf16)(v[e] - (float)hi[e]);
    }
}

// One wave per query row: its two planes (zero beyond d and for rows beyond nq), its squared norm and its fp16 image.
// Clears the words that the passes behind it set.
__global__ __launch_bounds__(256) void split_queries_kernel(const float *__restrict__ q, int64_t ldq, int64_t nq, int64_t rows,
                                                            int d, int dp, __bf16 *__restrict__ qh, __bf16 *__restrict__ ql,
                                                            float *__restrict__ qn, _Float16 *__restrict__ qf,
                                                            int32_t *__restrict__ qe, int32_t *__restrict__ hard,
                                                            int32_t *__restrict__ again, float *__restrict__ nxsum)
{
    const int lane = threadIdx.x & 63;
    const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= rows) return;
    float ss = 0.0f;
    for (int c = lane; c < dp; c += 64) {
        const float v = (r < nq && c < d) ? q[r * ldq + c] : 0.0f;
        const __bf16 hi = (__bf16)v;
        qh[r * dp + c] = hi;
        ql[r * dp + c] = (__bf16)(v - (float)hi);
        ss = fmaf(v, v, ss);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
    // |q| 2^e lies in [1, 2); norms below 2^-50 count as zero
    const int e = ss >= 0x1p-100f && ss <= HUGE_NORM ? -(ilogbf(ss) >> 1) : NO_SCALE;
    for (int c = lane; c < dp; c += 64) {
        const float v = (r < nq && c < d && e != NO_SCALE) ? q[r * ldq + c] : 0.0f;
        qf[r * dp + c] = (_Float16)ldexpf(v, e == NO_SCALE ? 0 : e);
    }
    if (lane == 0) {
        qn[r] = ss;
        qe[r] = e;
        again[r] = 0;
        if (r % 128 == 0) hard[r / 128] = 0;
        if (r == 0) *nxsum = 0.0f;
    }
}

// What a workgroup of a scan does first: which of its queries it has work for, and their thresholds.  Returns what rows are
// scaled by (as a power of two).
template <int QT, bool FP16>
__device__ __forceinline__ int scan_begin(const FilterIo &o, int *ctl, float *thr_l, int *fill, float *h_l, int s, int64_t q_tile)
{
    const int tid = threadIdx.x;
    if (tid < CTL_WORDS) ctl[tid] = 0;
    __syncthreads();
    // FP16: the tile's rows are scaled by two to the mean of its queries' scales
    int xe = 0;
    // More than a quarter of the tiles are hard: the others are left to the second scan, too, which takes two rounds of
    // workgroups for all.  Up to a quarter one round is enough, beyond, it may be two behind the first scan: 1M x 128, some tiles hard and
    // all, ms: 3000 queries, 6 of 24 2.3, 8 2.2 or 3.4, 10 3.6, all 2.8; 5000, 10 of 40 4.1, 12 4.0 or 6.1, all 4.6.
    bool leave = false;
    if (FP16) {
        const float mean = *o.nxsum * o.nxper;
        for (int i = tid; i < QT; i += FW * 64) {
            const int e = o.qe[q_tile + i];
            if (e != NO_SCALE) { atomicAdd(&ctl[CTL_SCALES], e); atomicAdd(&ctl[CTL_SCALED], 1); }
        }
        for (int64_t i = tid; 128 * i < o.nq; i += FW * 64)
            if (o.hard[i]) atomicAdd(&ctl[CTL_HARD], 1);
        __syncthreads();
        leave = 4 * ctl[CTL_HARD] > (o.nq + 127) >> 7;
        const int scaled = ctl[CTL_SCALED];
        xe = __builtin_amdgcn_readfirstlane(scaled ? ctl[CTL_SCALES] / scaled : 0);
        if (xe >= NEAR_ONE_LO && xe <= NEAR_ONE_HI && mean <= NEAR_ONE_ROWS) xe = 0;
        xe = __builtin_amdgcn_readfirstlane(xe);
    }
    for (int i = tid; i < QT; i += FW * 64) {
        const int64_t q = q_tile + i;
        float t = NAN;                                         // nothing compares: a slot that never collects
        const bool hard = q < o.nq && o.hard[q >> 7];
        // (The second scan may take two rounds of workgroups.  What overflowed in the first is left out of the other: where
        // all do (1M x 128, 1000 queries, inner product, 1 % of the rows 10 000 times as long) 6.86 -> 6.65 ms.)
        const int again = FP16 || q >= o.nq ? 0 : __hip_atomic_load(&o.again[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        bool mine = q < o.nq && (FP16 ? !hard : hard || again);
        if (mine && !(again & DIRECT) && o.qn[q] <= HUGE_NORM) {
            const int32_t kth = o.kth[q];
            const float bound = kth == INT32_MIN ? -INFINITY : sortable_to_float(kth);
            if (FP16) {
                // (a norm of up to 2^-50 taken as zero is off by 2^-50 |x| <= 2^(-35 - xe), scaled by 2^2 xe)
                const bool zero = o.qe[q] == NO_SCALE;
                const int e = zero ? xe : o.qe[q];
                if (e - xe > HALF_RANGE || xe - e > HALF_RANGE || (zero && xe > ZERO_SCALE) || leave) {
                    mine = false;
                    atomicOr(&o.again[q], AGAIN);
                } else {
                    t = ldexpf(bound - 0.5f * (o.c + o.ch) * o.qn[q] * 1.00001f - 0x1p-110f, xe + e) - f32_half_filter_small(o.d);
                    h_l[i] = ldexpf(o.h, e - xe);
                    if (s == 0) o.qx[q] = xe + e;
                }
            } else {
                t = bound - o.c * o.qn[q] * 1.00001f - 0x1p-110f;
            }
        }
        if (t != t) atomicAdd(&ctl[CTL_DONE], 1);
        thr_l[i] = t;
        fill[i] = mine ? (again & DIRECT ? o.Cs + 1 : 0) : -1;
    }
    return xe;
}

// What it does last: the rows set aside, and how many rows its queries have collected.
template <int QT, bool FP16>
__device__ __forceinline__ void scan_end(const FilterIo &o, int *ctl, const float *thr_l, int *fill, const float *h_l, int s, int64_t q_tile,
                                         int xe, float xscale)
{
    const int tid = threadIdx.x, S = o.S;
    cand_t *cbase = o.cbuf + ((size_t)q_tile * S + s) * o.Cs;
    const size_t qstride = (size_t)S * o.Cs;
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));   // (left early: the query copies on their way land before the LDS is given back)
    __syncthreads();
    // The rows set aside, summed in fp32 (off by less than the constant lets the rounded rows be): eight lanes to a row
    // and query, eight values each at a time.  1M x 128, 1000 queries, one such row: 0.45 ms (L2) and 0.52 in all, as
    // without it (the split's scan alone: 0.92; the first given up for it and the split's behind: 1.27).
    const bool any = FP16 && ctl[CTL_ANY];
#pragma clang loop unroll(disable)
    for (int w = 0; any && w < FW; ++w) {
        const int rows = ctl[CTL_ASIDE + w] < ASIDE ? ctl[CTL_ASIDE + w] : ASIDE, sub = tid & 7;
        for (int at = tid >> 3; at < QT * rows; at += FW * 8) {
            const int i = at % QT, tr = ctl[CTL_ROWS + w * ASIDE + at / QT];
            const int64_t row = ((int64_t)s + (int64_t)(tr / TILE_ROWS) * S) * TILE_ROWS + tr % TILE_ROWS;
            const _Float16 *qr = o.qf + (q_tile + i) * o.dp;
            const float *xr = o.x + row * o.ldx;
            float u = 0.0f, p = 0.0f;
#pragma clang loop unroll(disable)
            for (int c = 8 * sub; c < o.d; c += 64) {
                const v8h qv = *reinterpret_cast<const v8h *>(qr + c);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float v = c + e < o.d ? xr[c + e] * xscale : 0.0f;
                    u = fmaf((float)qv[e], v, u);
                    p = fmaf(v, v, p);
                }
            }
#pragma unroll
            for (int m = 1; m < 8; m <<= 1) {
                u += __shfl_xor(u, m, 64);
                p += __shfl_xor(p, m, 64);
            }
            if (!(p <= LONG_NORM)) ctl[CTL_DONE] = ALL_LOST;
            if (!(ldexpf(p, -2 * xe) <= HUGE_NORM)) ctl[CTL_HUGE] = 1;
            u = fmaf(-h_l[i], p, u);
            if (sub == 0 && u >= thr_l[i]) {
                const int pos = atomicAdd(&fill[i], 1);
                if (pos < o.Cs) cbase[(size_t)i * qstride + pos] = make_cand(~float_to_sortable(u), (uint32_t)row);
            }
        }
    }
    if (any) __syncthreads();                     // (the same in every thread)
    // a row the bounds do not hold for: all queries of the tile overflow
    const bool lost = ctl[CTL_DONE] >= ALL_LOST || ctl[CTL_HUGE];
    for (int i = tid; i < QT; i += FW * 64) {
        const int64_t q = q_tile + i;
        if (q >= o.nq || (!FP16 && fill[i] < 0)) continue;
        const int have = fill[i] < 0 ? 0 : (lost ? o.Cs + 1 : fill[i]);
        o.ccnt[(size_t)q * S + s] = have;
        if (have > o.Cs) atomicOr(&o.again[q], !FP16 || ctl[CTL_HUGE] ? DIRECT : AGAIN);
    }
}

template <bool SEED, int WQ, bool WIDE, bool FP16, bool EVEN>
__global__ __launch_bounds__(FW * 64, 2) void filter_f32_kernel(FilterIo o)
{
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int WR = FW / WQ, RB = WQ, QT = 64 * WQ;
    constexpr int NP = FP16 ? 1 : 2;                      // planes
    constexpr int AP = TILE_ROWS * PB, BP = QT * PB;      // bytes of a plane: items, queries
    constexpr int STAGE = NP * (AP + BP);                 // xh, xl, qh, ql
    constexpr int BC = NP * BP / 1024;                    // query copies per stage: 16 rows of one plane each
    using frag_t = std::conditional_t<FP16, v8h, v8b>;
    constexpr int DUMPS = FDUMPS;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
    const int wr = wave / WQ, wq = wave % WQ;

    // each XCD gets a contiguous range of (split, query tile) pairs: the query tiles of a split share its L2
    const int S = o.S, total = o.qtiles * S, per = total / 8, b = blockIdx.x;
    const int wk = (b < per * 8) ? (b % 8) * per + b / 8 : b;
    // ... in another order for each split: the second scan has work for some of the tiles only, and workgroups go to the
    // shader engines in turn, free or not (1M x 128, 1000 queries, 3 of 8 tiles hard: 743 us
    // with the same order for all, as long as for 6 tiles; 482 now)
    const int s = wk / o.qtiles, qt = (wk + s) % o.qtiles;

    float *nx = reinterpret_cast<float *>(smem + 2 * STAGE);       // [4][256] squared norms, by tile & 3
    float *thr_l = nx + 4 * TILE_ROWS;                             // [QT]
    int *fill = reinterpret_cast<int *>(thr_l + QT);               // [QT]; below 0: not a query of this scan
    float *h_l = reinterpret_cast<float *>(fill + QT);             // [QT] FP16: what a scaled norm is multiplied by
    int *ctl = fill + 2 * QT;                                      // [CTL_WORDS]
    float *dval = reinterpret_cast<float *>(ctl + CTL_WORDS) + wave * (DUMPS * 20);
    v4i *dmeta = reinterpret_cast<v4i *>(dval + DUMPS * 16);
    const int64_t q_tile = (int64_t)qt * QT, q_first = q_tile + wq * 64;

    int xe = 0;                       // FP16: rows are scaled by two to this
    if (!SEED) xe = scan_begin<QT, FP16>(o, ctl, thr_l, fill, h_l, s, q_tile);
    const float xscale = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(ldexpf(1.0f, xe))));
    __syncthreads();
    // Nothing to collect (to the second scan: the first has resolved all of them)?  The next barrier comes before any row
    // can be found lost, which is written to the same word.
    const bool none = !SEED && ctl[CTL_DONE] >= QT;
    __syncthreads();
    float gm[2] = {-INFINITY, -INFINITY};

    const int nt = (!none && o.tiles > s) ? (o.tiles - s + S - 1) / S : 0;
    const int kst = o.kst, T = nt * kst;

    // ---- items: registers -> two planes in LDS --------------------------------------------------
    // Eight lanes share a row of a stage (16 bytes each); a wave loads rows wave * 32 + 8 i + lane / 8.
    // Chunk c (16 bytes of a plane) of row r sits in slot c ^ ((r >> 2) & 3).
    const int lrow = lane >> 3, lcol = (lane & 7) * 4;
    v4f pre[2][4];                    // stages on their way, stage t in set t & 1
    // a lane's four rows: where they start in the tile's rows (the scan, whose tiles lie together), or in memory
    const float *src[4];
    const float *tile_rows = o.x;
    unsigned src_off[4];
    float part[4] = {0.f, 0.f, 0.f, 0.f}, sum = 0.0f;
    int ft = 0, fk = 0;               // tile (of this split) and stage of the tile that is fetched next
    int pt = 0, pk = 0;               // ... and that goes to LDS next
    auto fetch_tile = [&]() LPQF_INLINE {
        const int64_t t0 = ((int64_t)s + (int64_t)ft * S) * o.tile_stride;
        const int last = (int)(o.n - 1 - t0 < TILE_ROWS ? o.n - 1 - t0 : TILE_ROWS);   // rows past the end: any row, rejected later
        if (!SEED) tile_rows = o.x + t0 * o.ldx;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (SEED) {
                int64_t row = t0 + (int64_t)(wave * 2 + (i >> 1)) * o.run_gap + (i & 1) * 8 + lrow;
                src[i] = o.x + (row < o.n ? row : o.n - 1) * o.ldx;
            } else {
                const int r = wave * 32 + i * 8 + lrow;
                src_off[i] = (unsigned)(r < last ? r : last) * (unsigned)o.ldx;
            }
        }
    };
    // Loads of stage (ft, fk), LOADS of them on every path: only then does the compiler wait for one stage's loads
    // without waiting for those issued after them.  (With a branch between them, and with a stage that fetched
    // nothing, it waited for all, a memory round trip per stage.  It still does where stages of either parity merge: in the
    // sample and the second scan of an odd number of stages.)  What lies past a row's end is loaded from its
    // last four values and put right in fix; past the last stage the last tile's are fetched again.
    constexpr int LOADS = WIDE ? 4 : 16;
    auto fetch = [&](v4f (&to)[4]) LPQF_INLINE {
        const int c = fk * KF + lcol;
        if (WIDE) {
            const int at = c < o.d - 4 ? c : o.d - 4;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                to[i] = *reinterpret_cast<const v4f_any *>(SEED ? src[i] + at : tile_rows + (src_off[i] + (unsigned)at));
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int at = c + e < o.d ? c + e : 0;
                    to[i][e] = SEED ? src[i][at] : tile_rows[src_off[i] + (unsigned)at];
                }
        }
        if (++fk == kst) {
            fk = 0;
            if (ft + 1 < nt) { ++ft; fetch_tile(); }
        }
    };
    auto fix = [&](v4f v) LPQF_INLINE {           // the last stage of a row, and rows that are scaled
        const int left = o.d - (pk * KF + lcol);
        if (WIDE && left < 4) {
            v = left == 3 ? v4f{v[1], v[2], v[3], 0.f} : left == 2 ? v4f{v[2], v[3], 0.f, 0.f} : v4f{v[3], 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = e < left ? (FP16 ? v[e] * xscale : v[e]) : 0.0f;
        return v;
    };
    auto fix_stage = [&](v4f (&from)[4]) LPQF_INLINE {
        if ((pk + 1) * KF > o.d || (FP16 && xe != 0)) {
#pragma unroll
            for (int i = 0; i < 4; ++i) from[i] = fix(from[i]);
        }
    };
    auto put = [&](v4f (&from)[4], int slot) LPQF_INLINE {   // a fetched stage goes to LDS (fix_stage comes first)
        unsigned char *base = smem + slot * STAGE;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = wave * 32 + i * 8 + lrow;
            const int at = r * PB + (((lane & 7) >> 1) ^ ((r >> 2) & 3)) * 16 + (lane & 1) * 8;
            v4f v = from[i];
            if constexpr (FP16) {
                v4h f;
#pragma unroll
                for (int e = 0; e < 4; ++e) f[e] = (_Float16)v[e];
                *reinterpret_cast<v4h *>(base + at) = f;
            } else {
                v4b hi, lo;
                split4(v, hi, lo);
                *reinterpret_cast<v4b *>(base + at) = hi;
                *reinterpret_cast<v4b *>(base + AP + at) = lo;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) part[i] = fmaf(v[e], v[e], part[i]);
        }
    };
    auto put_done = [&]() LPQF_INLINE {           // ... and, at the end of a tile, its rows' norms
        if (++pk == kst) {
            constexpr float LIMIT = FP16 ? HALF_NORM : HUGE_NORM;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                part[i] += __int_as_float(dpp_move<DPP_XOR1>(__float_as_int(part[i])));
                part[i] += __int_as_float(dpp_move<DPP_XOR2>(__float_as_int(part[i])));
                part[i] += __int_as_float(dpp_move<DPP_HALF_MIRROR>(__float_as_int(part[i])));
                if (SEED) sum += part[i];
            }
            const int i = lane & 3;              // lanes 0 to 3 of the eight that share a row write the four rows' norms
            float p = part[0];
#pragma unroll
            for (int e = 1; e < 4; ++e) {
                const float pe = part[e];
                p = i == e ? pe : p;
            }
            if (FP16) {
                // set aside: without a norm no score of the row reaches a threshold
                const unsigned long long far = __ballot(!(p <= LIMIT));
                p = p <= LIMIT ? p : NAN;
                if (__builtin_expect(far != 0, 0)) {
                    int lane_ = lane;                                 // (as in drain)
                    asm volatile("" : "+v"(lane_));
                    const int at = wave * 32 + (lane_ & 3) * 8 + (lane_ >> 3);
                    const unsigned row = ((unsigned)s + (unsigned)(pt * S)) * TILE_ROWS + (unsigned)at;
                    if (((far >> lane_) & 1) && (lane_ & 4) == 0 && row < (unsigned)o.n) {   // (not a copy of the last row)
                        const int pos = atomicAdd(&ctl[CTL_ASIDE + wave], 1);
                        ctl[CTL_ANY] = 1;
                        if (pos < ASIDE) ctl[CTL_ROWS + wave * ASIDE + pos] = pt * TILE_ROWS + at;
                        else ctl[CTL_DONE] = ALL_LOST;
                    }
                }
            } else if (!SEED && !(p <= LIMIT)) {
                ctl[CTL_DONE] = ALL_LOST;
            }
            if ((lane & 4) == 0) nx[(pt & 3) * TILE_ROWS + wave * 32 + i * 8 + lrow] = p;
#pragma unroll
            for (int e = 0; e < 4; ++e) part[e] = 0.0f;
            pk = 0;
            ++pt;
        }
    };

    // ---- queries: asynchronous copies -----------------------------------------------------------
    // Copy instruction i of a stage brings 64 bytes of 16 rows of one plane.
    const unsigned lds0 = lds_offset(smem);
    const unsigned q_off = (unsigned)(((lane >> 2) * o.dp) * 2 + (((lane & 3) ^ ((lane >> 4) & 3)) * 16));
    int qk = 0;
    auto copy_queries = [&](int slot) LPQF_INLINE {
#pragma unroll
        for (int e = 0; e < (BC + FW - 1) / FW; ++e) {
            const int i = wave + e * FW, plane = i / (QT / 16), r16 = i % (QT / 16);
            if (BC % FW != 0 && i >= BC) break;
            const void *base = (FP16 ? (const char *)o.qf : (const char *)(plane ? o.ql : o.qh)) +
                               2 * ((q_tile + r16 * 16) * o.dp + qk * KF);
            const unsigned dst = lds0 + slot * STAGE + NP * AP + plane * BP + r16 * 1024;
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(q_off), "s"(base) : "memory");
        }
        qk = qk + 1 == kst ? 0 : qk + 1;
    };

    // ---- fragments ------------------------------------------------------------------------------
    const int sw = (half ^ ((col >> 2) & 3)) * 16;
    const int a_off = (wr * RB * 32 + col) * PB + sw, b_off = NP * AP + (wq * 64 + col) * PB + sw;
    frag_t A[2][NP][RB], B[2][NP][2]; // [k-step][plane][block]
#define LPQF_LOAD(SLOT, KSTEP, F)                                                                       \
    do {                                                                                                \
        const unsigned char *sb_ = smem + (SLOT) * STAGE;                                               \
        const unsigned char *pa_ = sb_ + (a_off ^ ((KSTEP) * 32)), *pb_ = sb_ + (b_off ^ ((KSTEP) * 32)); \
        _Pragma("unroll") for (int p = 0; p < NP; ++p) {                                                \
            _Pragma("unroll") for (int j = 0; j < 2; ++j) B[F][p][j] = *reinterpret_cast<const frag_t *>(pb_ + p * BP + j * 32 * PB); \
            _Pragma("unroll") for (int i = 0; i < RB; ++i) A[F][p][i] = *reinterpret_cast<const frag_t *>(pa_ + p * AP + i * 32 * PB); \
        }                                                                                               \
    } while (0)
    v16f acc[RB][2];                  // (a tile's first matrix instructions start from zero)
    constexpr v16f ZERO = {};
    auto mfma = [](frag_t a, frag_t b, v16f c) LPQF_INLINE {
        if constexpr (FP16) return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
        else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
    };
#define LPQF_MFMA(F, FIRST)                                                                                  \
    _Pragma("unroll") for (int pp = 0; pp < 2 * NP - 1; ++pp)   /* xh qh, xh ql, xl qh */               \
        _Pragma("unroll") for (int i = 0; i < RB; ++i)                                                  \
            _Pragma("unroll") for (int j = 0; j < 2; ++j)                                               \
                acc[i][j] = mfma(A[F][pp == 2][i], B[F][pp == 1][j], (FIRST) && pp == 0 ? ZERO : acc[i][j])

#define LPQF_ORDER() __builtin_amdgcn_sched_barrier(0)
    const int G = S * o.SEG * 2 * WR;
    auto flush_segment = [&](int seg) LPQF_INLINE {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            o.gmax[(size_t)(q_first + j * 32 + col) * G + (((size_t)s * o.SEG + seg) * WR + wr) * 2 + half] = float_to_sortable(gm[j]);
            gm[j] = -INFINITY;
        }
    };
    if (SEED) {   // segments this split never reaches keep the neutral value
        for (int g = 0; g < o.SEG; ++g) flush_segment(g);
    }
    cand_t *cbase = SEED ? nullptr : o.cbuf + ((size_t)q_tile * S + s) * o.Cs;
    const size_t qstride = (size_t)S * o.Cs;
    auto drain = [&](int dumps) LPQF_INLINE {     // queued scores that reach their query's threshold go to its region
        wave_lds_sync();
        for (int base = 0; base < dumps * 16; base += 64) {
            // (Nothing formed of the lane is kept for the whole scan: no register is left for it in tiles of 256 queries, and
            // a reload from scratch waited for both stages on their way, at nearly every tile.)
            int lane_ = lane;
            asm volatile("" : "+v"(lane_));
            const int at = base + lane_;
            if (at < dumps * 16) {
                const float u = dval[at];
                const v4i m4 = dmeta[at >> 4];
                const int ql = m4[1] & 255, r = at & 15;
                const unsigned row = (unsigned)m4[0] + 8 * (r >> 2) + 4 * (m4[1] >> 8) + (r & 3);
                if (u >= thr_l[ql] && row < (unsigned)o.n) {
                    const int pos = atomicAdd(&fill[ql], 1);
                    if (__builtin_expect(pos < o.Cs, 1)) {
                        cbase[(size_t)ql * qstride + pos] = make_cand(~float_to_sortable(u), row);
                    } else if (__builtin_expect(pos == o.Cs, 0)) {   // the direct kernel takes this query: collect no more for it
                        thr_l[ql] = NAN;
                        atomicAdd(&ctl[CTL_DONE], 1);
                    }
                }
            }
        }
        wave_lds_sync();
    };

    if (T > 0) {
        fetch_tile();
        fetch(pre[0]);
        copy_queries(0);
        fix_stage(pre[0]);
        put(pre[0], 0);
        put_done();
        if (T > 1) copy_queries(1);
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        fetch(pre[1]);
        fetch(pre[0]);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();
        LPQF_LOAD(0, 0, 0);
    }
    int t = 0, tile = 0, seg = 0, partial = 0;
    // Stage t, whose parity P is a constant: the sets of registers cannot be indexed at run time.
    auto stage = [&](auto parity, auto first) LPQF_INLINE {
        constexpr int P = decltype(parity)::value;
        constexpr bool FIRST = decltype(first)::value;
        fix_stage(pre[P ^ 1]);                // (a branch: not among what the matrix instructions cover)
        __builtin_amdgcn_s_waitcnt(0xC07F);   // the first k-step's fragments are there; do not wait for the second's below
        LPQF_LOAD(P, 1, 1);
        LPQF_MFMA(0, FIRST);
        // stage t + 1 goes into the other slot, which was read out before the last barrier (after the
        // last stage: stale values that nobody reads)
        put(pre[P ^ 1], P ^ 1);
        if (FP16) {   // the second k-step's fragments first, then the vector work of the split between the matrix instructions
            __builtin_amdgcn_sched_group_barrier(0x100, 2 + RB, 0);
#pragma unroll
            for (int i = 0; i < 2 * RB; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x2, 48 / (2 * RB), 0);
            }
        }
        LPQF_ORDER();
        if (t + 1 < T) put_done();
        // My reads of stage t, my writes and my query copies of stage t + 1 are complete; of the vector
        // memory operations only the loads of stage t + 2 are newer than those copies.
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(LOADS));
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();
        LPQF_LOAD(P ^ 1, 0, 0);               // (after the last stage: whatever the slot holds, unused)
        if (t + 2 < T) copy_queries(P);
        fetch(pre[P ^ 1]);
        LPQF_MFMA(1, false);
        ++t;
    };
    // For the epilogue of the next tile, read in this one: how many queries are done, and how many wave 0 said are
    // done in the epilogue before this one.  Everyone has passed the barriers of a tile since, and that word is
    // written again only behind those of the next, so all threads of the workgroup get the same.
    int done = 0, said = 0, known = 0, next = 0;
    auto look = [&]() LPQF_INLINE {
        done = ctl[CTL_DONE];
        said = ctl[CTL_SAID + next];
        next ^= 1;
    };
    if (!SEED) look();
    // The end of a tile; false when nothing is left to do.
    auto finish_tile = [&]() LPQF_INLINE -> bool {
        __builtin_amdgcn_sched_barrier(0);        // nothing of the contraction drifts down into the epilogue
        const int64_t row0 = ((int64_t)s + (int64_t)tile * S) * o.tile_stride;
        int dumps = 0;
        float thr[2], hq[2] = {o.h, o.h};        // (read here: registers are what the contraction is short of)
        if (!SEED) {
            thr[0] = thr_l[wq * 64 + col];
            thr[1] = thr_l[wq * 64 + 32 + col];
            if (FP16) { hq[0] = h_l[wq * 64 + col]; hq[1] = h_l[wq * 64 + 32 + col]; }
            const int now = __builtin_amdgcn_readfirstlane(said);
            if (__builtin_expect(now != known, 0)) {
                if (now >= QT) return false;     // nothing left to collect
                known = now;
            }
            if (tid == 0) ctl[CTL_SAID + (next ^ 1)] = done;
            look();                              // (here, not behind the epilogue: the next stage waits for all LDS reads at once)
        }
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            const float *np = nx + (tile & 3) * TILE_ROWS + (wr * RB + i) * 32 + 4 * half;
            v4f nv[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) nv[g] = *reinterpret_cast<const v4f *>(np + 8 * g);
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                v16f v = acc[i][j];
#pragma unroll
                for (int e = 0; e < 16; ++e) v[e] = fmaf(-hq[j], nv[e >> 2][e & 3], v[e]);
                float m = v[0];
#pragma unroll
                for (int e = 1; e < 16; ++e) m = fmaxf(m, v[e]);
                if (SEED) {
                    gm[j] = fmaxf(gm[j], m);
                } else {
                    unsigned long long mask = __ballot(m >= thr[j]);
                    while (__builtin_expect(mask != 0, 0)) {   // queue the 16 scores of the lanes that pass
                        int lane_ = lane;
                        asm volatile("" : "+v"(lane_));
                        const int at = dumps + __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                                                         __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
                        const bool put_ = ((mask >> lane_) & 1) && at < DUMPS;
                        if (put_) {
                            v4f *dst = reinterpret_cast<v4f *>(dval + at * 16);
#pragma unroll
                            for (int g = 0; g < 4; ++g) dst[g] = v4f{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
                            dmeta[at] = v4i{(int)(row0 + (wr * RB + i) * 32), (wq * 64 + j * 32 + (lane_ & 31)) | ((lane_ >> 5) << 8), 0, 0};
                        }
                        const unsigned long long done = __ballot(put_);
                        dumps += __popcll(done);
                        mask &= ~done;
                        if (mask) { drain(dumps); dumps = 0; }
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (!SEED && dumps) drain(dumps);
        if (SEED) {   // tile i belongs to segment i SEG / nt
            partial += o.SEG;
            if (partial >= nt || tile + 1 == nt) flush_segment(seg);
            for (; partial >= nt; partial -= nt) ++seg;
        }
        return ++tile < nt;
    };
    constexpr std::integral_constant<int, 0> P0;
    constexpr std::integral_constant<int, 1> P1;
    bool more = T > 0;
#pragma clang loop unroll(disable)
    while (more) {
        if constexpr (EVEN) {         // an even number of stages to a tile: the parities alternate in the code, too
            stage(P0, std::true_type());
            stage(P1, std::false_type());
#pragma clang loop unroll(disable)
            for (int k = 2; k < kst; k += 2) {
                stage(P0, std::false_type());
                stage(P1, std::false_type());
            }
        } else {
#pragma unroll
            for (int i = 0; i < RB; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = ZERO;
            int k = kst;
            if (t & 1) { stage(P1, std::false_type()); --k; }
#pragma clang loop unroll(disable)
            for (; k >= 2; k -= 2) {
                stage(P0, std::false_type());
                stage(P1, std::false_type());
            }
            if (k) stage(P0, std::false_type());
        }
        more = finish_tile();
    }
#undef LPQF_LOAD
#undef LPQF_MFMA
#undef LPQF_ORDER

    if (!SEED) scan_end<QT, FP16>(o, ctl, thr_l, fill, h_l, s, q_tile, xe, xscale);
    if (SEED) {
#pragma unroll
        for (int o_ = 32; o_ > 0; o_ >>= 1) sum += __shfl_xor(sum, o_, 64);
        __syncthreads();                          // (nobody reads the norms any more)
        if (lane == 0) nx[wave] = sum;
        __syncthreads();
        if (tid == 0) {                           // one atomic operation per workgroup: they all go to one word
#pragma unroll
            for (int i = 1; i < FW; ++i) sum += nx[i];
            atomicAdd(o.nxsum, sum);
        }
    }
}

// ---- the first scan of 65 to 128 features, queries kept in registers ---------------------------------
// Eight waves on 512 queries, 64 to a wave, whose fp16 fragments stay in 64 registers; a stage is 64 whole rows, rounded
// into one of two LDS slots and read by every wave.  Against the kernel above rows are rounded for 512 queries instead of
// 256, the queries are not copied again for each tile of rows, and there is half a barrier to a matrix instruction: 1M x 128,
// 1000 queries 390 -> 305 us (0.66 -> 0.84 PFLOP/s).  What bounds it is the power limit: 305 us in the first searches, 360
// after a dozen, and neither epilogues that run during the next block's matrix instructions nor waits for one stage's loads
// only (both built, 256 registers) changed it.
constexpr int RQT = 512, RSR = 64, RKS = 8, RDP = 16 * RKS;
constexpr size_t resident_lds_bytes()
{
    return (size_t)2 * RSR * RDP * 2 + 2 * RSR * 4 + (size_t)RQT * 12 + CTL_WORDS * 4 + (size_t)FW * FDUMPS * 80;
}

template <int FIX>   // rows shorter than 128 values, or scaled: decided once per workgroup
__device__ __forceinline__ void resident_scan(const FilterIo &o, unsigned char *smem, float *nx, float *thr_l, int *fill, float *h_l, int *ctl,
                                              int s, int64_t q_tile, int xe, float xscale, bool none)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
    const int S = o.S;
    float *dval = reinterpret_cast<float *>(ctl + CTL_WORDS) + wave * (FDUMPS * 20);
    v4i *dmeta = reinterpret_cast<v4i *>(dval + FDUMPS * 16);
    const int nt = (!none && o.tiles > s) ? (o.tiles - s + S - 1) / S : 0, T = nt * (TILE_ROWS / RSR);

    v8h B[2][RKS];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int ks = 0; ks < RKS; ++ks)
            B[j][ks] = *reinterpret_cast<const v8h *>(o.qf + (q_tile + wave * 64 + j * 32 + col) * RDP + ks * 16 + half * 8);

    // ---- rows: registers -> fp16 in LDS ------------------------------------------------------------
    // Eight lanes share a row, 16 bytes of each 128; chunk c (16 bytes in fp16) of row r sits in slot c ^ (r & 15).
    const int lrow = tid >> 3, lcol = (tid & 7) * 4;
    v4f pre[2][4];                    // stages on their way, stage t in set t & 1
    int ft = 0, fb = 0;               // tile (of this split) and quarter of the tile that is fetched next
    int pt = 0, pb = 0;               // ... and that goes to LDS next
    auto fetch = [&](v4f (&to)[4]) LPQF_INLINE {
        const int64_t t0 = ((int64_t)s + (int64_t)ft * S) * TILE_ROWS;
        const int last = (int)(o.n - 1 - t0 < TILE_ROWS ? o.n - 1 - t0 : TILE_ROWS);   // rows past the end: any row, rejected later
        const int r = fb * RSR + lrow;
        const float *tile_rows = o.x + t0 * o.ldx;
        const unsigned off = (unsigned)(r < last ? r : last) * (unsigned)o.ldx;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int c = j * 32 + lcol;
            to[j] = *reinterpret_cast<const v4f_any *>(tile_rows + (off + (unsigned)(FIX && c > o.d - 4 ? o.d - 4 : c)));
        }
        const bool more = ft + 1 < nt;    // past the last stage the last tile's are fetched again
        fb = fb + 1 == TILE_ROWS / RSR ? 0 : fb + 1;
        ft += fb == 0 && more;
    };
    float part = 0.0f;
    auto put = [&](v4f (&from)[4], int slot) LPQF_INLINE {
        unsigned char *row = smem + slot * (RSR * RDP * 2) + lrow * (RDP * 2) + (tid & 1) * 8;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            v4f v = from[j];
            if (FIX) {
                const int left = o.d - (j * 32 + lcol);
                if (left < 4) v = left == 3 ? v4f{v[1], v[2], v[3], 0.f} : left == 2 ? v4f{v[2], v[3], 0.f, 0.f} : v4f{v[3], 0.f, 0.f, 0.f};
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = e < left ? v[e] * xscale : 0.0f;
            }
            v4h f;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                f[e] = (_Float16)v[e];
                part = fmaf(v[e], v[e], part);
            }
            *reinterpret_cast<v4h *>(row + (((j * 4 + ((tid & 7) >> 1)) ^ (lrow & 15)) * 16)) = f;
        }
    };
    auto put_done = [&](int slot) LPQF_INLINE {   // ... and the rows' norms
        float p = part;
        part = 0.0f;
        p += __int_as_float(dpp_move<DPP_XOR1>(__float_as_int(p)));
        p += __int_as_float(dpp_move<DPP_XOR2>(__float_as_int(p)));
        p += __int_as_float(dpp_move<DPP_HALF_MIRROR>(__float_as_int(p)));
        // set aside: without a norm no score of the row reaches a threshold
        const unsigned long long far = __ballot(!(p <= HALF_NORM));
        if (__builtin_expect(far != 0, 0)) {
            const int at = pb * RSR + lrow;
            const unsigned row = ((unsigned)s + (unsigned)(pt * S)) * TILE_ROWS + (unsigned)at;
            if (((far >> lane) & 1) && (lane & 7) == 0 && row < (unsigned)o.n) {   // (not a copy of the last row)
                const int pos = atomicAdd(&ctl[CTL_ASIDE + wave], 1);
                ctl[CTL_ANY] = 1;
                if (pos < ASIDE) ctl[CTL_ROWS + wave * ASIDE + pos] = pt * TILE_ROWS + at;
                else ctl[CTL_DONE] = ALL_LOST;
            }
        }
        if ((lane & 7) == 0) nx[slot * RSR + lrow] = p <= HALF_NORM ? p : NAN;
        pb = pb + 1 == TILE_ROWS / RSR ? 0 : pb + 1;
        pt += pb == 0;
    };

    cand_t *cbase = o.cbuf + ((size_t)q_tile * S + s) * o.Cs;
    const size_t qstride = (size_t)S * o.Cs;
    auto drain = [&](int dumps) LPQF_INLINE {     // queued scores that reach their query's threshold go to its region
        wave_lds_sync();
        for (int base = 0; base < dumps * 16; base += 64) {
            const int at = base + lane;
            if (at < dumps * 16) {
                const float u = dval[at];
                const v4i m4 = dmeta[at >> 4];
                const int ql = m4[1] & (RQT - 1), r = at & 15;
                const unsigned row = (unsigned)m4[0] + 8 * (r >> 2) + 4 * (m4[1] / RQT) + (r & 3);
                if (u >= thr_l[ql] && row < (unsigned)o.n) {
                    const int pos = atomicAdd(&fill[ql], 1);
                    if (__builtin_expect(pos < o.Cs, 1)) {
                        cbase[(size_t)ql * qstride + pos] = make_cand(~float_to_sortable(u), row);
                    } else if (__builtin_expect(pos == o.Cs, 0)) {   // the second scan takes this query: collect no more for it
                        thr_l[ql] = NAN;
                        atomicAdd(&ctl[CTL_DONE], 1);
                    }
                }
            }
        }
        wave_lds_sync();
    };

    const int a_base = col * (RDP * 2) + ((half ^ (col & 15)) * 16);
    v8h A0[RKS], A1[RKS];
    auto load = [&](v8h (&A)[RKS], int slot, int block) LPQF_INLINE {
        const unsigned char *sb = smem + slot * (RSR * RDP * 2) + block * (32 * RDP * 2);
#pragma unroll
        for (int ks = 0; ks < RKS; ++ks) A[ks] = *reinterpret_cast<const v8h *>(sb + (a_base ^ (ks * 32)));
    };
    float thr[2], hq[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        thr[j] = thr_l[wave * 64 + j * 32 + col];
        hq[j] = h_l[wave * 64 + j * 32 + col];
    }
    constexpr v16f ZERO = {};
    int dumps = 0, t = 0;
    auto block = [&](v8h (&A)[RKS], int slot, int blk, auto between) LPQF_INLINE {
        v16f acc[2];
#pragma unroll
        for (int ks = 0; ks < RKS; ++ks)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(A[ks], B[j][ks], ks ? acc[j] : ZERO, 0, 0, 0);
        between();
        const float *np = nx + slot * RSR + blk * 32 + 4 * half;
        v4f nv[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) nv[g] = *reinterpret_cast<const v4f *>(np + 8 * g);
        __builtin_amdgcn_sched_barrier(0);        // nothing of the contraction drifts down into the epilogue
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            v16f v = acc[j];
#pragma unroll
            for (int e = 0; e < 16; ++e) v[e] = fmaf(-hq[j], nv[e >> 2][e & 3], v[e]);
            float m = v[0];
#pragma unroll
            for (int e = 1; e < 16; ++e) m = fmaxf(m, v[e]);
            unsigned long long mask = __ballot(m >= thr[j]);
            while (__builtin_expect(mask != 0, 0)) {   // queue the 16 scores of the lanes that pass
                const int at = dumps + __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
                const bool put_ = ((mask >> lane) & 1) && at < FDUMPS;
                if (put_) {
                    v4f *dst = reinterpret_cast<v4f *>(dval + at * 16);
#pragma unroll
                    for (int g = 0; g < 4; ++g) dst[g] = v4f{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
                    const int row0 = (s + (t / (TILE_ROWS / RSR)) * S) * TILE_ROWS + (t % (TILE_ROWS / RSR)) * RSR + blk * 32;
                    dmeta[at] = v4i{row0, (wave * 64 + j * 32 + col) | (half * RQT), 0, 0};
                }
                const unsigned long long done = __ballot(put_);
                dumps += __popcll(done);
                mask &= ~done;
                if (mask) { drain(dumps); dumps = 0; }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    if (T > 0) {
        fetch(pre[0]);
        fetch(pre[1]);
        put(pre[0], 0);
        put_done(0);
        fetch(pre[0]);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();
        load(A0, 0, 0);
    }
    auto stage = [&](auto parity) LPQF_INLINE {
        constexpr int P = decltype(parity)::value;
        load(A1, P, 1);
        // stage t + 1 goes into the other slot, which was read out before the last barrier (after the last stage: stale
        // values that nobody reads)
        block(A0, P, 0, [&]() LPQF_INLINE { put(pre[P ^ 1], P ^ 1); });
        fetch(pre[P ^ 1]);
        block(A1, P, 1, [&]() LPQF_INLINE { if (t + 1 < T) put_done(P ^ 1); });
        ++t;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // my reads of stage t and my writes of the next are complete
        __syncthreads();
        load(A0, P ^ 1, 0);                                  // (after the last stage: whatever the slot holds, unused)
    };
    constexpr std::integral_constant<int, 0> P0;
    constexpr std::integral_constant<int, 1> P1;
    int done = 0, said = 0, known = 0, next = 0;             // as in the kernel above
    auto look = [&]() LPQF_INLINE {
        done = ctl[CTL_DONE];
        said = ctl[CTL_SAID + next];
        next ^= 1;
    };
    look();
#pragma clang loop unroll(disable)
    while (t < T) {
        stage(P0);
        stage(P1);
        stage(P0);
        stage(P1);
        if (dumps) { drain(dumps); dumps = 0; }
        const int now = __builtin_amdgcn_readfirstlane(said);
        if (__builtin_expect(now != known, 0)) {
            if (now >= RQT) break;               // nothing left to collect
            known = now;
#pragma unroll
            for (int j = 0; j < 2; ++j) thr[j] = thr_l[wave * 64 + j * 32 + col];
        }
        if (tid == 0) ctl[CTL_SAID + (next ^ 1)] = done;
        look();
    }
}

__global__ __launch_bounds__(FW * 64, 2) void resident_scan_kernel(FilterIo o)
{
    extern __shared__ __align__(16) unsigned char smem[];
    const int total = o.qtiles * o.S, per = total / 8, b = blockIdx.x;
    const int wk = (b < per * 8) ? (b % 8) * per + b / 8 : b;         // as in the kernel above
    const int s = wk / o.qtiles, qt = (wk + s) % o.qtiles;
    float *nx = reinterpret_cast<float *>(smem + 2 * RSR * RDP * 2);
    float *thr_l = nx + 2 * RSR;
    int *fill = reinterpret_cast<int *>(thr_l + RQT);
    float *h_l = reinterpret_cast<float *>(fill + RQT);
    int *ctl = fill + 2 * RQT;
    const int64_t q_tile = (int64_t)qt * RQT;
    const int xe = scan_begin<RQT, true>(o, ctl, thr_l, fill, h_l, s, q_tile);
    const float xscale = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(ldexpf(1.0f, xe))));
    __syncthreads();
    const bool none = ctl[CTL_DONE] >= RQT;      // nothing to collect
    __syncthreads();
    if (o.d == RDP && xe == 0) resident_scan<0>(o, smem, nx, thr_l, fill, h_l, ctl, s, q_tile, xe, xscale, none);
    else resident_scan<1>(o, smem, nx, thr_l, fill, h_l, ctl, s, q_tile, xe, xscale, none);
    scan_end<RQT, true>(o, ctl, thr_l, fill, h_l, s, q_tile, xe, xscale);
}

hipError_t launch_resident(const FilterIo &o, hipStream_t st)
{
    if (o.dp != RDP || o.d < 4) return hipErrorInvalidValue;
    static bool attr_set = false;
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(resident_scan_kernel),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    resident_scan_kernel<<<(unsigned)(o.qtiles * o.S), FW * 64, resident_lds_bytes(), st>>>(o);
    return hipGetLastError();
}

template <bool SEED, int WQ, bool FP16>
hipError_t launch_filter(const FilterIo &o, hipStream_t st)
{
    const bool wide = o.d >= 4;       // (16-byte loads need no more than the rows' own alignment of 4)
    const bool even = o.kst % 2 == 0;
    if (FP16 && !even) return hipErrorInvalidValue;
    auto kern = !wide ? filter_f32_kernel<SEED, WQ, false, FP16, FP16>
                      : (even ? filter_f32_kernel<SEED, WQ, true, FP16, true> : filter_f32_kernel<SEED, WQ, true, FP16, FP16>);
    static bool attr_set[3] = {false, false, false};
    const int which = wide ? 1 + even : 0;
    if (!attr_set[which]) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set[which] = true;
    }
    kern<<<(unsigned)(o.qtiles * o.S), FW * 64, filter_lds_bytes(WQ, SEED, FP16), st>>>(o);
    return hipGetLastError();
}

size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

}  // namespace

F32Filter f32_filter_plan(int64_t n, int64_t nq, int d, int k)
{
    F32Filter p;
    // (Few queries too: the direct kernel sorts its candidate buffers several times per workgroup, 0.2 ms
    // whatever the size.  One query, k = 10: 10 000 x 128 0.23 -> 0.04 ms, 1M x 128 0.28 -> 0.16.)
    if (nq < 1 || n < 4096) return p;
    p.wq = nq <= 64 ? 1 : 2;
    const int qt = 64 * p.wq, row_waves = FW / p.wq;
    p.qtiles = (int)ceil_div(nq, qt);
    // The first scan pays for its launch from about 4e9 multiplications on (20 000 x 100, 50 queries 42 us without it and
    // 45 with it, 10 000 x 64, 2000 queries 48 and 52; 1M x 128, 128 queries 197 and 159).
    p.half = (double)n * (double)round_up(nq, 64) * (double)round_up(d, 2 * KF) >= 4e9;
    p.wq_half = !p.half ? p.wq : nq <= 64 ? 1 : (nq <= 128 ? 2 : 4);
    // 65 to 128 features: queries in registers, where their padding to tiles of 512 is not more than a quarter above the one to 256
    // (whole searches on 1M x 128, tiles of 256 / this, us: 1000 queries 430 / 356, 500 249 / 210, 300 229 / 191; 700, not taken,
    // 333 / 329; 600 on 300 000 x 70, not taken, 154 / 170).
    if (p.half && round_up(d, 2 * KF) == RDP && nq > 256 && 4 * round_up(nq, RQT) <= 5 * round_up(nq, 256)) p.wq_half = RQT / 64;
    p.qtiles_half = (int)ceil_div(nq, 64 * p.wq_half);
    p.nq_pad = round_up(nq, p.wq_half == RQT / 64 ? RQT : 256);
    p.dp = (int)round_up(d, 2 * KF);
    // The sample costs a contraction per row and query (or, for few queries, the bytes of its rows), each
    // item it lets through - about k n / rows per query - the bytes of a row: least at rows ~ sqrt(k n)
    // (~ sqrt(nq k n); the factors are measured, 1M x 128: one query 0.16 ms with 19 000 rows, 0.18 with 8300).
    const double per = 1.5 * std::sqrt((double)nq);
    // Behind the fp16 scan an item let through costs little that grows with d, a sampled row d: the most goes with
    // sqrt(1 / d) (with 13 for all: 100 000 x 1024, 2000 queries, k = 50 0.99 ms, with 5 0.84; 300 000 x 771 0.89 and
    // 0.85; 2M x 24, 2000 queries 0.99, with 20 0.98).
    const double by_d = 13.0 * std::sqrt(128.0 / (double)d);
    const double most = !p.half ? 13.0 : (by_d < 5.0 ? 5.0 : (by_d < 20.0 ? by_d : 20.0)), least = most < 6.0 ? most : 6.0;
    const double by_cost = (per < least ? least : (per < most ? per : most)) * std::sqrt((double)k * (double)n);
    const double by_room = (double)k * (double)n / 1200.0;
    int64_t seed = (int64_t)(by_cost > by_room ? by_cost : by_room);
    if (seed > n / 4) seed = n / 4;
    if (seed < 64 * (int64_t)k) seed = 64 * (int64_t)k;
    p.seed_tiles = (int)ceil_div(seed, TILE_ROWS);
    if ((int64_t)p.seed_tiles * TILE_ROWS * 2 > n) return p;   // too few items to sample: the direct kernel
    const int slots = 256;                                      // one workgroup per CU
    int s1 = slots / p.qtiles;
    if (s1 > p.seed_tiles) s1 = p.seed_tiles;
    if (s1 > 2048 / (2 * row_waves)) s1 = 2048 / (2 * row_waves);
    const SampleShape shape = sample_that_covers(n, p.seed_tiles, 16, s1 < 1 ? 1 : s1);
    p.S1 = shape.splits;
    p.seed_tiles = (int)shape.per_split * p.S1;
    while ((int64_t)p.seed_tiles * TILE_ROWS > n) p.seed_tiles -= p.S1;
    if (p.seed_tiles < 1) return p;
    p.run_stride = n / (16 * (int64_t)p.seed_tiles);
    p.SEG = mfma_seed_segments(p.S1, k, k, row_waves);
    p.G = mfma_seed_groups(p.S1, p.SEG, row_waves);
    if (p.G < k || p.G > 4096) return p;
    const int64_t tiles = ceil_div(n, TILE_ROWS);
    int64_t s2 = slots / p.qtiles_half;
    if (s2 > tiles) s2 = tiles;
    p.S2 = (int)(s2 < 1 ? 1 : s2);
    const double expect = 1.5 * (double)k * (double)n / ((double)p.seed_tiles * TILE_ROWS);
    if (expect > 3000.0) return p;                              // the selection sorts up to 4096
    // (64 at least, and 128 where half of 64 is used up, as few are not filled evenly: 1 357 103 x 37, 9019 queries, k = 2, seven regions
    // of 64 for 53: two dozen queries overflowed, 21 ms instead of 2.6, as the direct kernel takes 16 ms for one of so many.)
    const double each = 3.0 * expect / p.S2;
    int64_t cs = each > 32.0 ? 128 : 64;
    while ((double)cs < each && cs < 4096) cs <<= 1;
    p.Cs = (int)cs;
    size_t o = 0;
    p.off_qh = o;   o = align256(o + (size_t)p.nq_pad * p.dp * 2);
    p.off_ql = o;   o = align256(o + (size_t)p.nq_pad * p.dp * 2);
    p.off_qf = o;   o = align256(o + (size_t)p.nq_pad * p.dp * 2);
    p.off_qn = o;   o = align256(o + (size_t)p.nq_pad * 4);
    p.off_qe = o;   o = align256(o + (size_t)p.nq_pad * 4);
    p.off_qx = o;   o = align256(o + (size_t)p.nq_pad * 4);
    p.off_hard = o; o = align256(o + (size_t)p.nq_pad / 128 * 4 + 4);
    p.off_again = o; o = align256(o + (size_t)p.nq_pad * 4);
    p.off_gmax = o; o = align256(o + (size_t)p.nq_pad * p.G * 4);
    p.off_kth = o;  o = align256(o + (size_t)nq * 4);
    p.off_cbuf = o; o = align256(o + (size_t)nq * p.S2 * p.Cs * sizeof(cand_t));
    p.off_ccnt = o; o = align256(o + (size_t)nq * p.S2 * 4);
    p.off_over = o; o = align256(o + (size_t)nq * 4);
    p.total = o;
    p.use = true;
    return p;
}

hipError_t launch_f32_filter(const F32Filter &p, const float *x, int64_t n, int64_t ldx, const float *q, int64_t nq, int64_t ldq,
                             int d, int k, bool l2, char *ws, hipStream_t st)
{
    __bf16 *qh = reinterpret_cast<__bf16 *>(ws + p.off_qh), *ql = reinterpret_cast<__bf16 *>(ws + p.off_ql);
    float *qn = reinterpret_cast<float *>(ws + p.off_qn);
    int32_t *gmax = reinterpret_cast<int32_t *>(ws + p.off_gmax), *kth = reinterpret_cast<int32_t *>(ws + p.off_kth);
    _Float16 *qf = reinterpret_cast<_Float16 *>(ws + p.off_qf);
    int32_t *qe = reinterpret_cast<int32_t *>(ws + p.off_qe), *hard = reinterpret_cast<int32_t *>(ws + p.off_hard);
    float *nxsum = reinterpret_cast<float *>(hard + p.nq_pad / 128);
    int32_t *again = reinterpret_cast<int32_t *>(ws + p.off_again);
    split_queries_kernel<<<(unsigned)ceil_div(p.nq_pad, (int64_t)4), 256, 0, st>>>(q, ldq, nq, p.nq_pad, d, p.dp, qh, ql, qn, qf, qe,
                                                                                   hard, again, nxsum);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    FilterIo o = {};
    o.x = x; o.n = n; o.ldx = ldx; o.d = d; o.dp = p.dp;
    o.kst = (int)ceil_div(d, (int64_t)KF);
    o.qh = qh; o.ql = ql; o.qn = qn; o.nq = nq; o.qtiles = p.qtiles;
    o.c = f32_filter_constant(d);
    o.ch = f32_half_filter_constant(d);
    o.qf = qf; o.qe = qe; o.qx = reinterpret_cast<int32_t *>(ws + p.off_qx); o.hard = hard; o.again = again; o.nxsum = nxsum;
    // seeding pass: lower bounds of the scores of a sample (runs of 16 rows spread over the corpus)
    o.S = p.S1; o.SEG = p.SEG; o.gmax = gmax;
    o.tiles = p.seed_tiles; o.tile_stride = p.run_stride; o.run_gap = (int64_t)p.seed_tiles * p.run_stride;
    if (p.run_stride < RUN || ((int64_t)16 * p.seed_tiles - 1) * p.run_stride + RUN > n) return hipErrorInvalidValue;
    o.nxper = 1.0f / (8.0f * TILE_ROWS * (float)p.seed_tiles * (float)p.qtiles);
    o.h = l2 ? 0.5f * (1.0f + o.c) : 0.5f * o.c;
    e = p.wq == 1 ? launch_filter<true, 1, false>(o, st) : launch_filter<true, 2, false>(o, st);
    if (e != hipSuccess) return e;
    // Groups within the first scan's error of the bound, for a row of the sample's mean norm: beyond twice k and a few, the
    // query is left to the second scan (regions hold three times what the sample lets expect, so it would overflow).
    const float c2 = 0.5f * (o.c + o.ch) * 1.00001f;
    const HardQueries hq = {qn, nxsum, c2, c2 * o.nxper, p.half ? 2 * k + 8 : 0, hard};
    e = launch_seed_finalize(gmax, nq, p.G, k, k, nullptr, nullptr, st, nullptr, kth, nullptr, 0, 0, hq);
    if (e != hipSuccess) return e;
    // scans: every item whose upper bound reaches the k-th lower bound
    o.S = p.S2; o.kth = kth;
    o.cbuf = reinterpret_cast<cand_t *>(ws + p.off_cbuf); o.ccnt = reinterpret_cast<int32_t *>(ws + p.off_ccnt); o.Cs = p.Cs;
    o.tiles = (int)ceil_div(n, (int64_t)TILE_ROWS); o.tile_stride = TILE_ROWS; o.run_gap = RUN;
    if (p.half) {
        o.h = l2 ? 0.5f * (1.0f - o.ch) : -0.5f * o.ch;
        o.qtiles = p.qtiles_half; o.kst = p.dp / KF;
        e = p.wq_half == 1 ? launch_filter<false, 1, true>(o, st)
                           : (p.wq_half == 2 ? launch_filter<false, 2, true>(o, st)
                              : p.wq_half == 4 ? launch_filter<false, 4, true>(o, st) : launch_resident(o, st));
        if (e != hipSuccess) return e;
    }
    o.h = l2 ? 0.5f * (1.0f - o.c) : -0.5f * o.c;
    o.qtiles = p.qtiles; o.kst = (int)ceil_div(d, (int64_t)KF);
    return p.wq == 1 ? launch_filter<false, 1, false>(o, st) : launch_filter<false, 2, false>(o, st);
}

}  // namespace lpq
