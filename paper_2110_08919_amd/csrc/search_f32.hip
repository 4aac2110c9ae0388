// Exact search on the original fp32 vectors: the reference set S_E of the recall definition
// (Section 5.3).  The squared distance is summed directly as (q - x)^2 in fp32 (fused
// multiply-add, partial sums per lane combined by a tree), never through the norm identity,
// so near neighbours keep their relative accuracy.  One workgroup per (query tile, corpus split);
// selection and merge are the ones of the integer path, on an order-preserving integer image
// of the float.
#include "block_select.h"
#include "lpq_internal.h"
#include "wave_ops.h"

namespace lpq {

namespace {

constexpr int F32_THREADS = 256;
constexpr int F32_ROWS = F32_THREADS / 8;  // 8 lanes share a row, 4 floats each per step

// QT queries share one pass over the rows of a split and every lane group works on F32_R rows at
// once: the corpus is read once per QT queries, and a query value fetched from LDS feeds F32_R
// subtract/multiply-add pairs (with one row per group the LDS pipe, not the VALU, was the limit).
constexpr int F32_R = 4;
constexpr int F32_STEP = F32_ROWS * F32_R;   // rows per step of a workgroup

// One step of the halving butterfly over lane pairs: of its first CNT partial sums a lane keeps
// one half (the upper one if `upper`), adds the partner's partial sums of that half and leaves the
// results in red[0 .. CNT/2).  With a single sum left it is a plain exchange.  The partner is given
// by a DPP control (no LDS round trip): it must differ from the lane in the bit that `upper` tests
// and lie in the same group of 8 lanes; which other bits differ does not matter for the sums.
template <int CNT, int CTRL, int N>
__device__ __forceinline__ void halve_sums(float (&red)[N], bool upper)
{
    if constexpr (CNT > 1) {
        constexpr int H = CNT / 2;
#pragma unroll
        for (int i = 0; i < H; ++i) {
            const float mine = upper ? red[H + i] : red[i];
            const float theirs = upper ? red[i] : red[H + i];
            red[i] = mine + __int_as_float(dpp_move<CTRL>(__float_as_int(theirs)));
        }
    } else {
        red[0] += __int_as_float(dpp_move<CTRL>(__float_as_int(red[0])));
    }
}

// L2 is a template parameter: as a run-time flag the compiler computed both metrics for every pair
// and selected one (four vector operations per pair instead of two).
template <bool VEC, int QT, bool L2>
__global__ __launch_bounds__(F32_THREADS) void search_f32_kernel(
    const float *__restrict__ x, int64_t n, int64_t ldx, const float *__restrict__ qv, int64_t ldq, int64_t nq,
    int d, int k, int mode, int S, int64_t split_rows, cand_t *__restrict__ lists, int cap, const int32_t *__restrict__ only)
{
    extern __shared__ __align__(16) unsigned char smem[];
    cand_t *buf = reinterpret_cast<cand_t *>(smem);                 // [QT][cap]
    float *qs = reinterpret_cast<float *>(buf + (size_t)QT * cap);  // [QT][dp]
    __shared__ int s_count[2][QT];
    __shared__ cand_t s_thr[QT];

    // Workgroups are dealt round-robin to the 8 XCDs: give each XCD a contiguous range of (split,
    // query tile) pairs, split-major, so the query tiles that stream one split share that XCD's L2.
    const int tiles = gridDim.x / S, per = gridDim.x / 8, b = blockIdx.x;
    const int wk = (b < per * 8) ? (b % 8) * per + b / 8 : b;
    const int64_t q0 = (int64_t)(wk % tiles) * QT;
    const int s = wk / tiles;
    const int chunks = (d + 3) >> 2, dp = 4 * chunks;
    if (only) {   // only queries flagged by the filter; the same answer in every thread
        int any = 0;
        for (int j = 0; j < QT; ++j) any |= q0 + j < nq ? only[q0 + j] : 0;
        if (!any) return;
    }
    const int64_t rs = (int64_t)s * split_rows;
    const int64_t re = (rs + split_rows < n) ? rs + split_rows : n;
    constexpr bool l2 = L2;
    (void)mode;

    for (int i = threadIdx.x; i < QT * dp; i += F32_THREADS) {
        const int j = i / dp, c = i % dp;
        qs[i] = (c < d && q0 + j < nq) ? qv[(q0 + j) * ldq + c] : 0.0f;
    }
    for (int i = threadIdx.x; i < QT * cap; i += F32_THREADS) buf[i] = CAND_NONE;
    if (threadIdx.x < QT) s_thr[threadIdx.x] = CAND_NONE;
    if (threadIdx.x < 2 * QT) s_count[0][threadIdx.x] = 0;
    __syncthreads();

    const int sub = threadIdx.x & 7, grp = threadIdx.x >> 3;
    // which of the finished sums below are this lane's: all of one query's, whose buffer `at` is about
    constexpr int NACC = QT * F32_R;
    constexpr int PER = NACC >= 8 ? NACC / 8 : 1;
    static_assert(F32_R % PER == 0 && 8 % QT == 0, "a lane's sums are one query's, and every query has lanes of the eight");
    const int first = NACC >= 8 ? sub * PER : (sub >> 1), jl = first / F32_R;
    AppendSteps at;
    for (int64_t base = rs; base < re; base += F32_STEP) {
        float acc[QT][F32_R];
#pragma unroll
        for (int j = 0; j < QT; ++j)
#pragma unroll
            for (int r = 0; r < F32_R; ++r) acc[j][r] = 0.0f;
        // Four column chunks (of 4 floats) per lane at a time: all their loads are issued before the
        // arithmetic starts, so one memory round trip covers 16 loads per lane.
        for (int cb = sub; cb < chunks; cb += 32) {
            float xv[4][F32_R][4];
            // whole step inside the split and whole 16-byte chunks: plain loads, no per-value selects
            const bool plain = VEC && base + F32_STEP <= re && cb + 24 < chunks && 4 * (cb + 24) + 3 < d;
            if (plain) {
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int r = 0; r < F32_R; ++r) {
                        const float4 t = *reinterpret_cast<const float4 *>(x + (base + r * F32_ROWS + grp) * ldx + 4 * (cb + 8 * i));
                        xv[i][r][0] = t.x; xv[i][r][1] = t.y; xv[i][r][2] = t.z; xv[i][r][3] = t.w;
                    }
            } else
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int c = cb + 8 * i;
#pragma unroll
                for (int r = 0; r < F32_R; ++r) {
                    const int64_t row = base + r * F32_ROWS + grp;
                    const float *xr = x + row * ldx;
                    if (row >= re || c >= chunks) {
                        xv[i][r][0] = xv[i][r][1] = xv[i][r][2] = xv[i][r][3] = 0.0f;
                    } else if (VEC && 4 * c + 3 < d) {
                        const float4 t = *reinterpret_cast<const float4 *>(xr + 4 * c);
                        xv[i][r][0] = t.x; xv[i][r][1] = t.y; xv[i][r][2] = t.z; xv[i][r][3] = t.w;
                    } else {
#pragma unroll
                        for (int e = 0; e < 4; ++e) xv[i][r][e] = (4 * c + e < d) ? xr[4 * c + e] : 0.0f;
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int c = cb + 8 * i;
                if (c < chunks) {
#pragma unroll
                    for (int j = 0; j < QT; ++j) {
                        const float4 qq = *reinterpret_cast<const float4 *>(qs + j * dp + 4 * c);
                        const float qa[4] = {qq.x, qq.y, qq.z, qq.w};
#pragma unroll
                        for (int r = 0; r < F32_R; ++r)
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                if (l2) { const float t = qa[e] - xv[i][r][e]; acc[j][r] = fmaf(t, t, acc[j][r]); }
                                else acc[j][r] = fmaf(qa[e], xv[i][r][e], acc[j][r]);
                            }
                    }
                }
            }
        }
        // Sum over the 8 lanes of a row group by a halving butterfly: at each step a lane keeps one
        // half of its partial sums and receives the partner's partial sums of that half, so the
        // exchange costs QT * F32_R - 1 shuffles in all (not 3 per sum) and the finished sums end up
        // spread over the lanes: lane `sub` owns sums [sub * PER, sub * PER + PER) in (query, row)
        // order, and tests them against its queries' thresholds.
        float red[NACC];
#pragma unroll
        for (int j = 0; j < QT; ++j)
#pragma unroll
            for (int r = 0; r < F32_R; ++r) red[j * F32_R + r] = acc[j][r];
        halve_sums<NACC, DPP_HALF_MIRROR>(red, (sub & 4) != 0);               // partner 7 - sub: bit 2 differs
        halve_sums<(NACC > 1 ? NACC / 2 : 1), DPP_XOR2>(red, (sub & 2) != 0);
        halve_sums<(NACC > 3 ? NACC / 4 : 1), DPP_XOR1>(red, (sub & 1) != 0);
        // NACC >= 8: lane sub holds sums sub * PER + i.  NACC = 4 (one query): after the two halving
        // steps lanes 2p and 2p + 1 both hold sum p; the even lane acts.
        const bool acts = NACC >= 8 || (sub & 1) == 0;
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int r = (first + i) % F32_R;
            const int64_t row = base + r * F32_ROWS + grp;
            if (acts && row < re) {
                const float a = red[i];
                const cand_t c = make_cand(float_to_sortable(l2 ? a : -a), (uint32_t)row);
                if (c < s_thr[jl]) {
                    const int pos = at.held - at.before + atomicAdd(&s_count[at.turn][jl], 1);
                    buf[(size_t)jl * cap + pos] = c;
                }
            }
        }
        __syncthreads();
        at.step_done(s_count[at.turn][jl]);
#pragma unroll
        for (int j = 0; j < QT; ++j) {
            int h = __builtin_amdgcn_readlane(at.held, j * (8 / QT));   // of a lane of query j
            block_compact_if_full(buf + (size_t)j * cap, cap, k, F32_STEP, h, &s_thr[j]);
            at.held = jl == j ? h : at.held;
        }
    }
    for (int j = 0; j < QT; ++j) {
        block_bitonic_sort(buf + (size_t)j * cap, cap);
        if (q0 + j < nq) {
            cand_t *out = lists + ((q0 + j) * S + s) * k;
            for (int i = threadIdx.x; i < k; i += F32_THREADS) out[i] = buf[(size_t)j * cap + i];
        }
    }
}

// The k nearest of the rows the filter collected, one workgroup per query.  A candidate comes with the upper bound of
// its score: the k and a few with the highest are summed directly, the k-th of those distances says which upper bounds
// still matter, and only those rows are summed too: some 30 of 280 (1M x 128, k = 10), each 4 d bytes from far apart.
// Nothing is sorted on the way: a histogram of the bounds gives the highest, digit by digit where there are more than FIN_FEW
// candidates, and the rank of a distance is the number of those before it, counted by the thread that holds it (sorted are
// more than FIN_RANKED distances).  Directly summed: eight lanes per row, each with the same chunks of four features in the
// same order, the eight partial sums added in the same pairs, as in the kernel above, so a distance comes out with the same
// bits.  Bound by barriers and the latency of the rows.  1000 queries on 1M x 128, k = 10: 13 us, where summing all candidates
// took 37 and selecting among them 29 (sorting the bounds here: 37); k = 100, 700 candidates each: 28.
constexpr int FIN_CAP = 4096;       // candidates in LDS
// (ranks of 470 rows, two to a thread, took 16 us, their sort takes 5)
constexpr int FIN_FEW = FIN_CAP / 2, FIN_RANKED = F32_THREADS, FIN_BINS = F32_THREADS;
constexpr int FIN_REGIONS = F32_THREADS;
// A few short rows cost less than finding out which of them matter (8076 x 4, 3764 queries, k = 2 23 us, 13 now; of 500
// candidates they cost more: 1M x 16, 1000 queries, k = 10, the search 291 us and 302).
constexpr int FIN_SHORT = 16, FIN_ALL = 128;
struct FinishIo {
    const float *x, *q;
    int64_t ldx, ldq;
    int d, k, SS, Cs;
    int cap;                        // FIN_CAP, or as much as the regions can fill: twice a power of two of at least 32
    const int32_t *ccnt;            // [nq][SS]
    const cand_t *cbuf;             // [nq][SS][Cs] (~ image of the score's upper bound without the query's part, row)
    const float *qn;                // [nq] squared norms
    const int32_t *hard, *again;    // which scan a query's candidates are from
    const int32_t *qx;              // ... and by which power of two the first has scaled their scores
    float c, ch;                    // ... and the constants of their bounds
    int32_t *over;                  // [nq] set to 1 where the direct kernel has to search, else to 0
    int32_t *ids;
    float *dists;
};
template <bool VEC, bool L2>
__global__ __launch_bounds__(F32_THREADS) void f32_finish_kernel(FinishIo o)
{
    extern __shared__ __align__(16) unsigned char smem[];
    cand_t *buf = reinterpret_cast<cand_t *>(smem);           // [cap]
    float *qs = reinterpret_cast<float *>(buf + o.cap);       // the query, zero beyond d
    __shared__ int s_more, s_hist[FIN_BINS], s_wave[F32_THREADS / 64], s_cut, s_before;
    __shared__ float s_lo[F32_THREADS / 64], s_hi[F32_THREADS / 64];
    __shared__ cand_t s_kth;
    const int64_t q = blockIdx.x;
    const int tid = threadIdx.x, sub = tid & 7, grp = tid >> 3, chunks = (o.d + 3) >> 2, k = o.k;
    for (int i = tid; i < 4 * chunks; i += F32_THREADS) qs[i] = i < o.d ? o.q[q * o.ldq + i] : 0.0f;
    // The lanes of a region share its candidates, 256 lanes where there is one region.  (With a thread to a region, 10 000
    // queries on 1M x 128, 6 regions: k = 10 123 us, k = 100 144; 89 and 116 now.)
    static_assert(F32_THREADS == 256 && FIN_REGIONS == 256, "");
    const int share = __clz(o.SS - 1) - 24, per = 1 << share, region = tid >> share, part = tid & (per - 1);
    const int mine = region < o.SS ? o.ccnt[q * o.SS + region] : 0;
    int lost = mine > o.Cs;
    const int lane = tid & 63, wave = tid >> 6;
    auto scan = [&](int v) {                                  // inclusive sums over the lanes of a wave
#pragma unroll
        for (int w = 1; w < 64; w <<= 1) {
            const int up = __shfl_up(v, w, 64);
            if (lane >= w) v += up;
        }
        return v;
    };
    const int upto = scan(part ? 0 : mine);
    if (lane == 63) s_wave[wave] = upto;
    if (tid == 0) s_more = 0;
    s_hist[tid] = 0;
    lost = __syncthreads_or(lost);
    int before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < F32_THREADS / 64; ++w) {
        before += w < wave ? s_wave[w] : 0;
        total += s_wave[w];
    }
    if (lost || total < k) {                                  // the same in every thread
        if (tid == 0) o.over[q] = 1;
        return;
    }
    const cand_t *regions = o.cbuf + (size_t)q * o.SS * o.Cs;
    auto pow2 = [](int v) { return v <= 32 ? 32 : 1 << (32 - __clz(v - 1)); };
    auto sort = [&](cand_t *buf, int count) {                 // fills up to a power of two behind it
        for (int i = count + tid; i < pow2(count); i += F32_THREADS) buf[i] = CAND_NONE;
        __syncthreads();
        block_bitonic_sort(buf, pow2(count));
    };
    auto sum_directly = [&](cand_t *buf, int from, int to) {  // key halves of buf[from .. to) become the distances' images
        for (int i = from + grp; i < to; i += F32_ROWS) {
            const cand_t at = buf[i];
            if (at == CAND_NONE) continue;
            const uint32_t row = cand_id(at);
            const float *xr = o.x + (int64_t)row * o.ldx;
            float acc = 0.0f;
#pragma unroll 4
            for (int c = sub; c < chunks; c += 8) {
                float xa[4];
                if (VEC && 4 * c + 3 < o.d) {
                    const float4 t = *reinterpret_cast<const float4 *>(xr + 4 * c);
                    xa[0] = t.x; xa[1] = t.y; xa[2] = t.z; xa[3] = t.w;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) xa[e] = 4 * c + e < o.d ? xr[4 * c + e] : 0.0f;
                }
                const float4 qq = *reinterpret_cast<const float4 *>(qs + 4 * c);
                const float qa[4] = {qq.x, qq.y, qq.z, qq.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if (L2) { const float t = qa[e] - xa[e]; acc = fmaf(t, t, acc); }
                    else acc = fmaf(qa[e], xa[e], acc);
                }
            }
            acc += __int_as_float(dpp_move<DPP_HALF_MIRROR>(__float_as_int(acc)));
            acc += __int_as_float(dpp_move<DPP_XOR2>(__float_as_int(acc)));
            acc += __int_as_float(dpp_move<DPP_XOR1>(__float_as_int(acc)));
            if (sub == 0) buf[i] = make_cand(float_to_sortable(L2 ? acc : -acc), row);
        }
        __syncthreads();
    };

    // A row among the k nearest has a directly summed score of at least that of the k-th of some rows; its upper bound
    // is less than (C |q|^2) / 2 below that, C the constant of its scan.  The norm and the conversion of a distance
    // into a score are off by less than the split's constant allows.
    const bool half = !o.hard[q >> 7] && !o.again[q];
    const float qn = o.qn[q], c = half ? o.ch : o.c;
    auto limit_of = [&](cand_t kth_row) {
        const float kth = sortable_to_float(cand_key(kth_row));
        const float at = L2 ? 0.5f * (qn - kth) - 0.5f * (c + o.c) * qn * 1.00001f - 0.5f * o.c * kth - 0x1p-110f
                            : -kth - 0.5f * c * qn * 1.00001f - 0x1p-20f * fabsf(kth) - 0x1p-110f;
        return make_cand(~float_to_sortable(half ? ldexpf(at, o.qx[q]) - f32_half_filter_small(o.d) : at), 0xFFFFFFFFu);
    };
    auto emit = [&](cand_t best, int i) {
        const float v = sortable_to_float(cand_key(best));
        o.ids[q * k + i] = (int32_t)cand_id(best);
        o.dists[q * k + i] = L2 ? v : -v;
    };

    // up to FIN_FEW candidates are kept in LDS, more are read again from their regions
    const int half_cap = o.cap / 2;
    const bool kept = total <= half_cap;
    const bool every = total <= FIN_ALL && o.d <= FIN_SHORT;  // all candidates are summed at once
    cand_t *few = kept && !every ? buf + half_cap : buf;      // the rows that are summed
    const int room = kept ? half_cap : o.cap, want = k + k / 4 + 6 < total ? k + k / 4 + 6 : total;
    auto each = [&](auto f) {
        if (kept) { for (int i = tid; i < total; i += F32_THREADS) f(buf[i]); }
        else for (int i = part; i < mine; i += 4 * per) {     // four on their way at a time
            cand_t c[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) c[u] = regions[(size_t)region * o.Cs + (i + u * per < mine ? i + u * per : i)];
#pragma unroll
            for (int u = 0; u < 4; ++u) if (i + u * per < mine) f(c[u]);
        }
    };
    // the rank of a distance among all
    auto rank = [&](int i, int count) {
        const cand_t me = few[i];
        int r = 0;
#pragma unroll 8
        for (int j = 0; j < count; ++j) r += few[j] < me;
        return r;
    };
    auto emit_best = [&](int count) {
        if (count <= FIN_RANKED) {
            for (int i = tid; i < count; i += F32_THREADS) {
                const int r = rank(i, count);
                if (r < k) emit(few[i], r);
            }
        } else {
            sort(few, count);
            for (int i = tid; i < k; i += F32_THREADS) emit(few[i], i);
        }
    };
    if (every) {
        for (int i = part; i < mine; i += per) few[before + upto - mine + i] = regions[(size_t)region * o.Cs + i];
        __syncthreads();
        sum_directly(few, 0, total);
        emit_best(total);
        if (tid == 0) o.over[q] = 0;
        return;
    }
    auto find_cut = [&](int want) {                           // the bin up to which that many are, how many before it
        if (wave == 0) {
            int v[4], sum = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) { v[j] = s_hist[4 * lane + j]; sum += v[j]; }
            const int incl = scan(sum);
            if (lane == __ffsll((unsigned long long)__ballot(incl >= want)) - 1) {
                int at = incl - sum, j = 0;
                while (j < 3 && at + v[j] < want) at += v[j++];
                s_cut = 4 * lane + j;
                s_before = at;
            }
        }
        __syncthreads();
    };
    // near(candidate): one of the highest
    float hi = -INFINITY, scale = 0.0f;
    int cut = 0;
    uint32_t last = 0u;
    auto bound = [](cand_t cand) { return sortable_to_float(~cand_key(cand)); };
    auto bin = [&](cand_t cand) {                             // from the highest down
        const float at = (hi - bound(cand)) * scale;
        return at < (float)(FIN_BINS - 1) ? (int)at : FIN_BINS - 1;
    };
    auto near = [&](cand_t cand) { return kept ? bin(cand) <= cut : (uint32_t)(cand >> 32) <= last; };
    if (kept) {
        float lo = INFINITY;
        for (int i = part; i < mine; i += per) {
            const cand_t cand = regions[(size_t)region * o.Cs + i];
            buf[before + upto - mine + i] = cand;
            lo = fminf(lo, bound(cand));
            hi = fmaxf(hi, bound(cand));
        }
#pragma unroll
        for (int w = 32; w > 0; w >>= 1) {
            lo = fminf(lo, __shfl_xor(lo, w, 64));
            hi = fmaxf(hi, __shfl_xor(hi, w, 64));
        }
        if (lane == 0) { s_lo[wave] = lo; s_hi[wave] = hi; }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < F32_THREADS / 64; ++w) {
            lo = fminf(lo, s_lo[w]);
            hi = fmaxf(hi, s_hi[w]);
        }
        scale = (FIN_BINS - 1) / fmaxf(hi - lo, 0x1p-100f);
        each([&](cand_t cand) { atomicAdd(&s_hist[bin(cand)], 1); });
        __syncthreads();
        find_cut(want);
        cut = s_cut;
    } else {
        // (Sorting them FIN_CAP at a time took 0.36 ms for 10 000 a query, 64 queries, before too many were found to be left.)
        int rest = want;
        for (int shift = 24; shift >= 0; shift -= 8) {
            if (shift < 24) {
                s_hist[tid] = 0;
                __syncthreads();
            }
            each([&](cand_t cand) {
                const uint32_t key = (uint32_t)(cand >> 32);
                if (shift == 24 || (key ^ last) >> (shift + 8) == 0u) atomicAdd(&s_hist[(key >> shift) & 255u], 1);
            });
            __syncthreads();
            find_cut(rest);
            last |= (uint32_t)s_cut << shift;
            rest -= s_before;
        }
    }
    auto take = [&](cand_t cand) {
        const int at = atomicAdd(&s_more, 1);
        if (at < room) few[at] = cand;
    };
    each([&](cand_t cand) { if (near(cand)) take(cand); });
    __syncthreads();
    const int first = s_more;
    if (first > room) {                                       // (equal bounds)
        if (tid == 0) o.over[q] = 1;
        return;
    }
    sum_directly(few, 0, first);
    if (first <= FIN_RANKED) {
        for (int i = tid; i < first; i += F32_THREADS)
            if (rank(i, first) == k - 1) s_kth = few[i];
        __syncthreads();
    } else {
        sort(few, first);
        if (tid == 0) s_kth = few[k - 1];
        __syncthreads();
    }
    const cand_t limit = limit_of(s_kth);
    each([&](cand_t cand) { if (!near(cand) && cand <= limit) take(cand); });
    __syncthreads();
    int all = s_more;
    if (all > room) {
        if (tid == 0) o.over[q] = 1;
        return;
    }
    sum_directly(few, first, all);
    if (all > FIN_RANKED) {                                   // first without those beyond the k-th of before
        cand_t c[FIN_CAP / F32_THREADS];
#pragma unroll
        for (int u = 0; u < FIN_CAP / F32_THREADS; ++u) c[u] = tid + u * F32_THREADS < all ? few[tid + u * F32_THREADS] : CAND_NONE;
        if (tid == 0) s_more = 0;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < FIN_CAP / F32_THREADS; ++u) if (c[u] <= s_kth) take(c[u]);
        __syncthreads();
        all = s_more;
    }
    emit_best(all);
    if (tid == 0) o.over[q] = 0;
}

hipError_t launch_finish(bool vec, bool l2, int64_t nq, const FinishIo &o, hipStream_t st)
{
    auto kern = vec ? (l2 ? f32_finish_kernel<true, true> : f32_finish_kernel<true, false>)
                    : (l2 ? f32_finish_kernel<false, true> : f32_finish_kernel<false, false>);
    static bool attr_set[4] = {false, false, false, false};
    const int which = 2 * vec + l2;
    if (!attr_set[which]) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024);
        if (e != hipSuccess) return e;
        attr_set[which] = true;
    }
    const size_t lds = o.cap * sizeof(cand_t) + (size_t)((o.d + 3) / 4) * 16;
    if (o.SS > FIN_REGIONS || 2 * next_pow2(o.k) > FIN_CAP || lds > 128 * 1024) return hipErrorInvalidValue;
    kern<<<(unsigned)nq, F32_THREADS, lds, st>>>(o);
    return hipGetLastError();
}

int f32_cap(int k) { return next_pow2((2 * k > k + 2 * F32_STEP) ? 2 * k : k + 2 * F32_STEP); }

// queries per workgroup: as many as fit in 48 KB of LDS with their candidate buffers, at most 8
int f32_query_tile(int d, int k)
{
    const size_t per = (size_t)f32_cap(k) * sizeof(cand_t) + (size_t)((d + 3) / 4) * 16;
    int qt = 8;
    while (qt > 1 && qt * per > 48 * 1024) qt >>= 1;
    return qt;
}

int f32_splits(int64_t n, int64_t nq, int d, int k)
{
    const int64_t tiles = ceil_div(nq > 0 ? nq : 1, f32_query_tile(d, k));
    int64_t s = ceil_div(2048, tiles);
    const int64_t by_rows = n / 2048 > 0 ? n / 2048 : 1;
    if (s > by_rows) s = by_rows;
    if (s > merge_max_lists(k)) s = merge_max_lists(k);
    return (int)(s < 1 ? 1 : s);
}

template <int QT>
hipError_t launch_f32_tile(bool vec, unsigned blocks, size_t shmem, hipStream_t st, const float *x, int64_t n,
                           int64_t ldx, const float *q, int64_t ldq, int64_t nq, int d, int k, int mode, int S,
                           int64_t split_rows, cand_t *lists, int cap, const int32_t *only)
{
    const bool l2 = mode == MODE_F32_L2;
    auto kern = vec ? (l2 ? search_f32_kernel<true, QT, true> : search_f32_kernel<true, QT, false>)
                    : (l2 ? search_f32_kernel<false, QT, true> : search_f32_kernel<false, QT, false>);
    kern<<<blocks, F32_THREADS, shmem, st>>>(x, n, ldx, q, ldq, nq, d, k, mode, S, split_rows, lists, cap, only);
    return hipGetLastError();
}

}  // namespace

// Largest d a search for k results takes: one query's vector and candidate buffer, plus the kernel's
// 96 bytes of static LDS, must fit the 64 KB a workgroup may use without opting in to more.
int f32_max_d(int k)
{
    const int64_t room = 64 * 1024 - 128 - (int64_t)f32_cap(k) * (int64_t)sizeof(cand_t);
    return room < 16 ? 0 : (int)(room / 16 * 4);
}

static size_t f32_lists_bytes(int64_t n, int64_t nq, int d, int k)
{
    return ((size_t)nq * f32_splits(n, nq, d, k) * k * sizeof(cand_t) + 255) & ~size_t(255);
}

static size_t f32_batch_bytes(int64_t n, int64_t nq, int d, int k)
{
    return f32_lists_bytes(n, nq, d, k) + f32_filter_plan(n, nq, d, k).total;
}

// Queries searched at a time: as many as 256 MB of workspace hold, in parts of about the same size.  (Whole, 8192
// queries, k = 480 on 1M x 128 took 1.2 GB of candidate regions, where the direct kernel's lists take 31 MB.  A few
// thousand queries fill the tiles: 10 000, k = 100, 512 MB, 10.22 ms, in four parts of 141 MB 10.40.)
constexpr size_t F32_WORKSPACE = size_t(256) << 20;

static size_t f32_parts_bytes(int64_t n, int64_t nq, int64_t b, int d, int k)   // the largest part's workspace
{
    const int64_t last = nq > b ? nq % b : 0;
    const size_t full = f32_batch_bytes(n, b, d, k), rest = last ? f32_batch_bytes(n, last, d, k) : 0;
    return full > rest ? full : rest;
}

static int64_t f32_batch(int64_t n, int64_t nq, int d, int k)
{
    if (nq <= 256) return nq;
    for (int64_t parts = ceil_div(nq, 16384);; parts *= 2) {
        const int64_t b = parts == 1 ? nq : round_up(ceil_div(nq, parts), 128);
        if (b <= 256 || f32_parts_bytes(n, nq, b, d, k) <= F32_WORKSPACE) return b;
    }
}

size_t f32_workspace_bytes(int64_t n, int64_t nq, int d, int k)
{
    return f32_parts_bytes(n, nq, f32_batch(n, nq, d, k), d, k);
}

static hipError_t launch_f32_batch(const float *x, int64_t n, int64_t ldx, const float *q, int64_t nq, int64_t ldq,
                                   int d, int k, int metric, int32_t *ids, float *dists, void *ws, hipStream_t st)
{
    const int S = f32_splits(n, nq, d, k);
    const int qt = f32_query_tile(d, k);
    const int mode = metric == LPQ_METRIC_L2SQ ? MODE_F32_L2 : MODE_F32_IP;
    const int cap = f32_cap(k);
    const int64_t split_rows = round_up(ceil_div(n, S), F32_STEP);
    const size_t shmem = (size_t)qt * ((size_t)cap * sizeof(cand_t) + (size_t)((d + 3) / 4) * 16);
    if (d > f32_max_d(k) || shmem + 128 > 64 * 1024) return hipErrorInvalidValue;   // callers check f32_max_d first
    cand_t *lists = reinterpret_cast<cand_t *>(ws);
    const bool vec = ((uintptr_t)x % 16 == 0) && (ldx % 4 == 0);
    const unsigned blocks = (unsigned)(ceil_div(nq, qt) * S);
    hipError_t e;
    // Larger batches: the matrix-core filter, direct sums of what it leaves, selection; the direct kernel
    // then only works on query tiles that hold a query whose candidates did not fit.
    const F32Filter fp = f32_filter_plan(n, nq, d, k);
    const int32_t *only = nullptr;
    if (fp.use && ldx <= f32_filter_max_ld(d)) {
        char *fws = (char *)ws + f32_lists_bytes(n, nq, d, k);
        e = launch_f32_filter(fp, x, n, ldx, q, nq, ldq, d, k, mode == MODE_F32_L2, fws, st);
        if (e != hipSuccess) return e;
        FinishIo o = {};
        o.x = x; o.q = q; o.ldx = ldx; o.ldq = ldq; o.d = d; o.k = k; o.SS = fp.S2; o.Cs = fp.Cs;
        o.ccnt = reinterpret_cast<const int32_t *>(fws + fp.off_ccnt);
        o.cbuf = reinterpret_cast<const cand_t *>(fws + fp.off_cbuf);
        o.qn = reinterpret_cast<const float *>(fws + fp.off_qn);
        o.hard = reinterpret_cast<const int32_t *>(fws + fp.off_hard);
        o.again = reinterpret_cast<const int32_t *>(fws + fp.off_again);
        o.qx = reinterpret_cast<const int32_t *>(fws + fp.off_qx);
        // (LDS for no more than there can be lets more workgroups run at a time: 100 000 x 64, 10 000
        // queries, k = 10, six regions of 128: the search 451 -> 427 us)
        const int64_t most = (int64_t)fp.S2 * fp.Cs;
        o.cap = most >= FIN_FEW ? FIN_CAP : 2 * next_pow2(most < 32 ? 32 : (int)most);
        o.c = f32_filter_constant(d); o.ch = f32_half_filter_constant(d);
        int32_t *over = reinterpret_cast<int32_t *>(fws + fp.off_over);
        o.over = over; o.ids = ids; o.dists = dists;
        e = launch_finish(vec, mode == MODE_F32_L2, nq, o, st);
        if (e != hipSuccess) return e;
        only = over;
    }
    switch (qt) {
    case 8: e = launch_f32_tile<8>(vec, blocks, shmem, st, x, n, ldx, q, ldq, nq, d, k, mode, S, split_rows, lists, cap, only); break;
    case 4: e = launch_f32_tile<4>(vec, blocks, shmem, st, x, n, ldx, q, ldq, nq, d, k, mode, S, split_rows, lists, cap, only); break;
    case 2: e = launch_f32_tile<2>(vec, blocks, shmem, st, x, n, ldx, q, ldq, nq, d, k, mode, S, split_rows, lists, cap, only); break;
    default: e = launch_f32_tile<1>(vec, blocks, shmem, st, x, n, ldx, q, ldq, nq, d, k, mode, S, split_rows, lists, cap, only); break;
    }
    if (e != hipSuccess) return e;
    return launch_merge(lists, nq, S, k, nullptr, nullptr, nullptr, ids, reinterpret_cast<int32_t *>(dists),
                        nullptr, mode, st, true, only);
}

hipError_t launch_search_f32(const float *x, int64_t n, int64_t ldx, const float *q, int64_t nq, int64_t ldq,
                             int d, int k, int metric, int32_t *ids, float *dists, void *ws, hipStream_t st)
{
    const int64_t b = f32_batch(n, nq, d, k);
    for (int64_t q0 = 0; q0 < nq; q0 += b) {
        const hipError_t e = launch_f32_batch(x, n, ldx, q + q0 * ldq, nq - q0 < b ? nq - q0 : b, ldq, d, k, metric,
                                              ids + q0 * k, dists + q0 * k, ws, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace lpq
