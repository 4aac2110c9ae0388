// Generic integer search kernel: any padded dimension, any k <= MAX_K.  One workgroup scans
// one corpus split for one query with 4-way int8 dot products, keeps the candidates that
// beat the running k-th best in an LDS buffer and compacts the buffer by a bitonic sort
// whenever it could overflow.  It is the fallback for shapes the matrix-core kernel does
// not take and an independent second implementation of the same result.
#include <type_traits>

#include "block_select.h"
#include "lpq_internal.h"
#include "wave_ops.h"

namespace lpq {

namespace {

constexpr int GEN_THREADS = 256;
constexpr int GEN_ROWS = GEN_THREADS / 8;  // rows per step: 8 lanes share a row

// One (query, corpus split) pair by the whole workgroup; must be reached by all its threads.
__device__ __forceinline__ void generic_scan(const SearchArgs &a, int64_t rs, int64_t re, int64_t q, const cand_t *seeds,
                                             cand_t *out, int cap, cand_t *buf, uint4 *qs, int *s_count, cand_t *s_thr)
{
    const int chunks = a.d_pad >> 4;  // 16-byte chunks per row of int8 codes
    const bool l2 = a.metric == LPQ_METRIC_L2SQ;
    for (int c = threadIdx.x; c < chunks; c += GEN_THREADS)
        qs[c] = reinterpret_cast<const uint4 *>(a.qcodes + q * a.d_pad)[c];
    // Packed rows: a 16-byte chunk holds 32 codes, two to a byte, stored + 8; the low nibbles of a
    // dword meet one dword of the (permuted) query codes and its high nibbles the next one, as in
    // the matrix-core scan.  The result is dot(code + 8, q): the same key that scan produces.
    const int xchunks = a.packed ? chunks >> 1 : chunks;
    const int64_t row_bytes = a.packed ? a.d_pad >> 1 : a.d_pad;
    for (int i = threadIdx.x; i < cap; i += GEN_THREADS) buf[i] = CAND_NONE;
    if (threadIdx.x < 2) s_count[threadIdx.x] = 0;
    if (threadIdx.x == 0) *s_thr = seeds ? seeds[q] : CAND_NONE;
    __syncthreads();
    AppendSteps at;

    const int sub = threadIdx.x & 7, grp = threadIdx.x >> 3;
    for (int64_t base = rs; base < re; base += GEN_ROWS) {
        const int64_t row = base + grp;
        int dot = 0;
        if (row < re) {
            const uint4 *xr = reinterpret_cast<const uint4 *>(a.codes + row * row_bytes);
            if (a.packed) {
                for (int c = sub; c < xchunks; c += 8) {
                    const uint4 xv = xr[c], q0 = qs[2 * c], q1 = qs[2 * c + 1];
                    const unsigned m = 0x0F0F0F0Fu;
                    dot = __builtin_amdgcn_sdot4((int)(xv.x & m), (int)q0.x, dot, false);
                    dot = __builtin_amdgcn_sdot4((int)((xv.x >> 4) & m), (int)q0.y, dot, false);
                    dot = __builtin_amdgcn_sdot4((int)(xv.y & m), (int)q0.z, dot, false);
                    dot = __builtin_amdgcn_sdot4((int)((xv.y >> 4) & m), (int)q0.w, dot, false);
                    dot = __builtin_amdgcn_sdot4((int)(xv.z & m), (int)q1.x, dot, false);
                    dot = __builtin_amdgcn_sdot4((int)((xv.z >> 4) & m), (int)q1.y, dot, false);
                    dot = __builtin_amdgcn_sdot4((int)(xv.w & m), (int)q1.z, dot, false);
                    dot = __builtin_amdgcn_sdot4((int)((xv.w >> 4) & m), (int)q1.w, dot, false);
                }
            } else {
                for (int c = sub; c < chunks; c += 8) {
                    const uint4 xv = xr[c], qv = qs[c];
                    dot = __builtin_amdgcn_sdot4((int)xv.x, (int)qv.x, dot, false);
                    dot = __builtin_amdgcn_sdot4((int)xv.y, (int)qv.y, dot, false);
                    dot = __builtin_amdgcn_sdot4((int)xv.z, (int)qv.z, dot, false);
                    dot = __builtin_amdgcn_sdot4((int)xv.w, (int)qv.w, dot, false);
                }
            }
        }
        dot += __shfl_xor(dot, 4, 64);
        dot += __shfl_xor(dot, 2, 64);
        dot += __shfl_xor(dot, 1, 64);
        if (sub == 0 && row < re) {
            const int32_t key = (l2 ? a.norms[row] : 0) - 2 * dot;  // see cand_t
            const cand_t c = make_cand(key, (uint32_t)row);
            if (c < *s_thr) {
                const int pos = at.held - at.before + atomicAdd(&s_count[at.turn], 1);
                buf[pos] = c;
            }
        }
        __syncthreads();
        at.step_done(__builtin_amdgcn_readfirstlane(s_count[at.turn]));
        block_compact_if_full(buf, cap, a.k, GEN_ROWS, at.held, s_thr);
    }
    block_bitonic_sort(buf, cap);
    for (int i = threadIdx.x; i < a.k; i += GEN_THREADS) out[i] = buf[i];
    __syncthreads();   // buf and qs are free again
}

__global__ __launch_bounds__(GEN_THREADS) void search_generic_kernel(
    SearchArgs a, int64_t row0, int64_t row1, int S, int64_t split_rows, const cand_t *__restrict__ seeds,
    cand_t *__restrict__ lists, int cap)
{
    extern __shared__ __align__(16) unsigned char smem[];
    cand_t *buf = reinterpret_cast<cand_t *>(smem);
    uint4 *qs = reinterpret_cast<uint4 *>(buf + cap);
    __shared__ int s_count[2];
    __shared__ cand_t s_thr;
    const int64_t q = blockIdx.x / S;
    const int s = blockIdx.x % S;
    const int64_t rs = row0 + (int64_t)s * split_rows;
    const int64_t re = (rs + split_rows < row1) ? rs + split_rows : row1;
    generic_scan(a, rs, re, q, seeds, lists + ((int64_t)q * S + s) * a.k, cap, buf, qs, s_count, &s_thr);
}

// 64-bit minimum over the wave; every lane gets the result.
__device__ __forceinline__ cand_t wave_min_cand(cand_t c) { return wave_min_u64(c); }

// First candidate in (key, id) order that a bound taken from candidate c does not let through.
__device__ __forceinline__ cand_t next_bound(cand_t c) { return c + 1; }

// The same scan for a LIST of queries (the ones a collecting scan could not finish): the
// workgroups of a fixed-size grid share out the (listed query, split) pairs, so a handful of
// queries is spread over the whole chip and an empty list costs one tiny launch.  The workgroup that
// finishes a query's last split merges its lists: the flag of a query, 1 when listed, counts the finished ones (and
// stays non-zero), so no second launch is needed, and none waits for another.
// The merge takes no more LDS than eight workgroups of a CU have room for (with 32 KB to sort 4096 at once, 16 of 4000
// queries, k = 20, on 1M x 128 took 0.87 ms here, with 16 KB 0.72).
constexpr int LIST_MERGE_CAP = 2048;
__global__ __launch_bounds__(GEN_THREADS) void search_generic_list_kernel(
    SearchArgs a, int64_t row0, int64_t row1, int S, int64_t split_rows, RedoList first, int first_max, RedoList last,
    cand_t *lists, int cap, const cand_t *done_lists, int done_count, int32_t *__restrict__ ids, int32_t *__restrict__ dists,
    const int32_t *__restrict__ qnorms, int metric)
{
    extern __shared__ __align__(16) unsigned char smem[];
    cand_t *buf = reinterpret_cast<cand_t *>(smem);
    uint4 *qs = reinterpret_cast<uint4 *>(buf + cap);
    __shared__ int s_count[2], s_last;
    __shared__ cand_t s_thr;
    // the m candidates of a query's lists, up to 4096, sorted in two or three parts
    auto merge = [&](const cand_t *from_lists, int64_t q, int m) {
        for (int from = 0, kept = 0; from < m; kept = a.k) {
            const int take = m - from < LIST_MERGE_CAP - kept ? m - from : LIST_MERGE_CAP - kept;
            int mcap = 2;
            while (mcap < kept + take) mcap <<= 1;
            for (int i = kept + threadIdx.x; i < mcap; i += GEN_THREADS)
                buf[i] = i < kept + take ? from_lists[q * m + from + (i - kept)] : CAND_NONE;
            __syncthreads();
            block_bitonic_sort(buf, mcap);
            from += take;
        }
        for (int i = threadIdx.x; i < a.k; i += GEN_THREADS) emit_result(buf[i], q * a.k + i, q, ids, dists, qnorms, metric);
        __syncthreads();
    };
    const bool many = *first.count > first_max;             // same for every thread of the grid
    if (many && !last.queries) {                            // another kernel has searched them
        for (int64_t i = blockIdx.x; done_lists && i < *first.count; i += gridDim.x) merge(done_lists, first.queries[i], done_count * a.k);
        return;
    }
    const RedoList work = many ? last : first;
    const int64_t items = (int64_t)(*work.count) * S;
    for (int64_t item = blockIdx.x; item < items; item += gridDim.x) {
        const int64_t q = work.queries[item / S];
        const int s = (int)(item % S);
        const int64_t rs = row0 + (int64_t)s * split_rows;
        const int64_t re = (rs + split_rows < row1) ? rs + split_rows : row1;
        generic_scan(a, rs, re, q, nullptr, lists + ((int64_t)q * S + s) * a.k, cap, buf, qs, s_count, &s_thr);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");    // this wave's part of the list has reached the L2 ...
        __syncthreads();
        if (threadIdx.x == 0) {
            __threadfence();                                // ... and is visible to the chip, by one write-back for all
            s_last = atomicAdd(&work.flags[q], 1) == S;
            if (s_last) __threadfence();                    // the other lists are read as they are now
        }
        __syncthreads();
        if (s_last) merge(lists, q, S * a.k);               // the same answer in every thread of the workgroup
    }
}

// One workgroup per query: sort all candidates of its P lists (plus an optional extra list).
__global__ __launch_bounds__(256) void merge_kernel(
    const cand_t *__restrict__ lists, int P, int k, const cand_t *__restrict__ extra, int cap,
    cand_t *__restrict__ out_lists, cand_t *__restrict__ seeds_out, int32_t *__restrict__ ids,
    int32_t *__restrict__ dists, const int32_t *__restrict__ qnorms, int metric, const int32_t *__restrict__ only)
{
    extern __shared__ __align__(16) unsigned char smem[];
    cand_t *buf = reinterpret_cast<cand_t *>(smem);
    const int64_t q = blockIdx.x;
    if (only && !only[q]) return;   // same for the whole workgroup
    const int m = P * k;
    for (int i = threadIdx.x; i < cap; i += 256) {
        cand_t c = CAND_NONE;
        if (i < m) c = lists[q * m + i];
        else if (extra && i < m + k) c = extra[q * k + (i - m)];
        buf[i] = c;
    }
    __syncthreads();
    block_bitonic_sort(buf, cap);
    for (int i = threadIdx.x; i < k; i += 256) {
        const cand_t c = buf[i];
        if (out_lists) out_lists[q * k + i] = c;
        if (ids) emit_result(c, q * k + i, q, ids, dists, qnorms, metric);
    }
    if (seeds_out && threadIdx.x == 0) seeds_out[q] = buf[k - 1];
}

// Last step of the collecting scan for small k (<= 32) and at most 64 regions, one WAVE per query
// and no LDS: lane r owns region r.  In each pass every lane loads up to 8 more candidates of its
// region into registers; together with the k best kept so far (lane i keeps the i-th best) the
// wave takes the smallest k times, which become the kept ones of the next pass.  Any number of
// candidates the regions can hold is handled; a query with an overflowed region or fewer than k
// candidates is flagged in over[] instead.
__global__ __launch_bounds__(256) void collect_select_wave_kernel(
    const cand_t *__restrict__ cbuf, const int32_t *__restrict__ ccnt, int64_t nq, int SS, int Cs, int k,
    int32_t *__restrict__ over, int32_t *__restrict__ qlist, int32_t *__restrict__ qcount,
    int32_t *__restrict__ ids, int32_t *__restrict__ dists, const int32_t *__restrict__ qnorms, int metric)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t q = (int64_t)blockIdx.x * 4 + wave;
    if (q >= nq) return;                                   // wave-uniform
    const int c = (lane < SS) ? ccnt[q * SS + lane] : 0;
    const bool bad = c > Cs || c < 0;
    int total = bad ? 0 : c, most = total;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        total += __shfl_xor(total, o, 64);
        const int t = __shfl_xor(most, o, 64);
        most = t > most ? t : most;
    }
    if (__ballot(bad) || total < k) {
        if (lane == 0) { over[q] = 1; qlist[atomicAdd(qcount, 1)] = (int32_t)q; }
        return;
    }
    const cand_t *mine = cbuf + ((size_t)q * SS + (lane < SS ? lane : 0)) * Cs;
    cand_t keep = CAND_NONE;                               // lane i: the i-th best so far
    constexpr int E = 8;                                   // candidates a lane takes per pass
    for (int p0 = 0; p0 < most; p0 += E) {                 // wave-uniform trip count
        cand_t v[E + 1];
#pragma unroll
        for (int e = 0; e < E; ++e) v[e] = (p0 + e < c && !bad) ? mine[p0 + e] : CAND_NONE;
        v[E] = keep;
        cand_t next = CAND_NONE;
        for (int r = 0; r < k; ++r) {
            cand_t m = v[0];
#pragma unroll
            for (int e = 1; e <= E; ++e) m = v[e] < m ? v[e] : m;
            const cand_t mn = wave_min_cand(m);
            if (lane == r) next = mn;
            const int win = __ffsll((unsigned long long)__ballot(m == mn)) - 1;
            bool done = lane != win || mn == CAND_NONE;
#pragma unroll
            for (int e = 0; e <= E; ++e) {
                const bool hit = !done && v[e] == mn;
                v[e] = hit ? CAND_NONE : v[e];
                done = done || hit;
            }
        }
        keep = next;
    }
    if (lane < k) emit_result(keep, q * k + lane, q, ids, dists, qnorms, metric);
    if (lane == 0) over[q] = 0;
}

// 64-bit value of lane `src` (any lane), through two 32-bit shuffles.
__device__ __forceinline__ cand_t shfl_u64(cand_t v, int src)
{
    const unsigned lo = (unsigned)__shfl((int)(uint32_t)v, src, 64), hi = (unsigned)__shfl((int)(uint32_t)(v >> 32), src, 64);
    return ((cand_t)hi << 32) | lo;
}

// Ascending bitonic sort of 64 E candidates held E per lane by one wave, element e = E * lane + slot.
// Strides below E exchange registers of a lane, larger strides exchange with lane ^ (stride / E).
template <int E>
__device__ __forceinline__ void wave_sort(cand_t (&v)[E], int lane)
{
#pragma unroll
    for (int size = 2; size <= 64 * E; size <<= 1) {
#pragma unroll
        for (int stride = size >> 1; stride >= 1; stride >>= 1) {
            if (stride >= E) {
                const int lx = stride / E;
                const bool up = ((lane * E) & size) == 0;          // this run of `size` elements sorts ascending
                const bool low = (lane & lx) == 0;                 // this lane holds the lower element of each pair
                const bool take_min = up == low;
#pragma unroll
                for (int j = 0; j < E; ++j) {
                    const cand_t o = shfl_u64(v[j], lane ^ lx);
                    v[j] = take_min ? (o < v[j] ? o : v[j]) : (o > v[j] ? o : v[j]);
                }
            } else {
#pragma unroll
                for (int j = 0; j < E; ++j) {
                    if ((j & stride) == 0) {
                        const bool up = ((lane * E + j) & size) == 0;
                        const cand_t a = v[j], b = v[j | stride];
                        const bool swap = up ? (b < a) : (a < b);
                        v[j] = swap ? b : a;
                        v[j | stride] = swap ? a : b;
                    }
                }
            }
        }
    }
}

// A query whose regions overflowed: whatever the scan did collect for it are real items, so the k-th
// best of them bounds its final k-th best from above - and far more closely than the seeding pass did,
// since they all passed its bound.  The scan passes candidates strictly below a bound, and the k-th best
// itself must pass: the bound of the next round is the candidate right after it in (key, id) order, so ties
// of its key with larger ids do not pass (a region keeps its FIRST arrivals, the lowest ids among equal
// keys, which is what makes this converge on codes of few bits).
//
// By one workgroup, when there may be more candidates than the sort takes: every region gives its first
// min(count, Cs, maxc / SS) candidates; when the regions hold more, every candidate no worse than the k-th
// best of those - about k Cs / per of them - is sorted again, and the k-th best of ALL collected ones comes
// out.  (If even those do not fit, the first estimate stands: it is a valid bound either way.)
__device__ cand_t refined_bound(const cand_t *cbuf, const int32_t *ccnt, int64_t q, int SS, int Cs, int k, int maxc,
                                cand_t *buf, cand_t old_bound)
{
    __shared__ int s_n;
    const int tid = threadIdx.x;
    const int per = maxc / SS < Cs ? maxc / SS : Cs;           // slots per region, >= 1
    const int used = SS * per;
    int cap = 2;
    while (cap < used) cap <<= 1;
    __syncthreads();                                           // buf is free
    for (int i = tid; i < cap; i += 256) {
        cand_t c = CAND_NONE;
        if (i < used) {
            const int r = i / per, j = i - r * per;
            const int cnt = ccnt[q * SS + r];
            if (j < cnt) c = cbuf[((size_t)q * SS + r) * Cs + j];   // cnt > Cs: the region holds Cs, and j < per <= Cs
        }
        buf[i] = c;
    }
    __syncthreads();
    block_bitonic_sort(buf, cap);
    cand_t kth = (k <= cap) ? buf[k - 1] : CAND_NONE;   // the same value in every thread
    __syncthreads();
    if (per < Cs && kth != CAND_NONE) {
        if (tid == 0) s_n = 0;
        __syncthreads();
#pragma unroll 4
        for (int i = tid; i < SS * Cs; i += 256) {
            const int r = i / Cs;
            const cand_t c = i - r * Cs < ccnt[q * SS + r] ? cbuf[(size_t)q * SS * Cs + i] : CAND_NONE;
            if (c <= kth) {
                const int at = atomicAdd(&s_n, 1);
                if (at < maxc) buf[at] = c;
            }
        }
        __syncthreads();
        const int m = s_n;
        if (m >= k && m <= maxc) {
            int cap2 = 2;
            while (cap2 < m) cap2 <<= 1;
            for (int i = m + tid; i < cap2; i += 256) buf[i] = CAND_NONE;
            __syncthreads();
            block_bitonic_sort(buf, cap2);
            kth = buf[k - 1];
        }
    }
    return kth == CAND_NONE ? old_bound : next_bound(kth);
}

// One query of the kernel below by one wave: writes its result, or returns true if it has to be flagged.
__device__ bool collect_select_one(const cand_t *__restrict__ cbuf, const int32_t *__restrict__ ccnt, int64_t q, int SS, int Cs,
                                   int k, int32_t *__restrict__ ids, int32_t *__restrict__ dists,
                                   const int32_t *__restrict__ qnorms, int metric)
{
    const int lane = threadIdx.x & 63;
    const int count = lane < SS ? ccnt[q * SS + lane] : 0;
    const bool bad = count > Cs || count < 0;
    const int mine = bad ? 0 : count;
    int incl = mine;                                       // inclusive prefix sum over the lanes
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    const int total = __shfl(incl, 63, 64);
    if (__ballot(bad) || total < k) return true;           // wave-uniform
    const int excl = incl - mine;                          // index of the first candidate of this lane's region
    const cand_t *base = cbuf + (size_t)q * SS * Cs;
    // candidate number i of the query sits in the region of the first lane whose inclusive count exceeds i
    auto fetch = [&](int i) -> cand_t {
        int r = 0;
#pragma unroll
        for (int step = 32; step >= 1; step >>= 1)
            if (__shfl(incl, r + step - 1, 64) <= i) r += step;
        r = r > 63 ? 63 : r;
        const int at = i - __shfl(excl, r, 64);
        return i < total ? base[(size_t)r * Cs + at] : CAND_NONE;
    };
    auto put = [&](cand_t v, int e) {                      // the e-th best
        if (e < k) emit_result(v, q * k + e, q, ids, dists, qnorms, metric);
    };
    // few candidates: a smaller network (2 or 4 per lane) does
    auto small = [&](auto tag) {
        constexpr int E = decltype(tag)::value;
        cand_t v[E];
#pragma unroll
        for (int j = 0; j < E; ++j) v[j] = fetch(j * 64 + lane);
        wave_sort<E>(v, lane);
#pragma unroll
        for (int j = 0; j < E; ++j) put(v[j], lane * E + j);
    };
    if (total <= 128) {                                    // wave-uniform
        small(std::integral_constant<int, 2>{});
    } else if (total <= 256) {
        small(std::integral_constant<int, 4>{});
    } else {
        cand_t v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = fetch(j * 64 + lane);
        wave_sort<8>(v, lane);
        for (int done = 512; done < total; done += 384) {  // wave-uniform: the best 128 stay in lanes 0 .. 15
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const cand_t n = fetch(done + j * 48 + (lane - 16));   // (every lane takes part in the shuffles)
                if (lane >= 16) v[j] = n;
            }
            wave_sort<8>(v, lane);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) put(v[j], lane * 8 + j);
    }
    return false;
}

// Last step of the collecting scan for k <= 128 and at most 64 regions, one WAVE per query: lane r holds the
// count of region r; the wave loads up to 512 candidates (2, 4 or 8 per lane as needed, each
// found by a search over the prefix counts), sorts them in registers and keeps the best 128 in its first 16 lanes;
// further candidates come in 384 at a time through the other 48 lanes.  Any number of candidates the regions hold
// is handled; a query with an overflowed region or fewer than k candidates is flagged in over[] instead, and gets a
// tighter bound for the next round where bounds_out is given (zero for the others): by all four waves, as its
// regions hold thousands of candidates (one wave sorting them 384 at a time took 0.24 ms for 16 384).
constexpr int SORT_BOUND_BUF = 2048;   // of refined_bound: 16 KB, which leaves ten workgroups to a CU
__global__ __launch_bounds__(256) void collect_select_sort_kernel(
    const cand_t *__restrict__ cbuf, const int32_t *__restrict__ ccnt, int64_t nq, int SS, int Cs, int k,
    int32_t *__restrict__ over, int32_t *__restrict__ qlist, int32_t *__restrict__ qcount,
    int32_t *__restrict__ ids, int32_t *__restrict__ dists, const int32_t *__restrict__ qnorms, int metric,
    const cand_t *__restrict__ bounds_in, cand_t *__restrict__ bounds_out)
{
    __shared__ cand_t buf[SORT_BOUND_BUF];
    __shared__ int s_flagged[4];
    const int64_t first = (int64_t)blockIdx.x * 4;
    const bool flagged = first + (threadIdx.x >> 6) < nq &&
                         collect_select_one(cbuf, ccnt, first + (threadIdx.x >> 6), SS, Cs, k, ids, dists, qnorms, metric);
    if ((threadIdx.x & 63) == 0) s_flagged[threadIdx.x >> 6] = flagged;
    __syncthreads();
    for (int j = 0; j < 4 && first + j < nq; ++j) {        // the same in every thread
        const int64_t q = first + j;
        if (threadIdx.x == 0) {
            over[q] = s_flagged[j];
            if (s_flagged[j]) qlist[atomicAdd(qcount, 1)] = (int32_t)q;
        }
        if (!bounds_out) continue;
        const cand_t bound = s_flagged[j] ? refined_bound(cbuf, ccnt, q, SS, Cs, k, SORT_BOUND_BUF, buf, bounds_in[q]) : 0;
        if (threadIdx.x == 0) bounds_out[q] = bound;
    }
}

// The same with one workgroup per query, SS <= 256: nothing is sorted while the regions hold no more than
// RANK_FEW candidates.  A histogram of the keys between the best and the worst gives the few (k and the rest of a bin)
// that can belong, and the rank of each is the number of better ones, counted by the thread that holds it.  More
// candidates are sorted RANK_FEW at a time, the k best kept.  Against a wave per query that sorts in registers: k = 100,
// 450 candidates, 1000 queries 20 -> 11 us, 10 000 on 1M x 128 73 -> 47, on 4M x 256 107 -> 57; k = 10, 1000 queries on
// 1.2M x 100 9.8 -> 6.7, on 500 000 x 768 10.7 -> 7.6, on 200 000 x 2048 (350 candidates) 19.6 -> 7.8, 100 on 10 000 x 128
// 6.0 -> 4.3.  Large batches with few candidates stay with the wave, a quarter of a workgroup per query: 10 000 queries,
// k = 10, 90 candidates 21 us against 29 here.  RANK_TO_NQ is the line where there are 64 regions or fewer; on short rows that
// is from some 3600 queries on, where the wave is ahead (whole searches, k = 10, wave and here: 100 000 x 64, 3600 queries 92
// and 95 us, 50 000 778 and 816; 400 000 x 128, 4000 216 and 217, 10 000 485 and 492), so that the number decides for long rows
// alone, where the two hardly differ (500 000 x 768, 2600 queries 993 and 985, 6000 2144 and 2136; 1M x 256, 3000 671 and 670).
constexpr int RANK_FROM_K = 16, RANK_TO_NQ = 2048, RANK_FROM_EXPECTED = 192;
constexpr int RANK_FEW = 2048, RANK_COUNTED = 512, RANK_BINS = 256;
__global__ __launch_bounds__(256) void collect_select_rank_kernel(
    const cand_t *__restrict__ cbuf, const int32_t *__restrict__ ccnt, int SS, int Cs, int k,
    int32_t *__restrict__ over, int32_t *__restrict__ qlist, int32_t *__restrict__ qcount,
    int32_t *__restrict__ ids, int32_t *__restrict__ dists, const int32_t *__restrict__ qnorms, int metric,
    const cand_t *__restrict__ bounds_in, cand_t *__restrict__ bounds_out)
{
    __shared__ cand_t buf[RANK_FEW], few[RANK_COUNTED];
    __shared__ int s_end[256], s_hist[RANK_BINS], s_wave[4], s_cut, s_more;
    __shared__ uint32_t s_lo[4], s_hi[4];
    const int64_t q = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    auto scan = [&](int v) {                                   // inclusive sums over the lanes of a wave
#pragma unroll
        for (int w = 1; w < 64; w <<= 1) {
            const int up = __shfl_up(v, w, 64);
            if (lane >= w) v += up;
        }
        return v;
    };
    // The lanes of a region share its candidates, 256 lanes where there is one region.  (With a thread to a region whole
    // searches on 1M x 128, k = 100 took: 50 000 queries, 5 regions 7.9 ms, 100 000, 2 regions 19.7, 300 000, one 69.0;
    // 7.7, 19.1 and 65.5 now, and a wave's sort 7.9, 19.3 and 65.9.)
    const int share = __clz(SS - 1) - 24, per = 1 << share, region = tid >> share, sub = tid & (per - 1);
    const int mine = region < SS ? ccnt[q * SS + region] : 0;
    const int bad = mine > Cs || mine < 0;
    const int upto = scan(bad || sub ? 0 : mine);
    if (lane == 63) s_wave[wave] = upto;
    s_hist[tid] = 0;
    if (tid == 0) s_more = 0;
    const int lost = __syncthreads_or(bad);
    int end = upto, total = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        end += w < wave ? s_wave[w] : 0;
        total += s_wave[w];
    }
    const bool flagged = lost || total < k;                    // the same in every thread
    if (tid == 0) {
        over[q] = flagged;
        if (flagged) qlist[atomicAdd(qcount, 1)] = (int32_t)q;
    }
    if (bounds_out) {
        const cand_t bound = flagged ? refined_bound(cbuf, ccnt, q, SS, Cs, k, RANK_FEW, buf, bounds_in[q]) : 0;
        if (tid == 0) bounds_out[q] = bound;
    }
    if (flagged) return;
    const cand_t *regions = cbuf + (size_t)q * SS * Cs;
    if (total > RANK_FEW) {
        if (sub == 0) s_end[region] = end;
        __syncthreads();
        int kept = 0;
        for (int pos = 0; pos < total;) {
            const int take = total - pos < RANK_FEW - kept ? total - pos : RANK_FEW - kept;
            for (int i = tid; i < RANK_FEW - kept; i += 256) {
                cand_t c = CAND_NONE;
                if (i < take) {
                    int lo = 0, hi = SS - 1;                   // first region that ends beyond it
                    while (lo < hi) {
                        const int mid = (lo + hi) >> 1;
                        if (s_end[mid] > pos + i) hi = mid; else lo = mid + 1;
                    }
                    c = regions[(size_t)lo * Cs + (pos + i - (lo ? s_end[lo - 1] : 0))];
                }
                buf[kept + i] = c;
            }
            __syncthreads();
            block_bitonic_sort(buf, RANK_FEW);
            pos += take;
            kept = k;
        }
        for (int i = tid; i < k; i += 256) emit_result(buf[i], q * k + i, q, ids, dists, qnorms, metric);
        return;
    }
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
    for (int i = sub; i < mine; i += per) {
        const cand_t c = regions[(size_t)region * Cs + i];
        buf[end - mine + i] = c;
        const uint32_t key = (uint32_t)(c >> 32);
        lo = key < lo ? key : lo;
        hi = key > hi ? key : hi;
    }
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) {
        const uint32_t l = __shfl_xor(lo, w, 64), h = __shfl_xor(hi, w, 64);
        lo = l < lo ? l : lo;
        hi = h > hi ? h : hi;
    }
    if (lane == 0) { s_lo[wave] = lo; s_hi[wave] = hi; }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        lo = s_lo[w] < lo ? s_lo[w] : lo;
        hi = s_hi[w] > hi ? s_hi[w] : hi;
    }
    const int wide = 32 - __clz((int)(hi - lo)), shift = wide > 8 ? wide - 8 : 0;
    auto bin = [&](cand_t c) { return (int)(((uint32_t)(c >> 32) - lo) >> shift); };
    for (int i = tid; i < total; i += 256) atomicAdd(&s_hist[bin(buf[i])], 1);
    __syncthreads();
    if (wave == 0) {                                           // the bin that holds the k-th
        int v[4], sum = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) { v[j] = s_hist[4 * lane + j]; sum += v[j]; }
        const int incl = scan(sum);
        if (lane == __ffsll((unsigned long long)__ballot(incl >= k)) - 1) {
            int at = incl - sum, j = 0;
            while (j < 3 && at + v[j] < k) at += v[j++];
            s_cut = 4 * lane + j;
        }
    }
    __syncthreads();
    const int cut = s_cut;
    for (int i = tid; i < total; i += 256)
        if (bin(buf[i]) <= cut) {
            const int at = atomicAdd(&s_more, 1);
            if (at < RANK_COUNTED) few[at] = buf[i];
        }
    __syncthreads();
    const int count = s_more;
    if (count <= RANK_COUNTED) {
        for (int i = tid; i < count; i += 256) {
            const cand_t me = few[i];
            int r = 0;
            for (int j = 0; j < count; ++j) r += few[j] < me;
            if (r < k) emit_result(me, q * k + r, q, ids, dists, qnorms, metric);
        }
        return;
    }
    const int cap = next_pow2(total);                          // many in the last bin: sort
    for (int i = total + tid; i < cap; i += 256) buf[i] = CAND_NONE;
    __syncthreads();
    block_bitonic_sort(buf, cap);
    for (int i = tid; i < k; i += 256) emit_result(buf[i], q * k + i, q, ids, dists, qnorms, metric);
}

// Last step of the collecting scan, one workgroup per query: gather the query's regions into LDS,
// sort, write the k best.  A query with an overflowed region, more than `maxc` candidates or fewer
// than k is flagged in over[] instead and left to the generic kernel.
__global__ __launch_bounds__(256) void collect_select_kernel(
    const cand_t *__restrict__ cbuf, const int32_t *__restrict__ ccnt, int SS, int Cs, int k, int maxc,
    int32_t *__restrict__ over, int32_t *__restrict__ qlist, int32_t *__restrict__ qcount,
    int32_t *__restrict__ ids, int32_t *__restrict__ dists, const int32_t *__restrict__ qnorms, int metric,
    const int32_t *__restrict__ only, const int32_t *__restrict__ gate_count, int gate_min,
    const cand_t *bounds_in, cand_t *bounds_out /* may be the same array */)
{
    extern __shared__ __align__(16) unsigned char smem[];
    cand_t *buf = reinterpret_cast<cand_t *>(smem);            // [maxc]
    int *off = reinterpret_cast<int *>(buf + maxc);            // [SS + 1] first slot of each region
    __shared__ int tsum[256];
    __shared__ int s_bad;
    const int64_t q = blockIdx.x;
    const int tid = threadIdx.x;
    if (only) {   // second round: queries flagged in the first one, if they were more than gate_min
        if (*gate_count <= gate_min || !only[q]) {
            if (tid == 0) {
                over[q] = 0;
                if (bounds_out) bounds_out[q] = 0;
            }
            return;
        }
    }
    const int per = (SS + 255) / 256;                          // consecutive regions per thread
    const int r0 = tid * per, r1 = (r0 + per < SS) ? r0 + per : SS;
    if (tid == 0) s_bad = 0;
    __syncthreads();
    int local = 0;
    bool bad = false;
    for (int r = r0; r < r1; ++r) {
        const int c = ccnt[q * SS + r];
        bad |= c > Cs || c < 0;
        local += (c > Cs) ? Cs : (c < 0 ? 0 : c);
    }
    if (bad) s_bad = 1;
    tsum[tid] = local;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {                        // inclusive scan of the thread sums
        const int v = (tid >= o) ? tsum[tid - o] : 0;
        __syncthreads();
        tsum[tid] += v;
        __syncthreads();
    }
    const int M = tsum[255];
    if (s_bad || M > maxc || M < k) {
        if (tid == 0) { over[q] = 1; qlist[atomicAdd(qcount, 1)] = (int32_t)q; }
        if (bounds_out) {
            const cand_t b = refined_bound(cbuf, ccnt, q, SS, Cs, k, maxc, buf, bounds_in[q]);
            if (tid == 0) bounds_out[q] = b;
        }
        return;
    }
    int run = tsum[tid] - local;
    for (int r = r0; r < r1; ++r) {
        off[r] = run;
        const int c = ccnt[q * SS + r];
        run += c;
    }
    if (tid == 255) off[SS] = M;
    const int cap = next_pow2(M < 2 ? 2 : M);
    __syncthreads();
    for (int i = tid; i < cap; i += 256) {
        cand_t c = CAND_NONE;
        if (i < M) {
            int lo = 0, hi = SS;                               // last region with off[r] <= i
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (off[mid] <= i) lo = mid; else hi = mid;
            }
            c = cbuf[((size_t)q * SS + lo) * Cs + (i - off[lo])];
        }
        buf[i] = c;
    }
    __syncthreads();
    block_bitonic_sort(buf, cap);
    for (int i = tid; i < k; i += 256) emit_result(buf[i], q * k + i, q, ids, dists, qnorms, metric);
    if (tid == 0) {
        over[q] = 0;
        if (bounds_out) bounds_out[q] = 0;                     // nothing passes: this query is done
    }
}

// Merge of lists that are each sorted ascending, for k <= 32 and up to 1024 lists: one workgroup per
// query, LPL lists per thread.  The k-th smallest of the threads' smallest heads bounds the k-th best
// from above (k threads own one candidate at least as good), and only the candidates up to it - found
// by walking the few lists whose head is - are gathered and sorted: at most k threads' LPL lists of k.
// Two register sorts of 64 or 128 candidates give the bound.  The lists are not staged anywhere: a list
// costs one 8-byte load unless its head passes.  Measured on 512 lists of 10: 14.3 -> 6 us for one
// query against k rounds of "smallest head" per wave over all lists held in LDS.
constexpr int MERGE_SORTED_BUF = 4096;      // k * LPL * k candidates at most
template <int LPL, int E>
__global__ __launch_bounds__(256) void merge_sorted_kernel(
    const cand_t *__restrict__ lists, int P, int k, const cand_t *__restrict__ extra,
    cand_t *__restrict__ out_lists, cand_t *__restrict__ seeds_out, int32_t *__restrict__ ids,
    int32_t *__restrict__ dists, const int32_t *__restrict__ qnorms, int metric)
{
    extern __shared__ __align__(16) unsigned char smem[];
    cand_t *buf = reinterpret_cast<cand_t *>(smem);     // [MERGE_SORTED_BUF]
    __shared__ cand_t best[64 * E], bound;              // k <= 16 E smallest of each wave
    __shared__ int count;
    const int Pt = P + (extra ? 1 : 0);
    const int64_t q = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    cand_t head[LPL], mn = CAND_NONE;
#pragma unroll
    for (int j = 0; j < LPL; ++j) {
        const int l = threadIdx.x + 256 * j;
        head[j] = l < P ? lists[(q * P + l) * k] : (l < Pt ? extra[q * k] : CAND_NONE);
        mn = head[j] < mn ? head[j] : mn;
    }
    // lane i < k of the result: the i-th smallest of the lanes' values (all different, or CAND_NONE); the
    // shortest lists by k rounds of "smallest", which beat the sorting network up to k = 4
    auto smallest = [&](cand_t c) -> cand_t {
        if (k > 4) {
            cand_t v[1] = {c};
            wave_sort<1>(v, lane);
            return v[0];
        }
        cand_t out = CAND_NONE;
        for (int r = 0; r < k; ++r) {
            const cand_t m = wave_min_cand(c);
            if (lane == r) out = m;
            if (c == m) c = CAND_NONE;
        }
        return out;
    };
    const cand_t wbest = smallest(mn);
    if (lane < 16 * E) best[wave * 16 * E + lane] = wbest;
    if (threadIdx.x == 0) count = 0;
    __syncthreads();
    if (wave == 0 && E == 1) {
        const cand_t c = smallest(best[lane]);
        if (lane == k - 1) bound = c;
    } else if (wave == 0) {
        cand_t v[E];
#pragma unroll
        for (int j = 0; j < E; ++j) v[j] = best[E * lane + j];
        wave_sort<E>(v, lane);
#pragma unroll
        for (int j = 0; j < E; ++j)
            if (E * lane + j == k - 1) bound = v[j];
    }
    __syncthreads();
    const cand_t top = bound;
#pragma unroll
    for (int j = 0; j < LPL; ++j) {
        if (head[j] <= top && head[j] != CAND_NONE) {
            const int l = threadIdx.x + 256 * j;
            const cand_t *list = l < P ? lists + (q * P + l) * k : extra + q * k;
            cand_t c = head[j];
            for (int i = 1;; ++i) {
                const int at = atomicAdd(&count, 1);
                if (at < MERGE_SORTED_BUF) buf[at] = c;
                if (i == k) break;
                c = list[i];
                if (c > top || c == CAND_NONE) break;
            }
        }
    }
    __syncthreads();
    const int m = count < MERGE_SORTED_BUF ? count : MERGE_SORTED_BUF;   // >= k wherever the lists hold k candidates
    auto emit = [&](cand_t c, int r) {
        if (r >= k) return;
        if (out_lists) out_lists[q * k + r] = c;
        if (seeds_out && r == k - 1) seeds_out[q] = c;
        if (ids) emit_result(c, q * k + r, q, ids, dists, qnorms, metric);
    };
    auto sorted = [&](auto tag) {                       // up to 64 S candidates, by one wave in registers
        constexpr int S = decltype(tag)::value;
        cand_t v[S];
#pragma unroll
        for (int j = 0; j < S; ++j) { const int i = j * 64 + lane; v[j] = i < m ? buf[i] : CAND_NONE; }
        wave_sort<S>(v, lane);
#pragma unroll
        for (int j = 0; j < S; ++j) emit(v[j], lane * S + j);
    };
    if (m <= 64) {
        if (wave == 0) emit(smallest(lane < m ? buf[lane] : CAND_NONE), lane);
    } else if (m <= 128) {
        if (wave == 0) sorted(std::integral_constant<int, 2>{});
    } else if (m <= 256) {
        if (wave == 0) sorted(std::integral_constant<int, 4>{});
    } else {
        const int cap = next_pow2(m);
        for (int i = m + threadIdx.x; i < cap; i += 256) buf[i] = CAND_NONE;
        __syncthreads();
        block_bitonic_sort(buf, cap);
        for (int r = threadIdx.x; r < k; r += 256) emit(buf[r], r);
    }
}

// One workgroup per (query, group): sort the candidates of `group` consecutive lists.
__global__ __launch_bounds__(256) void merge_groups_kernel(const cand_t *__restrict__ lists, int P, int group, int groups,
                                                           int k, int cap, cand_t *__restrict__ out_lists)
{
    extern __shared__ __align__(16) unsigned char smem[];
    cand_t *buf = reinterpret_cast<cand_t *>(smem);
    const int64_t q = blockIdx.x / groups;
    const int g = blockIdx.x % groups;
    const int first = g * group, count = (first + group <= P ? group : P - first) * k;
    for (int i = threadIdx.x; i < cap; i += 256) buf[i] = (i < count) ? lists[(q * P + first) * k + i] : CAND_NONE;
    __syncthreads();
    block_bitonic_sort(buf, cap);
    for (int i = threadIdx.x; i < k; i += 256) out_lists[(q * groups + g) * k + i] = buf[i];
}

}  // namespace

hipError_t launch_merge_groups(const cand_t *lists, int64_t nq, int P, int group, int k, cand_t *out_lists,
                               hipStream_t st)
{
    if (nq <= 0) return hipSuccess;
    const int groups = (int)ceil_div(P, group);
    const int cap = next_pow2(group * k < 2 ? 2 : group * k);
    if (cap > 4096) return hipErrorInvalidValue;
    merge_groups_kernel<<<(unsigned)(nq * groups), 256, (size_t)cap * sizeof(cand_t), st>>>(lists, P, group, groups, k,
                                                                                          cap, out_lists);
    return hipGetLastError();
}

namespace {
}  // namespace

int merge_max_lists(int k) { return 4096 / k - 1; }

// Lists of k that are each sorted and short (k <= 32): at most 1024 of them, less one for an extra list.
int merge_max_sorted_lists(int k) { return k > 32 ? merge_max_lists(k) : 1023; }

hipError_t launch_collect_select(const cand_t *cbuf, const int32_t *ccnt, int64_t nq, int SS, int Cs, int k,
                                 int32_t *over, int32_t *qlist, int32_t *qcount, int32_t *ids, int32_t *dists,
                                 const int32_t *qnorms, int metric, hipStream_t st, int expected_candidates,
                                 const int32_t *only, const int32_t *gate_count, int gate_min, const cand_t *bounds_in,
                                 cand_t *bounds_out)
{
    if (nq <= 0) return hipSuccess;
    const int maxc = 4096;
    if (SS < 1 || SS > 2048 || k > maxc) return hipErrorInvalidValue;
    // (k rounds of "smallest in the wave" beat the sorting network only for the shortest lists: k = 1
    // 1.00 against 1.01 ms per search on the benchmark workload, k = 10 1.178 against 1.166, k = 32 1.446 against 1.375)
    if (!only && !bounds_out && expected_candidates > 0 && expected_candidates <= 256 && SS <= 64 && k <= 2) {
        collect_select_wave_kernel<<<(unsigned)ceil_div(nq, (int64_t)4), 256, 0, st>>>(cbuf, ccnt, nq, SS, Cs, k, over, qlist,
                                                                                 qcount, ids, dists, qnorms, metric);
        return hipGetLastError();
    }
    if (!only && k <= 128 && SS <= (nq > 64 ? 256 : 64)) {
        if (k > RANK_FROM_K || nq <= RANK_TO_NQ || expected_candidates > RANK_FROM_EXPECTED || SS > 64)
            collect_select_rank_kernel<<<(unsigned)nq, 256, 0, st>>>(cbuf, ccnt, SS, Cs, k, over, qlist, qcount, ids, dists, qnorms,
                                                                     metric, bounds_in, bounds_out);
        else   // one wave per query, sorted in registers
            collect_select_sort_kernel<<<(unsigned)ceil_div(nq, (int64_t)4), 256, 0, st>>>(cbuf, ccnt, nq, SS, Cs, k, over, qlist,
                                                                                         qcount, ids, dists, qnorms, metric,
                                                                                         bounds_in, bounds_out);
        return hipGetLastError();
    }
    const size_t lds = (size_t)maxc * sizeof(cand_t) + (size_t)(SS + 1) * sizeof(int);
    collect_select_kernel<<<(unsigned)nq, 256, lds, st>>>(cbuf, ccnt, SS, Cs, k, maxc, over, qlist, qcount, ids, dists,
                                                          qnorms, metric, only, gate_count, gate_min, bounds_in, bounds_out);
    return hipGetLastError();
}

hipError_t launch_search_generic(const SearchArgs &a, int64_t row0, int64_t row1, int S, const cand_t *seeds,
                                 cand_t *lists, hipStream_t st)
{
    if (a.nq <= 0 || row1 <= row0) return hipSuccess;
    const int cap = next_pow2((2 * a.k > a.k + 2 * GEN_ROWS) ? 2 * a.k : a.k + 2 * GEN_ROWS);
    const int64_t split_rows = round_up(ceil_div(row1 - row0, S), GEN_ROWS);
    const size_t shmem = (size_t)cap * sizeof(cand_t) + (size_t)a.d_pad;
    search_generic_kernel<<<(unsigned)(a.nq * S), GEN_THREADS, shmem, st>>>(a, row0, row1, S, split_rows,
                                                                              seeds, lists, cap);
    return hipGetLastError();
}

hipError_t launch_search_generic_list(const SearchArgs &a, int64_t row0, int64_t row1, int S, const RedoList &first,
                                      int first_max, const RedoList &last, cand_t *lists, int32_t *ids, int32_t *dists,
                                      const int32_t *qnorms, int metric, hipStream_t st, const cand_t *done_lists, int done_count)
{
    if (a.nq <= 0 || row1 <= row0) return hipSuccess;
    if ((int64_t)S * a.k > 4096 || (int64_t)done_count * a.k > 4096) return hipErrorInvalidValue;   // one workgroup merges a query's lists
    const int cap = next_pow2((2 * a.k > a.k + 2 * GEN_ROWS) ? 2 * a.k : a.k + 2 * GEN_ROWS);
    const int64_t split_rows = round_up(ceil_div(row1 - row0, S), GEN_ROWS);
    const size_t shmem = (size_t)cap * sizeof(cand_t) + (size_t)a.d_pad;
    const int longest = (done_count > S ? done_count : S) * a.k;
    const int merged = longest < 2 ? 2 : (longest < LIST_MERGE_CAP ? longest : LIST_MERGE_CAP);
    const size_t merge = (size_t)next_pow2(merged) * sizeof(cand_t);
    search_generic_list_kernel<<<2048, GEN_THREADS, shmem > merge ? shmem : merge, st>>>(
        a, row0, row1, S, split_rows, first, first_max, last, lists, cap, done_lists, done_count, ids, dists, qnorms, metric);
    return hipGetLastError();
}

hipError_t launch_merge(const cand_t *lists, int64_t nq, int P, int k, const cand_t *extra_lists,
                        cand_t *out_lists, cand_t *seeds_out, int32_t *ids, int32_t *dists,
                        const int32_t *qnorms, int metric, hipStream_t st, bool sorted_lists, const int32_t *only)
{
    if (nq <= 0) return hipSuccess;
    const int total = P * k + (extra_lists ? k : 0);
    // sorted lists of up to 32 (a sort of everything is as fast while it stays small: 39 lists of 10)
    if (!only && sorted_lists && k <= 32 && total > 256 && P <= merge_max_sorted_lists(k)) {
        const size_t lds = MERGE_SORTED_BUF * sizeof(cand_t);
        const int lpl = (int)ceil_div(P + (extra_lists ? 1 : 0), 256);   // lists a thread owns
        auto launch = [&](auto kern) -> hipError_t {
            kern<<<(unsigned)nq, 256, lds, st>>>(lists, P, k, extra_lists, out_lists, seeds_out, ids, dists, qnorms, metric);
            return hipGetLastError();
        };
        if (k <= 16) {
            if (lpl <= 1) return launch(merge_sorted_kernel<1, 1>);
            return lpl <= 2 ? launch(merge_sorted_kernel<2, 1>) : launch(merge_sorted_kernel<4, 1>);
        }
        if (lpl <= 1) return launch(merge_sorted_kernel<1, 2>);
        return lpl <= 2 ? launch(merge_sorted_kernel<2, 2>) : launch(merge_sorted_kernel<4, 2>);
    }
    const int cap = next_pow2(total < 2 ? 2 : total);
    if (cap > 4096) return hipErrorInvalidValue;
    merge_kernel<<<(unsigned)nq, 256, (size_t)cap * sizeof(cand_t), st>>>(
        lists, P, k, extra_lists, cap, out_lists, seeds_out, ids, dists, qnorms, metric, only);
    return hipGetLastError();
}

}  // namespace lpq
