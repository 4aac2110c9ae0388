// Last step of a search by group maxima (small batches).  The scan before it (search_mfma.hip, the seeding pass run over
// every row) has left one number per query and group of rows: the largest 2 dot - nx (the key negated) of the group, or the largest
// dot for inner products.  At least k items reach the k-th largest of the maxima, so the k nearest lie in groups that reach it, k of
// them and a few more; their rows are scored again and the k best kept.  Nothing was sampled and no candidate was collected on the
// way, so three launches make a search where five and eight did.  One query, k = 10, 1M x 128: scan 31 -> 22.7 us, what goes before
// and after it 24 -> 14 (sample 7, bound 5, merge 6 and encoding against 9 here and encoding), 55 -> 37 in all; 100 queries on
// 10 000 x 128 36 -> 18.5; 16 on 10M x 96 203 -> 188 (16 us here: 6700 rows a query, from memory).
// Ties.  The maxima are exact keys, so rows that tie with the k-th differ by their ids alone, and the lowest are found block by
// block from the first row on.  (With E = dot - ceil(nx / 2) in place of the key a row of odd norm was one nearer than its group's maximum said, and
// every group at the bound had half of its rows scored.)  16 queries, L2, k = 10, us, lists in registers / every group at the bound
// scored / now: half of 1M x 64 rows zero 91 / 129 / 48; one feature in twenty set, 1M x 32 55 / 62 / 41, 1M x 16 91 / 163 / 44, 64
// queries 107 / 601 / 48 and 196 / 510 / 51; each of 1000 vectors 1000 times, 1M x 64 47 / 62 / 42.
#include "block_select.h"
#include "lpq_internal.h"
#include "wave_ops.h"

namespace lpq {

namespace {

constexpr int MF_FLY = 8;             // 16-byte loads of rows a lane has in flight
constexpr int MF_UNITS = 1024;        // units worked off at a time; a unit is the 16 rows of a group in one stage
constexpr int MF_TIES = 256;          // candidates whose ranks are counted between two lists; more are sorted
constexpr int MF_WIDEST = 2048;       // blocks of 32 rows looked at together where many groups tie, at most
constexpr int MF_STEPS = 4;           // steps that a workgroup works off the groups that reach the bound in, before other ways are looked for
constexpr int MF_TAIL = 8;            // blocks of 32 rows behind the last whole stage, at most
constexpr int MF_MERGE = 2048;        // candidates of all helpers together, at most

// 16 bytes of a row with the query's codes at that place, its chunk c (packed rows: two codes + 8 to a byte, see generic_scan).
template <bool PACKED>
__device__ __forceinline__ int chunk_dot(uint4 xv, const uint4 *qs, int c)
{
    int dot = 0;
    if (PACKED) {
        const uint4 q0 = qs[2 * c], q1 = qs[2 * c + 1];
        const unsigned m = 0x0F0F0F0Fu;
        dot = __builtin_amdgcn_sdot4((int)(xv.x & m), (int)q0.x, dot, false);
        dot = __builtin_amdgcn_sdot4((int)((xv.x >> 4) & m), (int)q0.y, dot, false);
        dot = __builtin_amdgcn_sdot4((int)(xv.y & m), (int)q0.z, dot, false);
        dot = __builtin_amdgcn_sdot4((int)((xv.y >> 4) & m), (int)q0.w, dot, false);
        dot = __builtin_amdgcn_sdot4((int)(xv.z & m), (int)q1.x, dot, false);
        dot = __builtin_amdgcn_sdot4((int)((xv.z >> 4) & m), (int)q1.y, dot, false);
        dot = __builtin_amdgcn_sdot4((int)(xv.w & m), (int)q1.z, dot, false);
        dot = __builtin_amdgcn_sdot4((int)((xv.w >> 4) & m), (int)q1.w, dot, false);
    } else {
        const uint4 qv = qs[c];
        dot = __builtin_amdgcn_sdot4((int)xv.x, (int)qv.x, dot, false);
        dot = __builtin_amdgcn_sdot4((int)xv.y, (int)qv.y, dot, false);
        dot = __builtin_amdgcn_sdot4((int)xv.z, (int)qv.z, dot, false);
        dot = __builtin_amdgcn_sdot4((int)xv.w, (int)qv.w, dot, false);
    }
    return dot;
}

// One or more workgroups per query: each finds the same bound from the maxima, scores its share of the rows of the groups that
// reach it, and the one that ends last merges.  What bounds it is latency: a round trip to memory for the maxima (V 16-byte loads a
// thread, all in flight at once), one per step of 128 KB of rows (32 KB by 256 threads; a workgroup alone gets some 30 GB/s from memory),
// and two with the fences where helpers share the work.  LR lanes share a row, CPL times 16 bytes each.
template <int NT, bool PACKED, int LR, int CPL>
__global__ __launch_bounds__(NT) void maxima_finish_kernel(
    SearchArgs a, MaximaShape m, const int32_t *__restrict__ gmax, int helpers, int most_helpers, cand_t *lists, int32_t *counts,
    int32_t *done, int cap,
    int32_t *__restrict__ ids, int32_t *__restrict__ dists, const int32_t *__restrict__ qnorms, int metric)
{
    constexpr int ROWS = NT / LR, FLY = MF_FLY / CPL;               // rows side by side and behind one another in a step, 16 to a unit
    constexpr int V = 4;
    static_assert(FLY * ROWS % 16 == 0, "a step takes whole units");
    extern __shared__ __align__(16) unsigned char smem[];
    cand_t *buf = reinterpret_cast<cand_t *>(smem);                 // [max(cap, merge)]
    __shared__ uint4 qs[MAXIMA_MAX_D / 16];
    __shared__ int s_top[256], s_hit[MF_UNITS], s_over[MF_UNITS], s_unit[MF_UNITS];   // groups that reach the bound, groups above it; first rows of units
    __shared__ int s_count[2], s_bound, s_hits, s_above, s_units, s_last;
    __shared__ cand_t s_thr;
    const int64_t q = blockIdx.x / most_helpers;
    const int h = blockIdx.x % most_helpers, tid = threadIdx.x, lane = tid & 63, sub = tid % LR, grp = tid / LR;
    const bool l2 = a.metric == LPQ_METRIC_L2SQ;
    auto key_of = [&](int value) { return l2 ? -value : -2 * value; };   // the least key of a group with this maximum

    // ---- the bound: the k-th largest of the largest maxima of 256 foursomes of threads -----------
    const int4 *gm = reinterpret_cast<const int4 *>(gmax + q * m.G);
    // The four groups a thread loads at a time: a foursome's are 256 such units apart, as the neighbours of a group hold the rows beside
    // its own and a cluster stored in one piece is in few of them (427 queries, k = 10, 57 474 x 667 in clusters of 1646 rows: 213 us
    // with the sixteen of a foursome side by side, 78 so; by lists 65).
    auto unit_of = [&](int j) { return (NT == 256 ? tid : (tid & 3) * 256 + (tid >> 2)) + j * NT; };
    int4 v[V];
    int top = INT32_MIN;
#pragma unroll
    for (int j = 0; j < V; ++j) {
        const int i = unit_of(j);
        v[j] = i < m.G / 4 ? gm[i] : int4{INT32_MIN, INT32_MIN, INT32_MIN, INT32_MIN};
    }
    for (int i = tid; i < a.d_pad / 16; i += NT) qs[i] = reinterpret_cast<const uint4 *>(a.qcodes + q * a.d_pad)[i];
    for (int i = tid; i < cap; i += NT) buf[i] = CAND_NONE;
    if (tid < 2) s_count[tid] = 0;
    if (tid == 0) s_hits = s_above = s_units = 0;
#pragma unroll
    for (int j = 0; j < V; ++j) top = max(top, max(max(v[j].x, v[j].y), max(v[j].z, v[j].w)));
    const int own = top;
    if (NT > 256) {
        top = max(top, dpp_move<DPP_XOR1>(top));
        top = max(top, dpp_move<DPP_XOR2>(top));
    }
    if (NT == 256 || (tid & 3) == 0) s_top[NT == 256 ? tid : tid >> 2] = top;
    __syncthreads();
    if (tid < 64) {                                                 // bisection: the largest value that k of them reach
        int t[4], lo = INT32_MAX, hi = INT32_MIN;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            t[j] = s_top[lane + 64 * j];
            lo = min(lo, t[j] == INT32_MIN ? INT32_MAX : t[j]);     // (threads without a group; k have one, and each group has rows)
            hi = max(hi, t[j]);
        }
        int low = wave_min_i32(lo);
        for (unsigned wide = (unsigned)wave_max_i32(hi) - (unsigned)low; wide > 0;) {   // wave-uniform: it lies in [low, low + wide]
            const unsigned up = (wide + 1) / 2;
            int reach = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) reach += __popcll(__ballot(t[j] >= low + (int)up));
            low += reach >= a.k ? (int)up : 0;
            wide = reach >= a.k ? wide - up : up - 1;
        }
        if (lane == 0) {
            s_bound = low;
            s_thr = make_cand(key_of(low), 0xFFFFFFFFu);
        }
    }
    __syncthreads();
    const int bound = s_bound;

    // ---- rows of the groups that reach it --------------------------------------------------------
    AppendSteps at;
    int appended = 0;
    const uint4 *rows = reinterpret_cast<const uint4 *>(a.codes);
    const int chunks = a.d_pad >> (PACKED ? 5 : 4);
    // one step: `pick(i)` is the row of slot i (0 .. FLY * ROWS - 1) or -1
    auto step = [&](auto pick) {
        int row[FLY], nx[FLY];
        uint4 x[FLY][CPL];
#pragma unroll
        for (int u = 0; u < FLY; ++u) {                             // all loads in flight before the first is used
            row[u] = pick(grp + u * ROWS);
            const size_t r = row[u] >= 0 ? row[u] : 0;
#pragma unroll
            for (int c = 0; c < CPL; ++c) x[u][c] = rows[r * chunks + (sub + c * LR < chunks ? sub + c * LR : 0)];
            nx[u] = l2 ? a.norms[r] : 0;
        }
#pragma unroll
        for (int u = 0; u < FLY; ++u) {
            int dot = 0;
#pragma unroll
            for (int c = 0; c < CPL; ++c) dot += sub + c * LR < chunks ? chunk_dot<PACKED>(x[u][c], qs, sub + c * LR) : 0;
            dot += dpp_move<DPP_XOR1>(dot);
            dot += dpp_move<DPP_XOR2>(dot);
            dot += dpp_move<DPP_HALF_MIRROR>(dot);
            if (LR >= 16) dot += dpp_move<DPP_ROW_MIRROR>(dot);
            if (LR >= 32) dot += __shfl_xor(dot, 16, 64);
            if (LR >= 64) dot += __shfl_xor(dot, 32, 64);
            if (sub == 0 && row[u] >= 0) {
                const cand_t c = make_cand(nx[u] - 2 * dot, (uint32_t)row[u]);
                if (c < s_thr) buf[at.held - at.before + atomicAdd(&s_count[at.turn], 1)] = c;
            }
        }
        __syncthreads();
        const int count = __builtin_amdgcn_readfirstlane(s_count[at.turn]);
        appended += count - at.before;
        at.step_done(count);
        block_compact_if_full(buf, cap, a.k, FLY * ROWS, at.held, &s_thr);
    };
    auto work_off = [&]() {                                         // the units listed
        __syncthreads();
        const int units = s_units;
        __syncthreads();
        if (tid == 0) s_units = 0;
        for (int base = 0; base < units; base += FLY * ROWS / 16)
            step([&](int i) {
                const int j = i & 15, row = base + (i >> 4) < units ? s_unit[base + (i >> 4)] + 8 * (j >> 2) + (j & 3) : -1;
                return (unsigned)row < (unsigned)a.n ? row : -1;
            });
        __syncthreads();
    };
    auto tighten = [&]() {                                          // the k best of at least as many candidates, and their bound
        const int held = at.held;                                   // (the same in every thread)
        if (held < a.k) return;
        if (held <= MF_TIES) {
            const cand_t me = tid < held ? buf[tid] : CAND_NONE;
            int r = 0;
            for (int j = 0; tid < held && j < held; ++j) r += buf[j] < me;
            __syncthreads();
            if (tid >= a.k && tid < held) buf[tid] = CAND_NONE;
            if (tid < held && r < a.k) buf[r] = me;
            if (tid < held && r == a.k - 1 && me < s_thr) s_thr = me;
            at.held = a.k;
            __syncthreads();
        } else {
            block_compact_if_full(buf, cap, a.k, cap, at.held, &s_thr);
        }
    };
    auto stages_of = [&](int s) { return (m.stages - s + m.S - 1) / m.S; };
    if (own >= bound) {                                             // (few threads have a group that does)
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const int val[4] = {v[j].x, v[j].y, v[j].z, v[j].w}, first = 4 * unit_of(j);
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (val[c] >= bound && first + c < m.G) {
                    const int slot = atomicAdd(&s_hits, 1);
                    if (slot < MF_UNITS) s_hit[slot] = first + c;
                }
        }
    }
    __syncthreads();
    const int hits = s_hits, units = hits * m.seg_stages;
    // How many of the query's workgroups work, the same answer in each: all where there is more to do than the first have in a few
    // steps.  (The others then cost nothing; all of them always, with the fences and the merge, 2 us of 9 for one query on 1M x 128.
    // 64 queries, k = 100, 100 000 x 64: 59 us by the first alone, 46 by all.)
    constexpr int STEP_UNITS = FLY * ROWS / 16, STEPS = NT == 256 ? 2 * MF_STEPS : MF_STEPS;
    const int few = max(4 * a.k + 64, m.G / 32) < MF_UNITS ? max(4 * a.k + 64, m.G / 32) : MF_UNITS;
    int H = hits > few || units > STEPS * STEP_UNITS * helpers ? most_helpers : helpers;
    if (h >= H) return;
    int above = 0;
    bool walk = false, ties_only = false;
    int T0 = 0, all = 0;                                            // most stages of a split, and blocks of 32 rows in so many
    if (hits > few || units > STEPS * STEP_UNITS * H) {
        // Many groups: are they above the bound or at it?
        if (own > bound) {
#pragma unroll
            for (int j = 0; j < V; ++j) {
                const int val[4] = {v[j].x, v[j].y, v[j].z, v[j].w}, first = 4 * unit_of(j);
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (val[c] > bound) {
                        const int slot = atomicAdd(&s_above, 1);
                        if (slot < MF_UNITS) s_over[slot] = first + c;
                    }
            }
        }
        __syncthreads();
        above = s_above;
        const int ties = hits - above;
        ties_only = above <= 4 * a.k + 64;                          // (fewer than k are above the k-th largest maximum)
        // Walked if each workgroup's share of the groups at the bound is twice k or more, or where so many are at it that each
        // of them probably holds many such rows; otherwise scoring them all takes no more steps.
        walk = hits > MF_UNITS || ties > 2 * H * a.k || 4 * ties > m.G;
        T0 = stages_of(0);
        all = T0 * m.S * (m.parts / 2);
        if (ties_only && ties > 2 * H * a.k) {                      // each finds its k early, if they are spread evenly: one or a few do
            H = (all + 8191) / 8192 < H ? (all + 8191) / 8192 : H;
            if (h >= H) return;
        }
    }
    // The groups that reach the bound, or those above it where those at it are walked.  The helpers share the units, not the groups.
    const int *groups = walk ? s_over : s_hit;
    const int total = (walk ? (ties_only ? above : 0) : hits) * m.seg_stages, most = MF_UNITS - 2 * MF_TAIL;
    // the rows behind the last whole stage were not scanned: units of the same form
    const int tail = m.stages * m.stage_rows;
    auto list_tail = [&]() {
        if (h == 0 && tid < 2 * MF_TAIL && (tid >> 1) * 32 < (int)a.n - tail) s_unit[atomicAdd(&s_units, 1)] = tail + (tid >> 1) * 32 + (tid & 1) * 4;
    };
    if (!walk) list_tail();
    for (int from = 0; from == 0 || from < total; from += most) {
        const int to = from + most < total ? from + most : total;
        for (int u = from + tid; u < to; u += NT) {
            const int i = groups[u / m.seg_stages], nth = u % m.seg_stages;
            if (H > 1 && (i + nth) % H != h) continue;
            const int part = i % m.parts, seg = (i / m.parts) % m.SEG, s = i / (m.parts * m.SEG), T = stages_of(s);
            const int t = (int)(((int64_t)seg * T + m.SEG - 1) / m.SEG) + nth;
            if (t >= (int)(((int64_t)(seg + 1) * T + m.SEG - 1) / m.SEG)) continue;
            s_unit[atomicAdd(&s_units, 1)] = (s + m.S * t) * m.stage_rows + (part >> 1) * 32 + (part & 1) * 4;
        }
        work_off();
    }
    if (walk) {
        // Items that tie with the k-th by the hundreds or thousands (rows that repeat, features of few values).  What the groups
        // above the bound do not give is taken from those at it, lowest ids first: block by block, until k are held.  (Groups
        // above the bound in numbers, the nearest rows in few of the sets it was taken from: any group that can still win is taken.)
        if (tid == 0 && h == 0) atomicOr(&done[q], MAXIMA_MANY);
        const int longer = m.stages - (T0 - 1) * m.S;               // splits with T0 stages; the others have one less
        const int per_stage = m.parts / 2, share = (all + H - 1) / H;
        int better = 0;
        if (ties_only && above > 0) {
            if (tid == 0) s_hits = 0;
            __syncthreads();
            for (int i = tid; i < at.held; i += NT)
                if (cand_key(buf[i]) < key_of(bound)) atomicAdd(&s_hits, 1);
            __syncthreads();
            better = s_hits;
        }
        appended = 0;
        // The first look lists about a step's units, or an eighth of k, if groups at the bound are spread evenly.
        int width = ties_only ? (int)((int64_t)max(STEP_UNITS, a.k / 8) * m.G / (2 * (hits - above))) : 4;
        width = width < 4 ? 4 : width < MF_WIDEST ? width : MF_WIDEST;
        for (int from = 0; from < share && !(ties_only && better + appended >= a.k);) {
            if (!ties_only) tighten();
            const cand_t worst = s_thr;
            if (ties_only && make_cand(key_of(bound), (uint32_t)(from * H / per_stage * m.stage_rows)) >= worst) break;   // the same in every thread
            const int to = from + width < share ? from + width : share;
            for (int j = from + tid; j < to; j += NT) {
                const int u = j * H + (h + j) % H;                  // one of H blocks behind one another to each helper, in turn
                const int st = u / per_stage, s = st % m.S, t = st / m.S, T = s < longer ? T0 : T0 - 1;
                if (u >= all || t >= T) continue;
                const int2 pair = *reinterpret_cast<const int2 *>(gmax + q * m.G + (s * m.SEG + t * m.SEG / T) * m.parts + u % per_stage * 2);
#pragma unroll
                for (int part = 0; part < 2; ++part) {
                    const int largest = part ? pair.y : pair.x, row = st * m.stage_rows + u % per_stage * 32 + part * 4;
                    if (largest < bound || (ties_only ? largest > bound : make_cand(key_of(largest), (uint32_t)row) >= worst)) continue;
                    const int slot = atomicAdd(&s_units, 1);
                    if (slot < MF_UNITS) s_unit[slot] = row;
                }
            }
            __syncthreads();
            const int listed = s_units;
            if (listed > MF_UNITS) {                                // (half as many blocks always fit)
                __syncthreads();
                if (tid == 0) s_units = 0;
                width = MF_UNITS / 2;
                __syncthreads();
                continue;
            }
            const int had = appended;
            work_off();
            from = to;
            // The next: as many blocks as hold half as much again as is missing, if they hold as much each, at most four times as
            // many as now, or as list 256 units.
            int64_t next = 4 * width;
            if (ties_only && appended > had) next = min(next, (int64_t)width * 3 * (a.k - better - appended) / (2 * (appended - had)) + 1);
            if (listed > 0) next = min(next, (int64_t)width * (MF_UNITS / 4) / listed);
            width = (int)max((int64_t)4, min(next, (int64_t)MF_WIDEST));
        }
        list_tail();
        work_off();
    }

    // ---- the k best: ranks are counted, or where there are many candidates they are sorted -------
    auto finish = [&](int held, auto put) {
        if (held <= NT) {
            if (tid < held) {
                const cand_t me = buf[tid];
                int r = 0;
                for (int j = 0; j < held; ++j) r += buf[j] < me;
                if (r < a.k) put(r, me);
            }
            return;
        }
        const int pow2 = next_pow2(held);
        for (int i = held + tid; i < pow2; i += NT) buf[i] = CAND_NONE;
        __syncthreads();
        block_bitonic_sort(buf, pow2);
        for (int i = tid; i < a.k; i += NT) put(i, buf[i]);
    };
    int held = at.held;
    if (tid == 0) counts[q * most_helpers + h] = held < a.k ? held : a.k;
    if (H > 1) {
        cand_t *mine = lists + (q * most_helpers + h) * a.k;
        finish(held, [&](int r, cand_t c) { mine[r] = c; });
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");            // this wave's part has reached the L2 ...
        __syncthreads();
        if (tid == 0) {
            __threadfence();                                        // ... and is visible to the chip
            s_last = (atomicAdd(&done[q], 1) & (MAXIMA_MANY - 1)) == H - 1;
            if (s_last) __threadfence();                            // the other helpers' parts are read as they are now
            s_hits = 0;
        }
        __syncthreads();
        if (!s_last) return;                                        // the same in every thread of the workgroup
        for (int i = tid; i < H * a.k; i += NT)
            if (i % a.k < counts[q * most_helpers + i / a.k]) buf[atomicAdd(&s_hits, 1)] = lists[q * most_helpers * a.k + i];
        __syncthreads();
        held = s_hits;
    }
    finish(held, [&](int r, cand_t c) { emit_result(c, q * a.k + r, q, ids, dists, qnorms, metric); });
}

}  // namespace

hipError_t launch_maxima_finish(const SearchArgs &a, const MaximaShape &m, const int32_t *gmax, int threads, int helpers, int most_helpers, cand_t *lists,
                                int32_t *counts, int32_t *done, int32_t *ids, int32_t *dists, const int32_t *qnorms, int metric, hipStream_t st)
{
    if (a.nq <= 0) return hipSuccess;
    const int chunks = a.d_pad / (a.packed ? 32 : 16), lr = chunks <= 8 ? 8 : chunks <= 16 ? 16 : chunks <= 32 ? 32 : 64;
    const int per_lane = chunks <= 64 ? 1 : (chunks <= 128 ? 2 : 4), step = MF_FLY / per_lane * threads / lr;
    const int tops = threads == 256 ? m.G / 4 : m.G / 16;
    // the bound is the k-th of the (foursomes of) threads' maxima, the list of units has room for the rows behind the last
    // stage, and all that the helpers keep fits one merge
    if ((threads != 256 && threads != 1024) || a.k < 1 || a.k > MAXIMA_MAX_K || (threads == 256 && chunks > 16) ||
        (a.packed && chunks > 8) || a.d_pad > MAXIMA_MAX_D || helpers < 1 ||
        most_helpers < helpers || most_helpers * a.k > MF_MERGE || m.G % 16 || tops < a.k || m.G > 16 * threads ||
        a.n - (int64_t)m.stages * m.stage_rows > 32 * MF_TAIL || (m.stages / m.S + 1) * (int64_t)m.SEG > INT32_MAX ||
        ((int64_t)m.stages + m.S) * m.parts + most_helpers > INT32_MAX)
        return hipErrorInvalidValue;
    const int cap = next_pow2(a.k + step);
    const int most = most_helpers > 1 ? next_pow2(most_helpers * a.k) : cap;
    const size_t lds = (size_t)(cap > most ? cap : most) * sizeof(cand_t);
    auto launch = [&](auto kern) {
        kern<<<(unsigned)(a.nq * most_helpers), threads, lds, st>>>(a, m, gmax, helpers, most_helpers, lists, counts, done, cap, ids, dists, qnorms, metric);
        return hipGetLastError();
    };
    if (threads == 256) {
        if (a.packed) return launch(maxima_finish_kernel<256, true, 8, 1>);
        return lr == 8 ? launch(maxima_finish_kernel<256, false, 8, 1>) : launch(maxima_finish_kernel<256, false, 16, 1>);
    }
    if (a.packed) return launch(maxima_finish_kernel<1024, true, 8, 1>);
    switch (lr) {
    case 8: return launch(maxima_finish_kernel<1024, false, 8, 1>);
    case 16: return launch(maxima_finish_kernel<1024, false, 16, 1>);
    case 32: return launch(maxima_finish_kernel<1024, false, 32, 1>);
    default: break;
    }
    if (per_lane == 1) return launch(maxima_finish_kernel<1024, false, 64, 1>);
    return per_lane == 2 ? launch(maxima_finish_kernel<1024, false, 64, 2>) : launch(maxima_finish_kernel<1024, false, 64, 4>);
}

}  // namespace lpq
