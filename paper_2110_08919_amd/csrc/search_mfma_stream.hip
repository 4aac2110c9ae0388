// Matrix-core scan for rows too long for a wave to keep its queries in registers: both operands of
// the int8 contraction stream through LDS.
//
// A workgroup of eight waves computes tiles of 256 items x 64 WQ queries (WQ = 4, 2 or 1), the waves
// laid out 8 / WQ along the items and WQ along the queries, so a wave always holds WQ blocks of 32
// items by two blocks of 32 queries in accumulators.  A stage is 128 bytes (four k-steps of
// v_mfma_i32_32x32x32_i8) of every row of both operands, copied global->LDS asynchronously into a
// ring of two or three stages; the stages of consecutive tiles follow each other without a break, so
// the ring stays full across tile ends.  Only ceil(d / 128) stages of a row are read.
//
// Why this shape.  Rows of more than 1536 features had only the dot-product kernel; here the row
// length does not matter: a k-step of the 256 x 256 tile reads six fragments from LDS for eight matrix
// instructions.  200 000 x 2048, inner product, k = 10, whole search: 1000 queries 31.2 -> 0.42 ms, 10 000
// queries 3.9 ms = 2.1 POP/s.  Stages of 64 bytes (four in the ring) measured 10 % slower: half lines
// double the requests that the L2 serves.
//
// What bounds it: the matrix pipe is busy 64 % of the scan (1000 queries), the LDS 27 %, and the part is
// power-limited while it is, at 1.8 GHz (codes of few toggling bits run 10 % faster).  10 000 queries, same
// box: without the copies the search takes 3.0 ms instead of 3.9, without candidates 3.64.
//
// One workgroup barrier per stage, placed in front of its last k-step: by then every wave has read the
// stage (its reads were waited for), so the ring slot is refilled right behind the barrier, and the
// first fragments of the next stage are read while the last k-step is in the matrix core.
//
// Thresholds, keys, accumulator seeds and the collecting of candidates are those of the other
// matrix-core scans (see search_mfma.hip).  A tile ends only once per ceil(d / 128) stages, so its
// passing accumulators are queued and worked off there and then (appending each candidate from the
// accumulators, one block after the other, measured 8 % of the scan against 6 %).
#include "mfma_common.h"

namespace lpq {

namespace {

constexpr int SW = 8;                  // waves per workgroup
constexpr int TILE_ROWS = 256;         // items per tile
constexpr int KB = 128;                // bytes of a row per stage: whole 128-byte lines of the L2
constexpr int KS = KB / 32;            // k-steps per stage
constexpr int RUN = 16;                // a tile is 16 runs of 16 items, which the seeding pass takes from far apart
// Query codes an XCD's workgroups work on at a time: half of its 4 MB L2.
constexpr int64_t QGROUP_BYTES = 2 << 20;

struct StreamIo {
    const cand_t *seeds;   // [nq] thresholds of the collecting scan
    cand_t *cbuf;          // [nq][S][Cs] candidate regions
    int32_t *ccnt;         // [nq][S] candidates offered to each region
    int Cs;
    int32_t *gmax;         // seeding pass: [nq_pad][G] group maxima, G = S * SEG * 2 * (8 / WQ)
    int SEG;
    int tiles;             // tiles in all; split s takes tiles s, s + S, s + 2S, ...
    int64_t tile_stride;   // tile g starts at row g * tile_stride ...
    int64_t run_gap;       // ... and its runs of 16 items are this far apart (16: consecutive rows)
    int kst;               // stages per tile = ceil(d / 128)
    int qgroup;            // query tiles that one XCD works on at a time
    int32_t *done;         // search by group maxima (the pass reads every tile of consecutive rows, every segment has some): done[0 .. nq) = 0
};

// stages in the ring, and accumulator dumps a wave can queue: what 160 KB of LDS hold
constexpr int stream_stages(int wq) { return wq == 4 ? 2 : 3; }
constexpr int stream_dumps(int wq) { return wq == 2 ? 16 : 32; }
constexpr size_t stream_lds_bytes(int wq, bool seed)
{
    return (size_t)stream_stages(wq) * (TILE_ROWS + 64 * wq) * KB + 2 * (TILE_ROWS + 8) * 4 +
           (seed ? 0 : (size_t)64 * wq * 16 + (size_t)SW * stream_dumps(wq) * 80);
}
static_assert(stream_lds_bytes(4, false) <= 160 * 1024 && stream_lds_bytes(2, false) <= 160 * 1024 &&
              stream_lds_bytes(1, false) <= 160 * 1024, "one workgroup per CU");

// Asynchronous copy of 16 bytes per lane from base + off (base wave-uniform) to LDS.
__device__ __forceinline__ void async_copy16_at(const int8_t *base, unsigned off, unsigned lds_base)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_base), "v"(off), "s"(base) : "memory");
}

template <bool L2, bool SEED, int WQ>
__global__ __launch_bounds__(SW * 64, 2) void search_stream_kernel(SearchArgs a, int64_t row_end, int S,
                                                                                  int qtiles, StreamIo o)
{
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int WR = SW / WQ;                    // waves along the items
    constexpr int RB = WQ;                         // blocks of 32 items per wave: 256 / WR / 32
    constexpr int NST = stream_stages(WQ);
    constexpr int QT = 64 * WQ;
    constexpr int A_BYTES = TILE_ROWS * KB, STAGE = A_BYTES + QT * KB;
    constexpr int APW = TILE_ROWS / 8 / SW, BPW = QT / 8 / SW;   // copies per wave and stage: items, queries (8 rows each)
    constexpr int CPW = APW + BPW;
    constexpr int AUX = TILE_ROWS + 8;             // accumulator seeds and parity words of a tile

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
    const int wr = wave / WQ, wq = wave % WQ;

    // Order of (split, query tile) pairs.  Each XCD (workgroups are dealt to them round-robin) gets a
    // contiguous range, which walks the splits for a group of query tiles small enough to stay in its
    // L2 while the corpus streams by, then for the next group.
    const int total = qtiles * S, per = total / 8, b = blockIdx.x;
    const int wk = (b < per * 8) ? (b % 8) * per + b / 8 : b;
    const int grp = wk / (o.qgroup * S), in_grp = wk - grp * o.qgroup * S;
    const int gsize = qtiles - grp * o.qgroup < o.qgroup ? qtiles - grp * o.qgroup : o.qgroup;
    const int s = in_grp / gsize, qt = grp * o.qgroup + in_grp % gsize;

    unsigned char *ring = smem;
    int *aux = reinterpret_cast<int *>(smem + NST * STAGE);         // [2][AUX], by tile parity
    cand_t *thrC = reinterpret_cast<cand_t *>(aux + 2 * AUX);       // [QT] threshold candidates
    int *thrE = reinterpret_cast<int *>(thrC + QT);                 // [QT] the same on E, conservative
    int *fill = thrE + QT;                                          // [QT] candidates offered to this workgroup's regions
    constexpr int DUMPS = stream_dumps(WQ);
    int *dval = fill + QT + wave * (DUMPS * 20);                    // [DUMPS][16] accumulators this wave has queued
    v4i *dmeta = reinterpret_cast<v4i *>(dval + DUMPS * 16);        // [DUMPS] (first row, parity word, query | lane half << 8, -)
    const int64_t q_tile = (int64_t)qt * QT, q_first = q_tile + wq * 64;

    if constexpr (!SEED) {
        if (a.redo_flags) {   // a further round: only if the flagged queries are many, and only tiles that hold one
            if (*a.redo_count <= a.redo_min) return;   // the same answer in every thread of the grid
            int mine = 0;
            for (int64_t qq = q_tile + tid; qq < q_tile + QT && qq < a.nq; qq += SW * 64) mine |= a.redo_flags[qq];
            int *vote = reinterpret_cast<int *>(ring);   // the ring is still unused
            if (tid == 0) *vote = 0;
            __syncthreads();
            if (mine) atomicOr(vote, 1);
            __syncthreads();
            const int any = *vote;
            __syncthreads();   // everyone has read the vote before the ring is filled
            if (!any) return;  // the same answer in every thread of the workgroup
        }
        for (int i = tid; i < QT; i += SW * 64) {
            const cand_t sc = q_tile + i < a.nq ? o.seeds[q_tile + i] : 0;   // 0: a slot that never collects
            thrC[i] = sc;
            thrE[i] = thr_e(sc);
            fill[i] = 0;
        }
        __syncthreads();
    }

    int thr[2], gm[2] = {INT32_MIN, INT32_MIN};
    thr[0] = SEED ? INT32_MAX : thrE[wq * 64 + col];
    thr[1] = SEED ? INT32_MAX : thrE[wq * 64 + 32 + col];

    const int nt = (o.tiles > s) ? (o.tiles - s + S - 1) / S : 0;   // tiles of this split
    const int kst = o.kst, T = nt * kst;

    // ---- stage loader ---------------------------------------------------------------------------
    // A copy instruction brings 128 bytes of 8 rows; chunk c (16 bytes) of row r of a stage sits in slot
    // c ^ ((r >> 1) & 7) of the row, so that the 16 lanes that read one chunk column of 16 consecutive
    // rows touch all 64 banks.  The rows of odd instructions have bit 2 of r >> 1 set.
    const unsigned ring_lds = lds_offset(ring), aux_lds = lds_offset(aux);
    const unsigned off_even = (unsigned)((lane >> 3) * a.d_pad + ((lane & 7) ^ (lane >> 4)) * 16);
    const unsigned off_odd = (unsigned)((lane >> 3) * a.d_pad + ((lane & 7) ^ (lane >> 4) ^ 4) * 16);
    const unsigned off_wave = (wave & 1) ? off_odd : off_even;
    const int8_t *qsrc = a.qcodes + (q_tile + 8 * BPW * wave) * a.d_pad;
    int it = 0, ik = 0, islot = 0;     // the next stage to issue: tile (of this split), stage of the tile, ring slot
    auto first_row = [&](int t) {      // of the split's t-th tile
        const int64_t r = ((int64_t)s + (int64_t)S * t) * o.tile_stride;
        return SEED ? r + sample_shift((unsigned)(s + S * t), o.done ? 0 : o.tile_stride - RUN) : r;
    };
    int64_t irow = first_row(0);
    auto issue = [&]() {
        if (L2 && ik == 0) {           // a tile's first stage brings its accumulator seeds and parity words
            const unsigned dst = aux_lds + (it & 1) * AUX * 4;
            if (wave < 4) async_copy4(a.cinit + irow + (int64_t)(wave * 4 + (lane >> 4)) * o.run_gap + (lane & 15), dst + wave * 256);
            else if ((!SEED || o.done) && wave == 4 && lane < 8) async_copy4(a.parity + irow / 32 + lane, dst + TILE_ROWS * 4);
        }
        const unsigned dst = ring_lds + islot * STAGE;
        const int8_t *src = a.codes + (irow + (int64_t)(wave * APW / 2) * o.run_gap) * a.d_pad + ik * KB;
#pragma unroll
        for (int e = 0; e < APW; ++e)
            async_copy16_at(src + ((int64_t)(e / 2) * o.run_gap + (e & 1) * 8) * a.d_pad, (e & 1) ? off_odd : off_even,
                            dst + (wave * APW + e) * 1024);
#pragma unroll
        for (int e = 0; e < BPW; ++e)   // (one copy per wave: the parity of its rows is the wave's)
            async_copy16_at(qsrc + (int64_t)(8 * e) * a.d_pad + ik * KB,
                            BPW == 1 ? off_wave : ((e & 1) ? off_odd : off_even),
                            dst + A_BYTES + (wave * BPW + e) * 1024);
        islot = islot + 1 == NST ? 0 : islot + 1;
        if (++ik == kst) { ik = 0; irow = first_row(++it); }
    };

    // ---- fragments ------------------------------------------------------------------------------
    const int sw = (half ^ ((col >> 1) & 7)) * 16;   // k-step ks reads chunk 2 ks + half: exclusive-or with 32 ks
    const int a_off = (wr * RB * 32 + col) * KB + sw, b_off = A_BYTES + (wq * 64 + col) * KB + sw;
    v4i A[2][RB], B[2][2];                           // fragments of two consecutive k-steps
#define LPQS_LOAD(SLOT, KSTEP, F)                                                                       \
    do {                                                                                                \
        const unsigned char *sb_ = ring + (SLOT) * STAGE;                                               \
        const unsigned char *pa_ = sb_ + (a_off ^ ((KSTEP) * 32)), *pb_ = sb_ + (b_off ^ ((KSTEP) * 32)); \
        _Pragma("unroll") for (int j = 0; j < 2; ++j) B[F][j] = *reinterpret_cast<const v4i *>(pb_ + j * 32 * KB); \
        _Pragma("unroll") for (int i = 0; i < RB; ++i) A[F][i] = *reinterpret_cast<const v4i *>(pa_ + i * 32 * KB); \
    } while (0)
    v16i acc[RB][2];
#define LPQS_MFMA(F, I0, I1)                                                                            \
    _Pragma("unroll") for (int i = (I0); i < (I1); ++i)                                                 \
        _Pragma("unroll") for (int j = 0; j < 2; ++j)                                                   \
            acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A[F][i], B[F][j], acc[i][j], 0, 0, 0)
    // accumulators of a new tile start from its items' seeds
    auto start_tile = [&](int tile) {
        const int *cb = aux + (tile & 1) * AUX + wr * RB * 32;
#pragma unroll
        for (int i = 0; i < RB; ++i) {
            if (L2) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const v4i v = *reinterpret_cast<const v4i *>(cb + i * 32 + 8 * g + 4 * half);
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[i][0][4 * g + e] = acc[i][1][4 * g + e] = v[e];
                }
            } else {
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[i][0][e] = acc[i][1][e] = 0;
            }
            __builtin_amdgcn_sched_barrier(0);   // block by block: no reads hoisted into registers that are not there
        }
    };

    const int G = S * o.SEG * 2 * WR;
    auto flush_segment = [&](int seg) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            o.gmax[(size_t)(q_first + j * 32 + col) * G + (((size_t)s * o.SEG + seg) * WR + wr) * 2 + half] = gm[j];
            gm[j] = INT32_MIN;
        }
    };
    if (SEED && o.done) {
        if (blockIdx.x == 0)
            for (int i = tid; i < a.nq; i += SW * 64) o.done[i] = 0;
    } else if (SEED) {   // segments this split never reaches keep the neutral value
        for (int g = 0; g < o.SEG; ++g) flush_segment(g);
    }

    cand_t *cbase = SEED ? nullptr : o.cbuf + ((size_t)q_tile * S + s) * o.Cs;
    const size_t qstride = (size_t)S * o.Cs;

    // Empties this wave's queue of accumulator dumps: lanes cover (dump, accumulator) pairs, exact
    // candidates that beat their query's threshold go to the query's region.
    auto drain = [&](int dumps) {
        wave_lds_sync();
        for (int base = 0; base < dumps * 16; base += 64) {   // wave-uniform
            const int at = base + lane;
            if (at < dumps * 16) {
                const int e = dval[at];
                const v4i m4 = dmeta[at >> 4];
                const int ql = m4[2] & 255, r = at & 15;
                if (e >= thrE[ql]) {
                    const int off = 8 * (r >> 2) + 4 * (m4[2] >> 8) + (r & 3);
                    const int64_t row = (int64_t)(unsigned)m4[0] + off;
                    const cand_t c = make_cand(-(2 * e + (int)(((unsigned)m4[1] >> off) & 1u)), (uint32_t)row);
                    if (row < row_end && c < thrC[ql]) {
                        const int pos = atomicAdd(&fill[ql], 1);
                        if (pos < o.Cs) cbase[(size_t)ql * qstride + pos] = c;
                    }
                }
            }
        }
        wave_lds_sync();
    };

    // Only async copies (and stores, which make the counted waits more conservative) are outstanding
    // on the vector-memory counter from here on.
    __builtin_amdgcn_s_waitcnt(0x0F70);
    const int primed = T < NST ? T : NST;
    for (int st = 0; st < primed; ++st) issue();
    if (T > 0) {
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
        __syncthreads();
        LPQS_LOAD(0, 0, 0);
        start_tile(0);
    }
    int slot = 0, t = 0, seg = 0, part = 0;
    int64_t row0 = (int64_t)s * o.tile_stride;
#pragma clang loop unroll(disable)
    for (int tile = 0; tile < nt; ++tile, row0 += (int64_t)S * o.tile_stride) {
#pragma clang loop unroll(disable)
        for (int k = 0; k < kst; ++k, ++t) {
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                // the fragments of this k-step were asked for a k-step ago and are there; waiting for them
                // before the next ones are asked for keeps the compiler from waiting for those as well
                __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
                if (ks + 1 < KS) {
                    LPQS_LOAD(slot, ks + 1, (ks + 1) & 1);
                    LPQS_MFMA(ks & 1, 0, RB);
                    // the reads first, then the matrix instructions (left alone the compiler mixes them)
                    __builtin_amdgcn_sched_group_barrier(0x100, 2 + RB, 0);
                    __builtin_amdgcn_sched_group_barrier(0x008, 2 * RB, 0);
                    __builtin_amdgcn_sched_barrier(0);
                } else {
                    // my reads of stage t are complete.  Stages 0 .. t + NST - 1 have been issued and stage
                    // t + 1 must have landed: all but the copies of the NST - 2 newest stages; at the end of
                    // the split simply all of them
                    if (NST == 2 || t + NST > T) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
                    else __builtin_amdgcn_s_waitcnt(vmcnt_imm((NST - 2) * CPW));
                    asm volatile("" ::: "memory");
                    __syncthreads();
                    slot = slot + 1 == NST ? 0 : slot + 1;
                    LPQS_LOAD(slot, 0, 0);   // (after the last stage: whatever the ring holds, unused)
                    // the first matrix instructions go ahead of the copies' address arithmetic and issue
                    LPQS_MFMA(ks & 1, 0, 1);
                    __builtin_amdgcn_sched_barrier(0);
                    if (t + NST < T) issue();                            // refills the slot of stage t
                    __builtin_amdgcn_sched_barrier(0);
                    LPQS_MFMA(ks & 1, 1, RB);
                }
            }
        }
        __builtin_amdgcn_sched_barrier(0);   // nothing of the contraction drifts down into the epilogue
        const int *pw = aux + (tile & 1) * AUX + TILE_ROWS + wr * RB;
        int dumps = 0;
#pragma unroll
        for (int i = 0; i < RB; ++i) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                v16i v = acc[i][j];
                if (SEED && L2 && o.done) {   // 2 E, and 1 for an odd norm: what the key is the negative of
                    const unsigned odd = (unsigned)pw[i] >> (4 * half);
#pragma unroll
                    for (int r = 0; r < 16; ++r) v[r] = 2 * v[r] + (int)((odd >> (8 * (r >> 2) + (r & 3))) & 1u);
                }
                int m = max(max(v[0], v[1]), v[2]);
                m = max(max(m, v[3]), v[4]);
                m = max(max(m, v[5]), v[6]);
                m = max(max(m, v[7]), v[8]);
                m = max(max(m, v[9]), v[10]);
                m = max(max(m, v[11]), v[12]);
                m = max(max(m, v[13]), v[14]);
                m = max(m, v[15]);
                if (SEED) {
                    gm[j] = max(gm[j], m);
                } else {
                    unsigned long long mask = __ballot(m >= thr[j]);
                    while (__builtin_expect(mask != 0, 0)) {   // queue the 16 accumulators of the lanes that pass
                        int lane_ = lane;   // addresses are formed here, not carried through the loop in registers
                        asm volatile("" : "+v"(lane_));
                        const int at = dumps + __builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32),
                                                                         __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
                        const bool put = ((mask >> lane_) & 1) && at < DUMPS;
                        if (put) {
                            v4i *dst = reinterpret_cast<v4i *>(dval + at * 16);
#pragma unroll
                            for (int g = 0; g < 4; ++g) dst[g] = v4i{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
                            dmeta[at] = v4i{(int)(row0 + (wr * RB + i) * 32), L2 ? pw[i] : 0,
                                            (wq * 64 + j * 32 + (lane_ & 31)) | ((lane_ >> 5) << 8), 0};
                        }
                        const unsigned long long done = __ballot(put);
                        dumps += __popcll(done);
                        mask &= ~done;
                        if (mask) { drain(dumps); dumps = 0; }   // no room for the rest
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (!SEED && dumps) drain(dumps);
        start_tile(tile + 1);   // (after the last tile: seeds of no consequence)
        if (SEED) {             // tile i belongs to segment i SEG / nt: close it when the next tile is in another one
            part += o.SEG;
            if (part >= nt || tile + 1 == nt) flush_segment(seg);
            for (; part >= nt; part -= nt) ++seg;
        }
    }
#undef LPQS_LOAD
#undef LPQS_MFMA

    if (!SEED) {
        __syncthreads();   // every wave has appended its last candidates
        for (int i = tid; i < QT; i += SW * 64)
            if (q_tile + i < a.nq) o.ccnt[(size_t)(q_tile + i) * S + s] = fill[i];
    }
}

template <bool L2, bool SEED, int WQ>
hipError_t launch_wq(const SearchArgs &a, int64_t row_end, int S, StreamIo o, hipStream_t st)
{
    const int qtiles = (int)ceil_div(a.nq, 64 * WQ);
    const int64_t fit = QGROUP_BYTES / ((int64_t)64 * WQ * o.kst * KB);
    o.qgroup = (int)(fit < 1 ? 1 : (fit < qtiles ? fit : qtiles));
    auto kern = search_stream_kernel<L2, SEED, WQ>;
    static bool attr_set = false;  // per instantiation
    if (!attr_set) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        if (e != hipSuccess) return e;
        attr_set = true;
    }
    kern<<<(unsigned)(qtiles * S), SW * 64, stream_lds_bytes(WQ, SEED), st>>>(a, row_end, S, qtiles, o);
    return hipGetLastError();
}

template <bool SEED>
hipError_t launch_stream(const SearchArgs &a, int64_t row_end, int S, const StreamIo &o, hipStream_t st)
{
    if (a.nq <= 0 || row_end <= 0 || S < 1) return hipSuccess;
    // (a tile of fewer stages than the ring holds would let a tile's seeds overwrite those still in use)
    if (a.packed || a.d_pad % KB || o.kst < 3 || o.kst * KB > a.d_pad) return hipErrorInvalidValue;
    const bool l2 = a.metric == LPQ_METRIC_L2SQ;
    switch (mfma_stream_wq(a.nq)) {
    case 1: return l2 ? launch_wq<true, SEED, 1>(a, row_end, S, o, st) : launch_wq<false, SEED, 1>(a, row_end, S, o, st);
    case 2: return l2 ? launch_wq<true, SEED, 2>(a, row_end, S, o, st) : launch_wq<false, SEED, 2>(a, row_end, S, o, st);
    default: return l2 ? launch_wq<true, SEED, 4>(a, row_end, S, o, st) : launch_wq<false, SEED, 4>(a, row_end, S, o, st);
    }
}

}  // namespace

// Rows of 384 and 512 bytes stay with the long-row scan, whose waves hold 64 queries there (500K rows,
// 1000 queries: 0.236 and 0.291 ms against 0.247 and 0.298 here).  From 768 bytes on it held 32 and lost
// at every batch size (same corpus, L2: 768 bytes 0.458 -> 0.413 ms, 10 000 queries 4.08 -> 3.60, 16
// queries 0.141 -> 0.131; 300K x 1024, 10 000 queries: 3.22 -> 3.04; 300K x 1536, 1000 queries: 0.641 -> 0.498).
bool mfma_stream_rows(int d_pad) { return d_pad >= 768 && d_pad % KB == 0; }

// The narrowest tile that holds the batch: small batches are bound by the corpus bytes, and a wider
// tile would spend matrix time on queries that are not there.
int mfma_stream_wq(int64_t nq) { return nq <= 64 ? 1 : (nq <= 128 ? 2 : 4); }

int mfma_stream_row_waves(int64_t nq) { return SW / mfma_stream_wq(nq); }

hipError_t launch_stream_seed(const SearchArgs &a, int tiles, int64_t run_stride, int S, int SEG, int32_t *gmax,
                              hipStream_t st)
{
    // run i of tile g starts at row (i * tiles + g) * run_stride: every run lies inside the corpus
    if (!gmax || tiles < 1 || run_stride < RUN || ((int64_t)16 * tiles - 1) * run_stride + RUN > a.n) return hipErrorInvalidValue;
    StreamIo o = {};
    o.gmax = gmax; o.SEG = SEG;
    o.tiles = tiles; o.tile_stride = run_stride; o.run_gap = (int64_t)tiles * run_stride;
    o.kst = (int)ceil_div(a.d, KB);
    return launch_stream<true>(a, a.n, S, o, st);
}

hipError_t launch_maxima_stream(const SearchArgs &a, const MaximaShape &m, int32_t *gmax, int32_t *done, hipStream_t st)
{
    if (a.nq < 1 || !gmax || !done || m.S < 1 || m.SEG < 1 || m.SEG > m.stages / m.S || m.stage_rows != TILE_ROWS ||
        (int64_t)m.stages * TILE_ROWS > a.n || m.G != mfma_seed_groups(m.S, m.SEG, SW))
        return hipErrorInvalidValue;
    StreamIo o = {};
    o.gmax = gmax; o.SEG = m.SEG; o.done = done;
    o.tiles = m.stages; o.tile_stride = TILE_ROWS; o.run_gap = RUN;
    o.kst = (int)ceil_div(a.d, KB);
    if (a.packed || a.d_pad % KB || o.kst < 3) return hipErrorInvalidValue;   // (as launch_stream)
    return a.metric == LPQ_METRIC_L2SQ ? launch_wq<true, true, 1>(a, (int64_t)m.stages * TILE_ROWS, m.S, o, st)
                                       : launch_wq<false, true, 1>(a, (int64_t)m.stages * TILE_ROWS, m.S, o, st);
}

hipError_t launch_stream_collect(const SearchArgs &a, int S, const cand_t *seeds, cand_t *cbuf, int32_t *ccnt, int Cs,
                                 hipStream_t st)
{
    if (!seeds || !cbuf || !ccnt || Cs < 1) return hipErrorInvalidValue;
    StreamIo o = {};
    o.seeds = seeds; o.cbuf = cbuf; o.ccnt = ccnt; o.Cs = Cs;
    o.tiles = (int)ceil_div(a.n, TILE_ROWS); o.tile_stride = TILE_ROWS; o.run_gap = RUN;
    o.kst = (int)ceil_div(a.d, KB);
    return launch_stream<false>(a, a.n, S, o, st);
}

}  // namespace lpq
