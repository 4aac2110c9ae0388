// Workgroup-level selection helpers shared by the scan kernels and the merge kernel.
#pragma once

#include "lpq_internal.h"

namespace lpq {

// Ascending bitonic sort of buf[0..cap) (cap a power of two) by all threads of the block.
__device__ inline void block_bitonic_sort(cand_t *buf, int cap)
{
    for (int size = 2; size <= cap; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int i = threadIdx.x; i < (cap >> 1); i += blockDim.x) {
                const int lo = 2 * i - (i & (stride - 1));
                const int hi = lo + stride;
                const bool up = (lo & size) == 0;
                const cand_t a = buf[lo], b = buf[hi];
                if ((a > b) == up) { buf[lo] = b; buf[hi] = a; }
            }
            __syncthreads();
        }
    }
}

// A buffer that all threads of a block append to, in steps with one barrier each.  Behind the barrier every thread has to
// come to the same answer whether the buffer is compacted, while faster waves may already append in the next step: even and
// odd steps have a counter each, which is read before the next barrier and written again behind it only.  Neither is ever
// cleared; `before` is what the step's counter stood at, `after` the other one.
struct AppendSteps {
    int held = 0, turn = 0, before = 0, after = 0;
    __device__ __forceinline__ void step_done(int count)      // the step's counter, read behind its barrier
    {
        held += count - before;
        before = after;
        after = count;
        turn ^= 1;
    }
};

// Compacts such a buffer if the next step could overflow it: sort, keep the best k, tighten the threshold to the k-th best.
// Must be reached by all threads of the block; `held` candidates are in it, the same number in every thread, and `need` is
// the largest number of appends one step can make.
__device__ inline void block_compact_if_full(cand_t *buf, int cap, int k, int need, int &held, cand_t *s_thr)
{
    if (held + need > cap) {
        block_bitonic_sort(buf, cap);
        held = held < k ? held : k;
        for (int i = held + threadIdx.x; i < cap; i += blockDim.x) buf[i] = CAND_NONE;
        if (threadIdx.x == 0 && held == k && buf[k - 1] < *s_thr) *s_thr = buf[k - 1];
        __syncthreads();
    }
}

// Final id and distance of candidate c of query q, written at position `at`.
__device__ __forceinline__ void emit_result(cand_t c, int64_t at, int64_t q, int32_t *__restrict__ ids,
                                            int32_t *__restrict__ dists, const int32_t *__restrict__ qnorms, int metric)
{
    const int32_t key = cand_key(c);
    ids[at] = (c == CAND_NONE) ? -1 : (int32_t)cand_id(c);
    int32_t v;
    if (metric == MODE_I8_L2) v = key + qnorms[q];
    else if (metric == MODE_I8_IP) v = -(key / 2);
    else if (metric == MODE_I8_IP_ADJ) v = -(key / 2) + qnorms[q];
    else {
        const float f = sortable_to_float(key);
        v = __float_as_int(metric == MODE_F32_L2 ? f : -f);
    }
    dists[at] = v;
}

}  // namespace lpq
