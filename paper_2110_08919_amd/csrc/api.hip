// C ABI of liblpq.so: argument checks, handle lifetimes, workspace planning and the order
// in which the kernels of a search are enqueued.  No kernel lives here.
#include <atomic>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <cmath>
#include <vector>

#include "lpq_internal.h"

using namespace lpq;

// ------------------------------------------------------------------------ errors ----
static thread_local char g_err[512] = "";

static int fail(int code, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return code;
}

#define HIP_TRY(expr)                                                                        \
    do {                                                                                     \
        hipError_t e_ = (expr);                                                              \
        if (e_ != hipSuccess)                                                                \
            return fail(e_ == hipErrorOutOfMemory ? LPQ_ENOMEM : LPQ_EDEVICE, "%s: %s", #expr, \
                        hipGetErrorString(e_));                                              \
    } while (0)

extern "C" const char *lpq_last_error(void) { return g_err; }

// ------------------------------------------------------------------------ tuning ----
// Process-wide and read by every planning call: atomics, so that a thread changing a knob while
// others search is not a data race (a search still sees each knob at some moment of its planning;
// results never depend on them).
static std::atomic<int64_t> g_tune[LPQ_TUNE_COUNT_];
static inline int64_t tune(int key) { return g_tune[key].load(std::memory_order_relaxed); }

extern "C" int lpq_set_tuning(int key, int64_t value)
{
    if (key < 0 || key >= LPQ_TUNE_COUNT_) return fail(LPQ_EINVAL, "unknown tuning key %d", key);
#ifndef LPQ_ABLATION
    if (key == LPQ_TUNE_DRY_RUN && value != 0)
        return fail(LPQ_EINVAL, "LPQ_TUNE_DRY_RUN exists only in builds compiled with -DLPQ_ABLATION");
#endif
    g_tune[key].store(value, std::memory_order_relaxed);
    return LPQ_OK;
}

// --------------------------------------------------------------------- profiling ----
namespace {
// Event pairs are created when profiling is switched on, not inside the searches they time: a
// span only takes the next free pair (spans beyond the pool go untimed and are counted as dropped).
constexpr size_t PROFILE_POOL = 4096;
struct Profile {
    std::mutex mu;
    bool on = false;
    struct Span { hipEvent_t a, b; int kind; };
    std::vector<Span> pool;    // pairs created by lpq_profile_enable(1)
    size_t used = 0;           // pairs handed out so far
    int64_t dropped = 0;
    void clear()
    {
        for (auto &s : pool) { (void)hipEventDestroy(s.a); (void)hipEventDestroy(s.b); }
        pool.clear();
        used = 0;
        dropped = 0;
    }
};
Profile g_prof;

struct KernelSpan {  // brackets one kernel launch with two events while profiling is on
    hipEvent_t a = nullptr, b = nullptr;
    hipStream_t st;
    explicit KernelSpan(hipStream_t s, int kind_ = LPQ_PROFILE_SCAN) : st(s)
    {
        std::lock_guard<std::mutex> l(g_prof.mu);
        if (!g_prof.on) return;
        if (g_prof.used >= g_prof.pool.size()) { ++g_prof.dropped; return; }
        Profile::Span &sp = g_prof.pool[g_prof.used++];
        sp.kind = kind_;
        a = sp.a; b = sp.b;
        (void)hipEventRecord(a, st);
    }
    ~KernelSpan()
    {
        if (a) (void)hipEventRecord(b, st);
    }
};
}  // namespace

extern "C" int lpq_profile_enable(int on)
{
    std::lock_guard<std::mutex> l(g_prof.mu);
    g_prof.clear();
    g_prof.on = false;
    if (on) {
        g_prof.pool.reserve(PROFILE_POOL);
        for (size_t i = 0; i < PROFILE_POOL; ++i) {
            Profile::Span sp = {nullptr, nullptr, 0};
            hipError_t e = hipEventCreate(&sp.a);
            if (e == hipSuccess) e = hipEventCreate(&sp.b);
            if (e != hipSuccess) {
                if (sp.a) (void)hipEventDestroy(sp.a);
                g_prof.clear();
                return fail(LPQ_EDEVICE, "hipEventCreate: %s", hipGetErrorString(e));
            }
            g_prof.pool.push_back(sp);
        }
        g_prof.on = true;
    }
    return LPQ_OK;
}

static int profile_sum(int kind, int64_t *launches, double *total_ms)
{
    if (!launches || !total_ms) return fail(LPQ_EINVAL, "null output");
    std::lock_guard<std::mutex> l(g_prof.mu);
    double tot = 0.0;
    int64_t cnt = 0;
    for (size_t i = 0; i < g_prof.used; ++i) {
        const Profile::Span &s = g_prof.pool[i];
        if (kind >= 0 && s.kind != kind) continue;
        HIP_TRY(hipEventSynchronize(s.b));
        float ms = 0.f;
        HIP_TRY(hipEventElapsedTime(&ms, s.a, s.b));
        tot += ms;
        ++cnt;
    }
    *launches = cnt;
    *total_ms = tot;
    return LPQ_OK;
}

extern "C" int lpq_profile_read(int64_t *launches, double *total_ms) { return profile_sum(-1, launches, total_ms); }

extern "C" int lpq_profile_read_kind(int kind, int64_t *launches, double *total_ms)
{
    if (kind != LPQ_PROFILE_SCAN && kind != LPQ_PROFILE_SEED) return fail(LPQ_EINVAL, "unknown kernel kind %d", kind);
    return profile_sum(kind, launches, total_ms);
}

// ------------------------------------------------------------------------ probes ----
extern "C" int lpq_probe_mfma_i8(const void *operands_dev, size_t operand_bytes, int iters, double *tops, void *stream)
{
    if (!tops) return fail(LPQ_EINVAL, "null output");
    if (iters < 1 || iters > 10000000) return fail(LPQ_EINVAL, "iters = %d outside 1..10 000 000", iters);
    if (operands_dev && operand_bytes < 16) return fail(LPQ_EINVAL, "operand buffer smaller than 16 bytes");
    if (operands_dev && (uintptr_t)operands_dev % 16) return fail(LPQ_EINVAL, "operand buffer must be 16-byte aligned");
    *tops = 0.0;
    HIP_TRY(probe_mfma(operands_dev, operand_bytes, iters, tops, (hipStream_t)stream));
    return LPQ_OK;
}

extern "C" int lpq_probe_scan_core(const void *operands_dev, size_t operand_bytes, int stages, double *tops, void *stream)
{
    if (!tops) return fail(LPQ_EINVAL, "null output");
    if (stages < 1 || stages > 10000000) return fail(LPQ_EINVAL, "stages = %d outside 1..10 000 000", stages);
    if (operands_dev && operand_bytes < 16) return fail(LPQ_EINVAL, "operand buffer smaller than 16 bytes");
    if (operands_dev && (uintptr_t)operands_dev % 16) return fail(LPQ_EINVAL, "operand buffer must be 16-byte aligned");
    *tops = 0.0;
    HIP_TRY(probe_scan_core(operands_dev, operand_bytes, stages, tops, (hipStream_t)stream));
    return LPQ_OK;
}

extern "C" int lpq_probe_stream(const void *src_dev, size_t bytes, int mode, int reps, double *gbps, void *stream)
{
    if (!src_dev || !gbps) return fail(LPQ_EINVAL, "null argument");
    if (mode != 0 && mode != 1) return fail(LPQ_EINVAL, "unknown mode %d", mode);
    if (bytes < 4096 || reps < 1 || reps > 10000) return fail(LPQ_EINVAL, "bytes < 4096 or reps outside 1..10 000");
    if ((uintptr_t)src_dev % 16) return fail(LPQ_EINVAL, "buffer must be 16-byte aligned");
    *gbps = 0.0;
    HIP_TRY(probe_stream(src_dev, bytes / 4096 * 4096, mode, reps, gbps, (hipStream_t)stream));
    return LPQ_OK;
}

// --------------------------------------------------------------------- quantizer ----
struct lpq_quantizer {
    int d = 0, bits = 0;
    bool ready = false;
    float *params = nullptr;   // device [4][d]: k, S_b, S_e, m
    float *staging = nullptr;  // device [4][d]: calibration result before it is committed
    int *flag = nullptr;       // device: non-finite value seen
    void *windows = nullptr;   // of a quantile calibration
    void *block = nullptr;     // the allocation all of these lie in
    void *scratch = nullptr;   // calibration partials, from the first calibration that is not by windows on
};

static QuantParams view(const float *params, int d, int bits)
{
    QuantParams qp;
    qp.k = params; qp.sb = params + d; qp.se = params + 2 * d; qp.m = params + 3 * d;
    qp.d = d; qp.bits = bits;
    return qp;
}

extern "C" void lpq_quantizer_destroy(lpq_quantizer *q)
{
    if (!q) return;
    (void)hipFree(q->block);
    (void)hipFree(q->scratch);
    delete q;
}

extern "C" int lpq_quantizer_create(lpq_quantizer **out, int d, int bits)
{
    if (!out) return fail(LPQ_EINVAL, "out is null");
    if (d < 1) return fail(LPQ_EINVAL, "d = %d < 1", d);
    if (bits < 1 || bits > 8) return fail(LPQ_EINVAL, "bits = %d outside 1..8", bits);
    if (d > MAX_D) return fail(LPQ_ERANGE, "d = %d > %d", d, (int)MAX_D);
    lpq_quantizer *q = new (std::nothrow) lpq_quantizer;
    if (!q) return fail(LPQ_ENOMEM, "host allocation failed");
    q->d = d; q->bits = bits;
    // One allocation: each and its release cost tens of microseconds, which a program that calibrates often pays
    // every time.
    const size_t set = ((size_t)4 * d * sizeof(float) + 255) & ~size_t(255);
    const hipError_t e = hipMalloc(&q->block, 256 + 2 * set + calib_windows_bytes(d));
    if (e != hipSuccess) {
        lpq_quantizer_destroy(q);
        return fail(e == hipErrorOutOfMemory ? LPQ_ENOMEM : LPQ_EDEVICE, "hipMalloc: %s", hipGetErrorString(e));
    }
    char *p = static_cast<char *>(q->block);
    q->flag = reinterpret_cast<int *>(p);
    q->params = reinterpret_cast<float *>(p + 256);
    q->staging = reinterpret_cast<float *>(p + 256 + set);
    q->windows = p + 256 + 2 * set;
    *out = q;
    return LPQ_OK;
}

extern "C" int lpq_quantizer_calibrate(lpq_quantizer *q, const float *x_dev, int64_t n, int64_t ld, int mode,
                                       int scope, float sigma_mult, void *stream)
{
    if (!q || !x_dev) return fail(LPQ_EINVAL, "null argument");
    if (n < 1) return fail(LPQ_EINVAL, "n = %lld < 1", (long long)n);
    if (ld < q->d) return fail(LPQ_EINVAL, "ld = %lld < d = %d", (long long)ld, q->d);
    if (mode < LPQ_CALIB_MINMAX || mode > LPQ_CALIB_QUANTILE) return fail(LPQ_EINVAL, "unknown calibration mode %d", mode);
    if (mode == LPQ_CALIB_QUANTILE && !(sigma_mult >= 0.0f && sigma_mult < 0.5f)) return fail(LPQ_EINVAL, "clip fraction must be in [0, 0.5)");
    if (scope != LPQ_SCOPE_PER_FEATURE && scope != LPQ_SCOPE_GLOBAL && scope != LPQ_SCOPE_SHARED_WIDTH) return fail(LPQ_EINVAL, "unknown scope %d", scope);
    if (mode == LPQ_CALIB_GAUSS && !(sigma_mult > 0.0f)) return fail(LPQ_EINVAL, "sigma_mult must be > 0");
    hipStream_t st = (hipStream_t)stream;
    // A quantile's windows come with lists of 16 MB at most.  They are held during the call only, a quantizer lives as
    // long as its index does; allocated, with the partials, while the sample is taken (1M x 128, create to
    // destroy, 255 us with both held for good, 240 so; a second calibration 218 and 237).  Without the room for them
    // the general path does.
    char *temp = nullptr;
    const size_t lists_bytes = calib_lists_bytes(n, q->d, mode, scope, (double)sigma_mult);
    const size_t scratch_bytes = (calib_scratch_bytes(q->d) + 255) & ~size_t(255);
    if (lists_bytes) {
        HIP_TRY(launch_calib_windows(x_dev, n, ld, q->d, (double)sigma_mult, q->windows, st));
        if (hipMalloc(&temp, scratch_bytes + lists_bytes) != hipSuccess) {
            temp = nullptr;
            (void)hipGetLastError();
        }
    }
    if (!temp && !q->scratch) {
        const hipError_t e = hipMalloc(&q->scratch, scratch_bytes);
        if (e != hipSuccess) {
            q->scratch = nullptr;
            return fail(e == hipErrorOutOfMemory ? LPQ_ENOMEM : LPQ_EDEVICE, "hipMalloc: %s", hipGetErrorString(e));
        }
    }
    int bad = 0;
    auto attempt = [&](uint32_t *lists) -> hipError_t {
        hipError_t e = launch_calibrate(x_dev, n, ld, q->d, q->bits, mode, scope, (double)sigma_mult, temp ? temp : q->scratch,
                                        q->staging, q->params, q->flag, st, q->windows, lists);
        if (e == hipSuccess) e = hipMemcpyAsync(&bad, q->flag, sizeof(int), hipMemcpyDeviceToHost, st);
        const hipError_t w = hipStreamSynchronize(st);   // in any case: what was launched may still use the memory
        return e != hipSuccess ? e : w;
    };
    hipError_t e = attempt(temp ? reinterpret_cast<uint32_t *>(temp + scratch_bytes) : nullptr);
    if (e == hipSuccess && temp && bad == 2) e = attempt(nullptr);   // a window missed its quantile
    if (temp) (void)hipFree(temp);
    HIP_TRY(e);
    if (bad & 1) return fail(LPQ_ENONFINITE, "calibration data holds a NaN or an infinity");
    q->ready = true;
    return LPQ_OK;
}

extern "C" int lpq_quantizer_set_params(lpq_quantizer *q, const float *k, const float *s_b, const float *s_e)
{
    if (!q || !k || !s_b || !s_e) return fail(LPQ_EINVAL, "null argument");
    const size_t bytes = sizeof(float) * q->d;
    HIP_TRY(hipMemcpy(q->params, k, bytes, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(q->params + q->d, s_b, bytes, hipMemcpyHostToDevice));
    HIP_TRY(hipMemcpy(q->params + 2 * q->d, s_e, bytes, hipMemcpyHostToDevice));
    HIP_TRY(launch_derive_m(q->params, q->d, q->bits, nullptr));
    HIP_TRY(hipDeviceSynchronize());
    q->ready = true;
    return LPQ_OK;
}

extern "C" int lpq_quantizer_get_params(const lpq_quantizer *q, float *k, float *s_b, float *s_e, float *m)
{
    if (!q || !k || !s_b || !s_e) return fail(LPQ_EINVAL, "null argument");
    if (!q->ready) return fail(LPQ_ESTATE, "quantizer has no constants yet");
    const size_t bytes = sizeof(float) * q->d;
    HIP_TRY(hipDeviceSynchronize());
    float *all = static_cast<float *>(std::malloc(4 * bytes));   // the four arrays in one copy
    if (!all) return fail(LPQ_ENOMEM, "host allocation failed");
    const hipError_t e = hipMemcpy(all, q->params, 4 * bytes, hipMemcpyDeviceToHost);
    if (e == hipSuccess) {
        std::memcpy(k, all, bytes);
        std::memcpy(s_b, all + q->d, bytes);
        std::memcpy(s_e, all + 2 * (size_t)q->d, bytes);
        if (m) std::memcpy(m, all + 3 * (size_t)q->d, bytes);
    }
    std::free(all);
    HIP_TRY(e);
    return LPQ_OK;
}

extern "C" int lpq_encode(const lpq_quantizer *q, const float *x_dev, int64_t n, int64_t ld, int8_t *codes_dev,
                          int64_t ld_codes, int32_t *norms_dev, void *stream)
{
    if (!q || !x_dev || !codes_dev) return fail(LPQ_EINVAL, "null argument");
    if (n < 0) return fail(LPQ_EINVAL, "n < 0");
    if (ld < q->d || ld_codes < q->d) return fail(LPQ_EINVAL, "row stride smaller than d = %d", q->d);
    if (!q->ready) return fail(LPQ_ESTATE, "encode before calibrate/set_params");
    HIP_TRY(launch_encode(view(q->params, q->d, q->bits), x_dev, n, ld, codes_dev, ld_codes, 0, norms_dev,
                          (hipStream_t)stream));
    return LPQ_OK;
}

// ------------------------------------------------------------------------- index ----
struct lpq_index {
    int d = 0, d_pad = 0, bits = 0;
    bool packed = false;         // two 4-bit codes per byte: rows of d_pad / 2 bytes
    int64_t capacity = 0, cap_rows = 0, size = 0;
    float *params = nullptr;     // device copy of the quantizer constants
    int8_t *codes = nullptr;     // [cap_rows][d_pad], zero padded
    int32_t *norms = nullptr;    // [cap_rows]
    int32_t *cinit = nullptr;    // [cap_rows]   accumulator seeds of the matrix-core kernel
    uint32_t *parity = nullptr;  // [cap_rows/32]
    int8_t *stage = nullptr;     // packed only: [PACK_STAGE_ROWS][d_pad] int8 codes on their way to nibbles
};
constexpr int64_t PACK_STAGE_ROWS = 65536;

extern "C" void lpq_index_destroy(lpq_index *idx)
{
    if (!idx) return;
    (void)hipFree(idx->params);
    (void)hipFree(idx->codes);
    (void)hipFree(idx->norms);
    (void)hipFree(idx->cinit);
    (void)hipFree(idx->stage);
    (void)hipFree(idx->parity);
    delete idx;
}

// Row length an index stores d features in: a length the matrix-core scans have where one exists.
static int padded_row_length(int d)
{
    // up to 1536 features: the row lengths of the scans that keep queries in registers; beyond: whole
    // stages of the scan that streams them
    return d <= 64 ? 64 : d <= 96 ? 96 : d <= 128 ? 128 : d <= 192 ? 192 : d <= 256 ? 256
           : d <= 384 ? 384 : d <= 512 ? 512 : d <= 768 ? 768 : d <= 1024 ? 1024 : d <= 1536 ? 1536 : (int)round_up(d, 128);
}

static int index_create_impl(lpq_index **out, const lpq_quantizer *q, int64_t capacity, bool packed)
{
    if (!out || !q) return fail(LPQ_EINVAL, "null argument");
    if (!q->ready) return fail(LPQ_ESTATE, "quantizer has no constants yet");
    if (packed && q->bits > 4) return fail(LPQ_EINVAL, "packed storage needs a quantizer of at most 4 bits (has %d)", q->bits);
    if (packed && q->d > MAX_D_PACKED)
        return fail(LPQ_ERANGE, "packed storage is searched for at most %d features (has %d)", (int)MAX_D_PACKED, q->d);
    if (capacity < 1) return fail(LPQ_EINVAL, "capacity < 1");
    if (capacity >= (int64_t(1) << 31) - 1024) return fail(LPQ_ERANGE, "capacity must stay below 2^31 - 1024");
    lpq_index *idx = new (std::nothrow) lpq_index;
    if (!idx) return fail(LPQ_ENOMEM, "host allocation failed");
    idx->d = q->d; idx->bits = q->bits;
    idx->packed = packed;
    // Rows are zero padded to a length the matrix-core scans have (64, 96, 128, 192 or 256 bytes):
    // up to 256 features never fall back to the generic kernel, which is ~100x slower on large
    // batches; the price is up to 2x the row bytes for d <= 32 and 20 % for 129..160.
    idx->d_pad = padded_row_length(q->d);
    idx->capacity = capacity;
    idx->cap_rows = round_up(capacity, 256) + 256;  // whole tiles may be read past the last item
    const size_t code_bytes = (size_t)idx->cap_rows * idx->d_pad / (packed ? 2 : 1);
    hipError_t e = hipMalloc(&idx->params, sizeof(float) * 4 * idx->d);
    if (e == hipSuccess) e = hipMalloc(&idx->codes, code_bytes);
    if (e == hipSuccess && packed) e = hipMalloc(&idx->stage, (size_t)PACK_STAGE_ROWS * idx->d_pad);
    if (e == hipSuccess) e = hipMalloc(&idx->norms, sizeof(int32_t) * idx->cap_rows);
    if (e == hipSuccess) e = hipMalloc(&idx->cinit, sizeof(int32_t) * idx->cap_rows);
    if (e == hipSuccess) e = hipMalloc(&idx->parity, sizeof(uint32_t) * (idx->cap_rows / 32));
    if (e == hipSuccess) e = hipMemcpy(idx->params, q->params, sizeof(float) * 4 * idx->d, hipMemcpyDeviceToDevice);
    if (e == hipSuccess) e = hipMemset(idx->codes, packed ? 0x88 : 0, code_bytes);   // code 0 everywhere
    if (e == hipSuccess) e = hipMemset(idx->norms, 0, sizeof(int32_t) * idx->cap_rows);
    if (e == hipSuccess) e = hipMemset(idx->parity, 0, sizeof(uint32_t) * (idx->cap_rows / 32));
    if (e == hipSuccess) e = hipMemsetD32((hipDeviceptr_t)idx->cinit, CINIT_PAD, (size_t)idx->cap_rows);
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) {
        lpq_index_destroy(idx);
        return fail(e == hipErrorOutOfMemory ? LPQ_ENOMEM : LPQ_EDEVICE, "index allocation: %s", hipGetErrorString(e));
    }
    *out = idx;
    return LPQ_OK;
}

extern "C" int lpq_index_create(lpq_index **out, const lpq_quantizer *q, int64_t capacity)
{
    return index_create_impl(out, q, capacity, false);
}

extern "C" int lpq_index_create_packed(lpq_index **out, const lpq_quantizer *q, int64_t capacity)
{
    return index_create_impl(out, q, capacity, true);
}

// Packed index: rows [row0, row0 + n) from int8 codes (device), through the nibble packer.
static int index_pack_rows(lpq_index *idx, int64_t row0, const int8_t *codes, int64_t n, int64_t ld, hipStream_t st)
{
    HIP_TRY(launch_pack4(codes, n, ld, idx->d, reinterpret_cast<uint8_t *>(idx->codes) + (size_t)row0 * (idx->d_pad / 2),
                         idx->d_pad, idx->norms + row0, st));
    return LPQ_OK;
}

static int index_after_add(lpq_index *idx, int64_t n, hipStream_t st)
{
    const int64_t row0 = idx->size;
    idx->size += n;
    // Seeds for every row of every tile that can be touched: rows beyond size get the padding seed.
    HIP_TRY(launch_item_aux(idx->norms, row0, idx->size, idx->cinit, idx->parity, st));
    return LPQ_OK;
}

extern "C" int lpq_index_add_f32(lpq_index *idx, const float *x_dev, int64_t n, int64_t ld, void *stream)
{
    if (!idx || !x_dev) return fail(LPQ_EINVAL, "null argument");
    if (n < 0) return fail(LPQ_EINVAL, "n < 0");
    if (ld < idx->d) return fail(LPQ_EINVAL, "ld < d");
    if (idx->size + n > idx->capacity) return fail(LPQ_ERANGE, "index capacity %lld exceeded", (long long)idx->capacity);
    if (n == 0) return LPQ_OK;
    hipStream_t st = (hipStream_t)stream;
    if (idx->packed) {   // encode a chunk into the staging rows, pack it, next chunk
        for (int64_t r = 0; r < n; r += PACK_STAGE_ROWS) {
            const int64_t m = n - r < PACK_STAGE_ROWS ? n - r : PACK_STAGE_ROWS;
            HIP_TRY(launch_encode(view(idx->params, idx->d, idx->bits), x_dev + r * ld, m, ld, idx->stage, idx->d_pad,
                                  idx->d_pad, nullptr, st));
            const int rc = index_pack_rows(idx, idx->size + r, idx->stage, m, idx->d_pad, st);
            if (rc) return rc;
        }
        return index_after_add(idx, n, st);
    }
    HIP_TRY(launch_encode(view(idx->params, idx->d, idx->bits), x_dev, n, ld,
                          idx->codes + (size_t)idx->size * idx->d_pad, idx->d_pad, idx->d_pad,
                          idx->norms + idx->size, st));
    return index_after_add(idx, n, st);
}

extern "C" int lpq_index_add_i8(lpq_index *idx, const int8_t *codes_dev, int64_t n, int64_t ld, void *stream)
{
    if (!idx || !codes_dev) return fail(LPQ_EINVAL, "null argument");
    if (n < 0) return fail(LPQ_EINVAL, "n < 0");
    if (ld < idx->d) return fail(LPQ_EINVAL, "ld < d");
    if (idx->size + n > idx->capacity) return fail(LPQ_ERANGE, "index capacity %lld exceeded", (long long)idx->capacity);
    if (n == 0) return LPQ_OK;
    hipStream_t st = (hipStream_t)stream;
    if (idx->packed) {
        const int rc = index_pack_rows(idx, idx->size, codes_dev, n, ld, st);
        return rc ? rc : index_after_add(idx, n, st);
    }
    HIP_TRY(launch_repack_i8(codes_dev, n, ld, idx->d, idx->codes + (size_t)idx->size * idx->d_pad, idx->d_pad,
                             idx->d_pad, idx->norms + idx->size, st));
    return index_after_add(idx, n, st);
}

extern "C" int64_t lpq_index_size(const lpq_index *idx) { return idx ? idx->size : -1; }

extern "C" int lpq_index_data(const lpq_index *idx, const int8_t **codes_dev, int64_t *ld_codes,
                              const int32_t **norms_dev)
{
    if (!idx) return fail(LPQ_EINVAL, "null index");
    if (codes_dev) *codes_dev = idx->codes;
    if (ld_codes) *ld_codes = idx->packed ? idx->d_pad / 2 : idx->d_pad;
    if (norms_dev) *norms_dev = idx->norms;
    return LPQ_OK;
}

// -------------------------------------------------------------- candidate lists ----
extern "C" int lpq_gather_dist_i8(const lpq_index *idx, const int8_t *qcodes_dev, int64_t nq, int64_t ld,
                                  const int32_t *ids_dev, int m, int metric, int32_t *dist_dev, void *stream)
{
    if (!idx) return fail(LPQ_EINVAL, "null index");
    if (nq < 0 || m < 1) return fail(LPQ_EINVAL, "nq < 0 or m < 1");
    if (metric != LPQ_METRIC_L2SQ && metric != LPQ_METRIC_IP) return fail(LPQ_EINVAL, "unknown metric %d", metric);
    if (idx->size < 1) return fail(LPQ_ESTATE, "gather on an empty index");
    if (nq > 0 && (!qcodes_dev || !ids_dev || !dist_dev)) return fail(LPQ_EINVAL, "null argument");
    if (nq > 0 && ld < idx->d) return fail(LPQ_EINVAL, "ld < d");
    HIP_TRY(launch_gather_dist(idx->codes, idx->norms, idx->size, idx->d, idx->d_pad, qcodes_dev, nq, ld, ids_dev, m,
                               metric, dist_dev, (hipStream_t)stream, idx->packed));
    return LPQ_OK;
}

extern "C" int lpq_rerank_f32(const float *x_dev, int64_t n, int64_t ldx, const float *q_dev, int64_t nq, int64_t ldq,
                              int d, const int32_t *cand_ids_dev, int kc, int k, int metric, int32_t *ids_dev,
                              float *dist_dev, void *stream)
{
    if (d < 1 || n < 1 || nq < 0 || kc < 1 || k < 1) return fail(LPQ_EINVAL, "bad size");
    if (metric != LPQ_METRIC_L2SQ && metric != LPQ_METRIC_IP) return fail(LPQ_EINVAL, "unknown metric %d", metric);
    if (kc > 4096) return fail(LPQ_ERANGE, "kc = %d > 4096", kc);
    if (k > 4096) return fail(LPQ_ERANGE, "k = %d > 4096", k);
    if (ldx < d || (nq > 0 && ldq < d)) return fail(LPQ_EINVAL, "row stride < d");
    if (!x_dev || (nq > 0 && (!q_dev || !cand_ids_dev || !ids_dev || !dist_dev))) return fail(LPQ_EINVAL, "null argument");
    HIP_TRY(launch_rerank_f32(x_dev, n, ldx, q_dev, nq, ldq, d, cand_ids_dev, kc, k, metric, ids_dev, dist_dev,
                              (hipStream_t)stream));
    return LPQ_OK;
}

// ------------------------------------------------------------------------ search ----
namespace {

// How a search over n items is cut up, and where its intermediates live in the workspace.
enum PlanMode { PLAN_GENERIC = 0, PLAN_MFMA_LDS = 1, PLAN_MFMA_REG = 2, PLAN_MFMA_COLLECT = 3 };
struct Plan {
    int mode = PLAN_GENERIC;
    int64_t nq_pad = 0;
    int64_t seed_rows = 0;  // rows of the threshold-seeding pass (0 = none)
    int rank = 0;           // PLAN_MFMA_COLLECT: the bound of the first scan is the rank-th largest group maximum
    int S1 = 0, S2 = 0;     // corpus splits of the seeding pass and of the main pass
    int SEG = 0;            // PLAN_MFMA_REG: segments per split in the seeding pass
    int G = 0;              // PLAN_MFMA_REG: group maxima per query
    bool rsplit = false;    // PLAN_MFMA_REG, PLAN_MFMA_COLLECT: row-split workgroups (few queries)
    int rs_waves = 0;       // ... of this many waves (0 when not row-split)
    int merge_group = 0;    // lists merged per workgroup in the first merge pass (0 = single pass)
    int64_t seed_stride = 0;   // seeding pass: one stage every seed_stride rows (systematic sample)
    int seed_stages = 0;       // ... seed_stages of them per split
    int64_t piece_stride = 0;  // seeding pass: or runs of 8 rows every piece_stride rows, dealt round-robin to the splits
    int piece_stages = 0;      // ... eight runs to a stage, piece_stages stages per split
    int SS = 0, Cs = 0;     // PLAN_MFMA_COLLECT: regions per query, capacity of a region
    int Sg = 0;             // PLAN_MFMA_COLLECT: splits of the generic kernel for overflowed queries
    int Sr = 0;             // PLAN_MFMA_COLLECT: splits of the register-list kernel for many overflowed queries (0 = none)
    int rounds = 0;         // PLAN_MFMA_COLLECT: further rounds of the collecting scan, with tighter bounds, for overflowed queries
    int few = 0;            // ... unless no more than this many overflowed, which the generic kernel takes
    int wave_queries = 64;  // PLAN_MFMA_COLLECT: queries per wave of the scan
    bool stream = false;    // PLAN_MFMA_COLLECT: the scan that streams both operands (search_mfma_stream.hip)
    int seed_tiles = 0;     // ... its seeding pass: tiles of 256 rows, in runs of 16 rows
    int64_t run_stride = 0; // ... every run_stride rows
    int expect = 0;         // PLAN_MFMA_COLLECT: expected candidates per query
    bool maxima = false;    // in place of either: a search by group maxima of all rows, finished by helpers workgroups per query
    MaximaShape groups;
    int helpers = 0, most_helpers = 0, finish_threads = 0;
    size_t off_qcodes = 0, off_qnorms = 0, off_lists1 = 0, off_seedlist = 0, off_seeds = 0, off_lists2 = 0,
           off_gmax = 0, off_merge_tmp = 0, off_cbuf = 0, off_ccnt = 0, off_over = 0, off_qlist = 0, off_redo = 0, off_bounds2 = 0, off_over2 = 0,
           off_qlist2 = 0, total = 0;
};

size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

constexpr int WIDE_MIN_BITS = 2;
constexpr int64_t PACKED_BATCH_MIN = 128;  // packed index: larger batches take one collecting scan instead of tiles of 64 queries
constexpr int REFINE_ROUNDS = 2;        // further rounds of the collecting scan for queries that overflowed (k > 16)

// The bound of a collecting scan is the rank-th largest maximum of its sample.  With rank = k it is certain that k items
// reach it.  But the k nearest items are in a sample of a share s of the corpus in number like k draws that hit with
// probability s, and fewer than k items reach the bound only if rank of them or more are: the rank here is that number's
// mean, and as many standard deviations (with the term of its skew) as make it happen to one query in 100 nq: in one batch of a
// hundred, to one of 7000 queries at 70 and of 1M at 10 000.  (z is the normal quantile of that, 0.905 of sqrt(2 ln(100 nq)) within
// 4 % from 100 nq = 2e4 on.)  That takes the places of the nearest items for independent.  Samples are runs of 8 or 16 rows or whole stages, so
// neighbours stored side by side are hit together, and more queries fall short of k.
// Such a query is found by its count and searched again, as one whose region overflows is.
int seed_rank(int64_t n, int64_t rows, int64_t nq, int k)
{
    const double s = (double)rows / (double)n, mean = k * s;
    const double z = 0.905 * std::sqrt(2.0 * std::log(100.0 * (double)(nq > 1 ? nq : 1)));
    const double r = std::ceil(mean + z * std::sqrt(mean * (1.0 - s)) + (z * z - 1.0) / 6.0 * (1.0 - 2.0 * s) + 1.0);
    return r < (double)k ? (int)r : k;
}

// Small batches by group maxima (search_maxima.hip): three launches, no sample, no candidates on the way.  The scan splits
// rows between the waves of a workgroup, 64 queries each, so that every further 64 queries read the corpus again, and the
// finishing workgroups read about k groups of rows per query: the lines below bound both.  us, other scans / this one,
// 128 features, k = 10: one query on 1M rows 54 / 38, 16 on 10M x 96 202 / 188, 100 on 10 000 35 / 18, 1000 48 / 24, 100 on
// 200 000 42 / 30, 256 47 / 38, 600 57 / 51, 100 on 1M 67 / 48, 200 72 / 73, 128 on 5M x 96 173 / 162.  Rows of 384 bytes
// and more through the streaming scan: 16 on 300 000 x 512 94 / 45, 128 95 / 53, 16 on 500 000 x 768 108 / 94, 64, k = 100 122 /
// 127, 128 121 / 128, 100 on 1M x 384 152 / 125, 200 on 100 000 x 768 64 / 52, on 30 000 x 2048 75 / 59, 1 on 40 000 x 1500 51 / 34.
void plan_maxima(Plan &p, const lpq_index *idx, int64_t nq, int k)
{
    const int64_t n = idx->size;
    for (int key : {LPQ_TUNE_PATH, LPQ_TUNE_SPLITS, LPQ_TUNE_SEED_ROWS, LPQ_TUNE_WAVE_QUERIES, LPQ_TUNE_REGION_CAP})
        if (tune(key)) return;
    // (Codes of few bits go by lists.  The line is from when every group that ties with the k-th had its rows scored again, 16 queries on 1M
    // skewed integers of 24 features, 3 bits 46 / 341; with the ties found from the first row on it would be 44 / 30, and 0.53 of the time by
    // lists over 192 such shapes.)
    if (nq < 1 || nq > 4096 || idx->bits < 4 || (idx->bits < 6 && idx->d < 64) || k > MAXIMA_MAX_K || idx->d_pad > MAXIMA_MAX_D) return;
    const bool stream = idx->d_pad > 256;     // by the streaming scan, whose workgroups have eight waves and a CU to themselves
    if (nq > (idx->packed ? 64 : stream ? 512 : 4096)) return;
    const int waves = stream ? 8 : mfma_row_split_waves(idx->d_pad, idx->packed);
    const int64_t tiles = ceil_div(nq, 64), row_bytes = idx->packed ? idx->d_pad / 2 : idx->d_pad;
    if (idx->packed && idx->d_pad <= 128 && n > 3'000'000) return;   // (16 queries at 4 bits: 2M x 64 58 / 41; 10M x 96 139 / 155
    // when the line was drawn, 147 / 125 since up to 32 queries skip half of a tile)
    if (stream && tiles > 1 && tiles * n * row_bytes > int64_t(row_bytes < 768 ? 1024 : 420) << 20) return;
    if (!stream && tiles == 2 && tiles * n * row_bytes > int64_t(512) << 20) return;
    if (!stream && tiles > 2 && tiles * tiles * n * (row_bytes > 128 ? 2 * row_bytes : 128) > int64_t(512) << 20) return;
    MaximaShape m;
    m.parts = 2 * waves;
    m.stage_rows = 32 * waves;
    m.stages = (int)(n / m.stage_rows);
    if (m.stages < 16) return;
    const int slots = (int)((stream ? 256 : 512) / tiles);
    m.S = m.stages < slots ? m.stages : slots;
    // As many groups as the finishing threads hold, 16 each: workgroups of 256 where there are no more groups than that, or
    // where many queries need few rows each (a CU takes one of 1024 threads, or four).
    int threads = 1024;
    auto shape = [&]() {
        int64_t seg = 16 * threads / (m.S * m.parts);
        if (seg > m.stages / m.S) seg = m.stages / m.S;
        m.SEG = (int)(seg < 1 ? 1 : seg);
        m.G = m.S * m.SEG * m.parts;
        m.seg_stages = (int)ceil_div(ceil_div(m.stages, m.S), m.SEG);
        return 1.1 * (double)k * (double)n / (double)m.G;       // rows of the groups that reach the bound
    };
    double rows = shape();
    if (!stream && (m.G <= 16 * 256 || (tiles > 1 && 1.1 * (double)k * (double)n / (16.0 * 256.0) <= 768.0))) {
        threads = 256;
        rows = shape();
    }
    const int sets = m.G / (threads == 256 ? 4 : 16) < 256 ? m.G / (threads == 256 ? 4 : 16) : 256;
    // (Groups in sixteens, as the last kernel reads them: below 65 536 rows, where a stage is a split and a segment, an even number of stages of
    // 128 rows or a multiple of four of 64; half and a third of the corpora of 8000 to 65 536 rows keep the other scans.)
    if (m.G % 16 || m.G > 16 * threads || sets < k) return;
    // Streamed rows: the bound is the k-th largest of the maxima of so many sets of groups, and as many groups reach it as fall on k
    // sets if they fall on any set alike: up to all where k is near their number (64 queries, k = 50, 12 902 x 1913, 50 sets: 55 us by the
    // collecting scan, 119 here, 49 since neighbouring groups fall in different sets).  Of 1900 shapes of 257 to 4096 features (1 to 512 queries, k = 1 to 128) the 1686 within the line
    // take a median of 0.65 of the collecting scan's time and 18 of them 4 % more or worse, up to 23 %; from 160 to 300 MB on it is as
    // often slower, up to 1.7 times.  (On fewer than 8192 rows the other scan has little to sample: 4600 to 6600 rows, 163 to 384 MB 0.63 to 0.72.)
    const double reach = !stream ? rows : k == sets ? (double)n : std::fmin((double)n, -sets * std::log1p(-(double)k / sets) * (double)n / (double)m.G);
    const double finish_bytes = (double)nq * (reach * (double)row_bytes + 4.0 * m.G);
    // One tile of short rows, k up to 10, whose other scans cost least (register lists, or few candidates): a median of 0.81 of their time up to
    // 10 MB, 0.93 to 20, 0.97 to 30, 1.00 to 50.  k = 11 to 128: 0.76 to 40 MB, 0.88 to 110, 1.00 to 160, 1.08 to 250.
    const int most_mb = stream ? (n < 8192 ? 256 : 140) : tiles > 1 ? 32 : (k <= 10 ? 40 : 160);
    if (finish_bytes > (double)most_mb * (1 << 20)) return;
    int64_t h = (int64_t)(rows * (double)(row_bytes > 128 ? row_bytes : 128) / (768.0 * 128.0)), most = (threads == 256 ? 1024 : 256) / nq;
    if (most > 16) most = 16;
    if (most * k > 2048) most = 2048 / k;
    if (most < 1) most = 1;
    p.most_helpers = (int)most;      // (one query on 1M x 64, every second row zero: 2.9 ms by one workgroup)
    p.helpers = (int)(h < 1 ? 1 : (h > most ? most : h));
    p.finish_threads = threads;
    p.rsplit = !stream; p.rs_waves = waves;
    p.groups = m;
    p.maxima = true;
}

// compact: the plan for callers with a fixed workspace whose normal plan does not fit - fewer, larger splits
// (at least 512 rows), no collecting scan where another kernel needs less room.  Slower, the same results.
Plan make_plan(const lpq_index *idx, int64_t nq, int k, bool compact = false)
{
    Plan p;
    const int64_t n = idx->size;
    const int64_t want = tune(LPQ_TUNE_PATH);
    const bool regs = mfma_reg_supported(idx->d_pad, k), stream = !idx->packed && mfma_stream_rows(idx->d_pad) && !(compact && idx->d_pad > 1536);
    const bool coll = stream ? k <= MAX_K : mfma_collect_supported(idx->d_pad, k);
    // Large batches of short rows: the collecting variant with 128 queries per wave beats the
    // register lists at any k it takes (fewer LDS reads and less per-stage overhead per contraction).
    // (Not for codes of fewer than WIDE_MIN_BITS bits: there many items tie at the seed
    // threshold, all of them are collected, and queries spill to the exact redo.)
    const bool wide = coll && idx->bits >= WIDE_MIN_BITS && mfma_collect_wide(nq, idx->d_pad) &&
                      tune(LPQ_TUNE_WAVE_QUERIES) != 64;
    // Rows longer than 128 bytes: the register-list kernels hold 6 or 8 operand registers per query
    // block on top of the lists and spill; the collecting variant measured 1.6x (10 000 queries) to
    // 3.5x (16 queries) faster at d = 256 for every batch size and code width.
    const bool long_rows = coll && idx->d_pad > 128;
    // Lists of 11 to 16 entries: the 16-entry register lists cost more per accepted candidate than
    // collecting does; collecting measured 11 to 40 % faster at every batch size (d = 64 to 128).
    const bool long_lists = coll && k > 10;
    // Batches of 65 to 256 and 513 to 768 queries (the others are `wide`), lists of 5 to 10: the register lists
    // fill from nothing in every split, at a cost that grows with the candidates asked for and not with the
    // corpus, so the collecting scan wins from about one candidate in fifty items on.  Collecting / register
    // lists in us, 128 features, 8 bits: 5000 items, 65 queries, k = 10 42 / 55, 640 queries 49 / 63; 20 000, 256
    // queries, k = 10 39 / 45, k = 5 38 / 36; 100 000, 65 queries, k = 10 42 / 35, 640 49 / 51; 300 000, 640 65 / 66,
    // 256 50 / 50; a million, 65 68 / 62, 640 127 / 125.  k = 4 and less: the lists (50 000, 256 queries, k = 1 38 / 29).
    // (Of these batches 8-bit codes on small corpora go by group maxima first, see plan_maxima.)
    // (Codes of few bits tie at the bound and all that tie is collected.  1 bit always keeps the lists: a
    // million items, 100 queries 2.1 / 0.35 ms.  2 bits beyond 32 768 items too: 20 000, 256 queries 47 / 53 us,
    // 100 000 53 / 45, a million 114 / 78.  3 bits behave like 8.)
    const bool few_rows = coll && !compact && nq > 64 && k > 4 && nq * k * 50 >= n &&
                          idx->bits >= (n <= 32768 ? WIDE_MIN_BITS : 3);
    // Packed rows: the row-split register-list kernel (callers tile the queries by 64), or for large
    // batches the collecting scan over all queries at once; the generic kernel on request.
    // (lists of more than 16 entries: the collecting scan at every batch size; rows of 32 packed
    // bytes have no scan over more than 64 queries, their callers tile)
    const bool packed_batch = idx->packed && coll && idx->d_pad >= 96 && (nq > PACKED_BATCH_MIN || (!regs && nq > 64));
    const bool packed_collect = packed_batch || (idx->packed && coll && !regs && nq <= 64);
    if (idx->packed) p.mode = want == 1 ? PLAN_GENERIC : (packed_collect ? PLAN_MFMA_COLLECT
                                                          : (regs ? PLAN_MFMA_REG : PLAN_GENERIC));
    else if (want == 3 && coll) p.mode = PLAN_MFMA_COLLECT;
    else if (want != 1 && want != 4 && (wide || long_rows || long_lists || few_rows)) p.mode = PLAN_MFMA_COLLECT;
    else if (want != 1 && regs) p.mode = PLAN_MFMA_REG;
    else if (want != 1 && want != 4 && coll) p.mode = PLAN_MFMA_COLLECT;
    else if (want != 1 && mfma_lds_supported(idx->d_pad, k)) p.mode = PLAN_MFMA_LDS;
    // Corpora too small for any sample (below 4096 rows) and little work in all: the generic kernel
    // (1000 x 128, 1000 queries, k = 10: 0.05 ms against 0.29 ms for an unseeded matrix-core scan).
    if (want == 0 && n < 4096 && nq * n <= (int64_t(4) << 20)) p.mode = PLAN_GENERIC;
    p.nq_pad = round_up(nq > 0 ? nq : 1, 512);
    // A merge pass sorts up to 4096 candidates per workgroup; more lists than that are merged in
    // two passes, so the number of splits is bounded by max_lists^2 only.
    const int max_lists = merge_max_lists(k) * (merge_max_lists(k) > 1 ? merge_max_lists(k) : 1);
    const int64_t slots = 512;   // workgroups of the matrix-core kernels resident at once (2 per CU)

    // Seeding pass over a sample of the corpus: it yields, per query, an upper bound on the final
    // k-th best key, so the main pass rejects almost everything from its first tile on.
    // PLAN_MFMA_REG and PLAN_MFMA_COLLECT derive the bound from group maxima over chunks spread
    // evenly over the corpus (no candidates collected) and then scan ALL rows; PLAN_MFMA_LDS
    // searches a first slice exactly and scans the rest.  The collecting scan never tightens the
    // bound, so its sample is a fixed fraction of the corpus: about k n / seed_rows candidates
    // per query survive.
    const bool gm = p.mode == PLAN_MFMA_REG || p.mode == PLAN_MFMA_COLLECT;
    int64_t seed = 0;
    double room = 0.0;       // collecting scan: candidates per query that there is room for in any case
    if (tune(LPQ_TUNE_SEED_ROWS) > 0) seed = tune(LPQ_TUNE_SEED_ROWS);
    else if (tune(LPQ_TUNE_SEED_ROWS) == 0 && p.mode != PLAN_GENERIC) {
        // Few queries: the scan is bound by corpus bytes, so the sample stays small.  Otherwise a
        // larger sample pays for itself through fewer candidates in the main pass (measured).
        const bool few = gm && mfma_row_split(nq, idx->d_pad, idx->packed);
        seed = gm ? (few ? n / 16 : n / 8) : n / 64;
        // (corpora below 64K rows: the sample may go down to 1024 rows - without a seeding pass every
        // split spends its few hundred rows filling lists from empty thresholds: 10 000 x 128, 100
        // queries: 0.245 ms unseeded)
        const int64_t lo_gm = n >= 65536 ? 8192 : (n / 8 > 1024 ? n / 8 : 1024);
        const int64_t lo = gm ? lo_gm : 4096, hi = p.mode == PLAN_MFMA_COLLECT ? n : (gm ? (few ? 65536 : 131072) : 32768);
        seed = seed < lo ? lo : (seed > hi ? hi : seed);
        if (p.mode == PLAN_MFMA_COLLECT && few) {   // no tightening during the scan: the sample grows with k
            // (beyond k = 256 a quarter: an eighth would let about 9 k candidates through, more than the
            // 4096 the selection sorts)
            const int64_t by_k = n / 400 * k, least = n / 16, most = k > 512 ? n / 2 : (k > 256 ? n / 4 : n / 8);
            seed = by_k < least ? least : (by_k > most ? most : by_k);
        } else if (p.mode == PLAN_MFMA_COLLECT) {
            // The sample costs time in proportion to its rows, the rank n / rows candidates it lets through in proportion
            // to their number, one as much as 1200 sampled rows of 128 bytes (with 800 and 1700 within 1 % of that on 1M x 128
            // and 4M x 256, 10 000 queries, k = 10 and 100; with 300 and 2400 2 to 6 % slower).  No more than 1500 candidates
            // where that can be had, so that they stay well inside the 4096 the selection sorts; at most n / 4.
            // (k beyond 512: half the corpus; streamed rows up to two fifths: 33 527 x 904, 7013 queries, k = 76: 0.482 -> 0.450 ms)
            const int64_t most = k > 512 ? n / 2 : (stream ? n / 5 * 2 : n / 4);
            // What is best for the k-th largest maximum goes with sqrt(k n): compact plans keep it, others take no smaller
            // a sample than lets as many candidates through.  Their number is also the length of the shortest cluster stored in one piece
            // that still holds as many of the sample's groups as the bound's rank; the bound of a shorter one comes from another cluster,
            // and its queries are searched again.  With three quarters more, 92 random corpora of clusters of 30 to 5000 rows, k up to 16:
            // 20 slower than with the k-th maximum by 5 % or more, 1.4 % in the mean; as it is 8 slower and 4 % faster in the mean (770 rows,
            // 1.3M x 107, 2363 queries: 700 us, 1726, 697).  It costs a large batch on a corpus in no order 1 %: 1M x 128, 10 000 queries,
            // k = 10 1118 -> 1131 us; 1000 on 1.2M x 100 nothing.
            double by_k = 125000.0 * std::sqrt((double)n / 1e6 * (double)k / 10.0);
            if (stream && !compact) by_k *= std::sqrt(128.0 / (double)idx->d);
            const double by_room = (double)k * (double)n / 1500.0;
            const double want_rows = by_k > by_room ? by_k : by_room;
            seed = want_rows > (double)most ? most : (int64_t)want_rows;
            const double per_candidate = 1200.0 * 128.0 / (double)idx->d_pad;
            room = (double)k * (double)n / (double)(seed > 1 ? seed : 1);
            double best = INFINITY;
            for (double share = 0.5; !compact && share > 1.0 / 80.0; share *= 0.86) {
                const int64_t rows = (int64_t)((double)n * share);
                if (rows > most) continue;
                if (rows < lo) break;
                const double candidates = (double)seed_rank(n, rows, nq, k) / share;
                const double cost = (double)rows + per_candidate * (candidates > 1500.0 ? 100.0 : 1.0) * candidates;
                if (cost < best && candidates <= room) { best = cost; seed = rows; }
            }
            // Codes of few bits tie at the bound, and all that tie are collected: the sample that was best for the
            // k-th largest maximum (1M x 128, 1000 queries, k = 10, 2 bits: 159 us, 238 with the smaller one).
            if (idx->bits < 4 && (double)seed < want_rows) seed = want_rows > (double)most ? most : (int64_t)want_rows;
        }
    }
    seed = seed / 256 * 256;
    // A sample must hold at least 64 k rows for its k-th group maximum to mean something; a small
    // corpus may give up to half of its rows for that (20 000 x 128, 10 000 queries, k = 100: 0.5 ms
    // with such a sample against 2.3 ms through the generic kernel).
    if (p.mode == PLAN_MFMA_COLLECT && seed > 0 && seed < 64 * (int64_t)k) seed = round_up(64 * (int64_t)k, 256);
    if (seed < 64 * k || seed * 2 > n || (k <= 512 && p.mode != PLAN_MFMA_COLLECT && seed * 4 > n)) seed = 0;
    if (p.mode == PLAN_MFMA_COLLECT && !seed) {   // too few items to sample: exact paths
        // (longer lists without a sample: the generic kernel; the LDS-list matrix-core kernel measured
        // 10 to 70x slower on the corpora this happens for - 1000 x 128, k = 100, 1000 queries: 4.3 ms
        // against 0.06 ms - and stays reachable through LPQ_TUNE_PATH = 4)
        p.mode = (regs && want != 1) ? PLAN_MFMA_REG
                 : (want == 4 && mfma_lds_supported(idx->d_pad, k) && !idx->packed ? PLAN_MFMA_LDS : PLAN_GENERIC);
    }

    // lists one merge launch takes: the register-list scan's come out sorted, which allows more of them
    const int one_pass = p.mode == PLAN_MFMA_REG ? merge_max_sorted_lists(k) : merge_max_lists(k);
    auto splits_for = [&](int64_t rows, int64_t tiles_q, int64_t min_rows, int64_t slots, int64_t cap) {
        int64_t s;
        if (p.mode != PLAN_GENERIC) s = tune(LPQ_TUNE_SPLITS) > 0 ? tune(LPQ_TUNE_SPLITS) : slots / (tiles_q > 0 ? tiles_q : 1);
        else s = tune(LPQ_TUNE_SPLITS) > 0 ? tune(LPQ_TUNE_SPLITS) : ceil_div(2048, nq > 0 ? nq : 1);
        const int64_t by_rows = rows / min_rows > 0 ? rows / min_rows : 1;
        if (s > by_rows) s = by_rows;
        if (s > cap) s = cap;
        if (s < 1) s = 1;
        return (int)s;
    };
    const bool gmode = p.mode == PLAN_MFMA_REG || p.mode == PLAN_MFMA_COLLECT;
    int64_t qt = (p.mode == PLAN_MFMA_LDS && k > 16) ? 128 : 256;   // queries per workgroup
    int64_t slots_now = slots;
    bool long_scan = false;
    if (gmode) {
        // (rows of more than 128 bytes: the collecting scan only - the register lists do not fit beside them)
        const int waves = mfma_row_split_waves(idx->d_pad, idx->packed);
        p.rsplit = mfma_row_split(nq, idx->d_pad, idx->packed) && (waves == 4 || p.mode == PLAN_MFMA_COLLECT);
        p.rs_waves = p.rsplit ? waves : 0;
        if (p.mode == PLAN_MFMA_COLLECT && mfma_collect_wide(nq, idx->d_pad) && tune(LPQ_TUNE_WAVE_QUERIES) != 64)
            p.wave_queries = 128;
        if (p.mode == PLAN_MFMA_COLLECT && idx->packed)   // the packed scan has one variant per row length
            p.wave_queries = idx->d_pad <= 128 ? 128 : 64;
        qt = mfma_queries_per_workgroup(nq, idx->d_pad, p.wave_queries == 128);
        long_scan = p.mode == PLAN_MFMA_COLLECT && !idx->packed && !p.rsplit && mfma_long_rows(idx->d_pad, nq);
        if (long_scan) {   // the scan for long rows and its seeding pass have their own tiles
            p.wave_queries = mfma_long_wave_queries(idx->d_pad);
            qt = (int64_t)mfma_long_waves(idx->d_pad, nq) * p.wave_queries;
            if (qt > 512) p.nq_pad = round_up(nq > 0 ? nq : 1, qt);   // query rows (codes, group maxima) cover whole tiles
            if (mfma_long_waves(idx->d_pad, nq) == 8) slots_now = 256;   // one workgroup per CU
        }
        p.stream = p.mode == PLAN_MFMA_COLLECT && stream;
        if (p.stream) {
            qt = 64 * mfma_stream_wq(nq);
            slots_now = 256;   // one workgroup per CU
        }
    }
    const int64_t tiles_q = ceil_div(nq > 0 ? nq : 1, qt);
    // Fewest rows of a split.  Small corpora need every workgroup they can get: 10 000 x 128, k = 10, 1000
    // queries: 0.104 ms with splits of 512 rows, 0.065 with 256, 0.054 with 128; 100 queries 0.065 -> 0.041;
    // 30 000 x 128, 100 queries, k = 100: 0.127 -> 0.082; 64 rows gain nothing more.
    // (Packed rows: from 64K items on 128 splits are enough, more only spread the candidates thinner.)
    const int64_t min_rows = p.mode == PLAN_GENERIC ? 2048 : (compact || (idx->packed && n >= 65536) ? 512 : 128);
    // (A sample of a size asked for keeps the certain bound, and so do row-split launches: the number of candidates is not
    // what takes their time, and a query too few items pass for costs one of their rounds; and compact plans.)
    const bool by_rank = p.mode == PLAN_MFMA_COLLECT && !compact && !mfma_row_split(nq, idx->d_pad, idx->packed) &&
                         tune(LPQ_TUNE_SEED_ROWS) == 0;
    if (seed) {
        const int rank = by_rank ? seed_rank(n, seed, nq, k) : k;   // of the sample as asked for; it comes out a little larger or smaller
        // group maxima per query: 2 per split and segment (8 when rows are split), at most 2048 (4096 for k > 512)
        // (row-split launches with register lists: up to 128 splits; with 256 the 2048 maxima cost the
        // threshold kernel 3 us more than the pass gains.  Longer lists want the tighter bound: 1543 queries,
        // 97 candidates on 780K x 56 at 4 bits 2.05 ms with 128, 1.93 with 256)
        p.S1 = splits_for(seed, tiles_q, min_rows, slots_now, gmode ? (p.rsplit ? (p.mode == PLAN_MFMA_REG ? 128 : 256) : 1024) : merge_max_lists(k));
        if (p.stream) {
            // tiles of 256 rows made of runs of 16 rows spread evenly over the corpus
            const int row_waves = mfma_stream_row_waves(nq);
            const int most = 2048 / (2 * row_waves);
            if (p.S1 > most) p.S1 = most;
            const SampleShape shape = sample_that_covers(n, ceil_div(seed, 256), 16, p.S1);
            p.S1 = shape.splits;
            p.SEG = mfma_seed_segments(p.S1, k, rank, row_waves);
            p.G = mfma_seed_groups(p.S1, p.SEG, row_waves);
            p.seed_tiles = (int)shape.per_split * p.S1;
            if ((int64_t)p.seed_tiles * 256 > n) p.seed_tiles = (int)(seed / 256);
            p.run_stride = n / (16 * (int64_t)p.seed_tiles);
            seed = (int64_t)p.seed_tiles * 256;
        } else if (gmode) {
            SampleShape shape = {p.S1, ceil_div(seed / 64, p.S1)};
            if (!p.rsplit && !long_scan && !compact) shape = sample_that_covers(n, seed / 64, 8, p.S1);   // runs of 8 rows, see below
            p.S1 = shape.splits;
            p.SEG = mfma_seed_segments(p.S1, k, rank, p.rs_waves);
            p.G = mfma_seed_groups(p.S1, p.SEG, p.rs_waves);
            // systematic sample: one stage every seed_stride rows, shared out over the S1 splits
            const int64_t stage_rows = p.rsplit ? 32 * p.rs_waves : (long_scan ? mfma_long_stage_rows(idx->d_pad, nq) : 64);
            const int64_t stages = seed / stage_rows;
            p.seed_stages = (int)ceil_div(stages, p.S1);
            p.seed_stride = n / ((int64_t)p.seed_stages * p.S1) / 128 * 128;
            if (p.seed_stages < 1 || p.seed_stride < stage_rows) { p.seed_stages = 0; p.seed_stride = 0; }
            else seed = (int64_t)p.seed_stages * p.S1 * stage_rows;
            // Finer still (not for row-split launches): runs of 8 rows every piece_stride rows, dealt
            // round-robin to the splits, so that a run of neighbouring rows - a cluster stored
            // contiguously - is spread over many splits and hence over many groups of the pass.
            // (For k > 16 on a corpus sorted by norm a split's groups then span wide slices of the order
            // and up to a tenth of the queries overflow; the further rounds of the scan take those.)
            if (!p.rsplit && !long_scan) {
                const int64_t pstages = shape.per_split;                        // about as many rows as the stage-wise sample
                const int64_t pstride = pstages > 0 ? n / (8 * pstages * p.S1) : 0;   // all pieces inside the corpus
                if (pstride >= 16 && pstages >= 1) {
                    p.piece_stride = pstride;
                    p.piece_stages = (int)pstages;
                    seed = pstages * p.S1 * 64;
                }
            }
        }
    }
    p.seed_rows = seed;
    p.rank = by_rank ? seed_rank(n, seed, nq, k) : k;
    p.S2 = splits_for(gmode ? n : n - seed, tiles_q, min_rows, slots_now,
                      p.mode == PLAN_MFMA_COLLECT ? (p.rsplit ? 512 : 2048)
                                                  : (p.rsplit ? one_pass : max_lists));   // few queries: one merge pass
    // (The streaming scan's tiles hold 256 rows: no more splits than tiles, or the rest of them and of the regions stay
    // empty.  20 000 x 2048, one query 57.8 -> 54.5 us, 300 queries 80 -> 76; 40 000 x 768, 16 queries 51.8 -> 49.4.)
    if (p.stream && p.S2 > ceil_div(n, 256)) p.S2 = (int)ceil_div(n, 256);
    if (p.mode == PLAN_MFMA_COLLECT) {
        // expected candidates per query ~ k n / seed_rows, spread evenly over SS regions (the scan
        // deals its stages round-robin to the splits); a region holds three times its share, at
        // least 64, which leaves room for bounds several times looser than expected (a corpus stored
        // in sorted order).  Overflow is caught per query and redone exactly.
        // (Their size goes by the larger sample's candidates of the rule before the bound's rank: a further round's bound is the k-th best
        // of what the regions hold, and a cluster stored in one piece is in few of them.  With regions for the fewer candidates that are
        // expected now, 8080 queries, k = 200, 673 620 x 74 in clusters of 468 rows took 172 ms instead of 2.7, 4465, k = 100, 79 076 x 541
        // in clusters of 439 52 instead of 1.5.)
        p.SS = mfma_collect_regions(p.S2, p.rs_waves);
        const double candidates = 1.15 * (double)p.rank * (double)n / (double)seed;
        p.expect = (int)(candidates + 1.0);
        const double per_region = (!compact && 1.3 * room > candidates ? 1.3 * room : candidates) / p.SS;
        int64_t cs = 64;
        while ((double)cs < (compact && stream ? 1.5 : 3.0) * per_region && cs < 4096) cs <<= 1;
        p.Cs = (int)cs;
        if (tune(LPQ_TUNE_REGION_CAP) > 0) p.Cs = (int)(tune(LPQ_TUNE_REGION_CAP) < 4096 ? tune(LPQ_TUNE_REGION_CAP) : 4096);
        // splits of the redo scan: many, so that a few queries spread over the chip; bounded by the
        // single merge pass and by 256 MB of lists
        p.Sg = merge_max_lists(k) < 128 ? merge_max_lists(k) : 128;
        while (p.Sg > 4 && (size_t)nq * p.Sg * k * sizeof(cand_t) > (size_t(compact ? 16 : 256) << 20)) p.Sg /= 2;
    }

    if (!compact && gmode) plan_maxima(p, idx, nq, k);
    size_t o = 0;
    p.off_qcodes = o;   o = align256(o + (size_t)p.nq_pad * idx->d_pad);
    p.off_qnorms = o;   o = align256(o + (size_t)p.nq_pad * sizeof(int32_t));
    if (p.maxima) {
        p.off_lists1 = p.off_seedlist = p.off_seeds = o;
        p.off_lists2 = o;   o = align256(o + (size_t)nq * p.most_helpers * k * sizeof(cand_t));
        p.off_gmax = o;     o = align256(o + (size_t)(idx->d_pad > 256 ? round_up(nq, 64) : nq) * p.groups.G * sizeof(int32_t));
        p.off_merge_tmp = p.off_cbuf = o;
        p.off_ccnt = o;     o = align256(o + (size_t)nq * p.most_helpers * sizeof(int32_t));
        p.off_over = o;     o = align256(o + (size_t)nq * sizeof(int32_t));
        p.off_qlist = p.off_redo = p.off_bounds2 = p.off_over2 = p.off_qlist2 = p.total = o;
        return p;
    }
    p.off_lists1 = o;   o = align256(o + (gmode ? 0 : (size_t)nq * p.S1 * k * sizeof(cand_t)));
    p.off_seedlist = o; o = align256(o + (size_t)nq * k * sizeof(cand_t));
    p.off_seeds = o;    o = align256(o + (size_t)p.nq_pad * sizeof(cand_t));
    p.off_lists2 = o;
    o = align256(o + (size_t)nq * (p.mode == PLAN_MFMA_COLLECT ? p.Sg : p.S2) * k * sizeof(cand_t));
    p.off_gmax = o;
    if (gmode && seed) o = align256(o + (size_t)p.nq_pad * p.G * sizeof(int32_t));
    p.off_merge_tmp = o;
    if (p.mode != PLAN_MFMA_COLLECT && p.S2 > one_pass) {
        p.merge_group = merge_max_lists(k);
        o = align256(o + (size_t)nq * ceil_div(p.S2, p.merge_group) * k * sizeof(cand_t));
    }
    if (p.mode == PLAN_MFMA_COLLECT) {
        p.off_cbuf = o; o = align256(o + (size_t)nq * p.SS * p.Cs * sizeof(cand_t));
        p.off_ccnt = o; o = align256(o + (size_t)nq * p.SS * sizeof(int32_t));
        p.off_over = o; o = align256(o + (size_t)nq * sizeof(int32_t));
        p.off_qlist = o; o = align256(o + ((size_t)nq + 1) * sizeof(int32_t));   // redo list, then its counter
        // redo of many queries by the register-list kernel (k <= 16, 256 queries per workgroup): one
        // list per query and split, few enough splits for a single merge pass
        if (!p.rsplit && regs && !idx->packed) {
            int64_t sr = slots / ceil_div(nq, 256);
            if (sr > merge_max_lists(k)) sr = merge_max_lists(k);
            if (sr > n / 512) sr = n / 512;
            p.Sr = (int)(sr < 1 ? 1 : sr);
            p.off_redo = o; o = align256(o + (size_t)nq * p.Sr * k * sizeof(cand_t));
        }
        // longer lists: a second collecting scan of the flagged queries, bounded by what the first collected
        if (!p.Sr) {
            // A round takes as long as the scan of the whole batch, the generic kernel as long as the corpus over Sg
            // splits - fewer for longer lists - once, and up to twice that for 16 queries.  1 / 8 / 16 flagged, ms above a search with
            // none, generic kernel against rounds: 10 000 queries on 500K x 768, k = 10 0.8 / 1.0 / 1.7 against 3.7;
            // on 1M x 128, k = 32 0.63 / 0.72 / 0.75 against 1.15; 4000 queries there, k = 20 0.37 / 0.42 / 0.72 against 0.65;
            // 2048 on 500K x 768, k = 10 0.54 / 0.63 / 1.25 against 0.90; 1000 on 1M x 128, k = 100 0.72 against 0.20.
            if (k <= 32 && nq >= 2048) p.few = nq >= 8192 ? 16 : 8;
            p.rounds = p.rsplit ? 1 : REFINE_ROUNDS;   // few queries: every launch counts, and their many regions rarely overflow twice
            p.off_bounds2 = o; o = align256(o + (size_t)p.nq_pad * sizeof(cand_t));
            p.off_over2 = o;   o = align256(o + (size_t)p.rounds * nq * sizeof(int32_t));
            p.off_qlist2 = o;  o = align256(o + (size_t)p.rounds * (nq + 1) * sizeof(int32_t));   // per round: list, then its counter
        }
    }
    p.total = o;
    return p;
}

int check_search_args(const lpq_index *idx, const void *q, int64_t nq, int64_t ld, int k, int metric,
                      const void *ids, const void *dist)
{
    if (!idx) return fail(LPQ_EINVAL, "null index");
    if (nq < 0) return fail(LPQ_EINVAL, "nq < 0");
    if (k < 1) return fail(LPQ_EINVAL, "k = %d < 1", k);
    if (metric != LPQ_METRIC_L2SQ && metric != LPQ_METRIC_IP) return fail(LPQ_EINVAL, "unknown metric %d", metric);
    if (idx->size < 1) return fail(LPQ_ESTATE, "search on an empty index");
    if (k > idx->size) return fail(LPQ_ERANGE, "k = %d > number of items %lld", k, (long long)idx->size);
    if (k > MAX_K) return fail(LPQ_ERANGE, "k = %d > %d", k, (int)MAX_K);
    if (idx->packed && k > MAX_K_PACKED)
        return fail(LPQ_ERANGE, "k = %d > %d, the most a packed index is searched for", k, (int)MAX_K_PACKED);
    if (nq > 0 && (!q || !ids || !dist)) return fail(LPQ_EINVAL, "null argument");
    if (nq > 0 && ld < idx->d) return fail(LPQ_EINVAL, "ld < d");
    if (nq * (int64_t)k >= (int64_t(1) << 40)) return fail(LPQ_ERANGE, "nq too large");
    return LPQ_OK;
}

// Everything after the queries are codes in the workspace.
// qcodes / qnorms: the nq queries' codes (rows of d_pad bytes, zero rows up to a multiple of 512
// readable behind them) and the per-query term of the final distance; emit_mode: how the merge
// turns a key into a distance.
int search_core(const lpq_index *idx, const Plan &p, char *ws, const int8_t *qcodes, const int32_t *qnorms, int64_t nq,
                int k, int metric, int emit_mode, int32_t *ids, int32_t *dist, hipStream_t st)
{
    SearchArgs a;
    a.codes = idx->codes; a.norms = idx->norms; a.cinit = idx->cinit; a.parity = idx->parity;
    a.n = idx->size; a.d = idx->d; a.d_pad = idx->d_pad;
    a.packed = idx->packed;
    a.qcodes = qcodes;
    a.nq = nq; a.k = k; a.metric = metric;
#ifdef LPQ_ABLATION
    a.dry_run = (int)tune(LPQ_TUNE_DRY_RUN);
#endif
    a.work_order = (int)tune(LPQ_TUNE_WORK_ORDER);
    a.wave_queries = 64;
    a.rsplit = p.rsplit;
    a.rs_waves = p.rsplit ? p.rs_waves : 4;
    cand_t *lists1 = reinterpret_cast<cand_t *>(ws + p.off_lists1);
    cand_t *seedlist = reinterpret_cast<cand_t *>(ws + p.off_seedlist);
    cand_t *seeds = reinterpret_cast<cand_t *>(ws + p.off_seeds);
    cand_t *certain = p.mode == PLAN_MFMA_COLLECT ? seedlist : nullptr;   // bounds that k items are sure to reach, one per query
    cand_t *lists2 = reinterpret_cast<cand_t *>(ws + p.off_lists2);
    int32_t *gmax = reinterpret_cast<int32_t *>(ws + p.off_gmax);

    cand_t *merge_tmp = reinterpret_cast<cand_t *>(ws + p.off_merge_tmp);
    // Final merge of the main pass' S2 lists (plus an optional extra list), in one or two passes.
    const bool sorted = p.mode != PLAN_MFMA_LDS;   // that scan's lists come out in arrival order
    auto final_merge = [&](const cand_t *extra) -> hipError_t {
        if (!p.merge_group)
            return launch_merge(lists2, nq, p.S2, k, extra, nullptr, nullptr, ids, dist, qnorms, emit_mode, st, sorted);
        const int groups = (int)ceil_div(p.S2, p.merge_group);
        hipError_t e = launch_merge_groups(lists2, nq, p.S2, p.merge_group, k, merge_tmp, st);
        if (e != hipSuccess) return e;
        return launch_merge(merge_tmp, nq, groups, k, extra, nullptr, nullptr, ids, dist, qnorms, emit_mode, st, true);
    };
    auto scan = [&](int64_t r0, int64_t r1, int S, const cand_t *sd, cand_t *out) -> hipError_t {
        KernelSpan span(st);
        return p.mode == PLAN_GENERIC ? launch_search_generic(a, r0, r1, S, sd, out, st)
                                      : launch_search_mfma(a, r0, r1, S, sd, out, st);
    };
    auto seed_pass = [&]() -> hipError_t {
        {
            KernelSpan span(st, LPQ_PROFILE_SEED);
            a.wave_queries = p.wave_queries;   // same query tiling as the scan it seeds
            hipError_t e = p.stream ? launch_stream_seed(a, p.seed_tiles, p.run_stride, p.S1, p.SEG, gmax, st)
                           : p.piece_stride ? launch_seed_mfma(a, 0, a.n, p.S1, p.SEG, gmax, st, 0, 0, p.piece_stride, p.piece_stages)
                           : p.seed_stride ? launch_seed_mfma(a, 0, a.n, p.S1, p.SEG, gmax, st, p.seed_stride, p.seed_stages)
                                           : launch_seed_mfma(a, 0, p.seed_rows, p.S1, p.SEG, gmax, st);
            a.wave_queries = 64;
            if (e != hipSuccess) return e;
        }
        // (it also clears the counters of the redo lists)
        const bool coll = p.mode == PLAN_MFMA_COLLECT;
        return launch_seed_finalize(gmax, nq, p.G, k, coll ? p.rank : k, seeds, certain, st,
                                    coll ? reinterpret_cast<int32_t *>(ws + p.off_qlist) + nq : nullptr, nullptr,
                                    coll && p.rounds ? reinterpret_cast<int32_t *>(ws + p.off_qlist2) + nq : nullptr,
                                    coll ? p.rounds : 0, nq + 1);
    };
    if (p.maxima) {
        int32_t *done = reinterpret_cast<int32_t *>(ws + p.off_over);
        {
            KernelSpan span(st);
            HIP_TRY(idx->d_pad > 256 ? launch_maxima_stream(a, p.groups, gmax, done, st) : launch_maxima_mfma(a, p.groups, gmax, done, st));
        }
        HIP_TRY(launch_maxima_finish(a, p.groups, gmax, p.finish_threads, p.helpers, p.most_helpers, lists2, reinterpret_cast<int32_t *>(ws + p.off_ccnt), done, ids, dist,
                                     qnorms, emit_mode, st));
    } else if (p.mode == PLAN_MFMA_COLLECT) {
        cand_t *cbuf = reinterpret_cast<cand_t *>(ws + p.off_cbuf);
        int32_t *ccnt = reinterpret_cast<int32_t *>(ws + p.off_ccnt);
        int32_t *over = reinterpret_cast<int32_t *>(ws + p.off_over);
        auto collect = [&](SearchArgs &args, const cand_t *bounds) -> hipError_t {
            if (p.stream) return launch_stream_collect(args, p.S2, bounds, cbuf, ccnt, p.Cs, st);
            args.wave_queries = p.wave_queries;
            const hipError_t e = launch_collect_mfma(args, 0, args.n, p.S2, bounds, cbuf, ccnt, p.Cs, st);
            args.wave_queries = 64;
            return e;
        };
        HIP_TRY(seed_pass());
        {
            KernelSpan span(st);
            HIP_TRY(collect(a, seeds));
        }
        int32_t *qlist = reinterpret_cast<int32_t *>(ws + p.off_qlist), *qcount = qlist + nq;
        cand_t *bounds2 = p.rounds ? reinterpret_cast<cand_t *>(ws + p.off_bounds2) : nullptr;
        HIP_TRY(launch_collect_select(cbuf, ccnt, nq, p.SS, p.Cs, k, over, qlist, qcount, ids, dist, qnorms, emit_mode, st,
                                      p.expect, nullptr, nullptr, 0, certain, bounds2));
        // Queries whose candidates did not fit are searched again, exactly.  Short lists on short rows: a few
        // by the generic kernel, many (a corpus full of duplicates or ties) by a pass of the register-list
        // kernel over the query tiles that hold one; both are launched and the count on the device decides.  The generic
        // kernel's launch also merges the other's lists (in a launch of their own 2 us more on every search).
        if (p.Sr) {
            cand_t *lists_r = reinterpret_cast<cand_t *>(ws + p.off_redo);
            SearchArgs ar = a;
            ar.rsplit = false;
            ar.wave_queries = 64;
            ar.redo_flags = over; ar.redo_count = qcount; ar.redo_min = REDO_GENERIC_MAX;
            HIP_TRY(launch_search_mfma(ar, 0, a.n, p.Sr, certain, lists_r, st));
            HIP_TRY(launch_search_generic_list(a, 0, a.n, p.Sg, {qlist, qcount, over}, REDO_GENERIC_MAX, {}, lists2, ids, dist,
                                               qnorms, emit_mode, st, lists_r, p.Sr));
        }
        // Otherwise the selection has also left a bound per flagged query, taken from what the scan did
        // collect for it, and the scan runs again over the query tiles that hold one, up to p.rounds times
        // (what a round collects is the FIRST candidates of each region in scan order, not the best, so one
        // round may still leave too many: each cuts the number that pass by about k / (candidates the regions
        // hold)).  What overflows even then goes through the generic kernel, and so does at once what is flagged first
        // where no more than p.few queries are: a round takes as long as the scan of the whole batch, however few
        // they are.  All of it returns at once when nothing is flagged, so the number of these launches is what a
        // search pays: scan and selection per round and one more (with the bounds and the merge in launches of their own and the generic kernel in
        // front, ten instead of five, 1000 queries on 500K x 768 took 15 us longer).
        const int32_t *over_prev = over, *count_prev = qcount;
        for (int r = 0; r < p.rounds; ++r) {
            int32_t *over_r = reinterpret_cast<int32_t *>(ws + p.off_over2) + (size_t)r * nq;
            int32_t *qlist_r = reinterpret_cast<int32_t *>(ws + p.off_qlist2) + (size_t)r * (nq + 1), *count_r = qlist_r + nq;
            SearchArgs ar = a;
            ar.redo_flags = over_prev; ar.redo_count = count_prev; ar.redo_min = r ? 0 : p.few;
            HIP_TRY(collect(ar, bounds2));
            const bool last = r + 1 == p.rounds;
            HIP_TRY(launch_collect_select(cbuf, ccnt, nq, p.SS, p.Cs, k, over_r, qlist_r, count_r, ids, dist, qnorms,
                                          emit_mode, st, 0, over_prev, count_prev, ar.redo_min, bounds2, last ? nullptr : bounds2));
            over_prev = over_r; count_prev = count_r;
            if (last)
                HIP_TRY(launch_search_generic_list(a, 0, a.n, p.Sg, {qlist, qcount, over}, p.few, {qlist_r, count_r, over_r}, lists2,
                                                   ids, dist, qnorms, emit_mode, st));
        }
    } else if (p.mode == PLAN_MFMA_REG) {
        const cand_t *sd = nullptr;
        if (p.seed_rows) {
            HIP_TRY(seed_pass());
            sd = seeds;
        }
        HIP_TRY(scan(0, a.n, p.S2, sd, lists2));
        HIP_TRY(final_merge(nullptr));
    } else if (p.seed_rows) {
        HIP_TRY(scan(0, p.seed_rows, p.S1, nullptr, lists1));
        HIP_TRY(launch_merge(lists1, nq, p.S1, k, nullptr, seedlist, seeds, nullptr, nullptr, nullptr, metric, st, sorted));
        HIP_TRY(scan(p.seed_rows, a.n, p.S2, seeds, lists2));
        HIP_TRY(final_merge(seedlist));
    } else {
        HIP_TRY(scan(0, a.n, p.S2, nullptr, lists2));
        HIP_TRY(final_merge(nullptr));
    }
    return LPQ_OK;
}

// A packed index is searched in tiles of at most 64 queries by the row-split kernel; the workspace
// holds all queries' codes, their permuted copy and per-query terms, then one tile's plan.
struct PackedPlan {
    int64_t nq_pad;
    size_t off_qcodes, off_qnorms, off_qperm, off_qadj, off_tile, total;
};
constexpr int64_t PACKED_TILE = 64;

PackedPlan make_packed_plan(const lpq_index *idx, int64_t nq, int k, bool compact = false)
{
    PackedPlan pp;
    const int64_t full = nq < PACKED_TILE ? nq : PACKED_TILE, last = nq % PACKED_TILE;
    const Plan a = make_plan(idx, full, k, compact);
    size_t tile = a.total;
    int64_t tail = a.nq_pad;
    if (last) {
        const Plan b = make_plan(idx, last, k, compact);
        if (b.total > tile) tile = b.total;
        if (b.nq_pad > tail) tail = b.nq_pad;
    }
    pp.nq_pad = ceil_div(nq, PACKED_TILE) * PACKED_TILE + tail;   // every tile may read a whole padded tile
    const Plan whole = make_plan(idx, nq, k, compact);
    if (whole.mode == PLAN_MFMA_COLLECT && !whole.rsplit) {   // large batch: one scan over all queries
        tile = whole.total;
        if (whole.nq_pad > pp.nq_pad) pp.nq_pad = whole.nq_pad;
    }
    size_t o = 0;
    pp.off_qcodes = o; o = align256(o + (size_t)pp.nq_pad * idx->d_pad);
    pp.off_qnorms = o; o = align256(o + (size_t)pp.nq_pad * sizeof(int32_t));
    pp.off_qperm = o;  o = align256(o + (size_t)pp.nq_pad * idx->d_pad);
    pp.off_qadj = o;   o = align256(o + (size_t)pp.nq_pad * sizeof(int32_t));
    pp.off_tile = o;   o = align256(o + tile);
    pp.total = o;
    return pp;
}

int search_packed(const lpq_index *idx, const PackedPlan &pp, char *ws, int64_t nq, int k, int metric, int32_t *ids,
                  int32_t *dist, hipStream_t st, bool compact = false)
{
    int8_t *qperm = reinterpret_cast<int8_t *>(ws + pp.off_qperm);
    int32_t *qadj = reinterpret_cast<int32_t *>(ws + pp.off_qadj);
    HIP_TRY(launch_permute_queries(reinterpret_cast<const int8_t *>(ws + pp.off_qcodes), pp.nq_pad, idx->d_pad,
                                   metric == LPQ_METRIC_L2SQ, qperm, qadj, st));
    const int emit = metric == LPQ_METRIC_L2SQ ? MODE_I8_L2 : MODE_I8_IP_ADJ;
    const Plan whole = make_plan(idx, nq, k, compact);
    if (whole.mode == PLAN_MFMA_COLLECT && !whole.rsplit)
        return search_core(idx, whole, ws + pp.off_tile, qperm, qadj, nq, k, metric, emit, ids, dist, st);
    for (int64_t q0 = 0; q0 < nq; q0 += PACKED_TILE) {
        const int64_t nt = nq - q0 < PACKED_TILE ? nq - q0 : PACKED_TILE;
        const Plan pt = make_plan(idx, nt, k, compact);
        int rc = search_core(idx, pt, ws + pp.off_tile, qperm + q0 * idx->d_pad, qadj + q0, nt, k, metric, emit,
                             ids + q0 * k, dist + q0 * k, st);
        if (rc) return rc;
    }
    return LPQ_OK;
}

}  // namespace

namespace {

// An index that is only described: no device memory behind it.
int describe_index(int d, int bits, int packed, int64_t n_items, int64_t nq, int k, lpq_index &shape)
{
    if (d < 1 || bits < 1 || bits > 8) return fail(LPQ_EINVAL, "d < 1 or bits outside 1..8");
    if (d > MAX_D) return fail(LPQ_ERANGE, "d = %d > %d", d, (int)MAX_D);
    if (packed && (bits > 4 || d > MAX_D_PACKED)) return fail(LPQ_EINVAL, "packed storage: at most 4 bits and %d features", (int)MAX_D_PACKED);
    if (n_items < 1 || n_items >= (int64_t(1) << 31) - 1024) return fail(LPQ_ERANGE, "n_items outside 1 .. 2^31 - 1025");
    if (nq < 0 || k < 1) return fail(LPQ_EINVAL, "nq < 0 or k < 1");
    if (k > MAX_K || k > n_items || (packed && k > MAX_K_PACKED)) return fail(LPQ_ERANGE, "k = %d out of range", k);
    shape.d = d; shape.bits = bits; shape.packed = packed != 0;
    shape.d_pad = padded_row_length(d);
    shape.capacity = shape.size = n_items;
    return LPQ_OK;
}

// Its plan; a packed index is searched in tiles of 64 queries unless one collecting scan takes the whole batch.
Plan plan_of_tile(const lpq_index &shape, int64_t nq, int k)
{
    const Plan p = make_plan(&shape, nq, k);
    if (!shape.packed || (p.mode == PLAN_MFMA_COLLECT && !p.rsplit)) return p;
    return make_plan(&shape, nq < PACKED_TILE ? nq : PACKED_TILE, k);
}

}  // namespace

extern "C" int lpq_search_plan_info(int d, int bits, int packed, int64_t n_items, int64_t nq, int k, int64_t *out,
                                    int out_count)
{
    if (!out || out_count < LPQ_PLAN_INFO_COUNT) return fail(LPQ_EINVAL, "out must hold LPQ_PLAN_INFO_COUNT values");
    lpq_index shape;
    if (int rc = describe_index(d, bits, packed, n_items, nq, k, shape)) return rc;
    const Plan p = plan_of_tile(shape, nq, k);
    size_t total = p.total, base = 0;
    int64_t nq_rows = p.nq_pad;
    if (shape.packed) {
        const PackedPlan pp = make_packed_plan(&shape, nq, k);
        total = pp.total;
        base = pp.off_tile;
        nq_rows = pp.nq_pad;
    }
    const int64_t v[LPQ_PLAN_INFO_COUNT] = {
        p.mode, p.rsplit ? 1 : 0, p.rs_waves, p.wave_queries, nq_rows, p.seed_rows, p.S1, p.S2, p.SEG, p.G, p.SS, p.Cs,
        p.Sg, p.Sr, p.rounds, p.merge_group, (int64_t)total, (int64_t)base,
        (int64_t)p.off_qcodes, (int64_t)p.off_qnorms, (int64_t)p.off_lists1, (int64_t)p.off_seedlist, (int64_t)p.off_seeds,
        (int64_t)p.off_lists2, (int64_t)p.off_gmax, (int64_t)p.off_merge_tmp, (int64_t)p.off_cbuf, (int64_t)p.off_ccnt,
        (int64_t)p.off_over, (int64_t)p.off_qlist, (int64_t)p.off_redo, (int64_t)p.off_bounds2, (int64_t)p.off_over2,
        (int64_t)p.off_qlist2, (int64_t)p.total};
    for (int i = 0; i < LPQ_PLAN_INFO_COUNT; ++i) out[i] = v[i];
    return LPQ_OK;
}

extern "C" int lpq_search_maxima_info(int d, int bits, int packed, int64_t n_items, int64_t nq, int k, int64_t *out,
                                      int out_count)
{
    if (!out || out_count < LPQ_MAXIMA_INFO_COUNT) return fail(LPQ_EINVAL, "out must hold LPQ_MAXIMA_INFO_COUNT values");
    lpq_index shape;
    if (int rc = describe_index(d, bits, packed, n_items, nq, k, shape)) return rc;
    const Plan p = plan_of_tile(shape, nq, k);
    const MaximaShape m = p.maxima ? p.groups : MaximaShape();
    const int64_t v[LPQ_MAXIMA_INFO_COUNT] = {m.G, m.S, m.SEG, m.parts / 2, m.stage_rows, p.finish_threads, p.helpers, p.most_helpers};
    for (int i = 0; i < LPQ_MAXIMA_INFO_COUNT; ++i) out[i] = v[i];
    return LPQ_OK;
}

extern "C" size_t lpq_search_workspace_bytes(const lpq_index *idx, int64_t nq, int k, int metric)
{
    if (!idx || nq < 0 || k < 1 || k > MAX_K || idx->size < 1 || k > idx->size) return 0;
    (void)metric;
    if (idx->packed) return k > MAX_K_PACKED ? 0 : make_packed_plan(idx, nq, k).total + 256;
    return make_plan(idx, nq, k).total + 256;
}

static int search_f32_queries(const lpq_index *idx, const float *q_dev, int64_t nq, int64_t ld, int k, int metric,
                              int32_t *ids_dev, int32_t *dist_dev, void *workspace_dev, size_t workspace_bytes,
                              hipStream_t st, bool compact = false)
{
    char *ws = (char *)workspace_dev;
    if ((uintptr_t)workspace_dev % 256) return fail(LPQ_EINVAL, "workspace must be 256-byte aligned");
    if (idx->packed) {
        const PackedPlan pp = make_packed_plan(idx, nq, k, compact);
        if (!workspace_dev || workspace_bytes < pp.total) return fail(LPQ_ERANGE, "workspace of %zu bytes needed", pp.total);
        HIP_TRY(launch_encode(view(idx->params, idx->d, idx->bits), q_dev, nq, ld,
                              reinterpret_cast<int8_t *>(ws + pp.off_qcodes), idx->d_pad, idx->d_pad,
                              reinterpret_cast<int32_t *>(ws + pp.off_qnorms), st, pp.nq_pad));
        return search_packed(idx, pp, ws, nq, k, metric, ids_dev, dist_dev, st, compact);
    }
    const Plan p = make_plan(idx, nq, k, compact);
    if (!workspace_dev || workspace_bytes < p.total) return fail(LPQ_ERANGE, "workspace of %zu bytes needed", p.total);
    // Padding query rows [nq, nq_pad) are written as zero codes; their results are never written out.
    HIP_TRY(launch_encode(view(idx->params, idx->d, idx->bits), q_dev, nq, ld,
                          reinterpret_cast<int8_t *>(ws + p.off_qcodes), idx->d_pad, idx->d_pad,
                          reinterpret_cast<int32_t *>(ws + p.off_qnorms), st, p.nq_pad));
    return search_core(idx, p, ws, reinterpret_cast<const int8_t *>(ws + p.off_qcodes),
                       reinterpret_cast<const int32_t *>(ws + p.off_qnorms), nq, k, metric, metric, ids_dev, dist_dev, st);
}

extern "C" int lpq_search(const lpq_index *idx, const float *q_dev, int64_t nq, int64_t ld, int k, int metric,
                          int32_t *ids_dev, int32_t *dist_dev, void *workspace_dev, size_t workspace_bytes,
                          void *stream)
{
    int rc = check_search_args(idx, q_dev, nq, ld, k, metric, ids_dev, dist_dev);
    if (rc) return rc;
    if (nq == 0) return LPQ_OK;
    return search_f32_queries(idx, q_dev, nq, ld, k, metric, ids_dev, dist_dev, workspace_dev, workspace_bytes,
                              (hipStream_t)stream);
}

// ---- search without any allocation: the workspace is a device array of the library ----
// One copy of the array exists on every GPU the library is loaded on, at that GPU's own address;
// in host code the array's name is only a handle for hipGetSymbolAddress, never an address.
static __device__ __align__(256) unsigned char scratch[LPQ_STATIC_WORKSPACE_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[MAX_DEVICES];   // device address of `scratch` on device i, once looked up

// Device address of `scratch` on the current device (looked up once per device, with that device current).
int scratch_address(void **out)
{
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= MAX_DEVICES) return fail(LPQ_EDEVICE, "device ordinal %d outside 0..%d", dev, MAX_DEVICES - 1);
    std::lock_guard<std::mutex> l(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(LPQ_EDEVICE, "hipGetSymbolAddress returned a null address");
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return LPQ_OK;
}
}  // namespace

extern "C" int lpq_search_static(const lpq_index *idx, const float *q_dev, int64_t nq, int64_t ld, int k, int metric,
                                 int32_t *ids_dev, int32_t *dist_dev, void *stream)
{
    int rc = check_search_args(idx, q_dev, nq, ld, k, metric, ids_dev, dist_dev);
    if (rc) return rc;
    if (nq == 0) return LPQ_OK;
    const size_t limit = (size_t)LPQ_STATIC_WORKSPACE_BYTES;
    bool compact = false;
    auto bytes = [&](int64_t queries) {
        return idx->packed ? make_packed_plan(idx, queries, k, compact).total : make_plan(idx, queries, k, compact).total;
    };
    size_t need = bytes(nq);
    if (need > limit) {
        compact = true;
        need = bytes(nq);
    }
    // Rows beyond 1536 features are padded for the streaming scan, which the compact plan does not take; where only that
    // padding of the queries' codes is too much, half of them are searched at a time.
    int64_t part = nq;
    const size_t padding = idx->d_pad > 1536 ? (size_t)round_up(nq, 512) * (idx->d_pad - round_up(idx->d, 32)) : 0;
    if (need > limit && need - padding <= limit) {
        part = round_up(ceil_div(nq, 2), 512);
        need = bytes(part < nq ? part : nq);
    }
    if (need > limit)
        return fail(LPQ_ERANGE, "this search needs %zu bytes of workspace, the built-in one holds %zu: use lpq_search", need, limit);
    void *ws = nullptr;
    rc = scratch_address(&ws);
    if (rc) return rc;
    for (int64_t q0 = 0; q0 < nq; q0 += part) {
        const int64_t take = nq - q0 < part ? nq - q0 : part;
        rc = search_f32_queries(idx, q_dev + q0 * ld, take, ld, k, metric, ids_dev + q0 * k, dist_dev + q0 * k, ws, limit,
                                (hipStream_t)stream, compact);
        if (rc) return rc;
    }
    return LPQ_OK;
}

extern "C" int lpq_search_overflow_stats(const lpq_index *idx, int64_t nq, int k, int metric, const void *workspace_dev,
                                         int64_t *redone_queries, int64_t *max_region_fill)
{
    (void)metric;
    if (!idx || !workspace_dev || !redone_queries || !max_region_fill || nq < 1 || k < 1) return fail(LPQ_EINVAL, "bad argument");
    *redone_queries = 0;
    *max_region_fill = 0;
    const Plan p = make_plan(idx, nq, k);
    if (p.mode != PLAN_MFMA_COLLECT && !p.maxima) return LPQ_OK;
    HIP_TRY(hipDeviceSynchronize());
    std::vector<int32_t> over((size_t)nq), cnt((size_t)nq * (p.maxima ? p.most_helpers : p.SS));
    const char *ws = static_cast<const char *>(workspace_dev) + (idx->packed ? make_packed_plan(idx, nq, k).off_tile : 0);
    HIP_TRY(hipMemcpy(over.data(), ws + p.off_over, over.size() * sizeof(int32_t), hipMemcpyDeviceToHost));
    HIP_TRY(hipMemcpy(cnt.data(), ws + p.off_ccnt, cnt.size() * sizeof(int32_t), hipMemcpyDeviceToHost));
    if (p.maxima) {   // none is searched again, those that many groups tie for take longer; a query's first workgroup has always worked
        for (int32_t &v : over) v &= MAXIMA_MANY;
        for (size_t i = 0; i < cnt.size(); ++i)
            if (i % p.most_helpers) cnt[i] = 0;
    }
    for (int32_t v : over) *redone_queries += v != 0;
    for (int32_t v : cnt) if (v > *max_region_fill) *max_region_fill = v;
    return LPQ_OK;
}

extern "C" int lpq_search_overflow_left(const lpq_index *idx, int64_t nq, int k, int metric, const void *workspace_dev,
                                        int64_t *left_queries)
{
    (void)metric;
    if (!idx || !workspace_dev || !left_queries || nq < 1 || k < 1) return fail(LPQ_EINVAL, "bad argument");
    *left_queries = 0;
    const Plan p = make_plan(idx, nq, k);
    if (p.mode != PLAN_MFMA_COLLECT || p.maxima || !p.rounds) return LPQ_OK;
    HIP_TRY(hipDeviceSynchronize());
    std::vector<int32_t> over2((size_t)nq);
    const char *ws = static_cast<const char *>(workspace_dev) + (idx->packed ? make_packed_plan(idx, nq, k).off_tile : 0);
    HIP_TRY(hipMemcpy(over2.data(), ws + p.off_over2 + (size_t)(p.rounds - 1) * nq * sizeof(int32_t),
                      over2.size() * sizeof(int32_t), hipMemcpyDeviceToHost));
    for (int32_t v : over2) *left_queries += v != 0;
    return LPQ_OK;
}

extern "C" int lpq_search_i8(const lpq_index *idx, const int8_t *qcodes_dev, int64_t nq, int64_t ld, int k,
                             int metric, int32_t *ids_dev, int32_t *dist_dev, void *workspace_dev,
                             size_t workspace_bytes, void *stream)
{
    int rc = check_search_args(idx, qcodes_dev, nq, ld, k, metric, ids_dev, dist_dev);
    if (rc) return rc;
    if (nq == 0) return LPQ_OK;
    hipStream_t st = (hipStream_t)stream;
    char *ws = (char *)workspace_dev;
    if ((uintptr_t)workspace_dev % 256) return fail(LPQ_EINVAL, "workspace must be 256-byte aligned");
    if (idx->packed) {
        const PackedPlan pp = make_packed_plan(idx, nq, k);
        if (!workspace_dev || workspace_bytes < pp.total) return fail(LPQ_ERANGE, "workspace of %zu bytes needed", pp.total);
        HIP_TRY(launch_repack_i8(qcodes_dev, nq, ld, idx->d, reinterpret_cast<int8_t *>(ws + pp.off_qcodes), idx->d_pad,
                                 idx->d_pad, reinterpret_cast<int32_t *>(ws + pp.off_qnorms), st, pp.nq_pad));
        return search_packed(idx, pp, ws, nq, k, metric, ids_dev, dist_dev, st);
    }
    const Plan p = make_plan(idx, nq, k);
    if (!workspace_dev || workspace_bytes < p.total) return fail(LPQ_ERANGE, "workspace of %zu bytes needed", p.total);
    HIP_TRY(launch_repack_i8(qcodes_dev, nq, ld, idx->d, reinterpret_cast<int8_t *>(ws + p.off_qcodes), idx->d_pad,
                             idx->d_pad, reinterpret_cast<int32_t *>(ws + p.off_qnorms), st, p.nq_pad));
    return search_core(idx, p, ws, reinterpret_cast<const int8_t *>(ws + p.off_qcodes),
                       reinterpret_cast<const int32_t *>(ws + p.off_qnorms), nq, k, metric, metric, ids_dev, dist_dev, st);
}

// -------------------------------------------------------------------- fp32 exact ----
extern "C" size_t lpq_search_f32_workspace_bytes(int64_t n, int64_t nq, int d, int k)
{
    if (n < 1 || nq < 0 || d < 1 || k < 1 || k > MAX_K || k > n || d > f32_max_d(k)) return 0;
    return f32_workspace_bytes(n, nq, d, k) + 256;
}

extern "C" int lpq_search_f32(const float *x_dev, int64_t n, int64_t ldx, const float *q_dev, int64_t nq,
                              int64_t ldq, int d, int k, int metric, int32_t *ids_dev, float *dist_dev,
                              void *workspace_dev, size_t workspace_bytes, void *stream)
{
    if (d < 1) return fail(LPQ_EINVAL, "d < 1");
    if (n < 1) return fail(LPQ_ESTATE, "no items");
    if (nq < 0) return fail(LPQ_EINVAL, "nq < 0");
    if (k < 1) return fail(LPQ_EINVAL, "k < 1");
    if (metric != LPQ_METRIC_L2SQ && metric != LPQ_METRIC_IP) return fail(LPQ_EINVAL, "unknown metric %d", metric);
    if (k > n || k > MAX_K) return fail(LPQ_ERANGE, "k = %d out of range", k);
    if (n >= (int64_t(1) << 31) - 1024) return fail(LPQ_ERANGE, "n must stay below 2^31 - 1024");
    if (d > f32_max_d(k))
        return fail(LPQ_ERANGE, "d = %d: the fp32 search takes at most %d features for k = %d", d, f32_max_d(k), k);
    if (nq == 0) return LPQ_OK;
    if (!x_dev || !q_dev || !ids_dev || !dist_dev) return fail(LPQ_EINVAL, "null argument");
    if (ldx < d || ldq < d) return fail(LPQ_EINVAL, "row stride smaller than d");
    const size_t need = f32_workspace_bytes(n, nq, d, k);
    if (!workspace_dev || workspace_bytes < need) return fail(LPQ_ERANGE, "workspace of %zu bytes needed", need);
    if ((uintptr_t)workspace_dev % 256) return fail(LPQ_EINVAL, "workspace must be 256-byte aligned");
    HIP_TRY(launch_search_f32(x_dev, n, ldx, q_dev, nq, ldq, d, k, metric, ids_dev, dist_dev, workspace_dev,
                              (hipStream_t)stream));
    return LPQ_OK;
}
