// C ABI of the RSR Stage-2 library (declared in include/rsr.h): argument
// validation, handle construction (threshold computation, reference-row
// packing, graph upload), workspace management and kernel launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <memory>
#include <new>
#include <string>
#include <vector>

#include "rsr_internal.h"

using rsr::plane_words;
using rsr::sample_words;

namespace rsr {

// Allocations left before the injected failure (rsr_debug_fail_alloc); < 0:
// none armed.
static int64_t g_fail_countdown = -1;

static bool injected_failure() {
    if (g_fail_countdown < 0) return false;
    if (g_fail_countdown == 0) {
        g_fail_countdown = -1;
        return true;
    }
    --g_fail_countdown;
    return false;
}

hipError_t dev_malloc(void** p, size_t bytes) {
    if (injected_failure()) {
        *p = nullptr;
        return hipErrorOutOfMemory;
    }
    return hipMalloc(p, bytes);
}

hipError_t host_malloc(void** p, size_t bytes) {
    if (injected_failure()) {
        *p = nullptr;
        return hipErrorOutOfMemory;
    }
    return hipHostMalloc(p, bytes, hipHostMallocDefault);
}

rsr_status ensure_list(rsr_ctx* ctx, int64_t N) {
    if (ctx->ws.list_cap >= N) return RSR_OK;
    if (ctx->ws.list) {
        hipError_t e = hipFree(ctx->ws.list);
        ctx->ws.list = nullptr;
        ctx->ws.list_cap = 0;
        if (e != hipSuccess) return hip_error(ctx, e, "hipFree(unknown list)");
    }
    hipError_t e = dev_malloc(&ctx->ws.list, SampleList::bytes(N));
    if (e != hipSuccess) return hip_error(ctx, e, "unknown-sample list");
    ctx->ws.list_cap = N;
    return RSR_OK;
}

}  // namespace rsr

namespace {

struct DeviceGuard {
    int prev = -1;
    bool changed = false;
    explicit DeviceGuard(int dev) {
        if (hipGetDevice(&prev) == hipSuccess && prev != dev) {
            changed = hipSetDevice(dev) == hipSuccess;
        }
    }
    ~DeviceGuard() {
        if (changed) (void)hipSetDevice(prev);
    }
};

rsr_status fail(rsr_ctx* ctx, rsr_status st, const std::string& msg) {
    if (ctx) ctx->err = msg;
    return st;
}

rsr_status hip_fail(rsr_ctx* ctx, hipError_t e, const char* what) {
    std::string m = std::string(what) + ": " + hipGetErrorName(e) + " (" + hipGetErrorString(e) + ")";
    return fail(ctx, e == hipErrorOutOfMemory ? RSR_ENOMEM : RSR_EHIP, m);
}

#define RSR_HIP(ctx, call)                                  \
    do {                                                    \
        hipError_t e_ = (call);                             \
        if (e_ != hipSuccess) return hip_fail(ctx, e_, #call); \
    } while (0)

rsr_status validate_probs(rsr_ctx* ctx, int32_t n, int32_t K, const double* p) {
    if (n <= 0 || K < 2) return fail(ctx, RSR_EINVAL, "n must be > 0 and K >= 2");
    if (K > RSR_MAX_K) return fail(ctx, RSR_EUNSUPPORTED, "K exceeds RSR_MAX_K");
    if (static_cast<int64_t>(n) * (K - 1) > RSR_MAX_BITS)
        return fail(ctx, RSR_EUNSUPPORTED, "n*(K-1) exceeds RSR_MAX_BITS");
    if (!p) return fail(ctx, RSR_EINVAL, "p is NULL");
    for (int32_t i = 0; i < n; ++i) {
        double sum = 0.0;
        for (int32_t s = 0; s < K; ++s) {
            const double v = p[static_cast<size_t>(i) * K + s];
            if (!std::isfinite(v) || v < 0.0 || v > 1.0)
                return fail(ctx, RSR_EINVAL,
                            "p[" + std::to_string(i) + "][" + std::to_string(s) + "] not in [0,1]");
            sum += v;
        }
        if (std::fabs(sum - 1.0) > 1e-9)
            return fail(ctx, RSR_EINVAL, "row " + std::to_string(i) + " of p does not sum to 1");
    }
    return RSR_OK;
}

// Inverse-CDF thresholds: C[i][s-1] = min(floor(2^32 * cumulative), 2^32),
// with the cumulative probability summed left to right in fp64.
void compute_thresholds(int32_t n, int32_t K, const double* p, uint64_t* C) {
    const double two32 = 4294967296.0;
    for (int32_t i = 0; i < n; ++i) {
        double cum = 0.0;
        for (int32_t s = 1; s < K; ++s) {
            cum = cum + p[static_cast<size_t>(i) * K + (s - 1)];
            const double f = std::floor(cum * two32);
            uint64_t c = 0;
            if (f >= two32)
                c = 4294967296ull;
            else if (f > 0.0)
                c = static_cast<uint64_t>(f);
            C[static_cast<size_t>(i) * (K - 1) + (s - 1)] = c;
        }
    }
}


// A reference set is consistent when no upper row lies below a lower row:
// then no sample can be dominated on both sides and the LABEL cascade may stop
// at the first match.  Checked once on the device with the classification
// kernels themselves (upper rows as samples against the lower rows): the FP4
// form when the handle has matrix-core operands (0.72 against 7.15 ms for the
// popcount form at 2.5e4 rows of 590 bits per side; its 2.5e4 samples fill a
// fifth of the CUs), else the popcount form.  Synchronous.  Callers that know the
// rows to be consistent skip it.
rsr_status check_consistency(rsr_ctx* ctx, rsr_refs* refs, const std::vector<uint32_t>& up) {
    refs->consistent = true;
    if (refs->R_L == 0 || refs->R_U == 0) return RSR_OK;
    const int64_t RU = refs->R_U;
    const int W = refs->W, WR = refs->WR;
    std::vector<uint32_t> cols(static_cast<size_t>(W) * RU);
    for (int64_t r = 0; r < RU; ++r)
        for (int w = 0; w < W; ++w) cols[static_cast<size_t>(w) * RU + r] = up[r * WR + w];
    uint32_t* d_cols = nullptr;
    uint8_t* d_flags = nullptr;
    hipError_t e = rsr::dev_malloc(&d_cols, sizeof(uint32_t) * cols.size());
    if (e == hipSuccess) e = rsr::dev_malloc(&d_flags, static_cast<size_t>(RU));
    if (e == hipSuccess)
        e = hipMemcpyAsync(d_cols, cols.data(), sizeof(uint32_t) * cols.size(),
                           hipMemcpyHostToDevice, ctx->stream);
    if (e == hipSuccess) {
        rsr_refs lower_only = *refs;
        lower_only.R_U = 0;
        lower_only.TU = 0;
        lower_only.d_upper_bits = nullptr;
        lower_only.d_upper_frag = nullptr;
        lower_only.d_upper_frag4 = nullptr;
        lower_only.d_upper_frag32 = nullptr;
        lower_only.d_upper_cinit = nullptr;
        lower_only.d_upper_cinit4 = nullptr;
        e = refs->KS > 0 ? rsr::launch_dom_mfma(ctx->stream, &lower_only, d_cols, RU, RSR_LABEL, true,
                                                ctx->cu_count, d_flags, nullptr)
                         : rsr::launch_dom_bits(ctx->stream, &lower_only, d_cols, RU, RSR_LABEL,
                                                d_flags, nullptr);
    }
    std::vector<uint8_t> fl(static_cast<size_t>(RU));
    if (e == hipSuccess)
        e = hipMemcpyAsync(fl.data(), d_flags, fl.size(), hipMemcpyDeviceToHost, ctx->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(ctx->stream);
    if (d_cols) (void)hipFree(d_cols);
    if (d_flags) (void)hipFree(d_flags);
    if (e != hipSuccess) return hip_fail(ctx, e, "reference consistency check");
    for (uint8_t f : fl)
        if (f & 1u) {
            refs->consistent = false;
            break;
        }
    return RSR_OK;
}

// Byte offsets of a model's device arrays in its single allocation (and in
// its pinned staging buffer): thresholds u64 [n][K-1], probabilities f64
// [n][K], sampler thresholds u32 [PW][K-1][kPackWords], probabilities f32
// [n][K].  Every offset is a multiple of 8.
struct ModelLayout {
    size_t thresh, p64, pack, p32, total;
    ModelLayout(int n, int K) {
        const size_t nn = static_cast<size_t>(n), k1 = static_cast<size_t>(K - 1);
        thresh = 0;
        p64 = thresh + sizeof(uint64_t) * nn * k1;
        pack = p64 + sizeof(double) * nn * K;
        p32 = pack + sizeof(uint32_t) * plane_words(n) * k1 * rsr::kPackWords;
        total = p32 + sizeof(float) * nn * K;
    }
};

// The host images of a model's arrays (p already validated).  Padding
// components of the sampler form never set a bit.
void fill_model_stage(const ModelLayout& L, int n, int K, const double* p, void* stage) {
    char* base = static_cast<char*>(stage);
    uint64_t* C = reinterpret_cast<uint64_t*>(base + L.thresh);
    compute_thresholds(n, K, p, C);
    std::memcpy(base + L.p64, p, sizeof(double) * static_cast<size_t>(n) * K);
    uint32_t* pack = reinterpret_cast<uint32_t*>(base + L.pack);
    for (int wi = 0; wi < plane_words(n); ++wi)
        for (int s = 0; s < K - 1; ++s) {
            uint32_t* pw = pack + (static_cast<size_t>(wi) * (K - 1) + s) * rsr::kPackWords;
            std::fill(pw, pw + rsr::kPackWords, 0u);
            for (int k = 0; k < 32; ++k) {
                const int i = 32 * wi + k;
                const rsr::PackedThreshold t = rsr::pack_threshold(
                    i < n ? C[static_cast<size_t>(i) * (K - 1) + s] : uint64_t{1} << 32);
                pw[k / 2] |= static_cast<uint32_t>(t.s) << (16 * (k % 2));
                if (t.always) pw[16] |= 1u << k;
                if (t.low) pw[17] |= 1u << k;
            }
        }
    float* pf = reinterpret_cast<float*>(base + L.p32);
    for (size_t i = 0; i < static_cast<size_t>(n) * K; ++i) pf[i] = static_cast<float>(p[i]);
}

rsr_status ensure_cascade(rsr_ctx* ctx, int W, int64_t N, int64_t state_words = 0) {
    const int64_t words = 2 * static_cast<int64_t>(W) * N, idx = 4 * N;
    if (ctx->ws.casc_state_cap < state_words) {
        if (ctx->ws.casc_state) RSR_HIP(ctx, hipFree(ctx->ws.casc_state));
        ctx->ws.casc_state = nullptr;
        ctx->ws.casc_state_cap = 0;
        // Rounded to whole u64 (the state is cleared 8 bytes at a time).
        const int64_t cap = (state_words + 1) / 2 * 2;
        RSR_HIP(ctx, rsr::dev_malloc(&ctx->ws.casc_state, sizeof(uint32_t) * static_cast<size_t>(cap)));
        ctx->ws.casc_state_cap = cap;
    }
    if (ctx->ws.casc_words_cap < words) {
        if (ctx->ws.casc_words) RSR_HIP(ctx, hipFree(ctx->ws.casc_words));
        ctx->ws.casc_words = nullptr;
        ctx->ws.casc_words_cap = 0;
        RSR_HIP(ctx, rsr::dev_malloc(&ctx->ws.casc_words, sizeof(uint32_t) * static_cast<size_t>(words)));
        ctx->ws.casc_words_cap = words;
    }
    if (ctx->ws.casc_index_cap < idx) {
        if (ctx->ws.casc_index) RSR_HIP(ctx, hipFree(ctx->ws.casc_index));
        ctx->ws.casc_index = nullptr;
        ctx->ws.casc_index_cap = 0;
        RSR_HIP(ctx, rsr::dev_malloc(&ctx->ws.casc_index, sizeof(int32_t) * static_cast<size_t>(idx)));
        ctx->ws.casc_index_cap = idx;
    }
    return RSR_OK;
}

}  // namespace

extern "C" {

const char* rsr_status_str(rsr_status s) {
    switch (s) {
        case RSR_OK: return "RSR_OK";
        case RSR_EINVAL: return "RSR_EINVAL";
        case RSR_ENOMEM: return "RSR_ENOMEM";
        case RSR_EHIP: return "RSR_EHIP";
        case RSR_EUNSUPPORTED: return "RSR_EUNSUPPORTED";
    }
    return "unknown status";
}

const char* rsr_last_error(const rsr_ctx* ctx) { return ctx ? ctx->err.c_str() : "NULL context"; }

size_t rsr_words(int32_t n, int32_t K) {
    if (n <= 0 || K < 2) return 0;
    return static_cast<size_t>(sample_words(n, K));
}

rsr_status rsr_thresholds(int32_t n, int32_t K, const double* p, uint64_t* C) {
    rsr_status st = validate_probs(nullptr, n, K, p);
    if (st != RSR_OK) return st;
    if (!C) return RSR_EINVAL;
    compute_thresholds(n, K, p, C);
    return RSR_OK;
}

rsr_status rsr_ctx_create(int device, void* hip_stream, rsr_ctx** out) {
    if (!out) return RSR_EINVAL;
    *out = nullptr;
    int count = 0;
    if (hipGetDeviceCount(&count) != hipSuccess || count <= 0) return RSR_EHIP;
    if (device < 0 || device >= count) return RSR_EINVAL;
    rsr_ctx* ctx = new (std::nothrow) rsr_ctx();
    if (!ctx) return RSR_ENOMEM;
    ctx->device = device;
    ctx->stream = static_cast<hipStream_t>(hip_stream);
    DeviceGuard g(device);
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, device) != hipSuccess) {
        delete ctx;
        return RSR_EHIP;
    }
    ctx->cu_count = prop.multiProcessorCount;
    ctx->arch = prop.gcnArchName;
    rsr_status st = RSR_OK;
    if (rsr::dev_malloc(&ctx->ws.counters, sizeof(uint64_t) * 16) != hipSuccess ||
        rsr::dev_malloc(&ctx->ws.casc_counters,
                        sizeof(uint64_t) * rsr::CascadeBuffers::kCounterU64) != hipSuccess ||
        rsr::dev_malloc(&ctx->ws.count_part, sizeof(uint64_t) * rsr::kMaxReduceBlocks * 8) != hipSuccess ||
        rsr::dev_malloc(&ctx->ws.grad_part, sizeof(uint32_t) *
                                                (static_cast<size_t>(rsr::kMaxPaddedBits) + 1) *
                                                rsr::kMaxGradBlocks) != hipSuccess ||
        rsr::host_malloc(&ctx->ws.host_counts, sizeof(uint64_t) * 16) != hipSuccess)
        st = RSR_ENOMEM;
    if (st == RSR_OK && hipHostGetDevicePointer(reinterpret_cast<void**>(&ctx->ws.host_counts_dev),
                                                ctx->ws.host_counts, 0) != hipSuccess)
        st = RSR_EHIP;
    if (st == RSR_OK && rsr::noalloc_scratch(device, &ctx->noalloc_scratch) != hipSuccess)
        st = RSR_EHIP;
    // counters[15] is the ticket of the one-launch counts kernel, which
    // expects it at zero and leaves it there.
    if (st == RSR_OK && hipMemset(ctx->ws.counters, 0, sizeof(uint64_t) * 16) != hipSuccess)
        st = RSR_EHIP;
    if (st != RSR_OK) {
        rsr_ctx_destroy(ctx);
        return st;
    }
    *out = ctx;
    return RSR_OK;
}

rsr_status rsr_ctx_destroy(rsr_ctx* ctx) {
    if (!ctx) return RSR_EINVAL;
    DeviceGuard g(ctx->device);
    if (ctx->stream) (void)hipStreamSynchronize(ctx->stream);
    else (void)hipDeviceSynchronize();
    if (ctx->ws.counters) (void)hipFree(ctx->ws.counters);
    if (ctx->ws.casc_counters) (void)hipFree(ctx->ws.casc_counters);
    if (ctx->ws.casc_words) (void)hipFree(ctx->ws.casc_words);
    if (ctx->ws.casc_index) (void)hipFree(ctx->ws.casc_index);
    if (ctx->ws.casc_state) (void)hipFree(ctx->ws.casc_state);
    if (ctx->ws.list) (void)hipFree(ctx->ws.list);
    if (ctx->ws.count_part) (void)hipFree(ctx->ws.count_part);
    if (ctx->ws.grad_part) (void)hipFree(ctx->ws.grad_part);
    if (ctx->ws.host_counts) (void)hipHostFree(ctx->ws.host_counts);
    const rsr::CallbackStage& cb = ctx->ws.cb;
    if (cb.d_words) (void)hipFree(cb.d_words);
    if (cb.d_bytes) (void)hipFree(cb.d_bytes);
    if (cb.h_words) (void)hipHostFree(cb.h_words);
    if (cb.h_bytes) (void)hipHostFree(cb.h_bytes);
    if (cb.h_index) (void)hipHostFree(cb.h_index);
    delete ctx;
    return RSR_OK;
}

// ---- handles ---------------------------------------------------------------

rsr_status rsr_model_create(rsr_ctx* ctx, int32_t n, int32_t K, const double* p,
                            rsr_model** out) {
    if (!ctx || !out) return RSR_EINVAL;
    *out = nullptr;
    rsr_status st = validate_probs(ctx, n, K, p);
    if (st != RSR_OK) return st;
    DeviceGuard g(ctx->device);
    rsr_model* m = new (std::nothrow) rsr_model();
    if (!m) return fail(ctx, RSR_ENOMEM, "host allocation");
    m->ctx = ctx;
    m->n = n;
    m->K = K;
    const ModelLayout L(n, K);
    m->mem_bytes = L.total;
    hipError_t e = rsr::dev_malloc(&m->d_mem, L.total);
    if (e == hipSuccess) e = rsr::host_malloc(&m->h_stage, L.total);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&m->staged, hipEventDisableTiming);
    if (e != hipSuccess) {
        rsr_model_destroy(m);
        return hip_fail(ctx, e, "rsr_model_create allocation");
    }
    char* base = static_cast<char*>(m->d_mem);
    m->d_thresh = reinterpret_cast<uint64_t*>(base + L.thresh);
    m->d_p64 = reinterpret_cast<double*>(base + L.p64);
    m->d_pack = reinterpret_cast<uint32_t*>(base + L.pack);
    m->d_p = reinterpret_cast<float*>(base + L.p32);
    fill_model_stage(L, n, K, p, m->h_stage);
    e = hipMemcpyAsync(m->d_mem, m->h_stage, L.total, hipMemcpyHostToDevice, ctx->stream);
    if (e == hipSuccess) e = hipEventRecord(m->staged, ctx->stream);
    if (e == hipSuccess) e = hipEventSynchronize(m->staged);
    if (e != hipSuccess) {
        rsr_model_destroy(m);
        return hip_fail(ctx, e, "rsr_model_create upload");
    }
    *out = m;
    return RSR_OK;
}

rsr_status rsr_model_update(rsr_model* m, const double* p) {
    if (!m) return RSR_EINVAL;
    rsr_ctx* ctx = m->ctx;
    rsr_status st = validate_probs(ctx, m->n, m->K, p);
    if (st != RSR_OK) return st;
    DeviceGuard g(ctx->device);
    // The previous upload must have left the staging buffer before it is
    // overwritten (normally long done: any synchronising call since then
    // has waited for it).
    RSR_HIP(ctx, hipEventSynchronize(m->staged));
    fill_model_stage(ModelLayout(m->n, m->K), m->n, m->K, p, m->h_stage);
    RSR_HIP(ctx, hipMemcpyAsync(m->d_mem, m->h_stage, m->mem_bytes, hipMemcpyHostToDevice,
                                ctx->stream));
    RSR_HIP(ctx, hipEventRecord(m->staged, ctx->stream));
    return RSR_OK;
}

rsr_status rsr_model_destroy(rsr_model* m) {
    if (!m) return RSR_EINVAL;
    DeviceGuard g(m->ctx->device);
    if (m->staged) {
        (void)hipEventSynchronize(m->staged);
        (void)hipEventDestroy(m->staged);
    }
    if (m->d_mem) (void)hipFree(m->d_mem);
    if (m->h_stage) (void)hipHostFree(m->h_stage);
    delete m;
    return RSR_OK;
}

}  // extern "C"

namespace rsr {

void pack_rows(int n, int K, const uint8_t* rows, int64_t R, bool complement,
               std::vector<uint32_t>& bits) {
    constexpr uint64_t kOnes = 0x0101010101010101ull, kTop = 0x8080808080808080ull;
    const int PW = plane_words(n), W = sample_words(n, K), WR = dom_row_words(W);
    const size_t at = bits.size();
    bits.resize(at + static_cast<size_t>(R) * WR, 0u);
    for (int64_t r = 0; r < R; ++r) {
        const uint8_t* row = rows + r * n;
        uint32_t* dst = bits.data() + at + r * WR;
        // Eight components at a time: adding 128 - j to a byte sets its top
        // bit when the state is at least j (states are below 128), and a
        // product gathers the eight top bits.
        for (int i = 0; i < n; i += 8) {
            uint64_t x = 0;
            std::memcpy(&x, row + i, static_cast<size_t>(std::min(8, n - i)));
            for (int j = 1; j < K; ++j) {
                const uint64_t ge = ((x + kOnes * static_cast<uint64_t>(128 - j)) & kTop) >> 7;
                dst[(j - 1) * PW + i / 32] |=
                    static_cast<uint32_t>((ge * 0x0102040810204080ull) >> 56) << (i % 32);
            }
        }
        if (complement)  // within the planes' valid bits
            for (int w = 0; w < W; ++w) {
                const int valid = n - 32 * (w % PW);
                dst[w] = ~dst[w] & (valid >= 32 ? ~0u : (1u << valid) - 1u);
            }
    }
}

rsr_status pack_refs(rsr_ctx* ctx, int32_t n, int32_t K, const uint8_t* lower, int64_t R_L,
                     const uint8_t* upper, int64_t R_U, std::vector<uint32_t>& lo,
                     std::vector<uint32_t>& up) {
    if (n <= 0 || K < 2) return fail(ctx, RSR_EINVAL, "n must be > 0 and K >= 2");
    if (K > RSR_MAX_K || static_cast<int64_t>(n) * (K - 1) > RSR_MAX_BITS)
        return fail(ctx, RSR_EUNSUPPORTED, "n*(K-1) exceeds RSR_MAX_BITS or K > RSR_MAX_K");
    if (R_L < 0 || R_U < 0) return fail(ctx, RSR_EINVAL, "negative row count");
    if ((R_L > 0 && !lower) || (R_U > 0 && !upper))
        return fail(ctx, RSR_EINVAL, "NULL reference rows with a non-zero count");
    // Whether every state is below K, eight at a time.
    auto states_ok = [K](const uint8_t* v, int64_t count) {
        constexpr uint64_t kOnes = 0x0101010101010101ull, kTop = 0x8080808080808080ull;
        uint64_t bad = 0;
        int64_t i = 0;
        for (; i + 8 <= count; i += 8) {
            uint64_t x;
            std::memcpy(&x, v + i, 8);
            bad |= x | ((x & ~kTop) + kOnes * static_cast<uint64_t>(128 - K));
        }
        for (; i < count; ++i) bad |= v[i] >= K ? kTop : 0;
        return (bad & kTop) == 0;
    };
    if (!states_ok(lower, R_L * n)) return fail(ctx, RSR_EINVAL, "lower reference state >= K");
    if (!states_ok(upper, R_U * n)) return fail(ctx, RSR_EINVAL, "upper reference state >= K");
    if (dom_row_words(sample_words(n, K)) < 0)
        return fail(ctx, RSR_EUNSUPPORTED, "packed width not supported");
    pack_rows(n, K, lower, R_L, true, lo);
    pack_rows(n, K, upper, R_U, false, up);
    return RSR_OK;
}

static rsr_status build_refs(rsr_ctx* ctx, int32_t n, int32_t K, std::vector<uint32_t> lo,
                             std::vector<uint32_t> up, bool matrix_operands, bool consistent,
                             rsr_refs** out) {
    const int PW = plane_words(n);
    const int W = sample_words(n, K);
    const int WR = rsr::dom_row_words(W);
    const int64_t R_L = static_cast<int64_t>(lo.size() / WR);
    const int64_t R_U = static_cast<int64_t>(up.size() / WR);
    DeviceGuard g(ctx->device);
    // Store rows by increasing number of violation bits (stable): a row with
    // fewer constrained components dominates a larger region, so the LABEL
    // forms find most matches among the first rows.  Results do not depend
    // on the order.
    auto sort_rows = [&](std::vector<uint32_t>& rows, int64_t R, std::vector<int>& weight) {
        std::vector<int> of(R);
        std::vector<int64_t> next(static_cast<size_t>(W) * 32 + 2, 0);
        for (int64_t r = 0; r < R; ++r) {
            int c = 0;
            for (int w = 0; w < W; ++w) c += __builtin_popcount(rows[r * WR + w]);
            of[r] = c;
            next[c + 1] += 1;
        }
        for (size_t c = 1; c < next.size(); ++c) next[c] += next[c - 1];
        std::vector<uint32_t> sorted(rows.size());
        weight.resize(R);
        for (int64_t r = 0; r < R; ++r) {
            const int64_t to = next[of[r]]++;
            std::copy(rows.begin() + r * WR, rows.begin() + (r + 1) * WR, sorted.begin() + to * WR);
            weight[to] = of[r];
        }
        rows.swap(sorted);
    };
    std::vector<int> lo_weight, up_weight;
    sort_rows(lo, R_L, lo_weight);
    sort_rows(up, R_U, up_weight);
    // f(k) for every set bit k of a packed row.
    auto for_bits = [&](const uint32_t* row, auto f) {
        for (int w = 0; w < W; ++w)
            for (uint32_t m = row[w]; m; m &= m - 1) f(32 * w + __builtin_ctz(m));
    };

    // Matrix-core operands: fragment-ordered bytes and accumulator starts,
    // chosen so that a row matches exactly when its accumulator is negative.
    // Lower rows: bytes NOT t(r) in {0, 1}, start -1, so the result is
    // |t(x) & ~t(r)| - 1.  Upper rows: bytes -t(r) in {0, -1}, start
    // |t(r)| - 1, so the result is |t(r) & ~t(x)| - 1.  Pad rows and pad
    // tiles are all zero: result 0, never a match.
    const int KS = (W * 32 + 63) / 64;
    const bool with_mfma = matrix_operands && KS <= rsr::kMaxMfmaSteps;
    const int TL = static_cast<int>((R_L + 15) / 16), TU = static_cast<int>((R_U + 15) / 16);
    const int KS4 = (W * 32 + 127) / 128;
    std::vector<int8_t> lof, upf;
    std::vector<int32_t> loc, upc;
    std::vector<uint8_t> lof4, upf4, lof32, upf32;
    std::vector<float> loc4, upc4;
    if (with_mfma) {
        const int64_t TL32 = (R_L + 31) / 32, TU32 = (R_U + 31) / 32;
        lof.assign(static_cast<size_t>(TL) * KS * 1024, 0);
        upf.assign(static_cast<size_t>(TU) * KS * 1024, 0);
        loc.assign(static_cast<size_t>(TL) * 16, 0);
        upc.assign(static_cast<size_t>(TU) * 16, 0);
        lof4.assign(static_cast<size_t>(TL) * KS4 * 1024, 0);
        upf4.assign(static_cast<size_t>(TU) * KS4 * 1024, 0);
        loc4.assign(static_cast<size_t>(TL) * 16, 0.5f);
        upc4.assign(static_cast<size_t>(TU) * 16, 0.5f);
        lof32.assign(static_cast<size_t>(TL32) * KS * 1024, 0);
        upf32.assign(static_cast<size_t>(TU32) * KS * 1024, 0);
        // int8: 64 k per step; lane (group g, row rr) holds k = 64 s + 16 g ..
        // + 15.  FP4: 128 k per step; lane (group g, row rr) holds nibbles j =
        // 0..31 for k = 128 s + 32 g + j, two per byte, low nibble first.  FP4
        // on 32-row tiles: 64 k per step; lane (half h, row rr) holds nibbles j
        // for k = 64 s + 32 h + j, +1 on both sides (the kernel starts every
        // row at -1/2 and contracts upper rows with the complemented samples).
        auto frags = [&](const uint32_t* row, int64_t r, int8_t value, uint8_t nib,
                         std::vector<int8_t>& f8, std::vector<uint8_t>& f4,
                         std::vector<uint8_t>& f32) {
            int8_t* t8 = f8.data() + static_cast<size_t>(r / 16) * KS * 1024;
            uint8_t* t4 = f4.data() + static_cast<size_t>(r / 16) * KS4 * 1024;
            uint8_t* t32 = f32.data() + static_cast<size_t>(r / 32) * KS * 1024;
            const int r16 = static_cast<int>(r % 16), r32 = static_cast<int>(r % 32);
            for_bits(row, [&](int k) {
                const int s = k / 64, o = k % 64, s4 = k / 128, o4 = k % 128, j = k % 32;
                t8[(s * 64 + (o / 16) * 16 + r16) * 16 + o % 16] = value;
                t4[(s4 * 64 + (o4 / 32) * 16 + r16) * 16 + j / 2] |=
                    static_cast<uint8_t>(nib << (4 * (j % 2)));
                t32[(s * 64 + (o / 32) * 32 + r32) * 16 + j / 2] |=
                    static_cast<uint8_t>(0x2 << (4 * (j % 2)));
            });
        };
        for (int64_t r = 0; r < R_L; ++r) {
            frags(lo.data() + r * WR, r, 1, 0x2, lof, lof4, lof32);  // +1.0
            loc[r] = -1;
            loc4[r] = -0.5f;
        }
        for (int64_t r = 0; r < R_U; ++r) {
            frags(up.data() + r * WR, r, -1, 0xA, upf, upf4, upf32);  // -1.0
            upc[r] = up_weight[r] - 1;
            upc4[r] = static_cast<float>(upc[r]) + 0.5f;  // |t(r)| - 0.5
        }
    }
    // Sparse operands: the set bits of every row as column numbers, in slices
    // of 64 rows (see rsr_refs).
    auto slices = [&](int64_t R, const std::vector<int>& weight, std::vector<uint32_t>& off) {
        off.assign(1, 0u);
        for (int64_t r = 0; r < R; r += 64)  // the last row of a slice is its longest
            off.push_back(off.back() + static_cast<uint32_t>((weight[std::min(R, r + 64) - 1] + 3) / 4));
    };
    std::vector<uint32_t> lo_off, up_off;
    slices(R_L, lo_weight, lo_off);
    slices(R_U, up_weight, up_off);
    const double density =
        256.0 * (static_cast<double>(lo_off.back()) + up_off.back()) /
        std::max(1.0, 64.0 * n * (K - 1) * static_cast<double>(lo_off.size() + up_off.size() - 2));
    const bool sparse = (R_L == 0 || lo_weight[0] > 0) && (R_U == 0 || up_weight[0] > 0) &&
                        density <= rsr::sparse_density(n * (K - 1), std::max(R_L, R_U));
    std::vector<uint16_t> lo_idx, up_idx;
    auto columns = [&](const std::vector<uint32_t>& rows, int64_t R, const std::vector<uint32_t>& off,
                       std::vector<uint16_t>& idx) {
        std::vector<uint16_t> cols(static_cast<size_t>(W) * 32);
        idx.resize(static_cast<size_t>(off.back()) * 256);
        for (size_t sl = 0; sl + 1 < off.size(); ++sl) {
            const size_t places = static_cast<size_t>(off[sl + 1] - off[sl]) * 4;
            for (int64_t k = 0; k < 64; ++k) {
                const int64_t r = static_cast<int64_t>(sl) * 64 + k;
                uint16_t* dst = idx.data() + static_cast<size_t>(off[sl]) * 256 + k * 4;
                size_t c = 0;
                if (r < R) {
                    for_bits(rows.data() + r * WR, [&](int b) {
                        const int w = b / 32;
                        cols[c++] = static_cast<uint16_t>((w / PW) * n + b - 32 * (w - w % PW));
                    });
                    for (; c < places; ++c) cols[c] = cols[c - 1];
                }  // past the last row: its columns again
                for (size_t q = 0; q < places; ++q) dst[(q / 4) * 256 + q % 4] = cols[q];
            }
        }
    };
    if (sparse) {
        columns(lo, R_L, lo_off, lo_idx);
        columns(up, R_U, up_off, up_idx);
    }

    std::unique_ptr<rsr_refs, rsr_status (*)(rsr_refs*)> refs(new rsr_refs(), rsr_refs_destroy);
    refs->ctx = ctx;
    refs->n = n;
    refs->K = K;
    refs->W = W;
    refs->WR = WR;
    refs->R_L = R_L;
    refs->R_U = R_U;
    refs->chunks = static_cast<int64_t>(lo_off.back()) + up_off.back();
    // One allocation and one copy for all arrays, 256-byte aligned.
    struct Part {
        void** dst;
        const void* src;
        size_t bytes, at;
    };
    std::vector<Part> parts;
    size_t total = 0;
    auto part = [&](auto** dst, const auto& v) {
        const size_t bytes = sizeof(v[0]) * v.size();
        if (bytes == 0) return;
        parts.push_back({reinterpret_cast<void**>(dst), v.data(), bytes, total});
        total += (bytes + 255) / 256 * 256;
    };
    part(&refs->d_lower_nbits, lo);
    part(&refs->d_upper_bits, up);
    if (sparse) {
        refs->sparse = true;
        refs->sparse_count = density <= rsr::kSparseCountDensity &&
                             std::max(R_L, R_U) >= rsr::kSparseCountRows;
        part(&refs->d_lower_off, lo_off);
        part(&refs->d_lower_idx, lo_idx);
        part(&refs->d_upper_off, up_off);
        part(&refs->d_upper_idx, up_idx);
    }
    if (with_mfma) {
        refs->KS = KS;
        refs->TL = TL;
        refs->TU = TU;
        refs->KS4 = KS4;
        part(&refs->d_lower_frag, lof);
        part(&refs->d_lower_cinit, loc);
        part(&refs->d_upper_frag, upf);
        part(&refs->d_upper_cinit, upc);
        part(&refs->d_lower_frag32, lof32);
        part(&refs->d_upper_frag32, upf32);
        part(&refs->d_lower_frag4, lof4);
        part(&refs->d_lower_cinit4, loc4);
        part(&refs->d_upper_frag4, upf4);
        part(&refs->d_upper_cinit4, upc4);
    }
    if (total > 0) {
        std::vector<char> image(total);
        hipError_t e = rsr::dev_malloc(&refs->d_mem, total);
        if (e == hipSuccess) {
            for (const Part& q : parts) {
                std::memcpy(image.data() + q.at, q.src, q.bytes);
                *q.dst = static_cast<char*>(refs->d_mem) + q.at;
            }
            e = hipMemcpy(refs->d_mem, image.data(), total, hipMemcpyHostToDevice);
        }
        if (e != hipSuccess) return hip_fail(ctx, e, "rsr_refs_create upload");
    }
    refs->consistent = true;
    if (!consistent) {
        rsr_status st = check_consistency(ctx, refs.get(), up);
        if (st != RSR_OK) return st;
    }
    *out = refs.release();
    return RSR_OK;
}

rsr_status refs_from_packed(rsr_ctx* ctx, int32_t n, int32_t K, const std::vector<uint32_t>& lower,
                            const std::vector<uint32_t>& upper, bool consistent, rsr_refs** out) {
    return build_refs(ctx, n, K, lower, upper, false, consistent, out);
}

}  // namespace rsr

extern "C" {

rsr_status rsr_refs_consistent(const rsr_refs* refs, int32_t* out) {
    if (!refs || !out) return RSR_EINVAL;
    *out = refs->consistent ? 1 : 0;
    return RSR_OK;
}

rsr_status rsr_refs_create(rsr_ctx* ctx, int32_t n, int32_t K, const uint8_t* lower, int64_t R_L,
                           const uint8_t* upper, int64_t R_U, rsr_refs** out) {
    if (!ctx || !out) return RSR_EINVAL;
    *out = nullptr;
    try {
        std::vector<uint32_t> lo, up;
        rsr_status st = rsr::pack_refs(ctx, n, K, lower, R_L, upper, R_U, lo, up);
        if (st != RSR_OK) return st;
        return rsr::build_refs(ctx, n, K, std::move(lo), std::move(up), true, false, out);
    } catch (const std::bad_alloc&) {
        return fail(ctx, RSR_ENOMEM, "host allocation");
    }
}

rsr_status rsr_refs_destroy(rsr_refs* refs) {
    if (!refs) return RSR_EINVAL;
    DeviceGuard g(refs->ctx->device);
    if (refs->d_mem) (void)hipFree(refs->d_mem);
    delete refs;
    return RSR_OK;
}

rsr_status rsr_system_create(rsr_ctx* ctx, const rsr_system_desc* d, rsr_system** out) {
    if (!ctx || !out || !d) return RSR_EINVAL;
    *out = nullptr;
    if (d->kind == RSR_SYS_HOST_CALLBACK) {
        if (!d->phi) return fail(ctx, RSR_EINVAL, "RSR_SYS_HOST_CALLBACK without phi");
        if (d->n_edges <= 0 || d->K < 2) return fail(ctx, RSR_EINVAL, "n must be > 0 and K >= 2");
        if (d->K > RSR_MAX_K || static_cast<int64_t>(d->n_edges) * (d->K - 1) > RSR_MAX_BITS)
            return fail(ctx, RSR_EUNSUPPORTED, "n*(K-1) exceeds RSR_MAX_BITS or K > RSR_MAX_K");
        if (d->level < 1) return fail(ctx, RSR_EINVAL, "level must be >= 1");
        rsr_system* s = new (std::nothrow) rsr_system();
        if (!s) return fail(ctx, RSR_ENOMEM, "host allocation");
        s->ctx = ctx;
        s->kind = d->kind;
        s->n_edges = d->n_edges;
        s->K = d->K;
        s->level = d->level;
        s->phi = d->phi;
        s->user = d->user;
        *out = s;
        return RSR_OK;
    }
    if (d->kind != RSR_SYS_ST_CONNECTIVITY && d->kind != RSR_SYS_GLOBAL_CONNECTIVITY &&
        d->kind != RSR_SYS_MAX_FLOW)
        return fail(ctx, RSR_EINVAL, "unknown system kind");
    const bool global = d->kind == RSR_SYS_GLOBAL_CONNECTIVITY;
    const bool flow = d->kind == RSR_SYS_MAX_FLOW;
    if (d->n_nodes < 2 || d->n_edges <= 0 || d->K < 2 || !d->edge_u || !d->edge_v)
        return fail(ctx, RSR_EINVAL, "bad graph size or NULL edge arrays");
    if (d->n_nodes > RSR_MAX_NODES || d->K > RSR_MAX_K ||
        static_cast<int64_t>(d->n_edges) * (d->K - 1) > RSR_MAX_BITS)
        return fail(ctx, RSR_EUNSUPPORTED, "graph exceeds RSR_MAX_NODES / RSR_MAX_BITS");
    if (global) {
        if (d->level < 1 || d->level > 2) return fail(ctx, RSR_EINVAL, "level not in 1..2");
        // Edge list plus four waves' node sets, parents and depths in 64 KB of LDS.
        const int64_t words = d->n_edges + 4ll * (((d->n_nodes + 31) >> 5) + ((d->n_edges + 31) >> 5) +
                                                   2 * ((d->n_nodes + 1) >> 1));
        if (words * 4 > 64 * 1024)
            return fail(ctx, RSR_EUNSUPPORTED, "graph too large for the global-connectivity search");
    } else {
        if (d->source < 0 || d->source >= d->n_nodes || d->sink < 0 || d->sink >= d->n_nodes ||
            d->source == d->sink)
            return fail(ctx, RSR_EINVAL, "source/sink out of range or equal");
        if (flow ? (d->level < 1 || d->level > 255) : (d->level < 1 || d->level > d->K - 1))
            return fail(ctx, RSR_EINVAL, flow ? "demand not in 1..255" : "level not in 1..K-1");
        if (flow) {
            // Edge list plus four waves' marks, parents, capacities and flows in 64 KB.
            const int64_t words = d->n_edges + 4ll * (((d->n_nodes + 31) >> 5) + ((d->n_nodes + 1) >> 1) +
                                                       3 * ((d->n_edges + 3) >> 2));
            if (words * 4 > 64 * 1024)
                return fail(ctx, RSR_EUNSUPPORTED, "graph too large for the max-flow search");
        }
    }
    std::vector<uint32_t> packed(d->n_edges);
    for (int e = 0; e < d->n_edges; ++e) {
        const int32_t u = d->edge_u[e], v = d->edge_v[e];
        if (u < 0 || u >= d->n_nodes || v < 0 || v >= d->n_nodes)
            return fail(ctx, RSR_EINVAL, "edge endpoint out of range");
        packed[e] = static_cast<uint32_t>(u) | (static_cast<uint32_t>(v) << 16);
    }
    DeviceGuard g(ctx->device);
    rsr_system* s = new (std::nothrow) rsr_system();
    if (!s) return fail(ctx, RSR_ENOMEM, "host allocation");
    s->ctx = ctx;
    s->kind = d->kind;
    s->n_nodes = d->n_nodes;
    s->n_edges = d->n_edges;
    s->K = d->K;
    s->level = d->level;
    s->source = global ? 0 : d->source;
    s->sink = global ? 0 : d->sink;
    std::vector<int> degree(d->n_nodes, 0);
    for (uint32_t uv : packed) {
        ++degree[uv & 0xFFFFu];
        ++degree[uv >> 16];
    }
    s->tree_from = static_cast<int>(std::min_element(degree.begin(), degree.end()) - degree.begin());
    s->class_from = static_cast<int>(std::max_element(degree.begin(), degree.end()) - degree.begin());
    if (global && d->level == 2) {
        std::vector<uint8_t> near(d->n_nodes, 0);
        near[s->tree_from] = 1;
        std::vector<uint8_t> next = near;
        for (int step = 0; step <= rsr_system::kShallow && !s->shallow; ++step, near = next) {
            for (uint32_t uv : packed) {
                next[uv >> 16] |= near[uv & 0xFFFFu];
                next[uv & 0xFFFFu] |= near[uv >> 16];
            }
            s->shallow = next == near;
        }
    }
    hipError_t e = rsr::dev_malloc(&s->d_edges, sizeof(uint32_t) * packed.size());
    if (e == hipSuccess)
        e = hipMemcpy(s->d_edges, packed.data(), sizeof(uint32_t) * packed.size(),
                      hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        rsr_system_destroy(s);
        return hip_fail(ctx, e, "rsr_system_create upload");
    }
    *out = s;
    return RSR_OK;
}

rsr_status rsr_system_destroy(rsr_system* s) {
    if (!s) return RSR_EINVAL;
    DeviceGuard g(s->ctx->device);
    if (s->d_edges) (void)hipFree(s->d_edges);
    delete s;
    return RSR_OK;
}

// ---- hot path ----------------------------------------------------------------

rsr_status rsr_sample(rsr_ctx* ctx, const rsr_model* model, uint64_t seed, uint32_t stream_id,
                      uint64_t first_sample, int64_t N, uint32_t* d_samples) {
    if (!ctx) return RSR_EINVAL;
    if (!model || !d_samples) return fail(ctx, RSR_EINVAL, "NULL model or d_samples");
    if (N <= 0) return fail(ctx, RSR_EINVAL, "N must be > 0");
    DeviceGuard g(ctx->device);
    RSR_HIP(ctx, rsr::launch_sample(ctx->stream, model, seed, stream_id, first_sample, N,
                                    ctx->cu_count, d_samples));
    return RSR_OK;
}

rsr_status rsr_classify(rsr_ctx* ctx, const rsr_refs* refs, const uint32_t* d_samples, int64_t N,
                        int32_t mode, int32_t form, uint8_t* d_flags, uint32_t* d_match) {
    if (!ctx) return RSR_EINVAL;
    if (!refs || !d_samples || !d_flags) return fail(ctx, RSR_EINVAL, "NULL argument");
    if (N <= 0) return fail(ctx, RSR_EINVAL, "N must be > 0");
    if (mode != RSR_LABEL && mode != RSR_COUNT) return fail(ctx, RSR_EINVAL, "bad mode");
    if (form != RSR_AUTO && form != RSR_POPCOUNT && form != RSR_MFMA && form != RSR_MFMA_FP4 &&
        form != RSR_PERSIST)
        return fail(ctx, RSR_EINVAL, "bad form");
    if (refs->ctx->device != ctx->device) return fail(ctx, RSR_EINVAL, "refs on another device");
    DeviceGuard g(ctx->device);
    if ((form == RSR_MFMA && refs->KS == 0) ||
        ((form == RSR_MFMA_FP4 || form == RSR_PERSIST) && refs->KS4 == 0))
        return fail(ctx, RSR_EUNSUPPORTED, "matrix-core form needs n*(K-1) <= 1280");
    if (form == RSR_PERSIST &&
        (mode != RSR_LABEL || !refs->consistent || N > 0x7FFFFFFFll || !rsr::casc_persist_supported(refs)))
        return fail(ctx, RSR_EUNSUPPORTED,
                    "the persistent cascade takes LABEL mode on consistent rows, N <= 2^31-1");
    uint32_t* match = mode == RSR_COUNT ? d_match : nullptr;
    // RSR_AUTO: for LABEL on consistent rows (each sample stops at its first
    // match) the sparse form, or the cascade for dense or few rows; otherwise the
    // sparse count for many sparse rows, else the FP4 matrix-core form, which
    // makes the most tests per second in both modes; popcount beyond 1280 bits.
    if (form == RSR_AUTO && refs->sparse_count && (mode == RSR_COUNT || !refs->consistent) &&
        rsr::sparse_count_pays(mode, refs->n * (refs->K - 1), std::max(refs->R_L, refs->R_U), N,
                               ctx->cu_count)) {
        RSR_HIP(ctx, rsr::launch_sparse_count(ctx->stream, refs, d_samples, N, mode, ctx->cu_count,
                                              d_flags, match));
        return RSR_OK;
    }
    if (form == RSR_AUTO && refs->KS4 > 0 && (mode == RSR_COUNT || !refs->consistent))
        form = RSR_MFMA_FP4;
    const bool matrix = form == RSR_MFMA || form == RSR_MFMA_FP4;
    if (mode == RSR_LABEL && !matrix && refs->consistent && N <= 0x7FFFFFFFll) {
        // RSR_PERSIST runs the rounds after round 0 in one persistent
        // launch; the automatic and popcount forms run one launch per round.
        const int64_t n_max = refs->R_L > refs->R_U ? refs->R_L : refs->R_U;
        const bool persist = form == RSR_PERSIST;
        const int64_t stride = persist ? rsr::casc_persist_stride(refs, N, ctx->cu_count) : N;
        const int64_t state_words = persist ? rsr::casc_persist_state_words(stride, refs->KS) : 0;
        rsr_status st = ensure_cascade(ctx, refs->W, stride, state_words);
        if (st != RSR_OK) return st;
        rsr::CascadeBuffers cb;
        cb.words[0] = ctx->ws.casc_words;
        cb.words[1] = ctx->ws.casc_words + static_cast<int64_t>(refs->W) * stride;
        cb.index[0] = ctx->ws.casc_index;
        cb.index[1] = ctx->ws.casc_index + stride;
        cb.match[0] = reinterpret_cast<uint32_t*>(ctx->ws.casc_index + 2 * stride);
        cb.match[1] = reinterpret_cast<uint32_t*>(ctx->ws.casc_index + 3 * stride);
        cb.stride = stride;
        cb.set_counters(ctx->ws.casc_counters);
        if (form == RSR_AUTO && refs->sparse && rsr::sparse_label_pays(refs, N)) {
            RSR_HIP(ctx, rsr::launch_dom_sparse(ctx->stream, refs,
                                                rsr::single_src(d_samples, N, d_flags, nullptr),
                                                rsr::JobTiles(), cb, ctx->cu_count));
            return RSR_OK;
        }
        // The automatic form runs the rounds after round 0 in the FP4
        // matrix-core form when the handle has its operands, with faster
        // growing rounds from kWideRows rows per side on; the popcount form
        // stays popcount.
        const rsr::CascadeShape shape = form != RSR_AUTO || refs->KS4 == 0 ? rsr::CascadeShape{}
                                        : n_max >= rsr::kWideRows        ? rsr::mfma_wide_shape()
                                                                         : rsr::mfma_tail_shape();
        if (persist) {
            RSR_HIP(ctx, rsr::launch_fill_u64(ctx->stream, reinterpret_cast<uint64_t*>(ctx->ws.casc_state),
                                              (state_words + 1) / 2, 0));
            RSR_HIP(ctx, rsr::launch_casc_persist(ctx->stream, refs,
                                                  rsr::single_src(d_samples, N, d_flags, nullptr), cb,
                                                  rsr::mfma_head_shape(), ctx->ws.casc_state,
                                                  reinterpret_cast<unsigned long long*>(ctx->ws.counters + 14),
                                                  ctx->cu_count));
            return RSR_OK;
        }
        RSR_HIP(ctx, rsr::launch_fill_u64(ctx->stream, cb.counters, rsr::CascadeBuffers::kMaxRounds, 0));
        RSR_HIP(ctx, rsr::launch_dom_cascade(ctx->stream, refs,
                                             rsr::single_src(d_samples, N, d_flags, nullptr), cb,
                                             shape, ctx->cu_count * 8));
        return RSR_OK;
    }
    if (matrix)
        RSR_HIP(ctx, rsr::launch_dom_mfma(ctx->stream, refs, d_samples, N, mode,
                                          form == RSR_MFMA_FP4, ctx->cu_count, d_flags,
                                          match));
    else
        RSR_HIP(ctx, rsr::launch_dom_bits(ctx->stream, refs, d_samples, N, mode, d_flags, match));
    return RSR_OK;
}

rsr_status rsr_eval_unknown(rsr_ctx* ctx, const rsr_system* sys, const uint32_t* d_samples,
                            int64_t N, const uint8_t* d_flags, int32_t which, uint8_t* d_Y,
                            uint64_t* d_n_evaluated) {
    if (!ctx) return RSR_EINVAL;
    if (!sys || !d_samples || !d_Y) return fail(ctx, RSR_EINVAL, "NULL argument");
    if (N <= 0 || N > 0x7FFFFFFFll) return fail(ctx, RSR_EINVAL, "N must be in 1..2^31-1");
    if (which != RSR_UNKNOWN_ONLY && which != RSR_ALL) return fail(ctx, RSR_EINVAL, "bad which");
    if (which == RSR_UNKNOWN_ONLY && !d_flags)
        return fail(ctx, RSR_EINVAL, "d_flags is NULL with RSR_UNKNOWN_ONLY");
    DeviceGuard g(ctx->device);
    if (sys->kind == RSR_SYS_HOST_CALLBACK)
        return rsr::eval_callback(ctx, sys, d_samples, N, d_flags, which, d_Y, d_n_evaluated);
    const rsr::SegSrc seg = rsr::single_src(d_samples, N, const_cast<uint8_t*>(d_flags), d_Y);
    rsr::SampleList list;
    if (which == RSR_UNKNOWN_ONLY) {
        rsr_status st = rsr::ensure_list(ctx, N);
        if (st != RSR_OK) return st;
        list = rsr::SampleList(ctx->ws.list);
        RSR_HIP(ctx, rsr::launch_label(ctx->stream, seg, list));
    }
    RSR_HIP(ctx, rsr::launch_eval(ctx->stream, sys, seg, list, which, d_n_evaluated, ctx->cu_count));
    return RSR_OK;
}

rsr_status rsr_boundary_search(rsr_ctx* ctx, const rsr_system* sys, const uint32_t* d_samples,
                               int64_t N, const int64_t* d_pick, int64_t n_pick,
                               uint8_t* d_rows, uint8_t* d_side) {
    if (!ctx) return RSR_EINVAL;
    if (n_pick < 0) return fail(ctx, RSR_EINVAL, "n_pick must be >= 0");
    if (n_pick == 0) return RSR_OK;
    if (!sys || !d_samples || !d_pick || !d_rows || !d_side)
        return fail(ctx, RSR_EINVAL, "NULL argument");
    if (N <= 0 || N > 0x7FFFFFFFll) return fail(ctx, RSR_EINVAL, "N must be in 1..2^31-1");
    if (sys->kind == RSR_SYS_HOST_CALLBACK) {
        DeviceGuard g(ctx->device);
        return rsr::boundary_callback(ctx, sys, d_samples, N, d_pick, n_pick, d_rows, d_side);
    }
    if (rsr::boundary_lds_bytes(sys) > 64 * 1024)
        return fail(ctx, RSR_EUNSUPPORTED, "graph too large for the boundary search");
    DeviceGuard g(ctx->device);
    RSR_HIP(ctx, rsr::launch_boundary(ctx->stream, sys, d_samples, N, d_pick, n_pick, d_rows,
                                      d_side, ctx->cu_count * 8));
    return RSR_OK;
}

rsr_status rsr_estimate(rsr_ctx* ctx, const uint8_t* d_flags, const uint8_t* d_Y, int64_t N,
                        rsr_estimate_t* out) {
    if (!ctx) return RSR_EINVAL;
    if (!d_flags || !out) return fail(ctx, RSR_EINVAL, "NULL argument");
    if (N <= 0) return fail(ctx, RSR_EINVAL, "N must be > 0");
    DeviceGuard g(ctx->device);
    const bool aligned = (reinterpret_cast<uintptr_t>(d_flags) & 15u) == 0 &&
                         (reinterpret_cast<uintptr_t>(d_Y) & 15u) == 0;
    // host_counts[0..4] receive the counts and host_counts[5] the persistent
    // cascade's time-out flag (counters[14]); the one-launch kernel writes
    // them into the pinned buffer itself, the other path through a copy.
    uint64_t* c = ctx->ws.host_counts;
    if (aligned) {
        // The kernel's last block stores this call's sequence number into
        // c[6] after the counts (system-scope release), once every earlier
        // kernel of the stream and every other block of its own have ended:
        // the host returns as soon as it sees it, instead of waiting for the
        // end-of-kernel signal.  Past 10 ms of polling (a long queue ahead of
        // the counts) it synchronises the stream.
        const uint64_t seq = ++ctx->ws.estimate_seq;
        __atomic_store_n(&c[6], uint64_t{0}, __ATOMIC_RELAXED);
        RSR_HIP(ctx, rsr::launch_counts_vec(ctx->stream, d_flags, d_Y, N, ctx->ws.host_counts_dev,
                                            ctx->ws.count_part,
                                            reinterpret_cast<uint32_t*>(ctx->ws.counters + 15),
                                            ctx->ws.counters + 14, seq));
        const auto t0 = std::chrono::steady_clock::now();
        bool seen = false;
        for (uint32_t it = 1;; ++it) {
            if (__atomic_load_n(&c[6], __ATOMIC_ACQUIRE) == seq) {
                seen = true;
                break;
            }
            if ((it & 255u) == 0 &&
                std::chrono::steady_clock::now() - t0 > std::chrono::milliseconds(10))
                break;
        }
        if (!seen) RSR_HIP(ctx, hipStreamSynchronize(ctx->stream));
    } else {
        RSR_HIP(ctx, rsr::launch_counts(ctx->stream, d_flags, d_Y, N, ctx->ws.counters,
                                        ctx->ws.count_part));
        RSR_HIP(ctx, hipMemcpyAsync(c, ctx->ws.counters, sizeof(uint64_t) * 16,
                                    hipMemcpyDeviceToHost, ctx->stream));
        RSR_HIP(ctx, hipStreamSynchronize(ctx->stream));
        c[5] = c[14];
    }
    if (c[5] != 0) {
        // A persistent cascade since the last check could not synchronise its
        // blocks in time: its flags are not to be trusted.
        RSR_HIP(ctx, rsr::launch_fill_u64(ctx->stream, ctx->ws.counters + 14, 1, 0));
        return fail(ctx, RSR_EHIP, "a persistent classification timed out at a grid barrier");
    }
    out->n_L = c[0];
    out->n_U = c[1];
    out->n_u = c[2];
    out->n_both = c[3];
    out->n_u_up = c[4];
    out->N = static_cast<uint64_t>(N);
    const double Nd = static_cast<double>(N);
    out->p_L = static_cast<double>(out->n_L) / Nd;
    out->p_U = static_cast<double>(out->n_U) / Nd;
    out->p_u = static_cast<double>(out->n_u) / Nd;
    if (!d_Y) {
        out->P = out->se = out->cov = std::nan("");
        return RSR_OK;
    }
    const double P = static_cast<double>(out->n_U + out->n_u_up) / Nd;
    out->P = P;
    out->se = std::sqrt(P * (1.0 - P) / Nd);
    out->cov = P > 0.0 ? std::sqrt((1.0 - P) / (Nd * P)) : HUGE_VAL;
    return RSR_OK;
}

rsr_status rsr_grad(rsr_ctx* ctx, const rsr_model* model, const uint32_t* d_samples,
                    const uint8_t* d_Y, int64_t N, float* d_G, uint64_t* d_counts) {
    if (!ctx) return RSR_EINVAL;
    if (!model || !d_samples || !d_Y || !d_G) return fail(ctx, RSR_EINVAL, "NULL argument");
    if (N <= 0) return fail(ctx, RSR_EINVAL, "N must be > 0");
    DeviceGuard g(ctx->device);
    RSR_HIP(ctx, rsr::launch_grad(ctx->stream, model->n, model->K, model->d_p, d_samples, d_Y, N,
                                  ctx->ws.grad_part, d_G, d_counts));
    return RSR_OK;
}

rsr_status rsr_importance(rsr_ctx* ctx, const rsr_model* model, const uint32_t* d_samples,
                          const uint8_t* d_Y, int64_t N, float* d_I) {
    if (!ctx) return RSR_EINVAL;
    if (!model || !d_samples || !d_Y || !d_I) return fail(ctx, RSR_EINVAL, "NULL argument");
    if (N <= 0) return fail(ctx, RSR_EINVAL, "N must be > 0");
    if (model->K != 2) return fail(ctx, RSR_EINVAL, "the Birnbaum importance needs K = 2");
    DeviceGuard g(ctx->device);
    RSR_HIP(ctx, rsr::launch_importance(ctx->stream, model->n, model->d_p64, d_samples, d_Y, N,
                                        ctx->ws.grad_part, d_I));
    return RSR_OK;
}

rsr_status rsr_debug_barrier_timeout(int64_t ticks) {
    rsr::set_barrier_timeout(ticks);
    return RSR_OK;
}

rsr_status rsr_debug_fail_alloc(int64_t after) {
    rsr::g_fail_countdown = after < 0 ? -1 : after;
    return RSR_OK;
}

}  // extern "C"
