// Stage 1 of the RSR workflow (section 3.5, fig. rsr_alg): alternate sample
// classification and componentwise boundary search (section 3.4) until the
// unclassified fraction of a fresh sample set is small enough or the
// reference sets are large enough.  The sampling, classification, ordered
// pick of unclassified samples and the searches run on the device; the host
// keeps the rows (in discovery order), also packed, drops exact duplicates and
// builds the reference operands between iterations.
//
// What bounds a run is the host's share of an iteration.  So a row is packed
// once, when it is found; duplicates are found by the packed words; the
// device memory is one block and an iteration's rows and sides come in one
// copy; and a set that has only found rows is not checked for consistency.
// Five iterations of 100,000 samples and 1024 picks on 295 components:
// 1256 us, 1891 with every iteration's rows packed and checked anew.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "rsr_internal.h"

namespace {

rsr_status s1_fail(rsr_ctx* ctx, rsr_status st, const std::string& msg) {
    if (ctx) ctx->err = msg;
    return st;
}

rsr_status s1_hip(rsr_ctx* ctx, hipError_t e, const char* what) {
    return s1_fail(ctx, e == hipErrorOutOfMemory ? RSR_ENOMEM : RSR_EHIP,
                   std::string(what) + ": " + hipGetErrorName(e) + " (" + hipGetErrorString(e) + ")");
}

#define S1_HIP(ctx, call)                                 \
    do {                                                  \
        hipError_t e_ = (call);                           \
        if (e_ != hipSuccess) return s1_hip(ctx, e_, #call); \
    } while (0)

struct DeviceBuffer {
    void* p = nullptr;
    ~DeviceBuffer() {
        if (p) (void)hipFree(p);
    }
};

struct RefsHandle {
    rsr_refs* r = nullptr;
    ~RefsHandle() {
        if (r) (void)rsr_refs_destroy(r);
    }
};

struct CurrentDevice {
    int prev = -1;
    bool changed = false;
    explicit CurrentDevice(int dev) {
        if (hipGetDevice(&prev) == hipSuccess && prev != dev) changed = hipSetDevice(dev) == hipSuccess;
    }
    ~CurrentDevice() {
        if (changed) (void)hipSetDevice(prev);
    }
};

// The rows of one side in discovery order, packed too (words to a row; a row's
// packed form determines it), with a table of the distinct ones: open
// addressing, at most half full.
class RowSet {
  public:
    RowSet(int n, int K, bool lower)
        : n_(n), K_(K), lower_(lower),
          words_(rsr::dom_row_words(rsr::sample_words(n, K))), table_(1024, -1) {}

    int64_t size() const { return static_cast<int64_t>(rows_.size()) / n_; }
    const std::vector<uint8_t>& rows() const { return rows_; }
    const std::vector<uint32_t>& bits() const { return bits_; }

    // Takes the given rows, equal ones among them too.
    void start(const uint8_t* rows, int64_t R, std::vector<uint32_t> bits) {
        rows_.assign(rows, rows + R * n_);
        bits_ = std::move(bits);
        for (int64_t r = 0; r < R; ++r) enter(r);
    }

    // Appends a row unless it is there; whether it was appended.
    bool add(const uint8_t* row) {
        rsr::pack_rows(n_, K_, row, 1, lower_, bits_);
        if (!enter(size())) {
            bits_.resize(bits_.size() - words_);
            return false;
        }
        rows_.insert(rows_.end(), row, row + n_);
        return true;
    }

  private:
    // Enters packed row r into the table; false if an equal row is there.
    bool enter(int64_t r) {
        if (2 * (used_ + 1) > static_cast<int64_t>(table_.size())) {
            std::vector<int64_t> old(2 * table_.size(), -1);
            old.swap(table_);
            for (int64_t q : old)
                if (q >= 0) table_[place(q)] = q;
        }
        int64_t& at = table_[place(r)];
        if (at >= 0) return false;
        at = r;
        used_ += 1;
        return true;
    }

    // The slot of a row equal to packed row r, or the free one for it.
    size_t place(int64_t r) const {
        const uint32_t* row = bits_.data() + r * words_;
        uint64_t h = 0;
        for (int w = 0; w < words_; ++w) {
            h = (h ^ row[w]) * 0x9E3779B97F4A7C15ull;
            h ^= h >> 32;
        }
        size_t i = h & (table_.size() - 1);
        while (table_[i] >= 0 && std::memcmp(bits_.data() + table_[i] * words_, row,
                                             sizeof(uint32_t) * words_) != 0)
            i = (i + 1) & (table_.size() - 1);
        return i;
    }

    int n_, K_;
    bool lower_;
    int words_;
    std::vector<uint8_t> rows_;
    std::vector<uint32_t> bits_;
    std::vector<int64_t> table_;
    int64_t used_ = 0;
};

rsr_status run_stage1(rsr_ctx* ctx, const rsr_model* model, const rsr_system* sys,
                      const rsr_stage1_params* params, const uint8_t* lower0, int64_t R_L0,
                      const uint8_t* upper0, int64_t R_U0, uint8_t* lower, int64_t cap_L,
                      uint8_t* upper, int64_t cap_U, rsr_stage1_result* result) {
    if (!ctx) return RSR_EINVAL;
    if (!model || !sys || !params || !lower || !upper || !result)
        return s1_fail(ctx, RSR_EINVAL, "NULL argument");
    const rsr_stage1_params P = *params;
    if (model->n != sys->n_edges || model->K != sys->K)
        return s1_fail(ctx, RSR_EINVAL, "model and system differ in n or K");
    if (P.N <= 0 || P.N > 0x7FFFFFFFll) return s1_fail(ctx, RSR_EINVAL, "N must be in 1..2^31-1");
    if (P.picks < 1) return s1_fail(ctx, RSR_EINVAL, "picks must be >= 1");
    if (P.max_iters < 1) return s1_fail(ctx, RSR_EINVAL, "max_iters must be >= 1");
    if (!(P.eps_u >= 0.0)) return s1_fail(ctx, RSR_EINVAL, "eps_u must be >= 0");
    if (P.max_rows < 0 || cap_L < P.max_rows || cap_U < P.max_rows)
        return s1_fail(ctx, RSR_EINVAL, "max_rows must be >= 0 and cap_L, cap_U >= max_rows");
    if (R_L0 < 0 || R_U0 < 0 || (R_L0 > 0 && !lower0) || (R_U0 > 0 && !upper0))
        return s1_fail(ctx, RSR_EINVAL, "bad initial rows");
    if (R_L0 > cap_L || R_U0 > cap_U)
        return s1_fail(ctx, RSR_EINVAL, "initial rows exceed cap_L / cap_U");
    const int n = model->n, K = model->K;
    const size_t row = static_cast<size_t>(n);

    RowSet set_l(n, K, true), set_u(n, K, false);
    // The target is monotone for every system but a host callback: no found
    // upper row (a survival state) lies below a found lower row (a failure
    // state).  Given rows need not belong to the system.
    const bool consistent = R_L0 == 0 && R_U0 == 0 && sys->kind != RSR_SYS_HOST_CALLBACK;

    CurrentDevice guard(ctx->device);
    // No more than N samples can be picked, so room for N picks will do (and the
    // sizes below cannot overflow).
    const int64_t N = P.N, B = std::min<int64_t>(P.picks, N);
    // One block: samples, flags, picks, then an iteration's rows and, right
    // behind them, its sides.
    const auto aligned = [](size_t bytes) { return (bytes + 255) / 256 * 256; };
    const size_t at_flags = aligned(sizeof(uint32_t) * rsr::sample_words(n, K) * static_cast<size_t>(N));
    const size_t at_pick = at_flags + aligned(static_cast<size_t>(N));
    const size_t at_found = at_pick + aligned(sizeof(int64_t) * static_cast<size_t>(B));
    DeviceBuffer mem;
    S1_HIP(ctx, rsr::dev_malloc(&mem.p, at_found + (row + 1) * static_cast<size_t>(B)));
    char* base = static_cast<char*>(mem.p);
    uint32_t* samples = reinterpret_cast<uint32_t*>(base);
    uint8_t* flags = reinterpret_cast<uint8_t*>(base + at_flags);
    int64_t* pick = reinterpret_cast<int64_t*>(base + at_pick);
    uint8_t* found = reinterpret_cast<uint8_t*>(base + at_found);
    std::vector<uint8_t> found_h((row + 1) * static_cast<size_t>(B));
    {
        std::vector<uint32_t> lo, up;
        rsr_status st = rsr::pack_refs(ctx, n, K, lower0, R_L0, upper0, R_U0, lo, up);
        if (st != RSR_OK) return st;
        set_l.start(lower0, R_L0, std::move(lo));
        set_u.start(upper0, R_U0, std::move(up));
    }
    uint64_t* d_total = ctx->ws.counters + 12;
    uint64_t* h_total = ctx->ws.host_counts + 12;

    rsr_stage1_result res{};
    for (int32_t it = 0; it < P.max_iters; ++it) {
        const int64_t R_L = set_l.size(), R_U = set_u.size();
        RefsHandle refs;
        rsr_status st =
            rsr::refs_from_packed(ctx, n, K, set_l.bits(), set_u.bits(), consistent, &refs.r);
        if (st != RSR_OK) return st;
        st = rsr_sample(ctx, model, P.seed, static_cast<uint32_t>(it), 0, N, samples);
        if (st != RSR_OK) return st;
        st = rsr_classify(ctx, refs.r, samples, N, RSR_LABEL, RSR_AUTO, flags, nullptr);
        if (st != RSR_OK) return st;
        S1_HIP(ctx, rsr::launch_pick(ctx->stream, flags, N, B, pick, ctx->ws.count_part, d_total));
        S1_HIP(ctx, hipMemcpyAsync(h_total, d_total, sizeof(uint64_t), hipMemcpyDeviceToHost,
                                   ctx->stream));
        rsr_estimate_t est;
        st = rsr_estimate(ctx, flags, nullptr, N, &est);  // synchronises
        if (st != RSR_OK) return st;
        res.iterations = it + 1;
        res.p_u = est.p_u;
        if (est.p_u < P.eps_u || R_L + R_U >= P.max_rows || it + 1 == P.max_iters) break;
        const int64_t n_pick = std::min<int64_t>(static_cast<int64_t>(*h_total), B);
        if (n_pick == 0) break;
        const size_t rows_bytes = row * static_cast<size_t>(n_pick);
        st = rsr_boundary_search(ctx, sys, samples, N, pick, n_pick, found, found + rows_bytes);
        if (st != RSR_OK) return st;
        S1_HIP(ctx, hipMemcpyAsync(found_h.data(), found, rows_bytes + static_cast<size_t>(n_pick),
                                   hipMemcpyDeviceToHost, ctx->stream));
        S1_HIP(ctx, hipStreamSynchronize(ctx->stream));
        res.searches += n_pick;
        const uint8_t* side_h = found_h.data() + rows_bytes;
        int64_t total = R_L + R_U;
        for (int64_t j = 0; j < n_pick && total < P.max_rows; ++j) {
            if (side_h[j] > 1) return s1_fail(ctx, RSR_EHIP, "boundary search rejected a pick");
            if ((side_h[j] ? set_u : set_l).add(found_h.data() + j * row))
                total += 1;
            else
                res.duplicates += 1;
        }
    }
    res.R_L = set_l.size();
    res.R_U = set_u.size();
    if (res.R_L) std::memcpy(lower, set_l.rows().data(), set_l.rows().size());
    if (res.R_U) std::memcpy(upper, set_u.rows().data(), set_u.rows().size());
    *result = res;
    return RSR_OK;
}

}  // namespace

extern "C" rsr_status rsr_stage1(rsr_ctx* ctx, const rsr_model* model, const rsr_system* sys,
                                 const rsr_stage1_params* params, const uint8_t* lower0,
                                 int64_t R_L0, const uint8_t* upper0, int64_t R_U0,
                                 uint8_t* lower, int64_t cap_L, uint8_t* upper, int64_t cap_U,
                                 rsr_stage1_result* result) {
    try {
        return run_stage1(ctx, model, sys, params, lower0, R_L0, upper0, R_U0, lower, cap_L, upper,
                          cap_U, result);
    } catch (const std::bad_alloc&) {
        return s1_fail(ctx, RSR_ENOMEM, "host allocation");
    }
}
