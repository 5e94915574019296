// Monte Carlo sampler: 32-bit uniform words compared against integer
// inverse-CDF thresholds, written straight into the packed thermometer layout
// (word-major [W][N]; see rsr.h).
//
// The word of component i is two 16-bit halves at position i mod 8 of two
// Philox4x32-10 blocks (counter word 0 = i div 8, and the same with bit 31
// set).  Its high half decides u >= C unless it equals the high half of C,
// which happens with probability 2^-16 per threshold: only then is the second
// block drawn.  So one Philox block serves eight components, and the result
// is exactly that of comparing the full 32-bit word.
//
// One thread draws one sample (or, for few samples, a range of its words);
// the finished words are stored with coalesced 32-bit stores (lanes hold
// consecutive samples).  The thresholds are identical for every thread of a
// job, so they are read through the scalar cache.
//
// Bound: the vector ALU, by the 32 x 32 -> 64-bit products of Philox.  Two
// things keep them and the compares few:
//  * The counter of a block is (block, low(h), high(h), stream): only low(h)
//    differs between the lanes of a wave, and only `block` between the blocks
//    of a sample.  So the first round has no per-lane product at all, the
//    second one per sample (shared by its blocks), the third one and the
//    fourth to tenth two per block: 15 instead of 20 per eight components.
//    Everything else of the first rounds stays in scalar registers, which is
//    why those rounds use plain XORs: the three-input XOR builtin is a vector
//    instruction and would pull the uniform values into vector registers.
//  * A dword of a block is the high halves of two neighbouring components, so
//    packed 16-bit instructions compare both at once (classes2): three
//    instructions per pair give "above" and "tie" as a two-bit field.  Only a
//    threshold below 2^16 (a state less likely than 1.5e-5) is not decided by
//    its field 0, so such components come as a mask, and one of them that is
//    not "above" redraws its block, 2 in 2^16 times.  (1e6 samples of 295
//    components that fail with probability 1e-6: 65 us, 62 with 0.01; 247 where
//    every sample redraws the blocks of such a word.)
// Measured, against 20 products per block and one compare per component and
// threshold: 1e6 samples of 295 two-state components 84 -> 67 us, of 295
// three-state ones 114 -> 84 us; a plan's 48 jobs of 65536 samples of 240
// components 77 -> 57 us (there the keys and thresholds were vector loads).
#include "rsr_internal.h"

namespace rsr {
namespace {

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));

constexpr uint32_t kM0 = 0xD2511F53u, kM1 = 0xCD9E8D57u;
constexpr uint32_t kW0 = 0x9E3779B9u, kW1 = 0xBB67AE85u;

constexpr int kSampleBlock = 256;
// Waves per SIMD below which the words of a sample are split over blocks: one
// wave issues a product every few of its cycles, and 1e5 samples are 1.5 waves
// per SIMD, the second round half empty (1e5 samples of 295 components: 17.5 us
// whole, 11.5 us split).
constexpr int kWavesPerSimd = 8;

// Three-input XOR as one v_bitop3_b32 (truth table 0x96).
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ uint32_t hi32(uint64_t v) { return static_cast<uint32_t>(v >> 32); }
__device__ __forceinline__ uint32_t lo32(uint64_t v) { return static_cast<uint32_t>(v); }

struct Philox4 {
    uint32_t v[4];
};

// Philox4x32-10 (Salmon, Moraes, Dror & Shaw, SC'11, section 3.2) of any
// counter: the tie path only.
__device__ __forceinline__ Philox4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2,
                                                 uint32_t c3, uint32_t k0, uint32_t k1) {
#pragma unroll 1
    for (int round = 0; round < 10; ++round) {
        const uint64_t a = static_cast<uint64_t>(kM0) * c0;
        const uint64_t b = static_cast<uint64_t>(kM1) * c2;
        const uint32_t y0 = xor3(hi32(b), c1, k0);
        const uint32_t y2 = xor3(hi32(a), c3, k1);
        c1 = lo32(b);
        c3 = lo32(a);
        c0 = y0;
        c2 = y2;
        k0 += kW0;
        k1 += kW1;
    }
    return {{c0, c1, c2, c3}};
}

// What the Philox blocks of one sample share: the second round's product of
// the word that holds low(h).  ghi = high(h) is the same in every lane.
struct SampleKey {
    uint32_t k0, k1, ghi, stream;  // uniform
    uint32_t b1;                   // uniform: low word of round 1's second product
    uint32_t ah, al;               // per lane: round 2's first product
};

__device__ __forceinline__ SampleKey sample_key(uint32_t k0, uint32_t k1, uint32_t glo,
                                                uint32_t ghi, uint32_t stream) {
    SampleKey s;
    s.k0 = k0;
    s.k1 = k1;
    s.ghi = ghi;
    s.stream = stream;
    const uint64_t b = static_cast<uint64_t>(kM1) * ghi;
    s.b1 = lo32(b);
    const uint64_t a = static_cast<uint64_t>(kM0) * (glo ^ (hi32(b) ^ k0));
    s.ah = hi32(a);
    s.al = lo32(a);
    return s;
}

// Philox4x32-10 of counter (block, low(h), high(h), stream), `block` uniform.
__device__ __forceinline__ Philox4 philox_block(const SampleKey& s, uint32_t block) {
    // Round 1: both products uniform.
    const uint64_t a1 = static_cast<uint64_t>(kM0) * block;
    const uint32_t y2 = hi32(a1) ^ s.stream ^ s.k1, c3 = lo32(a1);
    // Round 2: the first product is the sample's, the second uniform.
    uint32_t k0 = s.k0 + kW0, k1 = s.k1 + kW1;
    const uint64_t b2 = static_cast<uint64_t>(kM1) * y2;
    const uint32_t t0 = hi32(b2) ^ s.b1 ^ k0;   // uniform
    const uint32_t t2 = s.ah ^ (c3 ^ k1);
    const uint32_t t1 = lo32(b2);               // uniform; the fourth word is s.al
    // Round 3: the first product uniform.
    k0 += kW0;
    k1 += kW1;
    const uint64_t a3 = static_cast<uint64_t>(kM0) * t0;
    const uint64_t b3 = static_cast<uint64_t>(kM1) * t2;
    uint32_t v0 = hi32(b3) ^ (t1 ^ k0), v1 = lo32(b3);
    uint32_t v2 = s.al ^ (hi32(a3) ^ k1);
    // Round 4: the fourth word is still uniform.
    k0 += kW0;
    k1 += kW1;
    const uint64_t a4 = static_cast<uint64_t>(kM0) * v0;
    const uint64_t b4 = static_cast<uint64_t>(kM1) * v2;
    v0 = xor3(hi32(b4), v1, k0);
    v2 = hi32(a4) ^ (lo32(a3) ^ k1);
    v1 = lo32(b4);
    uint32_t v3 = lo32(a4);
#pragma unroll
    for (int round = 4; round < 10; ++round) {
        k0 += kW0;
        k1 += kW1;
        const uint64_t a = static_cast<uint64_t>(kM0) * v0;
        const uint64_t b = static_cast<uint64_t>(kM1) * v2;
        v0 = xor3(hi32(b), v1, k0);
        v2 = xor3(hi32(a), v3, k1);
        v1 = lo32(b);
        v3 = lo32(a);
    }
    return {{v0, v1, v2, v3}};
}

// Runs f(u) for every distinct value u of v among the wave's active lanes, in
// the lanes that hold it, with u in a scalar register.  The loop's exit is
// uniform (left per lane, u would be a vector value behind it), and the empty
// asm hides that the argument equals v, which the compiler would otherwise use
// instead.
template <class F>
__device__ __forceinline__ void for_uniform(uint32_t v, F f) {
    uint64_t todo = __ballot(1);
    while (todo) {
        const uint32_t u =
            __builtin_amdgcn_readlane(v, __ffsll(static_cast<unsigned long long>(todo)) - 1);
        uint32_t scalar = u;
        asm("" : "+s"(scalar));
        const bool mine = v == u;
        todo &= ~__ballot(mine);
        if (mine) f(scalar);
    }
}

// min(max(u - s, 0), 2) of both 16-bit halves: 0 below, 1 tie, 2 above (see
// pack_threshold in rsr_internal.h).
__device__ __forceinline__ uint32_t classes2(uint32_t u, uint32_t s) {
    const u16x2 d = __builtin_elementwise_sub_sat(__builtin_bit_cast(u16x2, u),
                                                  __builtin_bit_cast(u16x2, s));
    const u16x2 two = {2, 2};
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(d, two));
}

// The tie path: the words of one sample again, in the blocks that hold a tie
// (bit q of `blocks`), by the full 32-bit compare.
template <int KM1>
__device__ __forceinline__ void redraw_blocks(const uint64_t* __restrict__ thresh, int n, int base,
                                           uint32_t blocks, uint32_t key0, uint32_t key1,
                                           uint32_t glo, uint32_t ghi, uint32_t stream,
                                           uint32_t (&acc)[KM1]) {
    while (blocks) {
        const int q = __ffs(static_cast<int>(blocks)) - 1;
        blocks &= blocks - 1;
        const int i0 = base + 8 * q;
        if (i0 >= n) return;
        const uint32_t c0 = static_cast<uint32_t>(i0 >> 3);
        const Philox4 hi = philox4x32_10(c0, glo, ghi, stream, key0, key1);
        const Philox4 lo = philox4x32_10(c0 | 0x80000000u, glo, ghi, stream, key0, key1);
#pragma unroll
        for (int s = 0; s < KM1; ++s) acc[s] &= ~(0xFFu << (8 * q));
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int shift = 16 * (k & 1);
            const uint32_t u = (((hi.v[k >> 1] >> shift) & 0xFFFFu) << 16) |
                               ((lo.v[k >> 1] >> shift) & 0xFFFFu);
            if (i0 + k >= n) break;
#pragma unroll
            for (int s = 0; s < KM1; ++s)
                if (u >= thresh[static_cast<int64_t>(i0 + k) * KM1 + s]) acc[s] |= 1u << (8 * q + k);
        }
    }
}

// Draws words [w0, w1) of every plane of sample index g (low(g) = glo; ghi
// uniform) and stores them in column h of the word-major [W][N] array out.
// KM1 = K - 1 thermometer planes; thresh and pack are the model's two forms of
// the thresholds (rsr_model).
template <int KM1>
__device__ __forceinline__ void draw_words(const uint64_t* __restrict__ thresh,
                                           const uint32_t* __restrict__ pack, int n, int PW,
                                           uint32_t key0, uint32_t key1, uint32_t stream,
                                           uint32_t glo, uint32_t ghi, int w0, int w1, int64_t h,
                                           int64_t N, uint32_t* __restrict__ out) {
    const SampleKey key = sample_key(key0, key1, glo, ghi, stream);
    for (int wi = w0; wi < w1; ++wi) {
        const uint32_t* pw = pack + static_cast<int64_t>(wi) * KM1 * kPackWords;
        // Two-bit fields: blocks 0 and 1 in A, 2 and 3 in B; field 4 (q mod 2)
        // + j of a 16-bit half holds the component of pair j in that half.
        uint32_t A[KM1], B[KM1];
#pragma unroll
        for (int s = 0; s < KM1; ++s) A[s] = B[s] = 0;
        const int groups = min(4, (n - wi * 32 + 7) >> 3);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (q >= groups) break;
            const Philox4 r = philox_block(key, static_cast<uint32_t>(4 * wi + q));
#pragma unroll
            for (int s = 0; s < KM1; ++s)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint32_t e = classes2(r.v[j], pw[s * kPackWords + 4 * q + j]);
                    if (q < 2) A[s] |= e << (2 * (4 * (q & 1) + j));
                    else B[s] |= e << (2 * (4 * (q & 1) + j));
                }
        }
        uint32_t acc[KM1], tie = 0, low = 0;
#pragma unroll
        for (int s = 0; s < KM1; ++s) {
            // "Above" is the upper bit of a field: A's to the even bits, B's at
            // the odd ones.  Bit 16 h + 8 (q mod 2) + 2 j + (q div 2) then
            // holds component 8 q + 2 j + h: swap index bits 4 and 0.
            const uint32_t t = ((A[s] >> 1) & 0x55555555u) | (B[s] & 0xAAAAAAAAu);
            const uint32_t x = ((t >> 15) ^ t) & 0x0000AAAAu;
            acc[s] = (t ^ x ^ (x << 15)) | pw[s * kPackWords + 16];
            tie |= (A[s] & 0x55555555u) | ((B[s] & 0x55555555u) << 1);
            low |= pw[s * kPackWords + 17] & ~acc[s];
        }
        if (tie | low) {
            // Tie bit 16 h + 8 (q mod 2) + 2 j + (q div 2): fold j and h.
            uint32_t f = tie | (tie >> 16);
            f |= f >> 4;
            f |= f >> 2;
            uint32_t blocks = (f & 1u) | ((f >> 7) & 2u) | ((f << 1) & 4u) | ((f >> 6) & 8u);
#pragma unroll
            for (int q = 0; q < 4; ++q) blocks |= (low >> (8 * q)) & 0xFFu ? 1u << q : 0u;
            redraw_blocks<KM1>(thresh, n, wi * 32, blocks, key0, key1, glo, ghi, stream, acc);
        }
#pragma unroll
        for (int s = 0; s < KM1; ++s) out[static_cast<int64_t>(s * PW + wi) * N + h] = acc[s];
    }
}

// blockIdx.y takes `per_y` words of every sample.
template <int KM1>
__global__ __launch_bounds__(kSampleBlock) void k_sample(const uint64_t* __restrict__ thresh,
                                                         const uint32_t* __restrict__ pack, int n,
                                                         int PW, int per_y, uint32_t key0,
                                                         uint32_t key1, uint32_t stream_id,
                                                         uint64_t first, int64_t N,
                                                         uint32_t* __restrict__ out) {
    const int64_t h = static_cast<int64_t>(blockIdx.x) * kSampleBlock + threadIdx.x;
    if (h >= N) return;
    const int w0 = static_cast<int>(blockIdx.y) * per_y;
    const int w1 = min(PW, w0 + per_y);
    const uint64_t g = first + static_cast<uint64_t>(h);
    const uint32_t ghi = hi32(g);
    // One pass, two where the wave's sample indices cross a multiple of 2^32.
    for_uniform(hi32(g), [&](uint32_t ghi) {
        draw_words<KM1>(thresh, pack, n, PW, key0, key1, stream_id, lo32(g), ghi, w0, w1, h, N, out);
    });
}

// Every sample of every job of a plan segment (same n and K), grid-stride
// over the segment's global index.
template <int KM1>
__global__ __launch_bounds__(kSampleBlock) void k_sample_jobs(const JobDev* __restrict__ jobs,
                                                              const int64_t* __restrict__ offsets,
                                                              int n_jobs, int64_t total, int n,
                                                              int PW) {
    SegSrc seg{};
    seg.jobs = jobs;
    seg.offsets = offsets;
    seg.n_jobs = n_jobs;
    seg.total = total;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kSampleBlock;
    for (int64_t g = static_cast<int64_t>(blockIdx.x) * kSampleBlock + threadIdx.x; g < total;
         g += stride) {
        int j;
        int64_t h;
        seg_locate(seg, g, j, h);
        // One pass per job among the wave's samples (one, but at job borders),
        // so that its key and thresholds are scalar.
        for_uniform(static_cast<uint32_t>(j), [&](uint32_t ju) {
            const JobDev& jd = jobs[ju];
            draw_words<KM1>(jd.thresh, jd.pack, n, PW, static_cast<uint32_t>(jd.seed),
                            static_cast<uint32_t>(jd.seed >> 32), jd.stream_id,
                            static_cast<uint32_t>(h), 0u, 0, PW, h, jd.N, jd.samples);
        });
    }
}

template <int KM1>
hipError_t launch_k(hipStream_t st, const rsr_model* m, uint64_t seed, uint32_t stream_id,
                    uint64_t first, int64_t N, int cus, uint32_t* d_samples) {
    const int PW = plane_words(m->n);
    const int64_t blocks = (N + kSampleBlock - 1) / kSampleBlock;
    // Few samples: their words are split over blocks until every SIMD has
    // about kWavesPerSimd waves.
    const int64_t want = static_cast<int64_t>(cus) * kWavesPerSimd;  // blocks: 4 waves on 4 SIMDs
    int64_t split = blocks >= want ? 1 : (want + blocks - 1) / blocks;
    if (split > PW) split = PW;
    const int per_y = static_cast<int>((PW + split - 1) / split);
    const dim3 grid(static_cast<unsigned>(blocks), static_cast<unsigned>((PW + per_y - 1) / per_y));
    hipLaunchKernelGGL(k_sample<KM1>, grid, dim3(kSampleBlock), 0, st, m->d_thresh, m->d_pack, m->n,
                       PW, per_y, static_cast<uint32_t>(seed), static_cast<uint32_t>(seed >> 32),
                       stream_id, first, N, d_samples);
    return hipGetLastError();
}

template <int KM1>
hipError_t launch_jobs_k(hipStream_t st, int n, const JobDev* jobs, const int64_t* offsets,
                         int n_jobs, int64_t total, int grid_cap) {
    int64_t blocks = (total + kSampleBlock - 1) / kSampleBlock;
    if (blocks > grid_cap) blocks = grid_cap;
    if (blocks < 1) blocks = 1;
    hipLaunchKernelGGL(k_sample_jobs<KM1>, dim3(static_cast<unsigned>(blocks)), dim3(kSampleBlock),
                       0, st, jobs, offsets, n_jobs, total, n, plane_words(n));
    return hipGetLastError();
}

}  // namespace

hipError_t launch_sample_jobs(hipStream_t st, int n, int K, const JobDev* jobs,
                              const int64_t* offsets, int n_jobs, int64_t total, int grid_cap) {
    switch (K - 1) {
#define RSR_K_CASE(k) \
    case k: return launch_jobs_k<k>(st, n, jobs, offsets, n_jobs, total, grid_cap);
        RSR_K_CASE(1) RSR_K_CASE(2) RSR_K_CASE(3) RSR_K_CASE(4) RSR_K_CASE(5) RSR_K_CASE(6)
        RSR_K_CASE(7) RSR_K_CASE(8) RSR_K_CASE(9) RSR_K_CASE(10) RSR_K_CASE(11) RSR_K_CASE(12)
        RSR_K_CASE(13) RSR_K_CASE(14) RSR_K_CASE(15)
#undef RSR_K_CASE
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_sample(hipStream_t st, const rsr_model* m, uint64_t seed, uint32_t stream_id,
                         uint64_t first, int64_t N, int cus, uint32_t* d_samples) {
    switch (m->K - 1) {
#define RSR_K_CASE(k) \
    case k: return launch_k<k>(st, m, seed, stream_id, first, N, cus, d_samples);
        RSR_K_CASE(1) RSR_K_CASE(2) RSR_K_CASE(3) RSR_K_CASE(4) RSR_K_CASE(5) RSR_K_CASE(6)
        RSR_K_CASE(7) RSR_K_CASE(8) RSR_K_CASE(9) RSR_K_CASE(10) RSR_K_CASE(11) RSR_K_CASE(12)
        RSR_K_CASE(13) RSR_K_CASE(14) RSR_K_CASE(15)
#undef RSR_K_CASE
        default: return hipErrorInvalidValue;
    }
}

}  // namespace rsr
