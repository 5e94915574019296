// LABEL-mode classification on a consistent reference set (no upper row lies
// below a lower row, so the first match on either side decides a sample; see
// k_cascade.hip) whose rows constrain few components.
//
// A reference row of s-t connectivity is a path or a cut: of the hundreds of
// packed bits it has to be tested on, a dozen or two are set.  The popcount
// and matrix-core forms test all of them.  Here the samples are transposed, so
// that one 32-bit word holds the same bit of 32 samples, and a row is tested
// by AND-ing the words of its own bits only: "x >= r" for 32 samples is the AND
// of the columns in t(r), "x <= r" the AND of the complements of the columns
// in NOT t(r).
//
// A block holds the columns of one tile of samples (128 << lg of them) in LDS,
// [column][4 << lg words].  A lane reads 16 bytes, 128 samples, of a column;
// 1 << lg neighbouring lanes share a row, so a wave tests 64 >> lg rows at once,
// which have about the same length, as rows are stored by increasing size.  A
// row is a list of 16-bit column numbers in chunks of four.  64 rows form a
// slice, [chunk][row], as long as its longest row: shorter rows repeat their
// last column and a last slice its last row, which changes no result.  So the
// chunks of a row are at a fixed stride, and a wave has those of its next rows
// in flight while it tests the present ones.  It leaves its rows once no sample
// they could decide is left: of a cut's edges only the first few are read.
//
// The rows are taken in rounds [0, first), [first, first * growth), ...  Round
// 0 tests every sample, writes every flag and lists the undecided samples;
// the next rounds test the listed ones, gathered into tiles again.  The tile
// size of a round is chosen on the device from the number of samples left, so
// that every block has one.  The lists need no counters: a block appends to a
// region of its own and leaves the region's extent, and the next round forms
// the prefix sums of the extents.  The last round shares the rows of a tile
// out over several blocks, since a decided sample's flag can be written by
// whoever finds the match (all of them write the same value).
//
// Bound: LDS reads, 16 bytes per 128 samples and bit.  Random columns of a tile
// read at 90 (128 samples) to 183 (2048 samples) bytes per clock and CU, and
// the rounds of 295-edge rows reach about 60 % of that; the rest is the chain
// of launch, prefix sums, gather and transpose of the short later rounds.
// Measured per LABEL call, against the cascade's popcount round 0 and FP4
// rounds: 119-node / 295-edge network, 1e4 rows per side, 1e6 samples 150 -> 62
// us; 500 / 1250, 4e4 rows, 262144 samples 343 -> 60 us; three-state edges,
// 2.5e4 rows, 1e6 samples 343 -> 91 us.
#include "bits.h"

namespace rsr {
namespace {

using namespace bits;

constexpr int kThreads = 512;
constexpr int kMinWaves = 4;  // per SIMD: two blocks in a CU
constexpr int kWaves = kThreads / 64;
static_assert(kSparseRegions <= kThreads, "a thread per region");
constexpr int kMaxLg = kSparseTiles - 1;  // tiles of at most 2048 samples
constexpr int kMaxWords = 4 << kMaxLg;
// Rows per side of round 0 (whole slices) and growth of the later rounds.  Round
// 0 takes 4 us more for 256 rows than for 128 at 1e6 samples and saves that in
// the later rounds (three-state case: 98 -> 91 us, the 295-edge one 61 -> 62);
// growth 8 adds a launch of 15 us on 2.5e4 rows and growth 32 leaves the last
// round too many samples (global connectivity: 113 -> 128 us).
constexpr int kFirst = 256;
constexpr int kGrowth = 16;
// Blocks per tile of the last round, and its least tile.
constexpr int kLastShare = 8;
constexpr int kLastLg = 2;

struct SparseRows {
    const uint32_t* off;    // [slices + 1] first chunk of a slice
    const uint2* chunks;    // [chunk][64 rows], four 16-bit columns each
    int s0, s1;             // the round's slices
};

// Sample words as the tiles take them: W words, PW per plane of n components.
struct SparseShape {
    int W, PW, n;
    int lg;                 // tile size (round 0) or the largest one
};

// The list of undecided samples, in per-block regions, by sample index.
struct SparseList {
    int2* regions;          // (start, count) of each block's region
    int32_t* h;             // index in its job
    int32_t* job;           // its job (only with a job table)
    uint32_t* words;        // [W][stride], or null: to be read from the job's array
    int64_t stride;
};

// LDS before the tile: match and valid masks and the waves' totals.
struct TileMasks {
    uint32_t low[kMaxWords], up[kMaxWords], valid[kMaxWords];
    uint32_t wave[kWaves];
};
static_assert(sizeof(TileMasks) % 16 == 0, "the tile behind it is read 16 bytes at a time");

__device__ __forceinline__ uint32_t nibble_bytes(uint32_t v) {
    return (v * 0x00204081u) & 0x01010101u;  // bit c -> byte c
}

// Four 32-bit words at a 4-byte aligned address.
struct __attribute__((packed, aligned(4))) Quad {
    uint32_t v[4];
};

// Takes every shares-th of one side's slices, from number `share` on, on the
// tile, the WAVES waves taking units of 64 >> lg rows in turn.  For each unit u
// start(a, u) gives the samples to test (four words per lane); UPPER rows keep
// those whose columns are all ones, lower rows those whose columns are all
// zeros, and done(a) takes what is left and says whether to stop.
template <bool UPPER, int WAVES, class Start, class Done>
__device__ __forceinline__ void test_rows(const SparseRows& rows, int share, int shares, int wave,
                                          const uint4* __restrict__ tile, int lg, Start start,
                                          Done done) {
    constexpr int kAhead = 4;  // chunks of a row that are loaded ahead
    const int lane = threadIdx.x & 63;
    const uint4* mine = tile + (lane & ((1 << lg) - 1));
    struct Unit {
        const uint2* at;
        int chunks;
        uint2 id[kAhead];
    };
    auto fetch = [&](Unit& un, int u) {
        const int slice = rows.s0 + share + (u >> lg) * shares;
        const uint32_t first = rows.off[slice];
        un.chunks = static_cast<int>(rows.off[slice + 1] - first);
        un.at = rows.chunks + static_cast<int64_t>(first) * 64 +
                (((u & ((1 << lg) - 1)) << (6 - lg)) + (lane >> lg));
#pragma unroll
        for (int k = 0; k < kAhead; ++k) un.id[k] = un.at[64 * min(k, un.chunks - 1)];
    };
    uint32_t a[4];
    auto test2 = [&](uint2 x, uint2 y) {
        const uint4 v0 = mine[(x.x & 0xFFFFu) << lg], v1 = mine[(x.x >> 16) << lg];
        const uint4 v2 = mine[(x.y & 0xFFFFu) << lg], v3 = mine[(x.y >> 16) << lg];
        const uint4 v4 = mine[(y.x & 0xFFFFu) << lg], v5 = mine[(y.x >> 16) << lg];
        const uint4 v6 = mine[(y.y & 0xFFFFu) << lg], v7 = mine[(y.y >> 16) << lg];
        // acc & p & q, or acc & ~p & ~q.
        auto both = [](uint32_t acc, uint32_t p, uint32_t q) {
            return __builtin_amdgcn_bitop3_b32(acc, p, q, UPPER ? 0x80 : 0x10);
        };
        a[0] = both(both(both(both(a[0], v0.x, v1.x), v2.x, v3.x), v4.x, v5.x), v6.x, v7.x);
        a[1] = both(both(both(both(a[1], v0.y, v1.y), v2.y, v3.y), v4.y, v5.y), v6.y, v7.y);
        a[2] = both(both(both(both(a[2], v0.z, v1.z), v2.z, v3.z), v4.z, v5.z), v6.z, v7.z);
        a[3] = both(both(both(both(a[3], v0.w, v1.w), v2.w, v3.w), v4.w, v5.w), v6.w, v7.w);
    };
    auto alive = [&] { return __any((a[0] | a[1] | a[2] | a[3]) != 0u) != 0; };
    const int units = ((rows.s1 - rows.s0 - share + shares - 1) / shares) << lg;
    int u = wave;
    if (u >= units) return;
    Unit next;
    fetch(next, u);
    for (; u < units; u += WAVES) {
        const Unit cur = next;
        if (u + WAVES < units) fetch(next, u + WAVES);
        start(a, u);
        test2(cur.id[0], cur.id[1]);
        if (cur.chunks > 2 && alive()) {
            uint2 more[2];
            more[0] = cur.at[64 * min(4, cur.chunks - 1)];
            more[1] = cur.at[64 * min(5, cur.chunks - 1)];
            test2(cur.id[2], cur.id[3]);
            for (int c = 4; c < cur.chunks && alive(); c += 2) {
                const uint2 x = more[0], y = more[1];
                more[0] = cur.at[64 * min(c + 2, cur.chunks - 1)];
                more[1] = cur.at[64 * min(c + 3, cur.chunks - 1)];
                test2(x, y);
            }
        }
        if (done(a)) return;
    }
}

// LABEL: open = this lane's undecided samples, hit = those a row matched.
template <bool UPPER>
__device__ __forceinline__ void test_side(const SparseRows& rows, int share, int shares, int wave,
                                          const uint4* __restrict__ tile, int lg,
                                          uint32_t (&open)[4], uint32_t (&hit)[4]) {
    test_rows<UPPER, kWaves>(
        rows, share, shares, wave, tile, lg,
        [&](uint32_t (&a)[4], int) {
#pragma unroll
            for (int q = 0; q < 4; ++q) a[q] = open[q];
        },
        [&](uint32_t (&a)[4]) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                hit[q] |= a[q];
                open[q] &= ~a[q];
            }
            return !__any((open[0] | open[1] | open[2] | open[3]) != 0u);
        });
}

// Clears the masks of a tile of `count` samples (1 << lg times 128 at most).
// Sample s of a tile is bit 4 (s / (4 words)) + s mod 4 of word (s / 4) mod
// words: four neighbouring samples of a word come with one 16-byte load, and
// a wave's loads are contiguous.
__device__ __forceinline__ void clear_masks(TileMasks& m, int lg, int count) {
    const int words = 4 << lg, tid = threadIdx.x;
    if (tid >= words) return;
    uint32_t v = 0xFFFFFFFFu;
    if (count < 32 * words) {
        v = 0;
#pragma unroll 1
        for (int b = 0; b < 32; ++b)
            if ((b >> 2) * 4 * words + 4 * tid + (b & 3) < count) v |= 1u << b;
    }
    m.valid[tid] = v;
    m.low[tid] = m.up[tid] = 0u;
}

// Columns of word w from the transposed words of position l.
__device__ __forceinline__ void put_columns(uint32_t (&a)[32], const SparseShape& p, int lg, int w,
                                            int l, uint32_t* tile) {
    transpose32(a);
    const int plane = w / p.PW, i0 = 32 * (w - plane * p.PW);
    const int bits = p.n - i0;
    uint32_t* at = tile + ((plane * p.n + i0) << (lg + 2)) + l;
    if (bits >= 32) {
#pragma unroll
        for (int k = 0; k < 32; ++k) at[k << (lg + 2)] = a[k];
    } else {
#pragma unroll
        for (int k = 0; k < 31; ++k)
            if (k < bits) at[k << (lg + 2)] = a[k];
    }
}

// The columns of samples h0 .. h0 + count - 1 of the array xs [W][N].
__device__ __forceinline__ void load_columns(const uint32_t* __restrict__ xs, int64_t N, int64_t h0,
                                             int count, const SparseShape& p, int lg,
                                             uint32_t* tile) {
    const int words = 4 << lg, size = 32 * words;
    for (int task = threadIdx.x; task < p.W << (lg + 2); task += blockDim.x) {
        const int w = task >> (lg + 2), l = task & (words - 1);
        const uint32_t* src = xs + w * N + h0;
        uint32_t a[32];
        if (count == size) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const Quad q = *reinterpret_cast<const Quad*>(src + 4 * l + i * 4 * words);
#pragma unroll
                for (int c = 0; c < 4; ++c) a[4 * i + c] = q.v[c];
            }
        } else {  // past the end: the last sample again, which is not valid
#pragma unroll
            for (int b = 0; b < 32; ++b)
                a[b] = src[min((b >> 2) * 4 * words + 4 * l + (b & 3), count - 1)];
        }
        put_columns(a, p, lg, w, l, tile);
    }
}

// Both sides' rows on the tile; the matches go to the masks.
__device__ __forceinline__ void test_tile(const SparseRows& low, const SparseRows& up, int share,
                                          int shares, const uint4* tile, int lg, TileMasks& m) {
    const int l4 = 4 * (threadIdx.x & ((1 << lg) - 1));
    uint32_t open[4], hit_l[4] = {0, 0, 0, 0}, hit_u[4] = {0, 0, 0, 0};
#pragma unroll
    for (int q = 0; q < 4; ++q) open[q] = m.valid[l4 + q];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // The lower side's units go round the waves the other way.
    test_side<true>(up, share, shares, wave, tile, lg, open, hit_u);
    test_side<false>(low, share, shares, kWaves - 1 - wave, tile, lg, open, hit_l);
    // One lane per word: lanes of a wave on one address would serialise.
    const bool first = (threadIdx.x & 63) < (1u << lg);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        hit_l[q] = or_rows(hit_l[q], lg);
        hit_u[q] = or_rows(hit_u[q], lg);
        if (first && hit_l[q]) atomicOr(&m.low[l4 + q], hit_l[q]);
        if (first && hit_u[q]) atomicOr(&m.up[l4 + q], hit_u[q]);
    }
}

// The tile's results for samples 4 tid .. 4 tid + 3, as four bits each.
struct Quartet {
    uint32_t low, up, left;
};
__device__ __forceinline__ Quartet quartet(const TileMasks& m, int lg) {
    Quartet r{0, 0, 0};
    const int tid = threadIdx.x, words = 4 << lg;
    if (tid < 8 * words) {
        const int l = tid & (words - 1), shift = 4 * (tid >> (lg + 2));
        r.low = (m.low[l] >> shift) & 15u;
        r.up = (m.up[l] >> shift) & 15u & ~r.low;
        r.left = (m.valid[l] >> shift) & 15u & ~(r.low | r.up);
    }
    return r;
}

// Rank of this thread's first set bit of `left` among the block's, in sample
// order; `all` = their number.  Every thread of the block must call it.
__device__ __forceinline__ uint32_t block_rank(uint32_t left, uint32_t* s_wave, uint32_t& all) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t rank = 0, wave_total = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const uint64_t m = __ballot((left >> c) & 1u);
        rank += static_cast<uint32_t>(__popcll(m & ((1ull << lane) - 1ull)));
        wave_total += static_cast<uint32_t>(__popcll(m));
    }
    if (lane == 0) s_wave[wave] = wave_total;
    __syncthreads();
    all = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const uint32_t t = s_wave[w];
        rank += w < wave ? t : 0u;
        all += t;
    }
    return rank;
}

// The job of tile t: the last one whose first tile is not behind it.  Every lane
// of the wave must call it, with one t.
__device__ __forceinline__ int job_of_tile(const int64_t* __restrict__ first_tile, int n_jobs,
                                           int64_t t) {
    int lo = 0, len = n_jobs;  // it is one of [lo, lo + len)
    while (len > 1) {
        const int step = (len + 63) >> 6, k = (threadIdx.x & 63) * step;
        const uint64_t before = __ballot(k == 0 || (k < len && first_tile[lo + k] <= t));
        const int at = (__popcll(before) - 1) * step;
        lo += at;
        len = min(step, len - at);
    }
    return lo;
}

// Round 0: every sample of the segment.  Tiles do not cross jobs; first_tile: see
// JobTiles (unused without a job table).  A block takes a range of tiles, whose
// samples are consecutive.
__global__ __launch_bounds__(kThreads, kMinWaves) void k_sparse_first(
    SegSrc seg, const int64_t* __restrict__ first_tile, int64_t tiles, SparseShape p,
    SparseRows low, SparseRows up, SparseList dst, int last) {
    extern __shared__ uint4 lds4[];
    TileMasks& m = *reinterpret_cast<TileMasks*>(lds4);
    uint4* tile = lds4 + sizeof(TileMasks) / 16;
    const int tid = threadIdx.x, lg = p.lg, words = 4 << lg, size = 32 * words;
    const int64_t per_block = (tiles + gridDim.x - 1) / gridDim.x;
    const int64_t t_end = min(tiles, (blockIdx.x + 1) * per_block);
    int64_t region = 0;
    uint32_t listed = 0;
    int64_t t = blockIdx.x * per_block;
    int job = 0;
    if (seg.jobs && t < t_end) job = job_of_tile(first_tile, seg.n_jobs, t);
    for (bool begin = true; t < t_end; ++t, begin = false) {
        if (seg.jobs && job + 1 < seg.n_jobs && first_tile[job + 1] <= t) ++job;
        const int64_t h0 = (t - (seg.jobs ? first_tile[job] : 0)) << (7 + lg);
        const uint32_t* xs = global_ptr(seg.jobs ? seg.jobs[job].samples : seg.samples);
        uint8_t* flags = global_ptr(seg.jobs ? seg.jobs[job].flags : seg.flags);
        const int64_t N = seg.jobs ? seg.jobs[job].N : seg.N;
        if (begin) region = (seg.jobs ? seg.offsets[job] : 0) + h0;
        const int count = static_cast<int>(min(static_cast<int64_t>(size), N - h0));
        clear_masks(m, lg, count);
        load_columns(xs, N, h0, count, p, lg, reinterpret_cast<uint32_t*>(tile));
        __syncthreads();
        test_tile(low, up, 0, 1, tile, lg, m);
        __syncthreads();
        const Quartet r = quartet(m, lg);
        const int s4 = 4 * tid;
        if (s4 < count) {
            const uint32_t f = nibble_bytes(r.low) | (nibble_bytes(r.up) << 1);
            uint8_t* fl = flags + h0 + s4;
            if (s4 + 4 <= count && (reinterpret_cast<uintptr_t>(fl) & 3u) == 0)
                *reinterpret_cast<uint32_t*>(fl) = f;
            else
                for (int c = 0; c < 4 && s4 + c < count; ++c) fl[c] = static_cast<uint8_t>(f >> (8 * c));
        }
        if (!last) {
            uint32_t all;
            int64_t slot = region + listed + block_rank(r.left, m.wave, all);
            for (uint32_t b = r.left; b; b &= b - 1, ++slot) {
                dst.h[slot] = static_cast<int32_t>(h0 + s4 + __ffs(static_cast<int>(b)) - 1);
                if (seg.jobs) dst.job[slot] = job;
            }
            listed += all;
        }
        __syncthreads();
    }
    if (!last && tid == 0)
        dst.regions[blockIdx.x] = make_int2(static_cast<int>(region), static_cast<int>(listed));
}

// A later round, on the listed samples.  The last round shares a tile's rows
// out over blocks (a decided sample's flag can be written by whoever finds the
// match, since all of them write the same value) and lists nothing.
__global__ __launch_bounds__(kThreads, kMinWaves) void k_sparse_list(SegSrc seg, SparseShape p,
                                                                     SparseRows low, SparseRows up,
                                                                     SparseList src, int n_src,
                                                                     SparseList dst, int last) {
    extern __shared__ uint4 lds4[];
    TileMasks& m = *reinterpret_cast<TileMasks*>(lds4);
    uint32_t* s_prefix = reinterpret_cast<uint32_t*>(lds4 + sizeof(TileMasks) / 16);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

    // Prefix sums of the source regions.
    const uint32_t extent = tid < n_src ? static_cast<uint32_t>(src.regions[tid].y) : 0u;
    uint32_t run = extent;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl_up(run, d);
        if (lane >= d) run += o;
    }
    if (lane == 63) m.wave[wave] = run;
    __syncthreads();
    uint32_t total = 0;
    run -= extent;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const uint32_t t = m.wave[w];
        run += w < wave ? t : 0u;
        total += t;
    }
    s_prefix[tid] = run;
    __syncthreads();

    // The smallest tile that gives every block at most one.  In the last
    // round the blocks share the tiles' rows instead, so there are fewer tiles.
    const int grid = static_cast<int>(gridDim.x);
    const int most = last ? (grid + kLastShare - 1) / kLastShare : grid;
    int lg = last ? min(kLastLg, p.lg) : 0;
    while (lg < p.lg && static_cast<int>((total + (128u << lg) - 1) >> (7 + lg)) > most) ++lg;
    const int words = 4 << lg, size = 32 * words;
    const int tiles = static_cast<int>((total + size - 1) >> (7 + lg));
    uint32_t* s_slot = s_prefix + kThreads;
    uint32_t* s_words = s_slot + size;             // [W][size]
    uint4* tile = reinterpret_cast<uint4*>(s_words + p.W * size);

    int shares = 1, item, item_end, item_step;
    if (last) {
        const int slices = max(low.s1 - low.s0, up.s1 - up.s0);
        shares = max(1, min(grid / max(tiles, 1), slices));
        item = blockIdx.x;
        item_end = tiles * shares;
        item_step = grid;
    } else {
        const int per_block = (tiles + grid - 1) / grid;
        item = blockIdx.x * per_block;
        item_end = min(tiles, item + per_block);
        item_step = 1;
    }
    const int64_t region = static_cast<int64_t>(item) << (7 + lg);
    uint32_t listed = 0;
    for (; item < item_end; item += item_step) {
        const int t = item / shares, share = item - t * shares;
        const uint32_t j0 = static_cast<uint32_t>(t) << (7 + lg);
        const int count = static_cast<int>(min(static_cast<uint32_t>(size), total - j0));
        clear_masks(m, lg, count);
        for (int s = tid; s < size; s += kThreads) {
            // Past the end: the last sample again, which is not valid.
            const uint32_t j = j0 + min(s, count - 1);
            int a = 0, b = n_src - 1;
            while (a < b) {
                const int mid = (a + b + 1) >> 1;
                if (s_prefix[mid] <= j) a = mid;
                else b = mid - 1;
            }
            s_slot[s] = static_cast<uint32_t>(src.regions[a].x) + (j - s_prefix[a]);
        }
        __syncthreads();
        // A thread reads every step-th word of a sample, eight in flight.
        const int lanes = min(size, kThreads), w0 = tid / lanes, step = kThreads / lanes;
        for (int s = tid & (lanes - 1); s < size; s += lanes) {
            const uint32_t slot = s_slot[s];
            const uint32_t* xs;
            int64_t stride = src.stride;
            if (src.words) {
                xs = src.words + slot;
            } else {
                xs = seg_words(seg, seg.jobs ? src.job[slot] : 0, stride) + src.h[slot];
            }
            xs = global_ptr(xs);
            for (int w = w0; w < p.W; w += 8 * step) {
                uint32_t v[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = xs[min(w + k * step, p.W - 1) * stride];
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    if (w + k * step < p.W) s_words[(w + k * step) * size + s] = v[k];
            }
        }
        __syncthreads();
        for (int task = tid; task < p.W << (lg + 2); task += kThreads) {
            const int w = task >> (lg + 2), l = task & (words - 1);
            const uint4* from = reinterpret_cast<const uint4*>(s_words + w * size) + l;
            uint32_t a[32];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const uint4 q = from[i * words];
                a[4 * i] = q.x;
                a[4 * i + 1] = q.y;
                a[4 * i + 2] = q.z;
                a[4 * i + 3] = q.w;
            }
            put_columns(a, p, lg, w, l, reinterpret_cast<uint32_t*>(tile));
        }
        __syncthreads();
        test_tile(low, up, share, shares, tile, lg, m);
        __syncthreads();
        const Quartet r = quartet(m, lg);
        for (uint32_t b = r.low | r.up; b; b &= b - 1) {
            const int c = __ffs(static_cast<int>(b)) - 1;
            const uint32_t slot = s_slot[4 * tid + c];
            seg_flags(seg, seg.jobs ? src.job[slot] : 0)[src.h[slot]] =
                static_cast<uint8_t>((r.low >> c) & 1u ? 1 : 2);
        }
        if (!last) {
            // The tile is done with: its place takes the survivors' numbers.
            uint16_t* s_list = reinterpret_cast<uint16_t*>(tile);
            uint32_t all;
            const int64_t base = region + listed;
            uint32_t rank = block_rank(r.left, m.wave, all);
            for (uint32_t b = r.left; b; b &= b - 1, ++rank) {
                const int s = 4 * tid + __ffs(static_cast<int>(b)) - 1;
                const uint32_t from = s_slot[s];
                dst.h[base + rank] = src.h[from];
                if (seg.jobs) dst.job[base + rank] = src.job[from];
                s_list[rank] = static_cast<uint16_t>(s);
            }
            __syncthreads();
            for (int w = wave; w < p.W; w += kWaves)
                for (uint32_t k = lane; k < all; k += 64)
                    dst.words[w * dst.stride + base + k] = s_words[w * size + s_list[k]];
            listed += all;
        }
        __syncthreads();
    }
    if (!last && tid == 0)
        dst.regions[blockIdx.x] = make_int2(static_cast<int>(region), static_cast<int>(listed));
}

// COUNT: every row against every sample.  A block of 16 waves has a CU to
// itself, with the largest tile that fits.  Measured against the FP4 matrix
// cores: 1e5 + 1e5 rows of 295 bits with 5 % and 10 % of them set, 1e6 samples,
// 17.4 -> 5.0 ms (LDS reads at about half their rate of 183 bytes per clock and
// CU, beside four vector instructions per read).
//
// The number of matching rows of each side is kept in bit-sliced form:
// bit i of s[l] is bit l of the count of this lane's sample i.  Rows come in
// one at a time; the first kPending levels pair them up before a full adder,
// so that most rows cost one or two of them and only every eighth ripples up.
constexpr int kCountThreads = 1024;
constexpr int kCountWaves = kCountThreads / 64;
constexpr int kCountBits = 8, kPending = 3;
struct RowCounter {
    uint32_t s[kCountBits][4], pending[kPending][4];
    int rows;  // added since the last flush (wave-uniform), below 1 << kCountBits

    __device__ __forceinline__ void clear() {
        rows = 0;
#pragma unroll
        for (int l = 0; l < kCountBits; ++l)
#pragma unroll
            for (int q = 0; q < 4; ++q) s[l][q] = 0;
    }
    // Adds c at level l and up.
    template <int L>
    __device__ __forceinline__ void ripple(uint32_t (&c)[4]) {
#pragma unroll
        for (int l = L; l < kCountBits; ++l)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t t = s[l][q] & c[q];
                s[l][q] ^= c[q];
                c[q] = t;
            }
    }
    template <int L>
    __device__ __forceinline__ void push(uint32_t (&c)[4]) {
        if constexpr (L == kPending) {
            ripple<L>(c);
        } else if ((rows >> L) & 1) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t a = s[L][q], b = pending[L][q];
                s[L][q] = __builtin_amdgcn_bitop3_b32(a, b, c[q], 0x96);  // sum
                c[q] = __builtin_amdgcn_bitop3_b32(a, b, c[q], 0xE8);     // carry
            }
            push<L + 1>(c);
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) pending[L][q] = c[q];
        }
    }
    template <int L>
    __device__ __forceinline__ void settle() {
        if constexpr (L < kPending) {
            if ((rows >> L) & 1) ripple<L>(pending[L]);
            settle<L + 1>();
        }
    }
    __device__ __forceinline__ void add(uint32_t (&a)[4]) {
        push<0>(a);
        ++rows;
    }
    // Adds the counts to the tile's and starts again.
    __device__ __forceinline__ void flush(uint32_t* counts, int lg) {
        if (rows == 0) return;
        settle<0>();
        const int l4 = 4 * (threadIdx.x & ((1 << lg) - 1)), stride = 16 << lg;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll 4
            for (int b = 0; b < 32; ++b) {
                uint32_t v = 0;
#pragma unroll
                for (int l = 0; l < kCountBits; ++l) v |= ((s[l][q] >> b) & 1u) << l;
                if (v) atomicAdd(&counts[(b >> 2) * stride + 4 * (l4 + q) + (b & 3)], v);
            }
        clear();
    }
};

template <bool UPPER>
__device__ __forceinline__ void count_side(const SparseRows& rows, int64_t R, int wave,
                                           const uint4* tile, int lg, const uint32_t (&valid)[4],
                                           uint32_t* counts) {
    const int in_unit = (threadIdx.x & 63) >> lg;
    RowCounter n;
    n.clear();
    test_rows<UPPER, kCountWaves>(
        rows, 0, 1, wave, tile, lg,
        [&](uint32_t (&a)[4], int u) {
            // The last slice repeats its last row.
            const bool row = (static_cast<int64_t>(u) << (6 - lg)) + in_unit < R;
#pragma unroll
            for (int q = 0; q < 4; ++q) a[q] = row ? valid[q] : 0u;
        },
        [&](uint32_t (&a)[4]) {
            if (__any((a[0] | a[1] | a[2] | a[3]) != 0u)) n.add(a);
            if (n.rows == (1 << kCountBits) - 1) n.flush(counts, lg);
            return false;
        });
    n.flush(counts, lg);
}

// Every row against every sample: counts of matching rows per side (match, or
// null) and the flags: both bits (COUNT), or the lower one's precedence (LABEL
// on rows that are not a consistent set).
__global__ __launch_bounds__(kCountThreads, 4) void k_sparse_count(
    const uint32_t* __restrict__ xs, int64_t N, SparseShape p, SparseRows low, int64_t R_L,
    SparseRows up, int64_t R_U, int label, uint8_t* __restrict__ flags, uint32_t* __restrict__ match) {
    extern __shared__ uint4 lds4[];
    TileMasks& m = *reinterpret_cast<TileMasks*>(lds4);
    const int tid = threadIdx.x, lg = p.lg, words = 4 << lg, size = 32 * words;
    uint32_t* n_low = reinterpret_cast<uint32_t*>(lds4 + sizeof(TileMasks) / 16);
    uint32_t* n_up = n_low + size;
    uint4* tile = reinterpret_cast<uint4*>(n_up + size);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t tiles = (N + size - 1) >> (7 + lg);
    for (int64_t t = blockIdx.x; t < tiles; t += gridDim.x) {
        const int64_t h0 = t << (7 + lg);
        const int count = static_cast<int>(min(static_cast<int64_t>(size), N - h0));
        clear_masks(m, lg, count);
        for (int s = tid; s < size; s += kCountThreads) n_low[s] = n_up[s] = 0;
        load_columns(xs, N, h0, count, p, lg, reinterpret_cast<uint32_t*>(tile));
        __syncthreads();
        uint32_t valid[4];
        const int l4 = 4 * (tid & ((1 << lg) - 1));
#pragma unroll
        for (int q = 0; q < 4; ++q) valid[q] = m.valid[l4 + q];
        count_side<true>(up, R_U, wave, tile, lg, valid, n_up);
        count_side<false>(low, R_L, kCountWaves - 1 - wave, tile, lg, valid, n_low);
        __syncthreads();
        for (int s = tid; s < count; s += kCountThreads) {
            const uint32_t nl = n_low[s], nu = n_up[s];
            flags[h0 + s] = static_cast<uint8_t>((nl ? 1 : 0) | (nu && !(label && nl) ? 2 : 0));
            if (match) {
                match[2 * (h0 + s)] = nl;
                match[2 * (h0 + s) + 1] = nu;
            }
        }
        __syncthreads();
    }
}

// LDS of a block with tiles of 128 << lg samples.  In a list round the tile's
// place also takes the survivors' numbers, two bytes a sample: more than the
// columns of fewer than 16 bits.
size_t lds_bytes(const rsr_refs* refs, int lg, bool first) {
    const size_t bits = static_cast<size_t>(refs->n) * (refs->K - 1);
    const size_t size = size_t{128} << lg;
    if (first) return sizeof(TileMasks) + (bits << (lg + 4));
    return sizeof(TileMasks) + ((bits < 16 ? 16 : bits) << (lg + 4)) +
           4 * (kThreads + size + refs->W * size);
}

// Largest tile whose block shares a CU's 160 KB of LDS with another one.
int largest_lg(const rsr_refs* refs, bool first) {
    int lg = kMaxLg;
    while (lg > 0 && lds_bytes(refs, lg, first) > 80 * 1024) --lg;
    return lg;
}

// LDS of a block of k_sparse_count, which has a CU to itself.
size_t count_lds(const rsr_refs* refs, int lg) {
    return sizeof(TileMasks) + 8 * (size_t{128} << lg) +
           (static_cast<size_t>(refs->n) * (refs->K - 1) << (lg + 4));
}

}  // namespace

hipError_t launch_sparse_count(hipStream_t st, const rsr_refs* refs, const uint32_t* d_samples,
                               int64_t N, int mode, int cus, uint8_t* d_flags, uint32_t* d_match) {
    SparseShape p{refs->W, plane_words(refs->n), refs->n, 0};
    // The largest tile that fits and leaves every CU one.
    while (p.lg < kMaxLg && count_lds(refs, p.lg + 1) <= 156 * 1024 &&
           ((N + (256 << p.lg) - 1) >> (8 + p.lg)) >= cus)
        ++p.lg;
    auto side = [](const uint32_t* off, const uint16_t* idx, int64_t R) {
        return SparseRows{off, reinterpret_cast<const uint2*>(idx), 0, static_cast<int>((R + 63) / 64)};
    };
    const int64_t tiles = (N + (128 << p.lg) - 1) >> (7 + p.lg);
    hipLaunchKernelGGL(k_sparse_count, dim3(static_cast<unsigned>(tiles < cus ? tiles : cus)),
                       dim3(kCountThreads), count_lds(refs, p.lg), st, d_samples, N, p,
                       side(refs->d_lower_off, refs->d_lower_idx, refs->R_L), refs->R_L,
                       side(refs->d_upper_off, refs->d_upper_idx, refs->R_U), refs->R_U,
                       mode == RSR_LABEL ? 1 : 0, d_flags, d_match);
    return hipGetLastError();
}

hipError_t launch_dom_sparse(hipStream_t st, const rsr_refs* refs, const SegSrc& seg,
                             const JobTiles& tiles, const CascadeBuffers& cb, int cus) {
    const int grid = 2 * cus < kSparseRegions ? 2 * cus : kSparseRegions;
    const int64_t rows = refs->R_L > refs->R_U ? refs->R_L : refs->R_U;
    int64_t lo = 0, hi = kFirst;
    SparseShape p{refs->W, plane_words(refs->n), refs->n, 0};
    int src_blocks = 0;
    for (int round = 0;; ++round) {
        // A round takes the rows that would leave the next one less than half
        // as many as its own.
        const bool last = hi + hi / 2 >= rows;
        auto side = [&](const uint32_t* off, const uint16_t* idx, int64_t R) {
            const int slices = static_cast<int>((R + 63) / 64);
            return SparseRows{off, reinterpret_cast<const uint2*>(idx),
                              static_cast<int>(lo / 64 < slices ? lo / 64 : slices),
                              static_cast<int>(last || hi / 64 > slices ? slices : hi / 64)};
        };
        const SparseRows low = side(refs->d_lower_off, refs->d_lower_idx, refs->R_L);
        const SparseRows up = side(refs->d_upper_off, refs->d_upper_idx, refs->R_U);
        auto list = [&](int k) {
            return SparseList{reinterpret_cast<int2*>(cb.sparse_regions[k & 1]), cb.index[k & 1],
                              reinterpret_cast<int32_t*>(cb.match[k & 1]),
                              k > 0 ? cb.words[k & 1] : nullptr, cb.stride};
        };
        if (round == 0) {
            const int largest = largest_lg(refs, true);
            int64_t n_tiles;
            for (;; ++p.lg) {
                n_tiles = seg.jobs ? tiles.host[p.lg * tiles.stride + seg.n_jobs]
                                   : (seg.total + (128 << p.lg) - 1) >> (7 + p.lg);
                if (p.lg == largest || n_tiles <= grid) break;
            }
            src_blocks = static_cast<int>(n_tiles < grid ? n_tiles : grid);
            hipLaunchKernelGGL(k_sparse_first, dim3(src_blocks), dim3(kThreads),
                               lds_bytes(refs, p.lg, true), st, seg,
                               seg.jobs ? tiles.dev + p.lg * tiles.stride : nullptr, n_tiles, p, low,
                               up, list(0), last ? 1 : 0);
        } else {
            p.lg = largest_lg(refs, false);
            hipLaunchKernelGGL(k_sparse_list, dim3(grid), dim3(kThreads),
                               lds_bytes(refs, p.lg, false), st, seg, p, low, up, list(round - 1),
                               src_blocks, list(round), last ? 1 : 0);
            src_blocks = grid;
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess || last) return e;
        lo = hi;
        hi *= kGrowth;
    }
}

}  // namespace rsr
