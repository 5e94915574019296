// Stage-2 evaluation of the system function on the samples left
// unclassified (section 3.5).
//
// k_label turns flags into Y (lower -> 0, upper -> 1) and lists the samples
// without a flag (sample_list.h).
//
// k_connect evaluates s-t connectivity at a level and global connectivity, 64
// samples per wavefront: an edge is a 64-bit word of the samples in which it is
// usable, a node one of the samples in which it is marked, and a step over an
// edge works on all 64 at once.  The lanes own the edges (lane l edges l, l +
// 64, ...) and sweep over them; the words of a sample are read by its lane and
// transposed through LDS.
//
//   s-t: two node sets grow, from the source and from the sink.  An edge
//     between them connects the sample; a set that stops growing is a whole
//     component, and then they never meet.
//   global, level 1: one set grows, from node `from`, and has to reach every
//     node.
//   global, level 2 (two-edge-connected): the first search also notes, per
//     sample, the edges that marked a node: a spanning tree.  Every other usable
//     edge lies on a cycle with tree edges, so its ends are joined by two
//     edge-disjoint paths, which is an equivalence.  A class grows from node
//     `to` over usable non-tree edges, and to a node with two usable edges into
//     it.  What is left outside hangs on by ears: one edge from the class into
//     the outside is taken as a seed, its component outside is searched
//     (noting every node's marking edge), and a node with an edge into the
//     class other than its marking edge closes a cycle and joins.  If none
//     does, the seed is a bridge.  A node with fewer than two usable edges
//     settles most of the others at the start.  Where ears would take many
//     rounds the samples go to k_walk2, one sample per wave (launch_global2).
//
// With few groups of samples a whole block works on one (a sweep is a chain of
// dependent LDS steps per 64 or 256 edges), else a wave.
//
// Bound: the latency of that chain for few samples, LDS throughput for many.
// Measured against one sample per wave with a bit per node and edge: plain
// Monte Carlo of 1e6 samples on 119 nodes / 295 edges 1188 -> 68 us; two-edge-
// connectivity of 125784 listed samples on 59 / 262, with the listing, 429 ->
// 84 us.  The listing took 32 to 67 us with one atomic per wave on a common
// counter and takes about 6 us for 1e6 flags.
#include <climits>

#include "bits.h"
#include "graph_search.h"
#include "sample_list.h"

namespace rsr {
namespace {

using namespace bits;

constexpr int kLabelBlock = 256;
constexpr int kLabelWaves = kLabelBlock / 64;
constexpr int kLabelTile = 4 * kLabelBlock;
// LDS that k_connect's blocks may take of a CU (160 KB less their static part).
constexpr size_t kConnectLds = 152 * 1024;
// A block works on one group up to this many groups per CU, from this many
// edges on: four waves shorten a sweep's chain, but every sweep then takes four
// block barriers (label and evaluation, block against wave per group: 1229
// samples of 1250 edges 29 / 41 us, 45 of 465 edges 20 / 21, 2696 of 295 edges
// 25 / 21).
constexpr int kBlockGroups = 2;
constexpr int kBlockEdges = 448;

__device__ __forceinline__ uint32_t flag_y(uint32_t f) {  // four flags at a time
    return (f >> 1) & ~f & 0x01010101u;
}

// A block takes `chunk` consecutive samples (whole tiles), four neighbouring
// ones per thread.
__global__ __launch_bounds__(kLabelBlock) void k_label(SegSrc seg, int64_t chunk, SampleList list) {
    __shared__ uint32_t s_wave[2][kLabelWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t begin = blockIdx.x * chunk;
    const int64_t end = begin + chunk < seg.total ? begin + chunk : seg.total;
    uint32_t listed = 0;
    int parity = 0;
    for (int64_t t0 = begin; t0 < end; t0 += kLabelTile, parity ^= 1) {
        const int64_t t1 = t0 + kLabelTile < end ? t0 + kLabelTile : end;
        const int64_t g = t0 + 4 * tid;
        // A tile usually lies in one job.
        int job = 0, job1 = 0;
        int64_t h0 = t0, h1;
        if (seg.jobs) {
            seg_locate(seg, t0, job, h0);
            seg_locate(seg, t1 - 1, job1, h1);
        }
        uint32_t f = 0x01010101u;
        const uint8_t* fl = seg_flags(seg, job) + h0 + 4 * tid;
        uint8_t* Y = seg_Y(seg, job) + h0 + 4 * tid;
        if (job == job1 && g + 4 <= t1 &&
            ((reinterpret_cast<uintptr_t>(fl) | reinterpret_cast<uintptr_t>(Y)) & 3u) == 0) {
            f = *reinterpret_cast<const uint32_t*>(fl);
            *reinterpret_cast<uint32_t*>(Y) = flag_y(f);
        } else {
            for (int c = 0; c < 4 && g + c < t1; ++c) {
                int j;
                int64_t h;
                seg_locate(seg, g + c, j, h);
                const uint32_t b = seg_flags(seg, j)[h];
                f = (f & ~(0xFFu << (8 * c))) | (b << (8 * c));
                seg_Y(seg, j)[h] = static_cast<uint8_t>(flag_y(b));
            }
        }
        const uint32_t open = ~(f | (f >> 1)) & 0x01010101u;  // bit 8 c: sample g + c
        uint32_t rank = 0, total = 0;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint64_t m = __ballot((open >> (8 * c)) & 1u);
            rank += static_cast<uint32_t>(__popcll(m & ((1ull << lane) - 1ull)));
            total += static_cast<uint32_t>(__popcll(m));
        }
        if (lane == 0) s_wave[parity][wave] = total;
        __syncthreads();
        total = 0;
#pragma unroll
        for (int w = 0; w < kLabelWaves; ++w) {
            const uint32_t t = s_wave[parity][w];
            rank += w < wave ? t : 0u;
            total += t;
        }
        int32_t* out = list.index + begin + listed + rank;
        for (uint32_t m = open; m; m &= m - 1)
            *out++ = static_cast<int32_t>(g + (__ffs(static_cast<int>(m)) - 1) / 8);
        listed += total;
    }
    if (tid == 0) list.regions[blockIdx.x] = make_int2(static_cast<int>(begin), static_cast<int>(listed));
    // The regions of the blocks that are not there are empty.
    if (blockIdx.x == 0)
        for (int r = gridDim.x + tid; r < kListRegions; r += kLabelBlock)
            list.regions[r] = make_int2(0, 0);
}

enum Connect { kSt, kGlobal1, kGlobal2 };

// Y of a sample that k_connect<kGlobal2> leaves to k_walk2.
constexpr uint32_t kOpen = 2;

// u64 words of a wave's edge table: the 32 edges of a packed word and two
// words of padding, so that the transpose's stores do not all hit one bank.
constexpr int kWordSlots = 34;
__host__ __device__ inline int edge_slots(int n_edges) { return ((n_edges + 31) >> 5) * kWordSlots; }
__device__ __forceinline__ int edge_slot(int e) { return e + 2 * (e >> 5); }

typedef uint32_t __attribute__((may_alias)) Word32;
typedef uint32_t Word128 __attribute__((ext_vector_type(4), may_alias));

// LDS of a group of samples in u64: usable edges and two node sets (one at
// level 1 of global connectivity); level 2 adds the tree, the edges that
// marked either end in an ear search, and the samples with a seed.
__host__ __device__ inline int connect_slots(int kind, int n_nodes, int n_edges) {
    const int slots = edge_slots(n_edges) * (kind == kGlobal2 ? 4 : 1) +
                      n_nodes * (kind == kGlobal1 ? 1 : 2) + (kind == kGlobal2 ? 1 : 0);
    return (slots + 1) & ~1;
}

__device__ __forceinline__ void or_into(uint64_t* p, uint64_t v) {
    atomicOr(reinterpret_cast<unsigned long long*>(p), static_cast<unsigned long long>(v));
}
__device__ __forceinline__ uint64_t or_fetch(uint64_t* p, uint64_t v) {
    return atomicOr(reinterpret_cast<unsigned long long*>(p), static_cast<unsigned long long>(v));
}
__device__ __forceinline__ uint64_t peek(const uint64_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The lanes that work on a group of samples: a wave, or (BLOCK) the block.
template <bool BLOCK>
struct Team {
    uint64_t* red;  // [waves] LDS
    __device__ int lane() const { return BLOCK ? threadIdx.x : threadIdx.x & 63; }
    __device__ int size() const { return BLOCK ? blockDim.x : 64; }
    __device__ void sync() const {
        if (BLOCK) __syncthreads();
        else graph::wave_sync();
    }
    // At the head of a loop whose body begins with a loop over nodes or edges:
    // makes the lanes without one wait for the others.  Otherwise the compiler may
    // send the lanes that skip a like loop before this one straight to the sync
    // behind it, and on, ahead of the lanes that still write (as with fewer than 64
    // nodes).
    __device__ void converge() const { __builtin_amdgcn_wave_barrier(); }
    __device__ bool any(bool b) const {  // also orders the LDS accesses
        if (BLOCK) return __syncthreads_or(b ? 1 : 0) != 0;
        graph::wave_sync();
        return __any(b) != 0;
    }
    __device__ uint64_t or_all(uint64_t v) const {
        uint64_t w = or_wave(v);
        if (!BLOCK) return w;
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = w;
        __syncthreads();
        w = 0;
        for (unsigned k = 0; k < blockDim.x >> 6; ++k) w |= red[k];
        __syncthreads();
        return w;
    }
};

struct Group {
    uint64_t* x;          // usable edges, by edge_slot
    const uint32_t* ends; // [n_edges] u | v << 16
    int n_edges, n_nodes;
};

template <bool BLOCK>
__device__ __forceinline__ uint64_t all_nodes(const Team<BLOCK>& tm, const Group& g,
                                              const uint64_t* set) {
    uint64_t missing = 0;
    for (int v = tm.lane(); v < g.n_nodes; v += tm.size()) missing |= ~peek(set + v);
    return ~tm.or_all(missing);
}

template <bool BLOCK>
__device__ __forceinline__ void set_nodes(const Team<BLOCK>& tm, const Group& g, uint64_t* set,
                                          int one) {
    for (int v = tm.lane(); v < g.n_nodes; v += tm.size()) set[v] = v == one ? ~0ull : 0ull;
}

// Samples whose source and sink the usable edges connect.
template <bool BLOCK>
__device__ __forceinline__ uint64_t st_connected(const Team<BLOCK>& tm, const Group& g, int source,
                                                 int sink, uint64_t* S, uint64_t* T) {
    set_nodes(tm, g, S, source);
    set_nodes(tm, g, T, sink);
    tm.sync();
    uint64_t conn = 0;
    while (true) {
        uint64_t meet = 0, grew_s = 0, grew_t = 0;
        for (int e = tm.lane(); e < g.n_edges; e += tm.size()) {
            const uint64_t use = g.x[edge_slot(e)] & ~conn;
            if (use == 0) continue;
            const uint32_t uv = g.ends[e], u = uv & 0xFFFFu, v = uv >> 16;
            const uint64_t su = peek(S + u), sv = peek(S + v), tu = peek(T + u), tv = peek(T + v);
            meet |= use & ((su & tv) | (sv & tu));
            const uint64_t ns = (su ^ sv) & use, nt = (tu ^ tv) & use;
            if (ns) {  // one end has it already
                or_into(S + u, ns);
                or_into(S + v, ns);
            }
            if (nt) {
                or_into(T + u, nt);
                or_into(T + v, nt);
            }
            grew_s |= ns;
            grew_t |= nt;
        }
        tm.sync();
        conn |= tm.or_all(meet);
        if ((tm.or_all(grew_s) & tm.or_all(grew_t) & ~conn) == 0) return conn;
    }
}

// Grows S over the usable edges until nothing changes; with TREE, notes the
// marking edges.
template <bool TREE, bool BLOCK>
__device__ __forceinline__ void grow_all(const Team<BLOCK>& tm, const Group& g, uint64_t* S,
                                         uint64_t* tree) {
    bool changed = true;
    while (changed) {
        changed = false;
        for (int e = tm.lane(); e < g.n_edges; e += tm.size()) {
            const uint64_t use = g.x[edge_slot(e)];
            const uint32_t uv = g.ends[e], u = uv & 0xFFFFu, v = uv >> 16;
            const uint64_t su = peek(S + u), sv = peek(S + v);
            const uint64_t to_u = sv & ~su & use, to_v = su & ~sv & use;
            if ((to_u | to_v) == 0) continue;
            changed = true;
            uint64_t won = 0;
            if (to_u) won |= to_u & ~or_fetch(S + u, to_u);
            if (to_v) won |= to_v & ~or_fetch(S + v, to_v);
            if (TREE) tree[edge_slot(e)] |= won;
        }
        changed = tm.any(changed);
    }
}

// Of the connected samples `open`, those without a bridge; on return `open` holds
// the ones that `ears` rounds of ears have not settled.  tree: a spanning tree's
// edges; S, T: node sets; by_u, by_v: edge tables; seeded: one word.
template <bool BLOCK>
__device__ __forceinline__ uint64_t bridgeless(const Team<BLOCK>& tm, const Group& g, int from,
                                               int ears, uint64_t& open, const uint64_t* tree,
                                               uint64_t* S, uint64_t* T, uint64_t* by_u,
                                               uint64_t* by_v, uint64_t* seeded) {
    // Two usable edges at every node?  S counts the first, T the second.
    set_nodes(tm, g, S, -1);
    set_nodes(tm, g, T, -1);
    tm.sync();
    for (int e = tm.lane(); e < g.n_edges; e += tm.size()) {
        const uint64_t use = g.x[edge_slot(e)];
        const uint32_t uv = g.ends[e], u = uv & 0xFFFFu, v = uv >> 16;
        if (u == v) continue;
        const uint64_t two_u = use & or_fetch(S + u, use), two_v = use & or_fetch(S + v, use);
        if (two_u) or_into(T + u, two_u);
        if (two_v) or_into(T + v, two_v);
    }
    tm.sync();
    open &= all_nodes(tm, g, T);
    if (open == 0) return 0;
    // The class of `from`, in S; T holds a node's first tree edge into it.
    set_nodes(tm, g, S, from);
    bool changed = true;
    while (changed) {
        tm.converge();
        set_nodes(tm, g, T, -1);
        tm.sync();
        changed = false;
        for (int e = tm.lane(); e < g.n_edges; e += tm.size()) {
            const uint64_t use = g.x[edge_slot(e)], in_tree = tree[edge_slot(e)];
            const uint32_t uv = g.ends[e], u = uv & 0xFFFFu, v = uv >> 16;
            const uint64_t su = peek(S + u), sv = peek(S + v);
            uint64_t to_u = sv & ~su & use, to_v = su & ~sv & use;
            if ((to_u | to_v) == 0) continue;
            const uint64_t tu = to_u & in_tree, tv = to_v & in_tree;
            to_u &= ~in_tree;
            to_v &= ~in_tree;
            if (tu) to_u |= tu & or_fetch(T + u, tu);
            if (tv) to_v |= tv & or_fetch(T + v, tv);
            if (to_u) or_into(S + u, to_u);
            if (to_v) or_into(S + v, to_v);
            changed = changed || (to_u | to_v) != 0;
        }
        changed = tm.any(changed);
    }
    uint64_t good = open & all_nodes(tm, g, S);
    open &= ~good;
    // Ears: T marks the searched nodes outside, by_u and by_v the edges that
    // marked their end u or v.
    for (int round = 0; open && round < ears; ++round) {
        tm.converge();
        set_nodes(tm, g, T, -1);
        for (int e = tm.lane(); e < g.n_edges; e += tm.size())
            by_u[edge_slot(e)] = by_v[edge_slot(e)] = 0;
        if (tm.lane() == 0) *seeded = 0;
        tm.sync();
        for (int e = tm.lane(); e < g.n_edges; e += tm.size()) {
            const uint32_t uv = g.ends[e], u = uv & 0xFFFFu, v = uv >> 16;
            const uint64_t su = S[u], sv = S[v], leaves = (su ^ sv) & g.x[edge_slot(e)] & open;
            if ((leaves & ~peek(seeded)) == 0) continue;
            const uint64_t won = leaves & ~or_fetch(seeded, leaves);
            const uint64_t to_u = won & sv, to_v = won & su;
            if (to_u) {
                or_into(T + u, to_u);
                by_u[edge_slot(e)] = to_u;
            }
            if (to_v) {
                or_into(T + v, to_v);
                by_v[edge_slot(e)] = to_v;
            }
        }
        tm.sync();
        uint64_t joined = 0;
        changed = true;
        while (changed) {
            changed = false;
            for (int e = tm.lane(); e < g.n_edges; e += tm.size()) {
                const int i = edge_slot(e);
                const uint64_t use = g.x[i] & open;
                const uint32_t uv = g.ends[e], u = uv & 0xFFFFu, v = uv >> 16;
                const uint64_t su = peek(S + u), sv = peek(S + v);
                const uint64_t near = use & ~(su & sv);
                if (near == 0) continue;  // inside the class
                const uint64_t cu = peek(T + u), cv = peek(T + v);
                // The search goes on outside; a marked node joins by an edge
                // from the class that is not its marking edge, any node by a
                // usable non-tree edge.
                const uint64_t mark_u = near & cv & ~cu & ~su & ~sv;
                const uint64_t mark_v = near & cu & ~cv & ~su & ~sv;
                const uint64_t in_tree = tree[i];
                const uint64_t join_u = near & sv & ~su & ((cu & ~by_u[i]) | ~in_tree);
                const uint64_t join_v = near & su & ~sv & ((cv & ~by_v[i]) | ~in_tree);
                if ((mark_u | mark_v | join_u | join_v) == 0) continue;
                changed = true;
                if (mark_u) by_u[i] |= mark_u & ~or_fetch(T + u, mark_u);
                if (mark_v) by_v[i] |= mark_v & ~or_fetch(T + v, mark_v);
                if (join_u) or_into(S + u, join_u);
                if (join_v) or_into(S + v, join_v);
                joined |= join_u | join_v;
            }
            changed = tm.any(changed);
        }
        // No node joined: the seed is a bridge.
        open &= tm.or_all(joined);
        const uint64_t whole = open & all_nodes(tm, g, S);
        good |= whole;
        open &= ~whole;
    }
    return good;
}

template <int KIND, bool BLOCK>
__device__ __forceinline__ void eval_groups(const SegSrc& seg, int PW, int plane, Group g, int from,
                                            int to, int ears, const SampleList& list,
                                            const uint32_t* before, int which, int64_t total,
                                            Team<BLOCK> tm) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6;
    const int slots = edge_slots(g.n_edges);
    uint64_t* tree = g.x + slots;
    uint64_t* S = KIND == kGlobal2 ? g.x + 4 * slots : tree;
    uint64_t* T = S + g.n_nodes;
    // The edge table is written and read in words of 4, 8 and 16 bytes.
    Word32* x32 = reinterpret_cast<Word32*>(g.x);
    const int64_t groups = (total + 63) >> 6;
    const int64_t first = BLOCK ? blockIdx.x : static_cast<int64_t>(blockIdx.x) * waves + wave;
    const int64_t step = BLOCK ? gridDim.x : static_cast<int64_t>(gridDim.x) * waves;
    for (int64_t group = first; group < groups; group += step) {
        // Lane = sample (past the end the last one again): its words, then the
        // transpose, in place, of 32 samples by 32 edges per lane.
        const int64_t j = group * 64 + lane;
        const bool valid = j < total;
        const int64_t jc = valid ? j : total - 1;
        const int64_t at = which == RSR_ALL ? jc : list_at(list, before, static_cast<uint32_t>(jc));
        int job;
        int64_t h, stride;
        seg_locate(seg, at, job, h);
        const uint32_t* xs = global_ptr(seg_words(seg, job, stride));
        xs += static_cast<int64_t>(plane) * PW * stride + h;
        const int w_step = BLOCK ? waves : 1;
        for (int w0 = BLOCK ? wave : 0; w0 < PW; w0 += 8 * w_step) {
            uint32_t v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = xs[min(w0 + k * w_step, PW - 1) * stride];
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (w0 + k * w_step < PW) x32[(w0 + k * w_step) * 2 * kWordSlots + lane] = v[k];
        }
        tm.sync();
        for (int t = tm.lane(); t < 2 * PW; t += tm.size()) {
            const int w = t >> 1, half = t & 1;
            uint32_t a[32];
            const Word128* rows = reinterpret_cast<const Word128*>(x32 + w * 2 * kWordSlots + 32 * half);
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const Word128 q = rows[i];
                a[4 * i] = q.x;
                a[4 * i + 1] = q.y;
                a[4 * i + 2] = q.z;
                a[4 * i + 3] = q.w;
            }
            transpose32(a);
            // Both halves of a word are read before either is written: they
            // are neighbouring lanes.
            graph::wave_sync();
#pragma unroll
            for (int k = 0; k < 32; ++k) x32[w * 2 * kWordSlots + 2 * k + half] = a[k];
        }
        tm.sync();

        uint64_t up, open = 0;
        if (KIND == kSt) {
            up = st_connected(tm, g, from, to, S, T);
        } else {
            if (KIND == kGlobal2)
                for (int e = tm.lane(); e < g.n_edges; e += tm.size()) tree[edge_slot(e)] = 0;
            set_nodes(tm, g, S, from);
            tm.sync();
            grow_all<KIND == kGlobal2>(tm, g, S, tree);
            up = all_nodes(tm, g, S);
            if (KIND == kGlobal2 && up) {
                open = up;
                up = bridgeless(tm, g, to, ears, open, tree, S, T, tree + slots, tree + 2 * slots,
                                T + g.n_nodes);
            }
        }
        if (valid && (!BLOCK || wave == 0))
            global_ptr(seg_Y(seg, job))[h] =
                static_cast<uint8_t>((open >> lane) & 1u ? kOpen : (up >> lane) & 1u);
        tm.sync();
    }
}

template <int KIND>
__global__ __launch_bounds__(256) void k_connect(SegSrc seg, int PW, int plane,
                                                 const uint32_t* __restrict__ edges, int n_edges,
                                                 int n_nodes, int from, int to, int ears,
                                                 SampleList list, int which, int block_groups,
                                                 int few,
                                                 unsigned long long* __restrict__ n_evaluated) {
    extern __shared__ uint64_t lds64[];
    __shared__ uint32_t before[kListRegions + 1];
    __shared__ uint64_t red[4];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = blockDim.x >> 6;
    const int64_t total = which == RSR_ALL ? seg.total : list_prefix(list, before);
    if (blockIdx.x == 0 && tid == 0 && n_evaluated)
        *n_evaluated = static_cast<unsigned long long>(total);
    if (KIND == kGlobal2 && total <= few) return;  // k_walk2 takes them all
    const int64_t groups = (total + 63) >> 6;
    const bool block = groups <= block_groups;
    if (static_cast<int64_t>(blockIdx.x) * (block ? 1 : waves) >= groups) return;  // per block

    uint32_t* s_edges = reinterpret_cast<uint32_t*>(lds64);
    for (int e = tid; e < n_edges; e += blockDim.x) s_edges[e] = edges[e];
    __syncthreads();
    uint64_t* x = lds64 + (((n_edges + 3) >> 2) << 1);
    if (block) {
        eval_groups<KIND>(seg, PW, plane, Group{x, s_edges, n_edges, n_nodes}, from, to, ears, list,
                          before, which, total, Team<true>{red});
    } else {
        x += wave * connect_slots(KIND, n_nodes, n_edges);
        eval_groups<KIND>(seg, PW, plane, Group{x, s_edges, n_edges, n_nodes}, from, to, ears, list,
                          before, which, total, Team<false>{red});
    }
}

constexpr int kWalkBlock = 256;
constexpr int kWalkWaves = kWalkBlock / 64;

// Two-edge-connectivity, one sample per wavefront by the tree-cycle walk of
// graph_search.h: all samples where there are at most `few`, else those that
// k_connect has left open.  Sample j is wave j's modulo the number of waves, so
// that neighbours, which are often open together, go to different ones.
__global__ __launch_bounds__(kWalkBlock) void k_walk2(
    SegSrc seg, const uint32_t* __restrict__ edges, int n_edges, int n_nodes, SampleList list,
    int which, int64_t few, unsigned long long* __restrict__ n_evaluated) {
    extern __shared__ uint32_t lds[];
    uint32_t* s_edges = lds;
    uint32_t* sets = lds + n_edges;
    uint32_t* before = sets + kWalkWaves * graph::global_words(n_nodes, n_edges);  // for a list
    const int64_t total = which == RSR_ALL ? seg.total : list_prefix(list, before);
    if (blockIdx.x == 0 && threadIdx.x == 0 && n_evaluated)
        *n_evaluated = static_cast<unsigned long long>(total);
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int64_t first = static_cast<int64_t>(blockIdx.x) * kWalkWaves;
    if (first >= total) return;  // uniform per block

    for (int e = threadIdx.x; e < n_edges; e += kWalkBlock) s_edges[e] = edges[e];
    __syncthreads();
    const graph::GlobalSets g = graph::global_sets(
        sets + wave * graph::global_words(n_nodes, n_edges), n_nodes, n_edges);
    const int edge_rounds = (n_edges + 63) >> 6;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kWalkWaves;
    for (int64_t j0 = first + wave; j0 < total; j0 += 64 * stride) {
        // Lane l looks at sample j0 + l * stride.
        const int64_t mine = j0 + lane * stride;
        bool todo = mine < total;
        int job = 0;
        int64_t h = 0;
        if (todo) {
            seg_locate(seg, which == RSR_ALL ? mine : list_at(list, before, static_cast<uint32_t>(mine)),
                       job, h);
            if (total > few) todo = global_ptr(seg_Y(seg, job))[h] == kOpen;
        }
        for (uint64_t left = __ballot(todo); left; left &= left - 1) {
            const int from = __ffsll(static_cast<unsigned long long>(left)) - 1;
            const int jb = __builtin_amdgcn_readlane(job, from);
            const int64_t at = static_cast<uint32_t>(
                __builtin_amdgcn_readlane(static_cast<int>(h), from));  // below 2^31
            int64_t xstride;
            const uint32_t* xs = seg_words(seg, jb, xstride);
            uint64_t usable = 0;  // plane 0 = [x >= 1]
            for (int k = 0; k < edge_rounds; ++k) {
                const int e = lane + 64 * k;
                if (e < n_edges) {
                    const uint32_t word = xs[static_cast<int64_t>(e >> 5) * xstride + at];
                    usable |= static_cast<uint64_t>((word >> (e & 31)) & 1u) << k;
                }
            }
            const bool up = graph::two_edge_connected(usable, s_edges, n_edges, n_nodes, g);
            if (lane == 0) seg_Y(seg, jb)[at] = up ? 1 : 0;
            graph::wave_sync();
        }
    }
}

// LDS of a block with the tables of `groups` groups.
size_t connect_lds(int kind, int n_nodes, int n_edges, int groups) {
    return 16 * (static_cast<size_t>(n_edges + 3) >> 2) +
           8 * static_cast<size_t>(connect_slots(kind, n_nodes, n_edges)) * groups;
}

template <int KIND>
hipError_t launch_connect(hipStream_t st, const rsr_system* sys, const SegSrc& seg, int plane,
                          int from, int to, const SampleList& list, int which,
                          uint64_t* d_n_evaluated, int cus, int ears = 0, int few = 0) {
    // Where the tables of a block's four waves would take more than half the LDS,
    // its waves work on one group always.  (With fewer waves a block instead, 20
    // samples of 4096 edges on 100 nodes took 31 us, 12 now, and 5e4 samples 69,
    // 27 now; a ladder of 2101 edges 2311 and 4923, 1053 and 2114 now.)
    constexpr int kWaves = 4;
    const bool one = connect_lds(KIND, sys->n_nodes, sys->n_edges, kWaves) > kConnectLds / 2;
    const size_t lds = connect_lds(KIND, sys->n_nodes, sys->n_edges, one ? 1 : kWaves);
    int per_cu = static_cast<int>(kConnectLds / lds);
    if (per_cu > 8) per_cu = 8;
    if (per_cu < 1) per_cu = 1;
    const int64_t need = (seg.total + 63) / 64, cap = static_cast<int64_t>(per_cu) * cus;
    hipLaunchKernelGGL(k_connect<KIND>, dim3(static_cast<unsigned>(need < cap ? need : cap)),
                       dim3(64 * kWaves), lds, st, seg, plane_words(sys->n_edges), plane,
                       sys->d_edges, sys->n_edges, sys->n_nodes, from, to, ears, list, which,
                       one ? INT_MAX : sys->n_edges >= kBlockEdges ? kBlockGroups * cus : 0, few,
                       reinterpret_cast<unsigned long long*>(d_n_evaluated));
    return hipGetLastError();
}

// Two-edge-connectivity: k_connect, then k_walk2 for what it leaves.
//
// A walk takes a wave the same time whatever the graph is like; k_connect takes 64
// samples at once but in sweeps, some for every step of the graph's depth and,
// with ears, for every round of them.  One round settles one ear per sample, so on
// a ladder or a chain of rings there are as many as links.  Hence:
//  * Ears only on graphs of three edges a node or more, where nearly every sample
//    is settled in a few rounds (5e4 samples, us without / with four rounds: 59
//    nodes and 262 edges 41 / 29, 200 / 800 119 / 42; but a 30 x 30 lattice with 1e3
//    samples 795 / 1069, a ladder of 1402 nodes 5698 / 12298, and 733419 until all
//    were settled).  59 / 262, 125784 listed samples, with the listing: 129 us with
//    two rounds, 99 with four, 84 with eight or more.
//  * All samples to the walk where its waves take them in one go, but on shallow
//    graphs of some size (1000 samples, us by walks / k_connect: 50 nodes and 120
//    edges 14 / 35, 59 / 262 20 / 24, ring of 500 588 / 780, roads of 288 nodes 124
//    / 163; but 119 / 295 33 / 26, 200 / 800 52 / 34, 500 / 1250 175 / 38).
//  * All samples to the walk where one group's tables exceed the LDS.
constexpr int kEars = 8;

hipError_t launch_global2(hipStream_t st, const rsr_system* sys, const SegSrc& seg,
                          const SampleList& list, int which, uint64_t* d_n_evaluated, int cus) {
    const size_t lds = sizeof(uint32_t) *
        (static_cast<size_t>(sys->n_edges) +
         kWalkWaves * static_cast<size_t>(graph::global_words(sys->n_nodes, sys->n_edges)) +
         (which == RSR_ALL ? 0 : kListRegions + 1));
    // The LDS of a CU, taken in pieces of 1280 bytes.
    int64_t per_cu = static_cast<int64_t>(160 * 1024 / ((lds + 1279) / 1280 * 1280));
    if (per_cu > 8) per_cu = 8;
    const int64_t cap = per_cu * cus;
    const int ears = sys->n_edges >= 3 * sys->n_nodes ? kEars : 0;
    const bool shallow = sys->n_nodes >= 96 && sys->n_edges >= 2 * sys->n_nodes && sys->shallow;
    int64_t few = shallow ? 0 : cap * kWalkWaves;
    if (connect_lds(kGlobal2, sys->n_nodes, sys->n_edges, 1) > kConnectLds) few = INT64_MAX;
    if (seg.total > few) {
        const hipError_t e =
            launch_connect<kGlobal2>(st, sys, seg, 0, sys->tree_from, sys->class_from, list, which,
                                     nullptr, cus, ears, static_cast<int>(few));
        if (e != hipSuccess) return e;
    }
    const int64_t need = (seg.total + kWalkWaves - 1) / kWalkWaves;
    hipLaunchKernelGGL(k_walk2, dim3(static_cast<unsigned>(need < cap ? need : cap)),
                       dim3(kWalkBlock), lds, st, seg, sys->d_edges, sys->n_edges, sys->n_nodes,
                       list, which, few, reinterpret_cast<unsigned long long*>(d_n_evaluated));
    return hipGetLastError();
}

}  // namespace

hipError_t launch_label(hipStream_t st, const SegSrc& seg, const SampleList& list) {
    const int64_t tiles = (seg.total + kLabelTile - 1) / kLabelTile;
    const int64_t per_block = (tiles + kListRegions - 1) / kListRegions;
    const int64_t blocks = (tiles + per_block - 1) / per_block;
    hipLaunchKernelGGL(k_label, dim3(static_cast<unsigned>(blocks)), dim3(kLabelBlock), 0, st, seg,
                       per_block * kLabelTile, list);
    return hipGetLastError();
}

hipError_t launch_eval(hipStream_t st, const rsr_system* sys, const SegSrc& seg,
                       const SampleList& list, int which, uint64_t* d_n_evaluated, int cus) {
    if (sys->kind == RSR_SYS_MAX_FLOW)
        return launch_flow_eval(st, sys, seg, list, which, d_n_evaluated, cus * 8);
    if (sys->kind == RSR_SYS_GLOBAL_CONNECTIVITY) {
        if (sys->level < 2)
            return launch_connect<kGlobal1>(st, sys, seg, 0, sys->class_from, 0, list, which,
                                            d_n_evaluated, cus);
        return launch_global2(st, sys, seg, list, which, d_n_evaluated, cus);
    }
    return launch_connect<kSt>(st, sys, seg, sys->level - 1, sys->source, sys->sink, list, which,
                               d_n_evaluated, cus);
}

}  // namespace rsr
