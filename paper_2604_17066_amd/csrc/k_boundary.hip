// Componentwise boundary search (section 3.4) for s-t connectivity at a level
// and for global connectivity, many start samples at once: one wavefront per
// start sample.
//
// The search visits the components (edges) in index order and moves each one
// state at a time towards K-1 (failure start) or 0 (survival start), undoing
// the step that changes the system side.  For these systems the side depends
// only on which edges are usable (state >= level; >= 1 for global
// connectivity), so a component's walk has one decisive step: for a failure
// start, making an unusable edge usable; for a survival start, making a usable
// edge unusable.  Every other step leaves the side unchanged and is taken.  The
// result is therefore fixed by the final usable set U':
//   failure start:  x'_i = K-1 if U'_i else level-1   (a maximal failure state)
//   survival start: x'_i = level if U'_i else 0       (a minimal survival state)
//
// s-t connectivity and level 1 of global connectivity need no search per step:
// U' follows from one spanning forest (k_boundary).
//  * Survival.  Deleting usable edges in index order unless the side changes
//    keeps, of all edge sets that preserve the side, the one that avoids the
//    low indices first: the minimum under the weights 2^-i.  A spanning forest
//    F of the usable edges that prefers HIGH indices is minimal for these
//    weights, cycle by cycle, so U' is the path of F from s to t (s-t), or F
//    itself (global).
//  * Failure, s-t.  Adding unusable edges in index order, an edge is refused
//    exactly when it would join the component of s with that of t.  Identify s
//    with t and take the usable edges, then the unusable ones by index, into a
//    spanning forest (Kruskal): its components are at every step those of the
//    walk, with s's and t's seen as one.  Split at s = t, the finished forest
//    has a part S* at s and a part T* at t, which hold the two components of
//    every earlier step; an edge between S* and T* was refused when its turn
//    came and every other edge was taken.
//  * Failure, global.  An edge is refused exactly when it would make the graph
//    connected, that is when two components are left and it joins them.  The
//    forest of the same order without the last (highest) of its unusable
//    edges has those two components.  If the forest does not span the nodes,
//    nothing is refused.
// The forest is built by Boruvka's rounds: every component picks its best
// edge, components hook along their picks, labels follow the hooks.  A start
// sample takes a few tens of wave-wide LDS passes whatever its states are,
// where a search for every decisive step took one pass per step and tree
// level.
//
// Bound: LDS latency, a chain of dependent reads in each pass; the wave's
// nodes and edges are spread over the lanes, and four edges of a lane are in
// flight together.  1024 starts on a graph of 119 nodes and 295 edges: 18.7 us,
// where searching step by step took 506 us.
#include "graph_search.h"

namespace rsr {
namespace {

using graph::wave_sync;

constexpr int kBoundaryBlock = 256;
constexpr int kBoundaryWaves = kBoundaryBlock / 64;

// A wave's LDS working set.
struct Forest {
    uint32_t* best;    // [n_nodes] of a component: hook << 16 | rank of its best edge
    uint16_t* label;   // [n_nodes] component of the node: one of its nodes
    uint16_t* before;  // [n_nodes] labels kept aside
    uint32_t* edges;   // [edge_words] the forest's edges
};

__host__ __device__ __forceinline__ int forest_words(int n_nodes, int n_edges) {
    return n_nodes + 2 * ((n_nodes + 1) >> 1) + ((n_edges + 31) >> 5);
}

__device__ __forceinline__ Forest forest_at(uint32_t* base, int n_nodes, int n_edges) {
    const int half_words = (n_nodes + 1) >> 1;
    Forest f;
    f.best = base;
    f.label = reinterpret_cast<uint16_t*>(base + n_nodes);
    f.before = reinterpret_cast<uint16_t*>(base + n_nodes + half_words);
    f.edges = base + n_nodes + 2 * half_words;
    return f;
}

// Joins the components of f.label along the lane's edges `cand` (edge
// lane + 64 k at bit k), best rank first, and adds the edges that joined two
// of them to f.edges.  The best rank is the highest edge index with `highest`,
// else the lowest.  The edges that a round's components pick form no cycle but
// the pair that picked one edge together: ranks are distinct, so along a chain
// of picks they rise.  Of such a pair the lower one stays a root.  Every
// component with an edge to another one is joined in every round, so there are
// at most log2(n_nodes) rounds.
__device__ void join(uint64_t cand, bool highest, const Forest& f,
                     const uint32_t* __restrict__ s_edges, int n_edges, int n_nodes) {
    const int lane = threadIdx.x & 63;
    while (true) {
        for (int v = lane; v < n_nodes; v += 64) f.best[v] = 0;
        wave_sync();
        uint64_t todo = cand;
        while (todo) {
            int k[4];
            uint32_t a[4], b[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {  // past the lane's last edge: its first again
                const bool more = q == 0 || todo;
                k[q] = more ? __ffsll(static_cast<unsigned long long>(todo)) - 1 : k[0];
                todo = more ? todo & (todo - 1) : todo;
                const uint32_t uv = s_edges[lane + 64 * k[q]];
                a[q] = uv & 0xFFFFu;
                b[q] = uv >> 16;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                a[q] = f.label[a[q]];
                b[q] = f.label[b[q]];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (a[q] == b[q]) {
                    cand &= ~(1ull << k[q]);  // inside a component from now on
                } else {
                    const int e = lane + 64 * k[q];
                    const uint32_t rank = static_cast<uint32_t>(highest ? e + 1 : n_edges - e);
                    atomicMax(&f.best[a[q]], rank);
                    atomicMax(&f.best[b[q]], rank);
                }
            }
        }
        if (!__any(cand != 0)) break;
        wave_sync();
        for (int r = lane; r < n_nodes; r += 64) {
            const uint32_t rank = f.best[r] & 0xFFFFu;
            if (!rank) continue;  // not a component, or one without an edge to another
            const int e = static_cast<int>(highest ? rank - 1 : n_edges - rank);
            const uint32_t uv = s_edges[e];
            const uint32_t a = f.label[uv & 0xFFFFu], b = f.label[uv >> 16];
            const uint32_t other = a == static_cast<uint32_t>(r) ? b : a;
            const bool mutual = (f.best[other] & 0xFFFFu) == rank;
            const uint32_t hook = mutual && static_cast<uint32_t>(r) < other ? r : other;
            f.best[r] = hook << 16 | rank;
            atomicOr(&f.edges[e >> 5], 1u << (e & 31));
        }
        wave_sync();
        for (int v = lane; v < n_nodes; v += 64) {
            uint32_t l = f.label[v];
            for (uint32_t h = f.best[l]; h && (h >> 16) != l; h = f.best[l]) l = h >> 16;
            f.label[v] = static_cast<uint16_t>(l);
        }
        wave_sync();
    }
    wave_sync();
}

// The lane's edges in the bit set f.edges.
__device__ __forceinline__ uint64_t own_edges(const Forest& f, int n_edges) {
    uint64_t own = 0;
    const int lane = threadIdx.x & 63;
    for (int k = 0; lane + 64 * k < n_edges; ++k) {
        const int e = lane + 64 * k;
        own |= static_cast<uint64_t>((f.edges[e >> 5] >> (e & 31)) & 1u) << k;
    }
    return own;
}

// Leaves of the forest f.edges only the path from s to t (nodes of one tree):
// cuts leaves other than s and t until none is left.  A node's word holds its
// degree (low half) and the sum of its edges' indices, so the one edge of a
// leaf can be read off.  A lane follows its cuts up the tree; a node that
// becomes a leaf is cut by whoever claims it first.
__device__ void trim_to_path(uint64_t own, const Forest& f, const uint32_t* __restrict__ s_edges,
                             int n_nodes, int s, int t) {
    const int lane = threadIdx.x & 63;
    uint32_t* node = f.best;
    for (int v = lane; v < n_nodes; v += 64) node[v] = v == s || v == t ? 2u : 0u;  // never a leaf
    wave_sync();
    while (own) {
        const int e = lane + 64 * (__ffsll(static_cast<unsigned long long>(own)) - 1);
        own &= own - 1;
        const uint32_t uv = s_edges[e], add = 1u + (static_cast<uint32_t>(e) << 16);
        atomicAdd(&node[uv & 0xFFFFu], add);
        atomicAdd(&node[uv >> 16], add);
    }
    wave_sync();
    for (int v = lane; v < n_nodes; v += 64) {
        uint32_t w = static_cast<uint32_t>(v), word = node[v];
        while ((word & 0xFFFFu) == 1u && atomicCAS(&node[w], word, 0u) == word) {
            const uint32_t e = word >> 16;
            atomicAnd(&f.edges[e >> 5], ~(1u << (e & 31)));
            w = graph::other_end(s_edges[e], w);
            word = atomicSub(&node[w], word) - word;
        }
    }
    wave_sync();
}

// s-t connectivity (global false) at `level`, or global connectivity at level
// 1 (global true; source, sink and level unused).
__global__ __launch_bounds__(kBoundaryBlock) void k_boundary(
    const uint32_t* __restrict__ xs, int64_t N, int PW, const uint32_t* __restrict__ edges,
    int n_edges, int n_nodes, bool global, int source, int sink, int K, int level,
    const int64_t* __restrict__ pick, int64_t n_pick, uint8_t* __restrict__ rows,
    uint8_t* __restrict__ side) {
    extern __shared__ uint32_t lds[];
    uint32_t* s_edges = lds;
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const int edge_words = (n_edges + 31) >> 5;
    const Forest f =
        forest_at(lds + n_edges + wave * forest_words(n_nodes, n_edges), n_nodes, n_edges);

    for (int e = threadIdx.x; e < n_edges; e += blockDim.x) s_edges[e] = edges[e];
    __syncthreads();

    const int rounds = (n_edges + 63) >> 6;
    const uint64_t all = lane + 64 * (rounds - 1) < n_edges
                             ? ~0ull >> (64 - rounds)
                             : (rounds > 1 ? ~0ull >> (65 - rounds) : 0ull);
    const int waves = blockDim.x >> 6;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * waves;
    for (int64_t j = static_cast<int64_t>(blockIdx.x) * waves + wave; j < n_pick; j += stride) {
        const int64_t h = pick[j];
        if (h < 0 || h >= N) {  // not a sample index: reported, nothing read
            if (lane == 0) side[j] = 0xFF;
            continue;
        }
        uint64_t usable = 0;
#pragma unroll 4
        for (int k = 0; k < rounds; ++k) {
            const int e = lane + 64 * k;
            if (e < n_edges) {
                const uint32_t word =
                    xs[static_cast<int64_t>((level - 1) * PW + (e >> 5)) * N + h];
                usable |= static_cast<uint64_t>((word >> (e & 31)) & 1u) << k;
            }
        }
        for (int v = lane; v < n_nodes; v += 64) f.label[v] = static_cast<uint16_t>(v);
        graph::fill(f.edges, edge_words, 0u);
        wave_sync();
        join(usable, true, f, s_edges, n_edges, n_nodes);

        bool survival;
        if (global) {
            bool apart = false;
            for (int v = lane; v < n_nodes; v += 64) apart = apart || f.label[v] != f.label[0];
            survival = !__any(apart);
        } else {
            survival = f.label[source] == f.label[sink];
        }
        if (survival) {
            usable = own_edges(f, n_edges);
            if (!global) {
                trim_to_path(usable, f, s_edges, n_nodes, source, sink);
                usable = own_edges(f, n_edges);
            }
        } else {
            const uint32_t ls = f.label[source], lt = f.label[sink];
            for (int v = lane; v < n_nodes; v += 64) {
                const uint16_t l = f.label[v];
                f.before[v] = l;
                if (!global && l == lt) f.label[v] = static_cast<uint16_t>(ls);
            }
            graph::fill(f.edges, edge_words, 0u);
            wave_sync();
            join(all & ~usable, false, f, s_edges, n_edges, n_nodes);
            uint64_t added = own_edges(f, n_edges);
            bool cut = true;  // whether the forest has two parts to keep apart
            if (global) {
                bool apart = false;
                for (int v = lane; v < n_nodes; v += 64) apart = apart || f.label[v] != f.label[0];
                cut = !__any(apart);
                if (cut) {  // without the highest of the added edges
                    int last = added ? lane + 64 * (63 - __clzll(added)) : -1;
                    for (int off = 32; off > 0; off >>= 1) last = max(last, __shfl_xor(last, off));
                    if (last >= 0 && (last & 63) == lane) added &= ~(1ull << (last >> 6));
                }
            }
            if (cut) {
                wave_sync();
                for (int v = lane; v < n_nodes; v += 64) f.label[v] = f.before[v];
                wave_sync();
                join(added, false, f, s_edges, n_edges, n_nodes);
                // s-t: the parts of s and t.  Global: there are but two.
                const uint32_t part_s = f.label[source], part_t = f.label[sink];
                uint64_t todo = all & ~usable;
                while (todo) {
                    const int k = __ffsll(static_cast<unsigned long long>(todo)) - 1;
                    todo &= todo - 1;
                    const uint32_t uv = s_edges[lane + 64 * k];
                    const uint32_t a = f.label[uv & 0xFFFFu], b = f.label[uv >> 16];
                    const bool refused = global ? a != b
                                                : (a == part_s && b == part_t) ||
                                                      (a == part_t && b == part_s);
                    if (!refused) usable |= 1ull << k;
                }
            } else {
                usable = all;
            }
        }

        const uint8_t hi = static_cast<uint8_t>(survival ? level : K - 1);
        const uint8_t lo = static_cast<uint8_t>(survival ? 0 : level - 1);
        uint8_t* out = rows + j * static_cast<int64_t>(n_edges);
        for (int k = 0; k < rounds; ++k) {
            const int e = lane + 64 * k;
            if (e < n_edges) out[e] = ((usable >> k) & 1u) ? hi : lo;
        }
        if (lane == 0) side[j] = survival ? 1 : 0;
        wave_sync();
    }
}

// Two-edge connectivity of all nodes (global connectivity at level 2; edges
// work at state >= 1): the walk step by step, with the system function
// evaluated from scratch at every decisive step (a search from node 0 and the
// bridge test).
__global__ __launch_bounds__(kBoundaryBlock) void k_boundary_global2(
    const uint32_t* __restrict__ xs, int64_t N, const uint32_t* __restrict__ edges, int n_edges,
    int n_nodes, int K, const int64_t* __restrict__ pick, int64_t n_pick,
    uint8_t* __restrict__ rows, uint8_t* __restrict__ side) {
    extern __shared__ uint32_t lds[];
    const int per_wave = graph::global_words(n_nodes, n_edges);
    uint32_t* s_edges = lds;
    const int wave = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63;
    const graph::GlobalSets g = graph::global_sets(lds + n_edges + wave * per_wave, n_nodes, n_edges);

    for (int e = threadIdx.x; e < n_edges; e += kBoundaryBlock) s_edges[e] = edges[e];
    __syncthreads();

    const int rounds = (n_edges + 63) >> 6;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBoundaryWaves;
    for (int64_t j = static_cast<int64_t>(blockIdx.x) * kBoundaryWaves + wave; j < n_pick;
         j += stride) {
        const int64_t h = pick[j];
        if (h < 0 || h >= N) {  // not a sample index: reported, nothing read
            if (lane == 0) side[j] = 0xFF;
            continue;
        }
        uint64_t usable = 0;  // plane 0 = [x >= 1]
        for (int k = 0; k < rounds; ++k) {
            const int e = lane + 64 * k;
            if (e < n_edges) {
                const uint32_t word = xs[static_cast<int64_t>(e >> 5) * N + h];
                usable |= static_cast<uint64_t>((word >> (e & 31)) & 1u) << k;
            }
        }
        const bool survival =
            graph::two_edge_connected(usable, s_edges, n_edges, n_nodes, g);
        for (int i = 0; i < n_edges; ++i) {
            const int owner = i & 63, k = i >> 6;
            const bool ui = (__shfl(usable, owner) >> k) & 1u;
            if (ui == !survival) continue;  // walks to K-1 (failure) or 0 (survival) unopposed
            const uint64_t flip = lane == owner ? (1ull << k) : 0ull;
            const uint64_t trial = survival ? (usable & ~flip) : (usable | flip);
            const bool after = graph::two_edge_connected(trial, s_edges, n_edges, n_nodes, g);
            if (after == survival) usable = trial;
        }
        const uint8_t hi = static_cast<uint8_t>(survival ? 1 : K - 1);
        uint8_t* out = rows + j * static_cast<int64_t>(n_edges);
        for (int k = 0; k < rounds; ++k) {
            const int e = lane + 64 * k;
            if (e < n_edges) out[e] = ((usable >> k) & 1u) ? hi : 0;
        }
        if (lane == 0) side[j] = survival ? 1 : 0;
        wave_sync();
    }
}

}  // namespace

// What the search may take of a CU's LDS, and so which graphs it accepts: the
// edge table, and node sets and parents for four waves.
size_t boundary_lds_bytes(const rsr_system* sys) {
    if (sys->kind == RSR_SYS_MAX_FLOW) return flow_lds_bytes(sys);
    const int n_nodes = sys->n_nodes, n_edges = sys->n_edges;
    size_t per_wave;
    if (sys->kind == RSR_SYS_GLOBAL_CONNECTIVITY) {
        per_wave = static_cast<size_t>(((n_nodes + 31) >> 5) + ((n_edges + 31) >> 5) +
                                       2 * ((n_nodes + 1) >> 1));
    } else {
        const int node_words = (n_nodes + 31) >> 5;
        const int edge_words = (n_edges + 31) >> 5;
        const int parent_words = (n_nodes + 1) >> 1;
        per_wave = static_cast<size_t>(2 * node_words + edge_words + parent_words);
    }
    return sizeof(uint32_t) * (static_cast<size_t>(n_edges) + kBoundaryWaves * per_wave);
}

hipError_t launch_boundary(hipStream_t st, const rsr_system* sys, const uint32_t* xs, int64_t N,
                           const int64_t* d_pick, int64_t n_pick, uint8_t* d_rows,
                           uint8_t* d_side, int grid_cap) {
    if (sys->kind == RSR_SYS_MAX_FLOW)
        return launch_boundary_flow(st, sys, xs, N, d_pick, n_pick, d_rows, d_side, grid_cap);
    const bool global = sys->kind == RSR_SYS_GLOBAL_CONNECTIVITY;
    const bool stepwise = global && sys->level >= 2;
    // The forests of four waves share a block's edge table where they fit the
    // 64 KiB that boundary_lds_bytes allows a graph; one wave's always does: it
    // takes 8 bytes a node, four waves' node sets and parents took 9.
    int waves = kBoundaryWaves;
    size_t lds = boundary_lds_bytes(sys);
    if (!stepwise) {
        const auto bytes = [&](int w) {
            return sizeof(uint32_t) * (static_cast<size_t>(sys->n_edges) +
                                       static_cast<size_t>(w) *
                                           forest_words(sys->n_nodes, sys->n_edges));
        };
        while (waves > 1 && bytes(waves) > 64 * 1024) waves >>= 1;
        lds = bytes(waves);
    }
    int64_t blocks = (n_pick + waves - 1) / waves;
    if (blocks > grid_cap) blocks = grid_cap;
    if (blocks < 1) blocks = 1;
    if (stepwise)
        hipLaunchKernelGGL(k_boundary_global2, dim3(static_cast<unsigned>(blocks)),
                           dim3(kBoundaryBlock), lds, st, xs, N, sys->d_edges, sys->n_edges,
                           sys->n_nodes, sys->K, d_pick, n_pick, d_rows, d_side);
    else
        hipLaunchKernelGGL(k_boundary, dim3(static_cast<unsigned>(blocks)), dim3(64 * waves), lds,
                           st, xs, N, plane_words(sys->n_edges), sys->d_edges, sys->n_edges,
                           sys->n_nodes, global, global ? 0 : sys->source, global ? 0 : sys->sink,
                           sys->K, global ? 1 : sys->level, d_pick, n_pick, d_rows, d_side);
    return hipGetLastError();
}

}  // namespace rsr
