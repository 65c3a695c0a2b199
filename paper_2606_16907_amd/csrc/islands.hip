// islands.hip -- GPU island construction from nodes (Sec. 4.1).
//
// An island holds nodes with the same GPU count whose compute, memory
// (Eq. 1) and intra-node bandwidth (Eq. 2) differ by at most a factor 1 + eps
// pairwise, and every member's links inside the island are at least as fast
// as its links leaving it (Eq. 3).  Steps (1)-(2): one block splits the nodes
// by GPU count, compute, memory and intra-node bandwidth, each split a block
// bitonic sort by (group, value, node) followed by a sweep that opens a new
// group at the first value above the group's smallest times (1 + eps).  Step
// (3): agglomerative clustering per group: the pair of clusters with the
// highest complete linkage (the least bandwidth between their nodes, a node
// pair counted by its slower direction; ties to the least pair of smallest
// node ids) is merged if the union satisfies Eq. 3 against every node outside
// it, else marked, until every pair is marked.  A union's Eq. 3 outcome
// depends only on its own nodes, so a failed pair stays failed while both
// clusters last, and the next merge is the highest pair whose union passes.
// The clustering runs in stages of falling thresholds.  Pairs linked at least
// as fast as a threshold lie in one component of the graph of such links, and
// what happens among them (linkages, marks, Eq. 3) touches no other component;
// the pairs above the threshold all come before the rest.  So a stage runs
// every component on a block of its own, over the pairs above its threshold
// only, and the next stage goes on from the clusters and marks it left: the
// same merges in the same order within each component as one serial run, most
// of them side by side (a leaf switch's nodes first, then a pod's, then what is
// left of the group).  A block works in rounds: each cluster's row keeps its
// best unmarked partner, known to pass (clean) or untested (dirty); when the
// best clean pair is above every dirty one it is merged, else every dirty pair
// above it is tested at once (a wave each) and the failures marked.  Linkage,
// marks and per-cluster least links (for each cluster and node, the node's
// slowest link into the cluster) sit in matrices over the group's node
// numbering; a cluster's members are one contiguous range of a permutation, so
// a test gives each lane a member: its slowest link inside the union from its
// own cluster's value and the other cluster's entry, its fastest link leaving
// from its bandwidth row sorted once (the first entry outside the union, from
// where its own cluster ends).  A finish pass numbers islands by their smallest
// node and reduces the island attributes and island-to-island bandwidths (least
// over node pairs).  Bound by the rounds' chains of dependent loads and
// barriers, so by the number of rounds in a row: 1024 nodes took 6.1 ms of
// clustering with a block per group, 0.57 ms in stages.
#include <stdint.h>

#include <cstring>
#include <type_traits>
#include <vector>

#include "tg_device.h"

#pragma clang fp contract(off)

namespace tg {

constexpr int kMaxNodes = 4096;
constexpr int kGroupThreads = 1024;
// Merge blocks: eight waves for a component of up to kSmallComp nodes (a leaf's
// pairs are tested at once, a wave each; one wave took 158 us over 1024 nodes'
// leaves, eight 91), sixteen above.
constexpr int kSmallComp = 64;
constexpr int kSmallThreads = 512;
constexpr int kMergeThreads = 1024;
// The stages' thresholds, as shares of the fastest link between two nodes.
// Where fabric levels differ by more than 2, the first separates the fastest
// level (leaves) and the second the next (pods); the last stage takes every pair
// of a group.  Levels of exactly 2:1 fall together two by two, which costs a part
// of the gain: 1024 nodes 7.8 ms in one stage and 2.2 in three, with levels of 4:1
// or 8:1 7.8 and 1.6.  Any shares give the same islands.
constexpr double kStageShare[] = {0.5, 0.125};
constexpr int kStages = 3;
// The stages cost two more rounds of launches, and a pair of clusters that waits
// for a slower link is looked for again.  One launch over whole groups it is
// where the largest group has fewer than kStagedNodes nodes, or kStagedOdd where
// links were measured one by one (most differ from their neighbour, and most
// unions fail Eq. 3), and where every link is above the first threshold's share of
// the fastest.  Stages against one launch: groups of 4 nodes 272 and 218 us, 8 326
// and 300, 12 and 16 behind levels of 4:1 361 and 374, 371 and 455; flat fabrics of
// 64 nodes 1559 and 1450, of 128 2215 and 1926; links measured one by one, 100
// nodes of six GPU types 911 and 720, 64 nodes of two types 789 and 943.  The last
// stage takes all its groups in one launch of sixteen waves: two launches, one
// after the other, took 2046 us on 197 nodes of four types, one 1480.
constexpr int kStagedNodes = 16, kStagedOdd = 48;
constexpr int kOneSmall = 32;  // nodes of a group up to which that launch has eight waves
constexpr double kNoPair = -__builtin_huge_val();

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// The call's scalars, uploaded and read back as one.
struct IslandState {
    int32_t err;               // a merge loop overran its round bound (an internal error)
    int32_t bad;               // first bad node_bw entry
    int32_t group;             // nodes of the largest group
    int32_t same;              // entries of the bandwidths equal to their right neighbour
    unsigned long long least;  // slowest and fastest link between two nodes (bits of a double)
    unsigned long long most;
};

struct IslandWs {
    int32_t *gpus;      // [n]
    double *val;        // [4][n] compute, memory, intra, host per node
    double *e;          // [n][n] node bandwidth, row = source
    int32_t *srt;       // [n][n] row u: the other nodes by bandwidth from u, fastest first
    int32_t *grp;       // [n] group after steps (1)-(2)
    int32_t *gstart;    // [n + 1] group g's nodes are gnodes[gstart[g] .. gstart[g + 1])
    int32_t *gnodes;    // [n]
    int32_t *ngroups;   // [1]
    int32_t *lq;        // [n] a node's number inside its group (its place in gnodes)
    int64_t *goff;      // [n + 1] where group g's nm x nm matrices start (sum of nm^2 before it)
    double *L;          // per group [nm][nm]: complete linkage between clusters (-inf: no pair)
    uint8_t *M;         // per group [nm][nm]: pairs whose union breaks Eq. 3
    double *XT;         // per group [nm][nm]: row c, column m: slowest link from node m into cluster c
    double *inown;      // [n] a node's slowest link into its own cluster (+inf alone)
    int32_t *pos;       // [n] first entry of the node's sorted row outside its own cluster
    int32_t *nxl;       // [n] that entry's number inside the group (-1: another group, or none)
    double *outv;       // [n] the node's bandwidth to it (-inf: none)
    int32_t *cl;        // [n] cluster (its smallest node) of each node
    int32_t *uf;        // [n] union-find parents of a stage's components
    int32_t *comp;      // [n] component of each node
    int32_t *lc;        // [n] its number inside the component
    int32_t *cstart;    // [n + 1] component c's nodes are cnodes[cstart[c] .. cstart[c + 1])
    int32_t *cnodes;    // [n]
    int32_t *ncomp;     // [1]
    IslandState *state; // [1]
    int32_t *island_of; // [n]
    int32_t *out_k;     // [1]
    int32_t *isl_gpus;  // [n]
    double *isl_val;    // [4][n] least compute, memory, intra, host
    double *isl_e;      // [n][n] (K x K used)
    size_t bytes;
};

static IslandWs carve_islands(int64_t n, void *base) {
    IslandWs w{};
    char *p = (char *)base;
    size_t off = 0;
    auto take = [&](size_t bytes) -> void * {
        void *r = base ? (void *)(p + off) : nullptr;
        off += align256(bytes > 0 ? bytes : 1);
        return r;
    };
    w.gpus = (int32_t *)take(4 * n);
    w.val = (double *)take(8 * 4 * n);
    w.e = (double *)take(8 * n * n);
    w.srt = (int32_t *)take(4 * n * n);
    w.grp = (int32_t *)take(4 * n);
    w.gstart = (int32_t *)take(4 * (n + 1));
    w.gnodes = (int32_t *)take(4 * n);
    w.ngroups = (int32_t *)take(4);
    w.lq = (int32_t *)take(4 * n);
    w.goff = (int64_t *)take(8 * (n + 1));
    w.L = (double *)take(8 * n * n);  // the groups' matrices together hold at most n^2 entries
    w.M = (uint8_t *)take(n * n);
    w.XT = (double *)take(8 * n * n);
    w.inown = (double *)take(8 * n);
    w.pos = (int32_t *)take(4 * n);
    w.nxl = (int32_t *)take(4 * n);
    w.outv = (double *)take(8 * n);
    w.cl = (int32_t *)take(4 * n);
    w.uf = (int32_t *)take(4 * n);
    w.comp = (int32_t *)take(4 * n);
    w.lc = (int32_t *)take(4 * n);
    w.cstart = (int32_t *)take(4 * (n + 1));
    w.cnodes = (int32_t *)take(4 * n);
    w.ncomp = (int32_t *)take(4);
    w.state = (IslandState *)take(sizeof(IslandState));
    w.island_of = (int32_t *)take(4 * n);
    w.out_k = (int32_t *)take(4);
    w.isl_gpus = (int32_t *)take(4 * n);
    w.isl_val = (double *)take(8 * 4 * n);
    w.isl_e = (double *)take(8 * n * n);
    w.bytes = off;
    return w;
}

size_t islands_ws_bytes(int n) { return carve_islands(n, nullptr).bytes; }

// Node bandwidths must be finite and non-negative: the first entry that is not
// into *bad (INT32_MAX if none; n^2 <= 2^24 entries).
// The first entry that is no bandwidth, the least and the greatest link, and how
// many entries equal their right neighbour (a wave's 64 entries have 63 pairs).
__global__ __launch_bounds__(256) void islands_check(int n, const double *__restrict__ e, IslandState *state) {
    __shared__ double wlo[256 / kWave], whi[256 / kWave];
    __shared__ int32_t wsame[256 / kWave];
    const uint32_t nn = (uint32_t)n * (uint32_t)n;  // at most 2^24
    double lo = __builtin_huge_val(), hi = 0.0;
    int32_t same = 0;
    const uint32_t step = gridDim.x * blockDim.x;
    constexpr int kAhead = 8;  // loads in flight
    for (uint32_t b0 = blockIdx.x * blockDim.x; b0 < nn; b0 += kAhead * step) {  // whole blocks
        double x[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) x[k] = e[min(b0 + threadIdx.x + k * step, nn - 1)];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            const uint32_t t = b0 + threadIdx.x + k * step;
            const double right = __shfl_down(x[k], 1);
            if (t >= nn) continue;
            if (!(x[k] >= 0.0) || !(x[k] < __builtin_huge_val())) {
                atomicMin(&state->bad, (int32_t)t);
            } else if (t % (uint32_t)(n + 1) != 0) {  // not a node's own entry
                lo = fmin(lo, fabs(x[k]));
                hi = fmax(hi, fabs(x[k]));
                same += wave_lane() < kWave - 1 && t + 1 < nn && x[k] == right;
            }
        }
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, off));
        hi = fmax(hi, __shfl_xor(hi, off));
        same += __shfl_xor(same, off);
    }
    if (wave_lane() == 0) {
        wlo[threadIdx.x / kWave] = lo;
        whi[threadIdx.x / kWave] = hi;
        wsame[threadIdx.x / kWave] = same;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < 256 / kWave; ++w) {
            lo = fmin(lo, wlo[w]);
            hi = fmax(hi, whi[w]);
            same += wsame[w];
        }
        // non-negative: the bits order like the values; a plain look first, so
        // that few blocks update
        const unsigned long long l = (unsigned long long)__double_as_longlong(lo),
                                 h = (unsigned long long)__double_as_longlong(hi);
        if (l < __hip_atomic_load(&state->least, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicMin(&state->least, l);
        if (h > __hip_atomic_load(&state->most, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicMax(&state->most, h);
        if (same) atomicAdd(&state->same, same);
    }
}

// ---------------------------------------------------------------------------
// steps (1)-(2): groups
// ---------------------------------------------------------------------------
// Order of nodes u, v by (group, value, node id); padding slots (>= n) last.
__device__ inline bool node_before(int u, int v, int n, const int32_t *g, const double *x) {
    if (u >= n) return false;
    if (v >= n) return true;
    if (g[u] != g[v]) return g[u] < g[v];
    if (x[u] != x[v]) return x[u] < x[v];
    return u < v;
}

__global__ __launch_bounds__(kGroupThreads) void islands_groups(int n, const int32_t *__restrict__ gpus,
                                                                const double *__restrict__ val, double eps_c,
                                                                double eps_m, double eps_i, int32_t *grp,
                                                                int32_t *gstart, int32_t *gnodes, int32_t *ngroups,
                                                                int32_t *lq, int64_t *goff, IslandState *state) {
    __shared__ int32_t ord[kMaxNodes];
    __shared__ int32_t g[kMaxNodes];
    __shared__ double x[kMaxNodes];
    __shared__ int32_t ng[kMaxNodes];      // new group of the t-th node in sorted order
    __shared__ int32_t gs[kMaxNodes + 1];  // group starts after the last split
    __shared__ int32_t nx[kMaxNodes];      // next opening position after an opening at t
    __shared__ int32_t scan_lds[kGroupThreads / 64 + 1];
    __shared__ int32_t s_groups;
    int np = 1;
    while (np < n) np <<= 1;
    for (int u = threadIdx.x; u < n; u += blockDim.x) g[u] = 0;
    // the split keys: GPU count (exact), compute, memory, intra-node bandwidth
    for (int f = 0; f < 4; ++f) {
        const double eps = f == 0 ? 0.0 : (f == 1 ? eps_c : (f == 2 ? eps_m : eps_i));
        for (int u = threadIdx.x; u < np; u += blockDim.x) {
            ord[u] = u;
            if (u < n) x[u] = f == 0 ? (double)gpus[u] : val[(int64_t)(f - 1) * n + u];
        }
        __syncthreads();
        for (int k = 2; k <= np; k <<= 1)
            for (int j = k >> 1; j > 0; j >>= 1) {
                for (int t = threadIdx.x; t < np; t += blockDim.x) {
                    const int q = t ^ j;
                    if (q > t) {
                        const int a = ord[t], b = ord[q];
                        const bool up = (t & k) == 0;
                        const bool swap = up ? node_before(b, a, n, g, x) : node_before(a, b, n, g, x);
                        if (swap) {
                            ord[t] = b;
                            ord[q] = a;
                        }
                    }
                }
                __syncthreads();
            }
        // the sweep: a new group opens at the first node of an old group and
        // at the first node whose value exceeds the opening node's times
        // (1 + eps).  From an opening position t the next one is the first
        // t' > t whose (old group, value) passes (g, x (1 + eps)) of t, found
        // by bisection in the sorted order; the openings are the chain of
        // such positions from 0, which thread 0 follows (one hop per group).
        for (int t = threadIdx.x; t < n; t += blockDim.x) {
            const int u = ord[t];
            const int gu = g[u];
            const double thr = x[u] * (1.0 + eps);
            int lo = t + 1, hi = n;  // first position past the run, in [t + 1, n]
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                const int v = ord[mid];
                if (g[v] > gu || (g[v] == gu && !(x[v] <= thr)))
                    hi = mid;
                else
                    lo = mid + 1;
            }
            nx[t] = lo;
            ng[t] = 0;
        }
        __syncthreads();
        if (threadIdx.x == 0)
            for (int t = 0; t < n; t = nx[t]) ng[t] = 1;
        __syncthreads();
        {  // new group of each position: openings up to it, less one
            int32_t carry = 0;
            for (int base = 0; base < n; base += blockDim.x) {
                const int t = base + (int)threadIdx.x;
                const int32_t f = t < n ? ng[t] : 0;
                int32_t tot;
                const int32_t ex = block_excl_scan<int32_t>(f, scan_lds, &tot);
                __syncthreads();
                if (t < n) ng[t] = carry + ex + f - 1;
                carry += tot;
            }
            if (threadIdx.x == 0) s_groups = carry;
        }
        __syncthreads();
        for (int t = threadIdx.x; t < n; t += blockDim.x) g[ord[t]] = ng[t];
        __syncthreads();
    }
    // group starts and member lists in sorted order (groups are numbered in it)
    const int G = s_groups;
    for (int t = threadIdx.x; t < n; t += blockDim.x)
        if (t == 0 || ng[t] != ng[t - 1]) gs[ng[t]] = t;
    if (threadIdx.x == 0) gs[G] = n;
    __syncthreads();
    if (threadIdx.x == 0) {
        *ngroups = G;
        int64_t off = 0, most = 0;
        for (int gg = 0; gg < G; ++gg) {
            goff[gg] = off;
            const int64_t nm = gs[gg + 1] - gs[gg];
            off += nm * nm;
            most = max(most, nm);
        }
        goff[G] = off;
        state->group = (int32_t)most;
    }
    for (int gg = threadIdx.x; gg <= G; gg += blockDim.x) gstart[gg] = gs[gg];
    for (int t = threadIdx.x; t < n; t += blockDim.x) {
        const int u = ord[t];
        gnodes[t] = u;
        grp[u] = ng[t];
        lq[u] = t - gs[ng[t]];
    }
}

// Row u of the node bandwidth sorted, fastest first (ties to the lesser
// node), u itself left out: the fastest link from u to a node outside a
// cluster is then the first entry outside it, a few entries in for a cluster
// whose own links are its fastest, as Eq. 3 asks.
__global__ __launch_bounds__(1024) void islands_sort_rows(int n, const double *__restrict__ e, int32_t *srt) {
    __shared__ double x[kMaxNodes];
    __shared__ int32_t id[kMaxNodes];
    const int u = blockIdx.x;
    int np = 1;
    while (np < n) np <<= 1;
    for (int t = threadIdx.x; t < np; t += blockDim.x) {
        id[t] = (t < n && t != u) ? t : n;  // n: after every real entry
        x[t] = t < n ? e[(int64_t)u * n + t] : 0.0;
    }
    __syncthreads();
    auto before = [&](int p, int q) {  // entry p sorts before entry q
        if (id[p] >= n) return false;
        if (id[q] >= n) return true;
        if (x[p] != x[q]) return x[p] > x[q];
        return id[p] < id[q];
    };
    for (int k = 2; k <= np; k <<= 1)
        for (int j = k >> 1; j > 0; j >>= 1) {
            for (int t = threadIdx.x; t < np; t += blockDim.x) {
                const int o = t ^ j;
                if (o > t) {
                    const bool up = (t & k) == 0;
                    if (up ? before(o, t) : before(t, o)) {
                        const double tx = x[t];
                        x[t] = x[o];
                        x[o] = tx;
                        const int32_t ti = id[t];
                        id[t] = id[o];
                        id[o] = ti;
                    }
                }
            }
            __syncthreads();
        }
    for (int t = threadIdx.x; t < n - 1; t += blockDim.x) srt[(int64_t)u * n + t] = id[t];
}

// The groups' matrices over their own node numbering: linkage of node pairs
// (the slower direction), no marks, and each node's slowest link into each
// single-node cluster; every node its own cluster.  Thread per node pair of
// the whole cluster; pairs in different groups do nothing.
__global__ __launch_bounds__(256) void islands_link_init(int n, const double *__restrict__ e,
                                                         const int32_t *__restrict__ grp,
                                                         const int32_t *__restrict__ gstart,
                                                         const int32_t *__restrict__ lq,
                                                         const int64_t *__restrict__ goff, double *L, uint8_t *M,
                                                         double *XT, double *inown, int32_t *pos, int32_t *cl,
                                                         int32_t *uf) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)n * n) return;
    const int u = (int)(t / n), v = (int)(t - (int64_t)u * n);
    if (v == 0) {
        cl[u] = u;
        inown[u] = __builtin_huge_val();
        pos[u] = 0;
        uf[u] = u;
    }
    const int g = grp[u];
    if (grp[v] != g) return;
    const int64_t nm = gstart[g + 1] - gstart[g];
    const int64_t qu = lq[u], qv = lq[v], base = goff[g];
    double l = kNoPair, x = __builtin_huge_val();
    if (u != v) {
        x = e[t];
        const double y = e[(int64_t)v * n + u];
        l = x < y ? x : y;
    }
    L[base + qu * nm + qv] = l;
    M[base + qu * nm + qv] = 0;
    XT[base + qv * nm + qu] = x;
}

// ---------------------------------------------------------------------------
// a stage's components
// ---------------------------------------------------------------------------
// Root of u; parents only ever move towards smaller nodes of the same
// component, so a stale read costs a step, not the result.
__device__ inline int uf_find(int32_t *uf, int u) {
    for (;;) {
        const int p = __hip_atomic_load(uf + u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (p == u) return u;
        u = p;
    }
}

// Joins the nodes of every pair of a group linked at least as fast as the
// stage's threshold.  Parents decrease, so each retry works on a smaller root:
// the loop ends.
__global__ __launch_bounds__(256) void islands_unite(int n, double tau, const double *__restrict__ e,
                                                     const int32_t *__restrict__ grp, int32_t *uf) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)n * n) return;
    const int u = (int)(t / n), v = (int)(t - (int64_t)u * n);
    if (u >= v || grp[u] != grp[v]) return;
    if (!(e[t] >= tau) || !(e[(int64_t)v * n + u] >= tau)) return;
    int a = uf_find(uf, u), b = uf_find(uf, v);
    while (a != b) {
        if (a < b) {
            const int x = a;
            a = b;
            b = x;
        }
        const int old = atomicCAS(&uf[a], a, b);
        if (old == a) break;
        a = uf_find(uf, old);
        b = uf_find(uf, b);
    }
}

// Component lists from the roots (one block).
__global__ __launch_bounds__(kGroupThreads) void islands_components(int n, int32_t *uf, int32_t *comp, int32_t *lc,
                                                                    int32_t *cstart, int32_t *cnodes,
                                                                    int32_t *ncomp) {
    __shared__ int32_t cnt[kMaxNodes];   // nodes of a root's component, then where its list starts
    __shared__ int32_t id[kMaxNodes];    // its number
    __shared__ int32_t scan_lds[kGroupThreads / kWave + 1];
    for (int u = threadIdx.x; u < n; u += kGroupThreads) cnt[u] = 0;
    __syncthreads();
    for (int u = threadIdx.x; u < n; u += kGroupThreads) {
        const int r = uf_find(uf, u);
        comp[u] = r;
        lc[u] = atomicAdd(&cnt[r], 1);
    }
    __syncthreads();
    int32_t carry = 0, numbered = 0;
    for (int base = 0; base < n; base += kGroupThreads) {
        const int u = base + (int)threadIdx.x;
        const int32_t c = u < n ? cnt[u] : 0;
        int32_t tot, roots;
        const int32_t at = block_excl_scan<int32_t>(c, scan_lds, &tot);
        const int32_t k = block_excl_scan<int32_t>(c > 0 ? 1 : 0, scan_lds, &roots);
        if (c > 0) {
            id[u] = numbered + k;
            cnt[u] = carry + at;
            cstart[numbered + k] = carry + at;
        }
        carry += tot;
        numbered += roots;
    }
    if (threadIdx.x == 0) {
        *ncomp = numbered;
        cstart[numbered] = n;
    }
    __syncthreads();
    for (int u = threadIdx.x; u < n; u += kGroupThreads) {
        const int r = comp[u];
        cnodes[cnt[r] + lc[u]] = u;
        comp[u] = id[r];
    }
}

// Linkage and least links between the clusters a stage starts from, for pairs
// inside one component: no pair has any yet, then each node pair lowers its
// clusters' entries (links are non-negative: their bits order like the
// values).
__global__ __launch_bounds__(256) void islands_stage_clear(int n, const int32_t *__restrict__ grp,
                                                           const int32_t *__restrict__ gstart,
                                                           const int32_t *__restrict__ lq,
                                                           const int64_t *__restrict__ goff,
                                                           const int32_t *__restrict__ comp,
                                                           const int32_t *__restrict__ cl, double *L, double *XT) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)n * n) return;
    const int u = (int)(t / n), v = (int)(t - (int64_t)u * n);
    if (comp[u] != comp[v] || cl[u] != u) return;
    const int g = grp[u];
    const int64_t nm = gstart[g + 1] - gstart[g], at = goff[g] + (int64_t)lq[u] * nm + lq[v];
    XT[at] = __builtin_huge_val();
    if (cl[v] == v) L[at] = u == v ? kNoPair : __builtin_huge_val();
}

__global__ __launch_bounds__(256) void islands_stage_links(int n, const double *__restrict__ e,
                                                           const int32_t *__restrict__ grp,
                                                           const int32_t *__restrict__ gstart,
                                                           const int32_t *__restrict__ lq,
                                                           const int64_t *__restrict__ goff,
                                                           const int32_t *__restrict__ comp,
                                                           const int32_t *__restrict__ cl, double *L, double *XT) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)n * n) return;
    const int u = (int)(t / n), v = (int)(t - (int64_t)u * n);  // the link from u to v
    if (u == v || comp[u] != comp[v]) return;
    const int g = grp[u], c = cl[u], d = cl[v];
    const int64_t nm = gstart[g + 1] - gstart[g], base = goff[g];
    const double x = e[t] == 0.0 ? 0.0 : e[t];
    const unsigned long long bits = (unsigned long long)__double_as_longlong(x);
    unsigned long long *xt = (unsigned long long *)&XT[base + (int64_t)lq[d] * nm + lq[u]];
    if (bits < __hip_atomic_load(xt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMin(xt, bits);
    if (c == d) return;
    unsigned long long *l1 = (unsigned long long *)&L[base + (int64_t)lq[c] * nm + lq[d]];
    unsigned long long *l2 = (unsigned long long *)&L[base + (int64_t)lq[d] * nm + lq[c]];
    if (bits < __hip_atomic_load(l1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMin(l1, bits);
    if (bits < __hip_atomic_load(l2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMin(l2, bits);
}

// ---------------------------------------------------------------------------
// step (3): agglomerative clustering, one block per component
// ---------------------------------------------------------------------------
// Pairs are ordered by linkage (higher first), then by the smaller node id of
// the pair's two clusters, then by the larger one: key (l, x, y), x < y the
// two ids.  No pair is (-inf, INT_MAX, INT_MAX), after every pair.
__device__ inline bool key_before(double l1, int x1, int y1, double l2, int x2, int y2) {
    return l1 > l2 || (l1 == l2 && (x1 < x2 || (x1 == x2 && y1 < y2)));
}

__device__ inline bool pair_before(double l1, int x1, int y1, double l2, int x2, int y2) {
    return key_before(l1, min(x1, y1), max(x1, y1), l2, min(x2, y2), max(x2, y2));
}

// The component's state in LDS, by node number inside it (q < nm).  A cluster is
// named by its representative, its node with the least id; its members are
// perm[st[c] .. st[c] + sz[c]).
template <int kMaxNodes, int kMergeWaves>
struct MergeLds {
    int32_t gid[kMaxNodes];  // node id of q
    int16_t mq[kMaxNodes];   // its number inside the group (the matrices' numbering)
    int16_t rep[kMaxNodes];  // representative of q's cluster
    int16_t perm[kMaxNodes];
    int16_t tmp[kMaxNodes];  // rotation buffer of perm
    int16_t st[kMaxNodes];
    int16_t sz[kMaxNodes];
    double rb[kMaxNodes];    // row c: linkage of its best unmarked partner
    int16_t ra[kMaxNodes];   // row c: that partner (-1: none)
    int16_t vp[kMaxNodes];   // row c: a partner whose union is known to pass (-1: none)
    uint8_t ok[kMaxNodes];   // row c: ra[c] is known to pass
    uint8_t redo[kMaxNodes]; // row c: its best partner was just marked
    int16_t list[kMaxNodes]; // rows to work on this round
    double wv_l[kMergeWaves];
    int32_t wv_x[kMergeWaves], wv_y[kMergeWaves], wv_q[kMergeWaves];
    int32_t cnt;
};

// The group's matrices.
struct MergeMat {
    double *L;   // linkage, row and column: cluster
    uint8_t *M;  // marked pairs
    double *XT;  // row: cluster, column: node
    int64_t nm;  // the group's nodes
};

// Row c's best unmarked partner among the component's clusters, linked at least
// as fast as tau, by one wave.
template <typename Lds>
__device__ inline void merge_row_best(Lds &S, int c, int nm, const MergeMat &A, double tau, int lane) {
    const double *Lr = A.L + (int64_t)S.mq[c] * A.nm;
    const uint8_t *Mr = A.M + (int64_t)S.mq[c] * A.nm;
    constexpr int kBatch = 16;  // row entries per lane with their loads in flight together
    double b = kNoPair;
    int a = -1;
    for (int v0 = lane; v0 < nm; v0 += kBatch * kWave) {
        double l[kBatch];
        uint8_t mk[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const int v = v0 + k * kWave;
            const int q = v < nm ? S.mq[v] : 0;
            l[k] = v < nm ? Lr[q] : kNoPair;
            mk[k] = v < nm ? Mr[q] : 1;
        }
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const int v = v0 + k * kWave;
            if (v < nm && v != c && S.rep[v] == v && !mk[k] && l[k] != kNoPair && l[k] >= tau &&
                (a < 0 || l[k] > b || (l[k] == b && S.gid[v] < S.gid[a]))) {
                b = l[k];
                a = v;
            }
        }
    }
    for (int off = kWave / 2; off > 0; off >>= 1) {
        const double b2 = __shfl_xor(b, off);
        const int a2 = __shfl_xor(a, off);
        if (a2 >= 0 && (a < 0 || b2 > b || (b2 == b && S.gid[a2] < S.gid[a]))) {
            b = b2;
            a = a2;
        }
    }
    if (lane == 0) {
        S.rb[c] = b;
        S.ra[c] = (int16_t)a;
        S.ok[c] = a >= 0 && a == S.vp[c];
    }
}

// Eq. 3 for the union of clusters c and d, by one wave: a lane per member.
template <typename Lds>
__device__ inline bool merge_eq3(const Lds &S, int c, int d, int g, int n, const MergeMat &A,
                                 const double *__restrict__ e, const int32_t *__restrict__ srt,
                                 const int32_t *__restrict__ grp, const int32_t *__restrict__ lq,
                                 const double *__restrict__ inown, const int32_t *__restrict__ pos,
                                 const int32_t *__restrict__ nxl, const double *__restrict__ outv, int lane) {
    bool pass = true;
    for (int side = 0; side < 2; ++side) {
        const int own = side ? d : c, oth = side ? c : d;
        const int t0 = S.st[own], t1 = t0 + S.sz[own];
        for (int t = t0 + lane; t < t1; t += kWave) {
            const int m = S.perm[t];
            const int gm = S.gid[m];
            const double x = A.XT[(int64_t)S.mq[oth] * A.nm + S.mq[m]];
            const double io = inown[gm];
            const double in = x < io ? x : io;
            // the fastest link leaving the union: the first entry past the own
            // cluster, unless it is in the other cluster (then scan on, past
            // both: an own node can follow an outside one of equal speed)
            const int x1 = nxl[gm];
            double out = outv[gm];
            if (x1 >= 0 && S.rep[x1] == oth) {
                const int32_t *row = srt + (int64_t)gm * n;
                out = kNoPair;
                for (int p = pos[gm] + 1; p < n - 1; ++p) {
                    const int w = row[p];
                    if (grp[w] != g) {
                        out = e[(int64_t)gm * n + w];
                        break;
                    }
                    const int r = S.rep[lq[w]];
                    if (r != oth && r != own) {
                        out = e[(int64_t)gm * n + w];
                        break;
                    }
                }
            }
            if (!(in >= out)) pass = false;
        }
    }
    return __ballot(!pass) == 0;
}

// A stage's components: lists, and each node's component and number inside it.
struct StageComps {
    const int32_t *of, *num, *start, *nodes, *count;
};

// One component of a stage (components of kMinNodes to kNodes nodes; the others
// leave).  grp, lq: the component and the number inside it of each node.
template <int kMergeThreads, int kMinNodes, int kNodes>
__global__ __launch_bounds__(kMergeThreads) void islands_merge(
    int n, double tau, const double *__restrict__ e, const int32_t *__restrict__ srt, StageComps comps,
    const int32_t *__restrict__ ggrp, const int32_t *__restrict__ glq, const int32_t *__restrict__ gstart,
    const int64_t *__restrict__ goff, double *Lg, uint8_t *Mg, double *XTg, double *inown, int32_t *pos,
    int32_t *nxl, double *outv, int32_t *cl, int32_t *err) {
    constexpr int kMergeWaves = kMergeThreads / kWave;
    __shared__ MergeLds<kNodes, kMergeWaves> S;
    __shared__ int32_t scan_lds[kMergeWaves + 1];
    const int g = blockIdx.x;
    if (g >= *comps.count) return;
    const int c0 = comps.start[g], nm = comps.start[g + 1] - c0;
    if (nm < kMinNodes || nm > kNodes) return;
    const int32_t *grp = comps.of, *lq = comps.num;
    const int gg0 = ggrp[comps.nodes[c0]];
    const MergeMat A{Lg + goff[gg0], Mg + goff[gg0], XTg + goff[gg0], gstart[gg0 + 1] - gstart[gg0]};
    auto at = [&](int c, int v) { return (int64_t)S.mq[c] * A.nm + S.mq[v]; };  // entry (c, v) of a matrix
    const int lane = threadIdx.x % kWave, wv = threadIdx.x / kWave;
    int32_t *cur = (int32_t *)S.rb;  // scratch until the rows are set
    for (int q = threadIdx.x; q < nm; q += kMergeThreads) {
        const int gm = comps.nodes[c0 + q];
        S.gid[q] = gm;
        S.mq[q] = (int16_t)glq[gm];
        S.vp[q] = -1;
        S.redo[q] = 0;
        S.ra[q] = -1;
        cur[q] = 0;
    }
    __syncthreads();
    // the clusters so far: representatives, sizes, member ranges
    for (int q = threadIdx.x; q < nm; q += kMergeThreads) {
        const int r = lq[cl[S.gid[q]]];
        S.rep[q] = (int16_t)r;
        S.tmp[q] = (int16_t)atomicAdd(&cur[r], 1);  // its place in the range
        // the first entry of its sorted row outside its own cluster
        const int gm = S.gid[q], p = pos[gm];
        if (p < n - 1) {
            const int w = srt[(int64_t)gm * n + p];
            nxl[gm] = grp[w] == g ? lq[w] : -1;
            outv[gm] = e[(int64_t)gm * n + w];
        } else {
            nxl[gm] = -1;
            outv[gm] = kNoPair;
        }
    }
    __syncthreads();
    int32_t carry = 0;
    for (int base = 0; base < nm; base += kMergeThreads) {
        const int q = base + (int)threadIdx.x;
        const int32_t z = q < nm ? cur[q] : 0;
        int32_t tot;
        const int32_t ex = block_excl_scan<int32_t>(z, scan_lds, &tot);
        if (q < nm) {
            S.sz[q] = (int16_t)z;
            S.st[q] = (int16_t)(carry + ex);
        }
        carry += tot;
    }
    __syncthreads();
    for (int q = threadIdx.x; q < nm; q += kMergeThreads) S.perm[S.st[S.rep[q]] + S.tmp[q]] = (int16_t)q;
    __syncthreads();
    for (int q = wv; q < nm; q += kMergeWaves)
        if (S.rep[q] == q) merge_row_best(S, q, nm, A, tau, lane);
    __syncthreads();
    // every round merges two clusters, or marks a pair or finds one that
    // passes (a row then stays clean until a merge touches it): at most nm - 1
    // merges, each followed by at most nm^2 marks and nm clean rows
    const int64_t max_rounds = (int64_t)nm * ((int64_t)nm * nm + nm + 1) + nm * (int64_t)nm + 1;
    for (int64_t round = 0;; ++round) {
        if (round >= max_rounds) {  // a broken invariant, not an input case
            if (threadIdx.x == 0) atomicExch(err, 1);
            break;
        }
        // the best clean pair: keys in registers, wave results in LDS, which
        // every thread then reduces itself
        double bl = kNoPair;
        int bx = INT_MAX, by = INT_MAX, bq = -1;
        for (int q = threadIdx.x; q < nm; q += kMergeThreads)
            if (S.rep[q] == q && S.ra[q] >= 0 && S.ok[q]) {
                const int a = S.gid[q], b = S.gid[S.ra[q]];
                const int x = min(a, b), y = max(a, b);
                if (key_before(S.rb[q], x, y, bl, bx, by)) {
                    bl = S.rb[q];
                    bx = x;
                    by = y;
                    bq = q;
                }
            }
        for (int off = kWave / 2; off > 0; off >>= 1) {
            const double l2 = __shfl_xor(bl, off);
            const int x2 = __shfl_xor(bx, off), y2 = __shfl_xor(by, off), q2 = __shfl_xor(bq, off);
            if (key_before(l2, x2, y2, bl, bx, by)) {
                bl = l2;
                bx = x2;
                by = y2;
                bq = q2;
            }
        }
        if (lane == 0) {
            S.wv_l[wv] = bl;
            S.wv_x[wv] = bx;
            S.wv_y[wv] = by;
            S.wv_q[wv] = bq;
        }
        if (threadIdx.x == 0) S.cnt = 0;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kMergeWaves; ++w)
            if (key_before(S.wv_l[w], S.wv_x[w], S.wv_y[w], bl, bx, by)) {
                bl = S.wv_l[w];
                bx = S.wv_x[w];
                by = S.wv_y[w];
                bq = S.wv_q[w];
            }
        const int bc = bq;
        // the dirty pairs above it
        for (int q = threadIdx.x; q < nm; q += kMergeThreads)
            if (S.rep[q] == q && S.ra[q] >= 0 && !S.ok[q]) {
                const int a = S.gid[q], b = S.gid[S.ra[q]];
                if (key_before(S.rb[q], min(a, b), max(a, b), bl, bx, by)) S.list[atomicAdd(&S.cnt, 1)] = (int16_t)q;
            }
        __syncthreads();
        const int nl = S.cnt;
        if (nl > 0) {
            for (int k = wv; k < nl; k += kMergeWaves) {
                const int c = S.list[k], d = S.ra[c];
                const bool pass = merge_eq3(S, c, d, g, n, A, e, srt, grp, lq, inown, pos, nxl, outv, lane);
                if (lane == 0) {
                    if (pass) {
                        S.ok[c] = 1;
                        S.vp[c] = (int16_t)d;
                    } else {
                        A.M[at(c, d)] = 1;
                        A.M[at(d, c)] = 1;
                        // the rows whose best partner this pair was look again
                        S.redo[c] = 1;
                        if (S.ra[d] == c) S.redo[d] = 1;
                    }
                }
            }
            if (threadIdx.x == 0) S.cnt = 0;
            __syncthreads();
            for (int q = threadIdx.x; q < nm; q += kMergeThreads)
                if (S.redo[q]) {
                    S.redo[q] = 0;
                    S.list[atomicAdd(&S.cnt, 1)] = (int16_t)q;
                }
            __syncthreads();
            const int nr = S.cnt;
            for (int k = wv; k < nr; k += kMergeWaves) merge_row_best(S, S.list[k], nm, A, tau, lane);
            __syncthreads();
            continue;
        }
        if (bc < 0) break;  // no pair left
        // merge d into c, the cluster with the smaller representative id
        int c = bc, d = S.ra[bc];
        if (S.gid[d] < S.gid[c]) {
            const int x = c;
            c = d;
            d = x;
        }
        const int sc = S.st[c], zc = S.sz[c], sd = S.st[d], zd = S.sz[d];
        // slowest links into the grown cluster, before its column of XT changes
        for (int t = threadIdx.x; t < zc + zd; t += kMergeThreads) {
            const int m = S.perm[t < zc ? sc + t : sd + t - zc];
            const double x = A.XT[at(t < zc ? d : c, m)];
            const int gm = S.gid[m];
            if (x < inown[gm]) inown[gm] = x;
        }
        // complete linkage is the lesser of the two rows; pairs with the grown
        // cluster are new pairs
        for (int v = threadIdx.x; v < nm; v += kMergeThreads) {
            if (v == c || v == d) continue;
            const double lc = A.L[at(c, v)], ld = A.L[at(d, v)];
            const double l = lc < ld ? lc : ld;
            A.L[at(c, v)] = l;
            A.L[at(v, c)] = l;
            A.M[at(c, v)] = 0;
            A.M[at(v, c)] = 0;
        }
        __syncthreads();
        for (int v = threadIdx.x; v < nm; v += kMergeThreads) {
            const double xc = A.XT[at(c, v)], xd = A.XT[at(d, v)];
            A.XT[at(c, v)] = xc < xd ? xc : xd;
        }
        for (int t = threadIdx.x; t < zd; t += kMergeThreads) S.rep[S.perm[sd + t]] = (int16_t)c;
        // the two member ranges side by side: rotate the stretch between them
        const int lo = sd > sc ? sc + zc : sd, hi = sd > sc ? sd + zd : sc + zc;
        for (int t = lo + (int)threadIdx.x; t < hi; t += kMergeThreads) S.tmp[t] = S.perm[t];
        __syncthreads();
        if (sd > sc) {  // d's range moves down to just after c's
            for (int t = lo + (int)threadIdx.x; t < hi; t += kMergeThreads)
                S.perm[t] = t < lo + zd ? S.tmp[sd + (t - lo)] : S.tmp[t - zd];
            for (int q = threadIdx.x; q < nm; q += kMergeThreads)
                if (S.rep[q] == q && q != c && S.st[q] >= lo && S.st[q] < sd) S.st[q] += zd;
        } else {  // d's range moves up to just after c's, which moves down
            for (int t = lo + (int)threadIdx.x; t < hi; t += kMergeThreads)
                S.perm[t] = t < hi - zd ? S.tmp[t + zd] : S.tmp[sd + (t - (hi - zd))];
            for (int q = threadIdx.x; q < nm; q += kMergeThreads)
                if (S.rep[q] == q && q != c && S.st[q] > sd && S.st[q] < sc) S.st[q] -= zd;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            if (sd < sc) S.st[c] = (int16_t)(sc - zd);
            S.sz[c] = (int16_t)(zc + zd);
            S.cnt = 0;
        }
        __syncthreads();
        // each member's first sorted-row entry outside the grown cluster,
        // kScan entries' loads in flight at a time
        for (int t = threadIdx.x; t < zc + zd; t += kMergeThreads) {
            constexpr int kScan = 8;
            const int gm = S.gid[S.perm[S.st[c] + t]];
            const int32_t *row = srt + (int64_t)gm * n;
            int p = pos[gm], w = -1;
            while (p < n - 1) {
                int ws[kScan], gg[kScan], ll[kScan];
#pragma unroll
                for (int k = 0; k < kScan; ++k) ws[k] = p + k < n - 1 ? row[p + k] : -1;
#pragma unroll
                for (int k = 0; k < kScan; ++k) {
                    gg[k] = ws[k] >= 0 ? grp[ws[k]] : -1;
                    ll[k] = ws[k] >= 0 ? lq[ws[k]] : 0;
                }
                int hit = -1;
#pragma unroll
                for (int k = 0; k < kScan; ++k)
                    if (hit < 0 && ws[k] >= 0 && (gg[k] != g || S.rep[ll[k]] != c)) hit = k;
                if (hit >= 0) {
                    w = ws[hit];
                    p += hit;
                    break;
                }
                p += kScan;  // all in the cluster, or past the row's end
            }
            if (p > n - 1) p = n - 1;
            pos[gm] = p;
            if (p < n - 1) {
                nxl[gm] = grp[w] == g ? lq[w] : -1;
                outv[gm] = e[(int64_t)gm * n + w];
            } else {
                nxl[gm] = -1;
                outv[gm] = kNoPair;
            }
        }
        // rows to look again: the grown cluster's, and those whose best partner
        // was one of the two; the others may now prefer the grown cluster
        for (int q = threadIdx.x; q < nm; q += kMergeThreads) {
            if (S.rep[q] != q) continue;
            if (q == c || S.vp[q] == c || S.vp[q] == d) S.vp[q] = -1;
            if (q == c || S.ra[q] == c || S.ra[q] == d) {
                S.list[atomicAdd(&S.cnt, 1)] = (int16_t)q;
            } else {
                const double l = A.L[at(q, c)];
                if (l != kNoPair && l >= tau &&
                    (S.ra[q] < 0 || pair_before(l, S.gid[q], S.gid[c], S.rb[q], S.gid[q], S.gid[S.ra[q]]))) {
                    S.rb[q] = l;
                    S.ra[q] = (int16_t)c;
                    S.ok[q] = 0;
                }
            }
        }
        __syncthreads();
        const int nr = S.cnt;
        for (int k = wv; k < nr; k += kMergeWaves) merge_row_best(S, S.list[k], nm, A, tau, lane);
        __syncthreads();
    }
    for (int q = threadIdx.x; q < nm; q += kMergeThreads) cl[S.gid[q]] = S.gid[S.rep[q]];
}

// ---------------------------------------------------------------------------
// numbering and island attributes
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(1024) void islands_number(int n, const int32_t *__restrict__ cl,
                                                       const int32_t *__restrict__ gpus,
                                                       const double *__restrict__ val, int32_t *island_of,
                                                       int32_t *out_k, int32_t *isl_gpus, double *isl_val) {
    __shared__ int32_t lds[1024 / kWave + 1];
    __shared__ int32_t id[kMaxNodes];
    // island id of a representative: representatives before it
    int32_t carry = 0;
    for (int base = 0; base < n; base += blockDim.x) {
        const int u = base + threadIdx.x;
        const int32_t rep = (u < n && cl[u] == u) ? 1 : 0;
        int32_t tot;
        const int32_t ex = block_excl_scan<int32_t>(rep, lds, &tot);
        if (u < n) id[u] = carry + ex;
        carry += tot;
    }
    __syncthreads();
    const int K = carry;
    for (int k = threadIdx.x; k < K; k += blockDim.x) {
        isl_gpus[k] = 0;
        for (int f = 0; f < 4; ++f) isl_val[(int64_t)f * n + k] = __builtin_huge_val();
    }
    __syncthreads();
    // GPU sums and least values: integer sums and minima do not depend on the
    // order of the updates; the values are non-negative (a zero taken as +0),
    // so their bit patterns order like the values
    for (int u = threadIdx.x; u < n; u += blockDim.x) {
        const int k = id[cl[u]];
        island_of[u] = k;
        atomicAdd(&isl_gpus[k], gpus[u]);
        for (int f = 0; f < 4; ++f) {
            const double v = val[(int64_t)f * n + u];
            atomicMin((unsigned long long *)&isl_val[(int64_t)f * n + k],
                      (unsigned long long)__double_as_longlong(v == 0.0 ? 0.0 : v));
        }
    }
    if (threadIdx.x == 0) *out_k = K;
}

// Island-to-island bandwidth: block u reduces its row per destination island
// in LDS, then one atomic per (u, island) into the K x K matrix.  The values
// are non-negative, so their bit patterns order like the values.
__global__ __launch_bounds__(256) void islands_inter_init(int64_t kk, int K, double *isl_e) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < kk) isl_e[t] = (t / K == t % K) ? 0.0 : __builtin_huge_val();
}

__global__ __launch_bounds__(256) void islands_inter(int n, const int32_t *__restrict__ out_k,
                                                     const double *__restrict__ e,
                                                     const int32_t *__restrict__ island_of, double *isl_e) {
    __shared__ unsigned long long m[kMaxNodes];
    const int u = blockIdx.x;
    const int K = *out_k;
    const int a = island_of[u];
    for (int k = threadIdx.x; k < K; k += blockDim.x) m[k] = 0x7FF0000000000000ull;  // +inf
    __syncthreads();
    for (int v = threadIdx.x; v < n; v += blockDim.x) {
        const int b = island_of[v];
        if (b != a) atomicMin(&m[b], (unsigned long long)__double_as_longlong(e[(int64_t)u * n + v]));
    }
    __syncthreads();
    for (int k = threadIdx.x; k < K; k += blockDim.x)
        if (k != a && m[k] != 0x7FF0000000000000ull)
            atomicMin((unsigned long long *)&isl_e[(int64_t)a * K + k], m[k]);
}

template <int N>
using Int = std::integral_constant<int, N>;

hipError_t launch_build_islands(int n, const tg_island *nodes_host, const double *e_host, double eps_c,
                                double eps_m, double eps_i, void *ws, hipStream_t s, int32_t *island_of,
                                tg_island *islands, double *inter_bw, int32_t *n_islands, int64_t *bad_bw) {
    const IslandWs w = carve_islands(n, ws);
    // node columns, uploaded from the caller's arrays
    std::vector<int32_t> hg(n);
    std::vector<double> hv((size_t)4 * n);
    for (int u = 0; u < n; ++u) {
        hg[u] = nodes_host[u].n_gpus;
        hv[u] = nodes_host[u].peak_flops;
        hv[n + u] = nodes_host[u].hbm_bytes;
        hv[2 * n + u] = nodes_host[u].intra_bw;
        hv[3 * n + u] = nodes_host[u].host_bw;
    }
    hipError_t e = hipMemcpyAsync(w.gpus, hg.data(), 4 * (size_t)n, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(w.val, hv.data(), 8 * 4 * (size_t)n, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(w.e, e_host, 8 * (size_t)n * n, hipMemcpyHostToDevice, s);
    IslandState state{0, INT32_MAX, 0, 0, 0x7FF0000000000000ull, 0};
    if (e == hipSuccess) e = hipMemcpyAsync(w.state, &state, sizeof(state), hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return e;
    const int64_t nn = (int64_t)n * n;
    // a block's two updates of the state go one after the other: 2048 blocks took
    // 22 us over 1024 nodes
    islands_check<<<dim3((unsigned)std::min<int64_t>((nn + 255) / 256, 256)), dim3(256), 0, s>>>(n, w.e, w.state);
    islands_groups<<<dim3(1), dim3(kGroupThreads), 0, s>>>(n, w.gpus, w.val, eps_c, eps_m, eps_i, w.grp, w.gstart,
                                                           w.gnodes, w.ngroups, w.lq, w.goff,
                                                           w.state);
    e = hipMemcpyAsync(&state, w.state, sizeof(state), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);  // the host staging arrays go away
    if (e != hipSuccess) return e;
    *bad_bw = state.bad == INT32_MAX ? -1 : state.bad;
    if (state.bad != INT32_MAX) return hipSuccess;
    double least, most;
    std::memcpy(&least, &state.least, 8);
    std::memcpy(&most, &state.most, 8);
    const int staged = 2 * (int64_t)state.same >= nn ? kStagedNodes : kStagedOdd;
    const int first = state.group < staged || least > kStageShare[0] * most ? kStages - 1 : 0;
    const dim3 pairs((unsigned)((nn + 255) / 256));
    islands_link_init<<<pairs, dim3(256), 0, s>>>(n, w.e, w.grp, w.gstart, w.lq, w.goff, w.L, w.M, w.XT, w.inown,
                                                  w.pos, w.cl, w.uf);
    islands_sort_rows<<<dim3((unsigned)n), dim3(1024), 0, s>>>(n, w.e, w.srt);
    for (int st = first; st < kStages; ++st) {
        const bool last = st == kStages - 1;
        const double tau = last ? kNoPair : kStageShare[st] * most;
        StageComps comps{w.comp, w.lc, w.cstart, w.cnodes, w.ncomp};
        if (last) {
            comps = StageComps{w.grp, w.lq, w.gstart, w.gnodes, w.ngroups};
        } else {
            islands_unite<<<pairs, dim3(256), 0, s>>>(n, tau, w.e, w.grp, w.uf);
            islands_components<<<dim3(1), dim3(kGroupThreads), 0, s>>>(n, w.uf, w.comp, w.lc, w.cstart, w.cnodes,
                                                                       w.ncomp);
        }
        if (st > first) {
            islands_stage_clear<<<pairs, dim3(256), 0, s>>>(n, w.grp, w.gstart, w.lq, w.goff, comps.of, w.cl, w.L,
                                                            w.XT);
            islands_stage_links<<<pairs, dim3(256), 0, s>>>(n, w.e, w.grp, w.gstart, w.lq, w.goff, comps.of, w.cl,
                                                            w.L, w.XT);
        }
        auto merge = [&](auto threads, auto fewest, auto most_nodes) {
            constexpr int NT = decltype(threads)::value;
            islands_merge<NT, decltype(fewest)::value, decltype(most_nodes)::value>
                <<<dim3((unsigned)n), dim3(NT), 0, s>>>(n, tau, w.e, w.srt, comps, w.grp, w.lq, w.gstart, w.goff, w.L,
                                                        w.M, w.XT, w.inown, w.pos, w.nxl, w.outv, w.cl,
                                                        &w.state->err);
        };
        if (last && state.group > kOneSmall) {
            merge(Int<kMergeThreads>{}, Int<2>{}, Int<kMaxNodes>{});
        } else {
            merge(Int<kSmallThreads>{}, Int<2>{}, Int<kSmallComp>{});
            if (state.group > kSmallComp) merge(Int<kMergeThreads>{}, Int<kSmallComp + 1>{}, Int<kMaxNodes>{});
        }
    }
    islands_number<<<dim3(1), dim3(1024), 0, s>>>(n, w.cl, w.gpus, w.val, w.island_of, w.out_k, w.isl_gpus,
                                                  w.isl_val);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    int32_t K = 0, merr = 0;
    e = hipMemcpyAsync(&K, w.out_k, 4, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipMemcpyAsync(&merr, &w.state->err, 4, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    if (merr) return hipErrorUnknown;
    const int64_t kk = (int64_t)K * K;
    islands_inter_init<<<dim3((unsigned)((kk + 255) / 256)), dim3(256), 0, s>>>(kk, K, w.isl_e);
    islands_inter<<<dim3((unsigned)n), dim3(256), 0, s>>>(n, w.out_k, w.e, w.island_of, w.isl_e);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    std::vector<int32_t> og(K > 0 ? K : 1);
    std::vector<double> ov((size_t)4 * n);
    e = hipMemcpyAsync(island_of, w.island_of, 4 * (size_t)n, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipMemcpyAsync(og.data(), w.isl_gpus, 4 * (size_t)K, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipMemcpyAsync(ov.data(), w.isl_val, 8 * 4 * (size_t)n, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipMemcpyAsync(inter_bw, w.isl_e, 8 * (size_t)kk, hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e == hipSuccess) {
        for (int k = 0; k < K; ++k) {
            islands[k].n_gpus = og[k];
            islands[k].reserved = 0;
            islands[k].peak_flops = ov[k];
            islands[k].hbm_bytes = ov[n + k];
            islands[k].intra_bw = ov[2 * n + k];
            islands[k].host_bw = ov[3 * n + k];
        }
        *n_islands = K;
    }
    return e;
}

}  // namespace tg
