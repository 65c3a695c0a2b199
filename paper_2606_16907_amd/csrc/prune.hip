// prune.hip -- the surviving set: incompatibility, infeasibility and
// dominance pruning (Sec. 5.1), as a frontier pass plus a stream compaction.
//
// Group G = (slice s, island k, micro-batch b).  A member p survives iff b
// divides the global batch, (s, k) passes imbalance pruning when it is on,
// d_max_p >= 1 and p has the least key (cost, -d_max, idx) among members whose
// d_max reaches d_max_p.  Equivalently the survivors are rep(G, d) for d = 1..K,
// the least-key member fitting at depth d: a member survives iff no other member
// at least as deep has a smaller key.
//
// Frontier: a wave owns 64 consecutive slices of one (island, b) group list;
// every lane walks the same members (a scalar loop) in ascending idx, reading
// one coalesced 64-byte row of depths per member and, where the depth can
// still matter, one 512-byte row of costs, eight members in flight.  On
// clusters of up to 32 islands with enough members a group each lane keeps the
// least cost of every depth in LDS (frontier_buckets); elsewhere each lane keeps
// the staircase of its group in registers (up to kStair entries of strictly
// increasing depth and key): a member is dropped when an entry at least as deep
// costs no more; otherwise it removes the entries it beats and takes a slot.
// When the slots are full the shallowest of them and the newcomer leaves and the
// pass ignores every member at or above its depth from then on: survival of a
// member depends only on members at least as deep, so the entries kept are
// exactly the survivors deeper than that depth.  A further pass (rare: more than
// kStair survivors in one group) settles the shallower ones, with the least kept
// entry as a cost cap.  Each pass records its entries in an LDS bit mask per
// member (lane bit = slice), 512 members at a time, written as whole 64-bit words
// of a bitmap with one row per compatible config (a later pass ORs into the words
// it wrote).
// Compaction: popcounts per tile of words, then each block adds up the counts
// of the tiles before its own (scanned first where there are many tiles) and
// writes its candidate indices in ascending order, dealt one by one in sparse
// tiles and word by word in dense ones.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "tg_device.h"

namespace tg {

constexpr int kFrontWaves = 4;
// Staircase entries a lane keeps per pass: 4 for groups of up to 64 members
// (64 VGPRs, 8 waves per SIMD), 8 above (86 VGPRs, 5 waves per SIMD), where
// staircases grow longer and a second pass would cost more than occupancy.
constexpr int kSmallGroup = 64;
constexpr int kMaskChunk = 512;   // members per LDS mask round when a pass is recorded
constexpr int kMemberBits = 23;   // an entry packs depth << kMemberBits | member
constexpr uint32_t kMemberMask = (1u << kMemberBits) - 1u;
constexpr int kEmitThreads = 256;
// Words a thread of the compaction takes: four, or one up to kFineWords words (a
// tile of rows that survive everywhere has 64 outputs a word, and with few
// tiles the densest sets the time: 24 -> 12 us on the 70B instance's 228,000
// words).  In a bitmap of at most kSmallWords words a block counts the words
// before its tile by itself (at most 32 a thread) and no count pass runs.
constexpr int64_t kSmallWords = 8192;
constexpr int64_t kFineWords = (int64_t)4096 * kEmitThreads;
// Tile counts a block adds up by itself, at most (32 a thread); above that a
// scan of the counts runs first.
constexpr int64_t kSumTiles = 8192;

static int words_per_thread(int64_t n_words) { return n_words <= kFineWords ? 1 : 4; }

// Offer member m (cost c, depth d >= 1, later in idx than every entry) to a
// lane's staircase.  Entry e beats m when d_e >= d and c_e <= c (equal cost:
// the deeper key is smaller, and equal depth: the earlier idx).
template <int R>
__device__ inline void stair_offer(double (&cv)[R], uint32_t (&pk)[R], double c, int d, int m, int &floor) {
    const uint32_t dk = (uint32_t)d << kMemberBits;
    bool beaten = false;
#pragma unroll
    for (int r = 0; r < R; ++r) beaten = beaten || (pk[r] >= dk && cv[r] <= c);  // empty slots hold 0
    if (beaten) return;
    const uint32_t dk1 = (uint32_t)(d + 1) << kMemberBits;
    const uint32_t x = dk | (uint32_t)m;
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (pk[r] < dk1 && cv[r] >= c) pk[r] = 0u;  // entries m beats
    bool placed = false;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const bool t = !placed && pk[r] == 0u;
        if (t) {
            pk[r] = x;
            cv[r] = c;
        }
        placed = placed || t;
    }
    if (placed) return;
    // full: the shallowest of the entries and m leaves, and its depth becomes the floor
    uint32_t lo = x;
#pragma unroll
    for (int r = 0; r < R; ++r) lo = min(lo, pk[r]);
    floor = (int)(lo >> kMemberBits);
    if (lo == x) return;
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (pk[r] == lo) {
            pk[r] = x;
            cv[r] = c;
        }
}

__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Writes the bitmap words of every member of the wave's group for its slice
// chunk: the lanes' entries set their bits in an LDS mask, kChunk members
// at a time.  After the first pass a word also keeps the bits it already
// has.
template <int kStair, int kChunk>
__device__ inline void record_pass(const DevProblem &P, uint64_t *mask, const uint32_t (&pk)[kStair], bool mine,
                                   int lane, int m0, int nm, int64_t sc, bool merge, uint64_t *bitmap) {
    for (int base = 0; base < nm; base += kChunk) {
        const int n = min(kChunk, nm - base);
        for (int m = lane; m < n; m += kWave) mask[m] = 0;
        wave_sync();
        if (mine) {
#pragma unroll
            for (int r = 0; r < kStair; ++r) {
                const int m = (int)(pk[r] & kMemberMask) - base;
                if (pk[r] != 0u && m >= 0 && m < n) atomicOr((unsigned long long *)&mask[m], 1ull << lane);
            }
        }
        wave_sync();
        for (int m = lane; m < n; m += kWave) {
            uint64_t *at = bitmap + (int64_t)P.kb_rows[m0 + base + m] * P.words + sc;
            *at = merge ? (*at | mask[m]) : mask[m];
        }
        wave_sync();
    }
}

// Members whose cost is no number (scores of this library are numbers; a
// caller's arrays may hold anything) survive where they fit at all and beat
// nobody: their bits are added to the words already recorded, by the lane that
// wrote them.
__device__ inline void nan_pass(const DevProblem &P, const double *__restrict__ cost,
                                const uint8_t *__restrict__ dmax, uint64_t *bitmap, bool need, int lane, int m0,
                                int nm, int64_t s, int64_t sc) {
    for (int m = 0; m < nm; ++m) {
        const int64_t at = (int64_t)P.kb_members[m0 + m] * P.NS + s;
        bool mine = false;
        if (need && dmax[at] > 0) {
            const double c = cost[at];
            mine = c != c;
        }
        const uint64_t word = __ballot(mine);
        if (word && lane == (m & (kWave - 1))) bitmap[(int64_t)P.kb_rows[m0 + m] * P.words + sc] |= word;
    }
}

// The register staircase of a wave: its 64 slices' groups (members m0 .. m0 + nm
// - 1) in as many passes as their survivors need, each recorded in the bitmap.
// `need` lanes have a group.  A cost that is no number is not offered (several
// of one depth would fill the slots in every pass, without end).  Inlined before
// anything is optimized: simplified as a function of its own first, the offers
// lose half of the branches by which a wave skips what no lane needs, and the
// extended space on 33 islands and 8 layers took 270 us a prune against 219.
template <int kStair, int kChunk>
__device__ __forceinline__ void stair_passes(const DevProblem &P, uint64_t *mask, const double *__restrict__ cost,
                                             const uint8_t *__restrict__ dmax, uint64_t *bitmap, bool need, int lane,
                                             int m0, int nm, int64_t s, int64_t sc) {
    const int64_t NS = P.NS;
    const bool grouped = need;
    bool nan = false;
    int hi = 1 << 30;  // members deeper than hi are settled (by an earlier pass)
    double cap = 0.0;  // least cost among the settled members, once there are any
    bool capped = false;
    bool merge = false;
    do {  // every wave records at least one pass: it writes all of its words
        double cv[kStair];
        uint32_t pk[kStair];
#pragma unroll
        for (int r = 0; r < kStair; ++r) {
            cv[r] = 0.0;
            pk[r] = 0u;
        }
        int floor = 0;  // members at or above this depth no longer matter in this pass
        for (int mb = 0; mb < nm; mb += 8) {
            int d[8];
            double c[8];
            const double *crow[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int64_t row = (int64_t)P.kb_members[m0 + min(mb + u, nm - 1)] * NS;
                crow[u] = cost + row;
                d[u] = (mb + u < nm && need) ? (int)dmax[row + s] : 0;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) c[u] = (d[u] > floor && d[u] <= hi) ? crow[u][s] : 0.0;
            uint64_t odd = 0;  // one check for two costs, acted on once a batch (a branch a member took 8% longer)
#pragma unroll
            for (int u = 0; u < 8; u += 2) odd |= __ballot(__builtin_isunordered(c[u], c[u + 1]));
            if (__builtin_expect(odd != 0, 0)) {
                nan = true;
#pragma unroll
                for (int u = 0; u < 8; ++u) d[u] = c[u] == c[u] ? d[u] : 0;
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (d[u] > floor && d[u] <= hi && !(capped && cap <= c[u]))
                    stair_offer<kStair>(cv, pk, c[u], d[u], mb + u, floor);
        }
        record_pass<kStair, kChunk>(P, mask, pk, need, lane, m0, nm, sc, merge, bitmap);
        merge = true;
        if (need) {
            if (floor == 0) {
                need = false;
            } else {  // the survivors at or above the floor are still to be found
                uint32_t lo = 0xFFFFFFFFu;
#pragma unroll
                for (int r = 0; r < kStair; ++r)
                    if (pk[r] != 0u && pk[r] < lo) {
                        lo = pk[r];
                        cap = cv[r];
                    }
                hi = floor;
                capped = true;
            }
        }
        // a further pass reads back the words this wave wrote (each lane the
        // same words, so program order already holds; the fence makes it plain)
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    } while (__ballot(need) != 0);
    if (__builtin_expect(nan, 0)) nan_pass(P, cost, dmax, bitmap, grouped, lane, m0, nm, s, sc);
}

template <int kStair>
__global__ __launch_bounds__(256) void frontier_kernel(DevProblem P, const double *__restrict__ cost,
                                                       const uint8_t *__restrict__ dmax, uint64_t *bitmap,
                                                       int64_t n_tiles) {
    __shared__ uint64_t smask[kFrontWaves][kMaskChunk];
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t tile = (int64_t)blockIdx.x * kFrontWaves + wv;
    if (tile >= n_tiles) return;  // whole waves leave; nothing below synchronises the block
    const int q = (int)(tile / P.words);
    const int64_t sc = tile - (int64_t)q * P.words;
    const int m0 = P.kb_off[q];
    const int nm = P.kb_off[q + 1] - m0;
    const int64_t s = sc * kWave + lane;
    bool need = s < P.NS;
    if (need && P.imb) {  // an unbalanced (slice, island) group has no survivors
        const uint32_t ij = P.sij[s];
        need = slice_balanced(P, P.pre, (int)(ij & 0xFFFFu), (int)(ij >> 16), P.kb_island[q]);
    }
    stair_passes<kStair, kMaskChunk>(P, smask[wv], cost, dmax, bitmap, need, lane, m0, nm, s, sc);
}

// The frontier by depth buckets, for clusters of at most kBucketDepths islands
// (depths 1..K): a wave keeps, per lane and depth, the least cost among the
// group's members that fit exactly that deep and the first member costing it,
// in LDS.  A member is one LDS minimum that returns the value before it, now and
// then a write, and a batch's eight are in flight together (a read, a compare
// and a write one after the other: 433 us a prune of the extended MoE instance,
// this way 394); the register staircase compares and moves up to eight entries
// (about 160 instructions a member; it was issue-bound at under 2 TB/s on the
// extended MoE instance).  Afterwards a sweep from the deepest bucket up keeps
// those cheaper than everything deeper: the survivors, whatever their number, in
// one pass.  Bound by the depth-then-cost loads of kBucketBatch members in flight
// (the next batch's depths load with this batch's costs) at the 7 to 13 waves a
// CU that 22 KB a wave (32 islands) to 12 KB (16) leave at most.  A wider cluster
// keeps the registers: with 80 layers of the MoE model a prune takes 299, 316 and
// 342 us on 36, 40 and 48 islands with the staircase and 329, 414 and 580 with
// buckets (33 islands: 283 and 271), though models too short to fill the card
// would gain (8 layers on 40 islands 103 and 67).  Groups go largest first, so the last blocks are short ones.
// This library's depths are at most K; a wave that meets a deeper one in a
// caller's arrays starts over with the staircase, which has no such limit (the
// LDS bounds the waves a CU holds, so its registers are free here).
// Register staircase -> buckets, frontier kernel: extended MoE 790 -> 370 us,
// extended 70B 385 -> 275, uneven 27 islands 113 -> 103, MoE 90 -> 64, 70B 38 ->
// 35, 8B 17 -> 13; batches of 12, 16 and 24 members within 3% either way.
constexpr int kBucketDepths = 32;
constexpr int kBucketMembers = 0xFFFE;  // a member's number in its group takes 16 bits
constexpr int kBucketBatch = 8;
static_assert(kMemberPad >= kBucketBatch - 1, "a batch reads past its group");
constexpr int kBucketChunk = 128;       // members per LDS mask round

// Buckets pay for setting up and sweeping K depths a group, so they take
// clusters whose groups average at least 1.5 K members: at 1.5 to 1.8 (uneven,
// 70B, MoE) they gain 8 to 40%, at 1.0 (18 islands, 125 layers, 18 members a
// group) the staircase took 123 us a call against 142.
static bool use_buckets(const DevProblem &P) {
    return P.K <= kBucketDepths && P.max_members <= kBucketMembers &&
           2 * (int64_t)P.n_rows >= 3 * (int64_t)P.K * P.n_kb;
}

static size_t bucket_lds(int K) { return (size_t)(K + 1) * kWave * (sizeof(double) + sizeof(uint16_t)); }

__global__ __launch_bounds__(kWave) void frontier_buckets(DevProblem P, const double *__restrict__ cost,
                                                          const uint8_t *__restrict__ dmax,
                                                          uint64_t *__restrict__ bitmap) {
    extern __shared__ double lds_best[];       // [K + 1][64] least cost of each depth; 0: what counts for nothing
    __shared__ uint64_t mask[kBucketChunk];
    const int K = P.K;
    const int lane = threadIdx.x;
    double *least_at = lds_best + lane;
    uint16_t *who_at = (uint16_t *)(lds_best + (int64_t)(K + 1) * kWave) + lane;
    double *best = least_at + kWave;           // depth d: best[(d - 1) * 64]
    uint16_t *who = who_at + kWave;
    constexpr uint16_t kNone = 0xFFFF;
    constexpr double kNever = __builtin_huge_val();
    const int qo = (int)(blockIdx.x / P.words);
    const int64_t sc = blockIdx.x - (int64_t)qo * P.words;
    const int q = P.kb_order[qo];
    const int m0 = P.kb_off[q];
    const int nm = P.kb_off[q + 1] - m0;
    const int64_t s = sc * kWave + lane;
    const int64_t NS = P.NS;
    bool need = s < NS;
    if (need && P.imb) {  // an unbalanced (slice, island) group has no survivors
        const uint32_t ij = P.sij[s];
        need = slice_balanced(P, P.pre, (int)(ij & 0xFFFFu), (int)(ij >> 16), P.kb_island[q]);
    }
    for (int d = 0; d <= K; ++d) {
        least_at[d * kWave] = kNever;
        who_at[d * kWave] = kNone;
    }
    const int64_t at = need ? s : 0;  // lanes that score nothing read row starts
    // the list has kMemberPad more entries: rows past this group's are read and
    // ignored, so a batch's members load together, with no end to check
    const int32_t *list = P.kb_members + m0;
    auto row = [&](int m) { return (int64_t)((uint64_t)(uint32_t)list[m] * (uint32_t)NS); };
    int deepest = 0;
    uint64_t nan = 0;  // lanes that met one
    int d[kBucketBatch];
    const int left = need ? nm : 0;
#pragma unroll
    for (int u = 0; u < kBucketBatch; ++u) {
        const int v = (dmax + row(u))[at];
        d[u] = u < left ? v : 0;
    }
    for (int mb = 0; mb < nm; mb += kBucketBatch) {
        double c[kBucketBatch];
        int dn[kBucketBatch];
#pragma unroll
        for (int u = 0; u < kBucketBatch; ++u) c[u] = d[u] > 0 ? (cost + row(mb + u))[at] : 0.0;
        const int next = mb + kBucketBatch < nm ? mb + kBucketBatch : mb;  // the last batch reads itself again
#pragma unroll
        for (int u = 0; u < kBucketBatch; ++u) {
            const int v = (dmax + row(next + u))[at];
            dn[u] = mb + kBucketBatch + u < left ? v : 0;
        }
        // a wave's LDS operations take effect in order: each member's atomic
        // returns the least cost before it, this batch's earlier members'
        // included, and all eight are in flight together
        double before[kBucketBatch];
        int slot[kBucketBatch];
        uint64_t odd = 0;
#pragma unroll
        for (int u = 0; u < kBucketBatch; ++u) {
            deepest = max(deepest, d[u]);
            odd |= __ballot(!(c[u] < kNever));
            slot[u] = (c[u] == c[u] ? min(d[u], K) : 0) * kWave;
            before[u] = __hip_atomic_fetch_min(&least_at[slot[u]], c[u] == c[u] ? c[u] : 0.0, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_WAVEFRONT);
        }
#pragma unroll
        for (int u = 0; u < kBucketBatch; ++u)
            if (!(before[u] <= c[u])) who_at[slot[u]] = (uint16_t)(mb + u);  // ties stay with the earlier member
        if (__builtin_expect(odd != 0, 0)) {  // an infinite cost takes a depth that has no member yet
#pragma unroll
            for (int u = 0; u < kBucketBatch; ++u) {
                nan |= __ballot(c[u] != c[u]);
                if (c[u] == kNever && who_at[slot[u]] == kNone) who_at[slot[u]] = (uint16_t)(mb + u);
            }
        }
#pragma unroll
        for (int u = 0; u < kBucketBatch; ++u) d[u] = dn[u];
    }
    if (__builtin_expect(__ballot(deepest > K) != 0, 0)) {
        if (P.max_members <= kSmallGroup)
            stair_passes<4, kBucketChunk>(P, mask, cost, dmax, bitmap, need, lane, m0, nm, s, sc);
        else
            stair_passes<8, kBucketChunk>(P, mask, cost, dmax, bitmap, need, lane, m0, nm, s, sc);
        return;
    }
    // a bucket survives if it is cheaper than every deeper one
    double least = __builtin_nan("");
    for (int e = K - 1; e >= 0; --e) {
        const double v = best[e * kWave];
        if (who[e * kWave] != kNone && !(least <= v))
            least = v;
        else
            who[e * kWave] = kNone;
    }
    for (int base = 0; base < nm; base += kBucketChunk) {
        const int n = min(kBucketChunk, nm - base);
        for (int m = lane; m < n; m += kWave) mask[m] = 0;
        wave_sync();
        for (int e = 0; e < K; ++e) {
            const int m = (int)who[e * kWave] - base;  // kNone is past every chunk
            if (m >= 0 && m < n) atomicOr((unsigned long long *)&mask[m], 1ull << lane);
        }
        wave_sync();
        for (int m = lane; m < n; m += kWave) bitmap[(int64_t)P.kb_rows[m0 + base + m] * P.words + sc] = mask[m];
        wave_sync();
    }
    if (__builtin_expect(nan != 0, 0)) {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
        nan_pass(P, cost, dmax, bitmap, need, lane, m0, nm, s, sc);
    }
}

template <int WPT>
__global__ __launch_bounds__(kEmitThreads) void count_kernel(const uint64_t *__restrict__ bitmap, int64_t n_words,
                                                             int64_t *tile_cnt) {
    __shared__ int64_t lds[kEmitThreads / kWave + 1];
    const int64_t base = (int64_t)blockIdx.x * kEmitThreads * WPT + (int64_t)threadIdx.x * WPT;
    int64_t c = 0;
#pragma unroll
    for (int w = 0; w < WPT; ++w)
        if (base + w < n_words) c += __popcll(bitmap[base + w]);
    int64_t total;
    block_excl_scan<int64_t>(c, lds, &total);
    if (threadIdx.x == 0) tile_cnt[blockIdx.x] = total;
}

// Exclusive scan of n int64 values in place by one block.
__global__ __launch_bounds__(1024) void scan_small_i64(int64_t *a, int64_t n) {
    __shared__ int64_t lds[1024 / kWave + 1];
    int64_t carry = 0;
    for (int64_t base = 0; base < n; base += blockDim.x) {
        const int64_t i = base + threadIdx.x;
        const int64_t v = i < n ? a[i] : 0;
        int64_t sum;
        const int64_t ex = block_excl_scan<int64_t>(v, lds, &sum);
        if (i < n) a[i] = carry + ex;
        carry += sum;
    }
}

// Position of the n-th set bit of w (from 0; w has more than n).
__device__ inline int nth_bit(uint64_t w, int n) {
    uint32_t x = (uint32_t)w;
    int pos = 0;
    int c = __popc(x);
    if (n >= c) {
        n -= c;
        x = (uint32_t)(w >> 32);
        pos = 32;
    }
#pragma unroll
    for (int half = 16; half > 0; half >>= 1) {
        c = __popc(x & ((1u << half) - 1u));
        if (n >= c) {
            n -= c;
            x >>= half;
            pos += half;
        }
    }
    return pos;
}

// Bitmap -> ascending candidate indices, and their number to *total and, when
// given, *total_host.  A sparse tile's outputs are dealt to its threads one by
// one (the word by bisection over the words' offsets in LDS, the bit by
// popcounts): a thread walking its own words' bits had up to 256 dependent
// stores.  A dense tile (kWalkBits bits a word) goes word by word, a lane per
// bit.  Both ways the stores are coalesced.  Dealing costs about 100 instructions
// an output and walking 12 a word: 28 rows of 8,256 slices of a narrow space
// (104,950 survivors, up to 64 a word) took 34 us dealt, 11 walked, and 21 with the
// thread walk.
// WPT: words a thread takes.  kFrom: where the bits before the tile come from.
constexpr int kWalkBits = 8;
enum class Before { kWords, kCounts, kScan };

template <int WPT, Before kFrom>
__global__ __launch_bounds__(kEmitThreads) void emit_kernel(DevProblem P, const uint64_t *__restrict__ bitmap,
                                                            int64_t n_words, const int64_t *__restrict__ tile_cnt,
                                                            int64_t *out, int64_t capacity, int64_t *total,
                                                            int64_t *total_host) {
    constexpr int kTile = kEmitThreads * WPT;
    __shared__ uint64_t sw[kTile];   // the words
    __shared__ int64_t sbase[kTile]; // candidate index of each word's bit 0
    __shared__ int32_t soff[kTile];  // set bits before each word in the tile
    __shared__ int32_t lds[kEmitThreads / kWave + 1];
    __shared__ int64_t wsum[kEmitThreads / kWave];
    const int64_t tile = blockIdx.x;
    const int64_t w0 = tile * kTile + (int64_t)threadIdx.x * WPT;
    uint64_t w[WPT];
    int32_t c = 0;
#pragma unroll
    for (int t = 0; t < WPT; ++t) w[t] = w0 + t < n_words ? bitmap[w0 + t] : 0ull;
    int64_t mine = 0;  // this thread's share of the bits before the tile
    if (kFrom == Before::kWords)
#pragma unroll 8
        for (int64_t t = threadIdx.x; t < tile * kTile; t += kEmitThreads) mine += __popcll(bitmap[t]);
    if (kFrom == Before::kCounts)
#pragma unroll 8
        for (int64_t t = threadIdx.x; t < tile; t += kEmitThreads) mine += tile_cnt[t];
    if (kFrom == Before::kScan && threadIdx.x == 0) mine = tile_cnt[tile];
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) mine += __shfl_xor(mine, off);
    if (wave_lane() == 0) wsum[threadIdx.x / kWave] = mine;
#pragma unroll
    for (int t = 0; t < WPT; ++t) c += __popcll(w[t]);
    int32_t count;
    int32_t off = block_excl_scan<int32_t>(c, lds, &count);
    int64_t row = w0 / P.words;
    int64_t sc = w0 - row * P.words;
#pragma unroll
    for (int t = 0; t < WPT; ++t) {
        const int at = (int)threadIdx.x * WPT + t;
        sw[at] = w[t];
        soff[at] = off;
        off += __popcll(w[t]);
        if (w[t]) sbase[at] = (int64_t)P.row_cfg[row] * P.NS + sc * kWave;
        if (++sc == P.words) {
            sc = 0;
            ++row;
        }
    }
    __syncthreads();
    int64_t before = 0;
#pragma unroll
    for (int u = 0; u < kEmitThreads / kWave; ++u) before += wsum[u];
    if (threadIdx.x == 0 && tile == gridDim.x - 1) {
        *total = before + count;
        if (total_host) *total_host = before + count;
    }
    if (count >= kWalkBits * kTile) {  // a wave takes its words in turn, a lane a bit
        const int lane = wave_lane(), a0 = (int)threadIdx.x / kWave * (kTile / (kEmitThreads / kWave));
#pragma unroll 4
        for (int at = a0; at < a0 + kTile / (kEmitThreads / kWave); ++at) {
            const uint64_t x = sw[at];
            const int64_t pos = before + soff[at] + __popcll(x & ((1ull << lane) - 1ull));
            if ((x >> lane & 1ull) && pos < capacity) out[pos] = sbase[at] + lane;
        }
        return;
    }
    for (int32_t r = threadIdx.x; r < count; r += kEmitThreads) {
        int at = 0;  // the last word whose offset is at most r
#pragma unroll
        for (int step = kTile / 2; step > 0; step >>= 1)
            if (soff[at + step] <= r) at += step;
        const int64_t pos = before + r;
        if (pos < capacity) out[pos] = sbase[at] + nth_bit(sw[at], r - soff[at]);
    }
}

__global__ void no_survivors(int64_t *total, int64_t *total_host) {
    *total = 0;
    if (total_host) *total_host = 0;
}

// Redundancy pruning: bit s of a row of the slice bitmap is bit cls[s] of
// the same row of the class bitmap (a class's staircase holds on every slice
// of the class).  A block keeps the classes of up to kExpandSlices slices in
// LDS and runs kExpandRows rows through them, a wave per row: a row without
// survivors (most are) is only cleared, else 64 slices' bits make a word by
// ballot, 64 words go out in one store.  Reading the classes per word from L2
// and dividing per word took 380 us on the 128-layer instance (4.2M words);
// this takes 73 us.
constexpr int kExpandSlices = (160 * 1024 / 8 - 256) / 4;  // eight blocks fill a CU; 256 bytes are the vote's
constexpr int kExpandRows = 8;
constexpr int kExpandWords = 8;  // words a wave builds at a time, their reads in flight together

__global__ __launch_bounds__(256) void expand_kernel(DevProblem P, const uint64_t *__restrict__ cbits,
                                                     int32_t cwords, uint64_t *bits, int pieces, int piece) {
    __shared__ uint32_t cls[kExpandSlices];
    const int pc = blockIdx.x % pieces;  // a piece: `piece` slices, whole words
    const int64_t r0 = (int64_t)(blockIdx.x / pieces) * kExpandRows;
    const int64_t r1 = min(r0 + kExpandRows, (int64_t)P.n_rows);
    const int64_t s0 = (int64_t)pc * piece;
    const int ns = (int)min((int64_t)piece, P.NS - s0);
    const int nw = (ns + kWave - 1) / kWave;
    const int lane = wave_lane(), wv = threadIdx.x / kWave;
    // the classes only once a row needs them
    bool any = false;
    for (int64_t t = r0 * cwords + threadIdx.x; t < r1 * cwords; t += 256) any = any || cbits[t] != 0;
    if (__syncthreads_or(any)) {
        for (int t = threadIdx.x; t < ns; t += 256) cls[t] = P.cls[s0 + t];
        __syncthreads();
    }
    for (int64_t row = r0 + wv; row < r1; row += 256 / kWave) {
        const uint64_t *cb = cbits + row * cwords;
        uint64_t *to = bits + row * P.words + s0 / kWave;
        bool live = false;
        for (int w = lane; w < cwords; w += kWave) live = live || cb[w] != 0;
        if (__ballot(live) == 0) {
            for (int w = lane; w < nw; w += kWave) to[w] = 0;
            continue;
        }
        for (int b0 = 0; b0 < nw; b0 += kWave) {
            uint64_t mine = 0;
            for (int k0 = 0; k0 < kWave && b0 + k0 < nw; k0 += kExpandWords) {
                uint32_t c[kExpandWords];
                uint64_t x[kExpandWords];
#pragma unroll
                for (int k = 0; k < kExpandWords; ++k) {
                    const int t = (b0 + k0 + k) * kWave + lane;
                    c[k] = cls[min(t, ns - 1)];
                }
#pragma unroll
                for (int k = 0; k < kExpandWords; ++k) x[k] = cb[c[k] >> 6];
#pragma unroll
                for (int k = 0; k < kExpandWords; ++k) {
                    const bool in = (b0 + k0 + k) * kWave + lane < ns;
                    const uint64_t word = __ballot(in && ((x[k] >> (c[k] & 63)) & 1ull));
                    if (lane == k0 + k) mine = word;
                }
            }
            if (b0 + lane < nw) to[b0 + lane] = mine;
        }
    }
}

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

static int64_t bitmap_words(const DevProblem &P) { return (int64_t)P.n_rows * P.words; }

// The prune workspace: the bitmap, the tile counts, the survivor count.
struct PruneWs {
    uint64_t *bitmap;
    int64_t *tiles, *total;
    int64_t n_words, n_tiles;
    size_t bytes;
};

static PruneWs carve_prune(const DevProblem &P, void *ws) {
    PruneWs w{};
    w.n_words = bitmap_words(P);
    const int64_t tile = (int64_t)kEmitThreads * words_per_thread(w.n_words);
    w.n_tiles = (w.n_words + tile - 1) / tile;
    const size_t tiles_at = align256(sizeof(uint64_t) * (size_t)(w.n_words > 0 ? w.n_words : 1));
    const size_t total_at = tiles_at + align256(sizeof(int64_t) * (size_t)(w.n_tiles + 1));
    w.bytes = total_at + align256(sizeof(int64_t));
    if (ws) {
        w.bitmap = (uint64_t *)ws;
        w.tiles = (int64_t *)((char *)ws + tiles_at);
        w.total = (int64_t *)((char *)ws + total_at);
    }
    return w;
}

size_t prune_ws_bytes(const DevProblem &P) { return carve_prune(P, nullptr).bytes; }

static hipError_t launch_frontier(const DevProblem &P, const double *cost, const uint8_t *dmax, uint64_t *bitmap,
                                  hipStream_t s) {
    const int64_t n_front = (int64_t)P.n_kb * P.words;
    if (n_front > 0 && use_buckets(P)) {
        frontier_buckets<<<dim3((unsigned)n_front), dim3(kWave), bucket_lds(P.K), s>>>(P, cost, dmax, bitmap);
    } else if (n_front > 0) {
        const int64_t blocks = (n_front + kFrontWaves - 1) / kFrontWaves;
        if (P.max_members <= kSmallGroup)
            frontier_kernel<4><<<dim3((unsigned)blocks), dim3(kFrontWaves * kWave), 0, s>>>(P, cost, dmax, bitmap,
                                                                                            n_front);
        else
            frontier_kernel<8><<<dim3((unsigned)blocks), dim3(kFrontWaves * kWave), 0, s>>>(P, cost, dmax, bitmap,
                                                                                            n_front);
    }
    return hipGetLastError();
}

// Survivor bitmap -> ascending candidate indices.
static hipError_t launch_compact(const DevProblem &P, const PruneWs &w, int64_t *surv, int64_t capacity,
                                 hipStream_t s, int64_t **d_total_out, int64_t *total_host = nullptr) {
    *d_total_out = w.total;
    const dim3 grid((unsigned)w.n_tiles), block(kEmitThreads);
    auto emit = [&](auto wpt, auto from) {
        emit_kernel<decltype(wpt)::value, decltype(from)::value><<<grid, block, 0, s>>>(
            P, w.bitmap, w.n_words, w.tiles, surv, capacity, w.total, total_host);
    };
    using One = std::integral_constant<int, 1>;
    using Four = std::integral_constant<int, 4>;
    if (w.n_words == 0) {
        no_survivors<<<dim3(1), dim3(1), 0, s>>>(w.total, total_host);
    } else if (w.n_words <= kSmallWords) {
        emit(One{}, std::integral_constant<Before, Before::kWords>{});
    } else if (words_per_thread(w.n_words) == 1) {
        count_kernel<1><<<grid, block, 0, s>>>(w.bitmap, w.n_words, w.tiles);
        emit(One{}, std::integral_constant<Before, Before::kCounts>{});
    } else {
        count_kernel<4><<<grid, block, 0, s>>>(w.bitmap, w.n_words, w.tiles);
        if (w.n_tiles <= kSumTiles) {
            emit(Four{}, std::integral_constant<Before, Before::kCounts>{});
        } else {
            scan_small_i64<<<dim3(1), dim3(1024), 0, s>>>(w.tiles, w.n_tiles);
            emit(Four{}, std::integral_constant<Before, Before::kScan>{});
        }
    }
    return hipGetLastError();
}

hipError_t launch_prune(const DevProblem &P, const double *cost, const uint8_t *dmax, int64_t *surv,
                        int64_t capacity, void *ws, hipStream_t s, int64_t **d_total_out, int64_t *total_host) {
    const PruneWs w = carve_prune(P, ws);
    hipError_t e = launch_frontier(P, cost, dmax, w.bitmap, s);
    if (e != hipSuccess) return e;
    return launch_compact(P, w, surv, capacity, s, d_total_out, total_host);
}

// Scratch of the prune variant that allocates nothing: a device array the
// code object carries, one copy per GPU, held until the process ends.  Host
// code never names it in a kernel argument or a copy (the name is a host-side
// stand-in there); it reaches the array through the device address that
// hipGetSymbolAddress returns for the current GPU, resolved once per GPU.
// Every call rewrites all the workspace it reads (each bitmap word, tile
// count and the total), so nothing needs clearing between calls.
static __device__ __align__(256) uint8_t scratch[kStaticScratchBytes];

hipError_t static_scratch(int device, void **out) {
    static std::mutex mu;
    static void *addr[kMaxScratchDevices] = {};
    if (device < 0 || device >= kMaxScratchDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[device]) {
        void *ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[device] = ptr;
    }
    *out = addr[device];
    return hipSuccess;
}

// Class bitmap after the slice-level workspace of launch_prune.
size_t prune_classes_ws_bytes(const DevProblem &P) {
    const DevProblem C = class_view(P);
    return prune_ws_bytes(P) + align256(sizeof(uint64_t) * (size_t)std::max<int64_t>(1, bitmap_words(C)));
}

hipError_t launch_prune_classes(const DevProblem &P, const double *cost, const uint8_t *dmax, int64_t *surv,
                                int64_t capacity, void *ws, hipStream_t s, int64_t **d_total_out) {
    const DevProblem C = class_view(P);
    const PruneWs w = carve_prune(P, ws);
    uint64_t *cbits = (uint64_t *)((char *)ws + prune_ws_bytes(P));
    hipError_t e = launch_frontier(C, cost, dmax, cbits, s);
    if (e != hipSuccess) return e;
    if (w.n_words > 0) {
        const int pieces = (int)((P.NS + kExpandSlices - 1) / kExpandSlices);
        const int piece = (int)((P.words + pieces - 1) / pieces) * kWave;
        const int64_t blocks = ((int64_t)P.n_rows + kExpandRows - 1) / kExpandRows * pieces;
        expand_kernel<<<dim3((unsigned)blocks), dim3(256), 0, s>>>(P, cbits, C.words, w.bitmap, pieces, piece);
    }
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_compact(P, w, surv, capacity, s, d_total_out);
}

}  // namespace tg
