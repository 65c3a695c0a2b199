// score.hip -- per-config coefficients, candidate scoring and decoding.
//
// Scoring is the analytic stand-in for the per-pair parallelizer query of
// Tab. 2 (profile() + parallelize()): a step-time cost per micro-batch and the
// deepest 1F1B position the pair fits at (Sec. 5.2).  Candidates are
// idx = g * NS + s (g: global config, s: slice).  A wave owns 64 consecutive
// slices and walks a run of 16 configs: the slice sums live in VGPRs for the
// whole run, the run's coefficients are staged once in LDS, and every
// config writes one coalesced 512-byte row of costs and 64 bytes of depths,
// the costs with streaming (nontemporal) stores, the depths too when their
// runs are 64-byte aligned.  Where slices repeat (equal layers) a second kernel
// evaluates each config once per slice class and writes its rows by lookup.
// Both are bound by HBM writes (9 bytes per candidate).
#include <algorithm>
#include <type_traits>

#include "tg_device.h"

#pragma clang fp contract(off)

namespace tg {

// ---------------------------------------------------------------------------
// coefficients of one config (exact operation order of the stated model)
// ---------------------------------------------------------------------------
__device__ inline double ring_share(int64_t D) { return (double)(D - 1) / (double)D; }

// bf16 bytes per parameter moved for data-parallel sync, per micro-batch
__device__ inline double sync_per_microbatch(int z, int64_t D) {
    if (z <= 1) return 0.0;
    if (z == 2) return 2.0 * ring_share(D);
    return 6.0 * ring_share(D);
}

// bf16 bytes per parameter moved for data-parallel sync, per iteration
__device__ inline double sync_per_iteration(int z, int64_t D) {
    if (z <= 1) return 4.0 * ring_share(D);
    if (z == 2) return 2.0 * ring_share(D);
    return 0.0;
}

// model-state bytes per parameter (bf16 weight + bf16 grad + fp32 master, m, v)
__device__ inline double state_per_param(int z, int64_t D) {
    if (z == 0) return 16.0;
    if (z == 1) return 4.0 + 12.0 / (double)D;
    if (z == 2) return 2.0 + 14.0 / (double)D;
    return 16.0 / (double)D;
}

// q = tp * cp GPUs share a micro-batch's tokens; the data-parallel group
// (gradient sync, ZeRO sharding) is dp * cp; recomputation runs the forward
// pass twice (compute passes nc = 4, forward-collective passes nt = 3).
// Bound by the 192 bytes it writes a config.
__global__ __launch_bounds__(256) void coef_kernel(DevProblem P, const Config *__restrict__ cfg,
                                                   Coef *__restrict__ coef) {
    const int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= P.ncfg) return;
    const Config in = cfg[g];
    Coef c{};
    c.k = in.k;
    c.tp = in.tp;
    c.cp = in.cp;
    c.dp = in.dp;
    c.ep = in.ep;
    c.z = in.z;
    c.rc = in.rc;
    c.of = in.of;
    c.mb = in.mb;
    c.b_idx = in.b_idx;
    c.row = in.row;
    const double F = P.peak[c.k], W = P.intra[c.k], M = P.hbm[c.k], Hb = P.host[c.k];
    const int64_t b = (int64_t)c.dp * c.mb;
    const int64_t Dd = (int64_t)c.dp * c.cp, De = (int64_t)(c.dp / c.ep) * c.cp;
    const double qd = (double)c.tp, qe = (double)((int64_t)c.tp * c.ep);
    const int64_t q = (int64_t)c.tp * c.cp;
    const double nc = c.rc ? 4.0 : 3.0;
    const int nt = c.rc ? 3 : 2;
    c.m_real = (double)P.B / (double)b;
    c.alpha = (nc * (double)c.mb) / (((double)q * F) * P.eta);
    c.beta = c.tp > 1 ? (((double)(2 * nt) * (double)c.mb) * (double)(c.tp - 1)) / ((double)q * W) : 0.0;
    c.gamma = c.ep > 1 ? (((double)nt * (double)c.mb) * (double)(c.ep - 1)) / (((double)c.ep * (double)q) * W)
                       : 0.0;
    c.kappa = c.cp > 1 ? (((double)(nt + 1) * (double)c.mb) * (double)(c.cp - 1)) /
                             (((double)c.cp * (double)c.tp) * W)
                       : 0.0;
    c.dd = ((sync_per_microbatch(c.z, Dd) / qd) / W) + (((sync_per_iteration(c.z, Dd) / qd) / W) / c.m_real);
    c.de = ((sync_per_microbatch(c.z, De) / qe) / W) + (((sync_per_iteration(c.z, De) / qe) / W) / c.m_real);
    c.mud = state_per_param(c.z, Dd) / qd;
    c.mue = state_per_param(c.z, De) / qe;
    c.rho = (double)c.mb / (double)q;
    c.omega = c.of ? (2.0 * (double)c.mb) / ((double)q * Hb) : 0.0;
    c.H = M * P.mem_frac;
    c.inv_rho = (double)q / (double)c.mb;
    coef[g] = c;
}

hipError_t launch_coef(const DevProblem &P, const Config *cfg, Coef *coef, hipStream_t s) {
    const int64_t blocks = (P.ncfg + 255) / 256;
    coef_kernel<<<dim3((unsigned)blocks), dim3(256), 0, s>>>(P, cfg, coef);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// scoring
// ---------------------------------------------------------------------------
constexpr int kScoreWaves = 4;     // waves per block
// Configs per wave tile: 16 where a wave's depth rows are line-aligned and go
// out as streaming stores (more rows a tile scatter those stores: the
// 128-layer instance took 1.74 -> 1.91 ms at 32), 32 elsewhere, where a
// tile's slice sums and coefficient staging then serve more configs (MoE
// 110 -> 105 µs, 70B 122 -> 114 µs).
constexpr int score_configs(bool nt_depth) { return nt_depth ? 16 : 32; }

// Largest d in 1..K with state + min(d, m) * A1 <= H, or 0.  fits() is
// monotone in d, so a first guess d0 from (H - state) / A1 (K once the
// stash saturates at m micro-batches) is the answer exactly when d0 fits and
// d0 + 1 does not; otherwise a short walk from d0 finds it.  Every decision
// is an exact evaluation of fits(); the guess only picks where to look.  The
// guess and both checks run on every lane without branches (in doubles: the
// guess is a small integer, so min(d0, m) and min(d0 + 1, m) are the values
// fits() takes); the wave walks only when a lane that scores a candidate
// (`live`) has a wrong guess, and the walk returns d0 to a lane whose guess
// is right.
__device__ inline int max_depth(double state, double A1, double H, double m_real, double guess_scale, int K,
                                bool live) {
    auto fits = [&](int d) -> bool {
        const double inflight = fmin((double)d, m_real);
        return state + inflight * A1 <= H;
    };
    const double Kd = (double)K;
    const double q = (H - state) * guess_scale;
    // floor(q) within [0, K] (NaN: 0)
    const double g = q >= m_real ? Kd : floor(fmin(fmax(q, 0.0), Kd));
    const bool lo_ok = g == 0.0 || state + fmin(g, m_real) * A1 <= H;
    const bool hi_ok = g == Kd || !(state + fmin(g + 1.0, m_real) * A1 <= H);
    const int d0 = (int)g;
    if (__builtin_expect(__ballot(live && !(lo_ok && hi_ok)) == 0, 1)) return d0;
    int d = d0 > K - 1 ? K - 1 : d0;
#pragma nounroll
    while (live && d > 0 && !fits(d)) --d;
#pragma nounroll
    while (live && d < K && fits(d + 1)) ++d;
    return d;
}

// Blocks are dispatched round-robin over the 8 XCDs.  Renumbering them so
// that consecutive tiles run on the same XCD keeps every cache line of the
// output (depth rows are not line-aligned) inside one L2, which merges the
// partial lines before they reach HBM.
constexpr int kXcds = 8;

// The coefficients a wave needs for its run of configs, staged in LDS: one
// coalesced load per lane at the start of the tile instead of scalar loads in
// every iteration (the coefficient table falls out of L2 under the streaming
// writes, and scalar misses would stall each iteration).
struct StagedCoef {
    double alpha, beta, gamma, dd, de, mud, mue, rho, H, m_real, inv_rho, kappa, omega;
    int32_t rc, of;
};

// Copies the coefficients the model reads from a config's row.
template <bool kExt>
__device__ inline StagedCoef stage_coef(const Coef &c) {
    StagedCoef x;
    x.alpha = c.alpha;
    x.beta = c.beta;
    x.gamma = c.gamma;
    x.dd = c.dd;
    x.de = c.de;
    x.mud = c.mud;
    x.mue = c.mue;
    x.rho = c.rho;
    x.H = c.H;
    x.m_real = c.m_real;
    x.inv_rho = c.inv_rho;
    if (kExt) {  // read only by the extended variants
        x.kappa = c.kappa;
        x.omega = c.omega;
        x.rc = c.rc;
        x.of = c.of;
    }
    return x;
}

// A slice's sums: exact int64 prefix differences, then one rounding to
// binary64.  The reciprocals only feed the depth guess.
struct SliceSums {
    double Fl = 0.0, Pd = 0.0, Pe = 0.0, Act = 0.0, Tb = 0.0, Ab = 0.0, inv_act = 0.0;
    double Oa = 0.0, Cb = 0.0, inv_oa = 0.0;
};

template <bool kDense, bool kExt>
__device__ inline SliceSums slice_sums(const DevProblem &P, uint32_t ij) {
    SliceSums u;
    const int i = (int)(ij & 0xFFFFu), j = (int)(ij >> 16);
    const int64_t *pre = P.pre;
    const int64_t Lp = P.L + 1;
    u.Fl = (double)(pre[j] - pre[i]);
    u.Pd = (double)(pre[Lp + j] - pre[Lp + i]);
    u.Act = (double)(pre[3 * Lp + j] - pre[3 * Lp + i]);
    u.Tb = (double)(pre[4 * Lp + j] - pre[4 * Lp + i]);
    if (!kDense) {
        u.Pe = (double)(pre[2 * Lp + j] - pre[2 * Lp + i]);
        u.Ab = (double)(pre[5 * Lp + j] - pre[5 * Lp + i]);
    }
    u.inv_act = 1.0 / u.Act;
    if (kExt) {
        u.Oa = (double)(pre[6 * Lp + j] - pre[6 * Lp + i]);
        u.Cb = (double)(pre[7 * Lp + j] - pre[7 * Lp + i]);
        u.inv_oa = 1.0 / u.Oa;
    }
    return u;
}

// The cost and depth of one (slice, config).  kExt: the space has context
// parallelism, recomputation or offloading (two more slice sums, two more cost
// terms, the stash and depth rules).  Every lane of the wave calls it; `live`
// lanes score a candidate.
template <bool kDense, bool kExt>
__device__ inline double score_one(const StagedCoef &c, const SliceSums &u, int K, bool live, int &dm) {
    // with recomputation only the layer boundaries (outputs) are stashed
    const double S = (kExt && c.rc) ? u.Oa : u.Act;
    double v = c.alpha * u.Fl;
    v = v + c.beta * u.Tb;
    if (!kDense) v = v + c.gamma * u.Ab;
    v = v + c.dd * u.Pd;
    if (!kDense) v = v + c.de * u.Pe;
    if (kExt) {
        v = v + c.kappa * u.Cb;
        v = v + c.omega * S;
    }
    double state = c.mud * u.Pd;
    if (!kDense) state = state + c.mue * u.Pe;
    const double A1 = c.rho * S;
    if (kExt && c.of)  // offloaded: one micro-batch on the device at every depth
        dm = (state + (fmin(1.0, c.m_real) * A1)) <= c.H ? K : 0;
    else
        dm = max_depth(state, A1, c.H, c.m_real, c.inv_rho * ((kExt && c.rc) ? u.inv_oa : u.inv_act), K, live);
    return v;
}

// kNtDepth: a wave's 64 depths of a row start on a 64-byte boundary (NS a
// multiple of 64) and go out with streaming stores like the costs; otherwise
// the run straddles segments that the neighbouring waves also write, and
// ordinary stores let L2 merge them.
template <bool kDense, bool kExt, bool kNtDepth>
__global__ __launch_bounds__(256) void score_kernel(DevProblem P, int64_t first, int64_t last, int64_t g_lo,
                                                    int64_t g_hi, int64_t n_stiles, int64_t n_tiles,
                                                    double *__restrict__ cost, uint8_t *__restrict__ dmax) {
    constexpr int kCfg = score_configs(kNtDepth);
    __shared__ StagedCoef cs[kScoreWaves][kCfg];
    const int64_t per_xcd = gridDim.x / kXcds;
    const int64_t blk = (int64_t)(blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t tile = blk * kScoreWaves + wv;
    if (tile >= n_tiles) return;
    const int64_t gt = tile / n_stiles;
    const int64_t st = tile - gt * n_stiles;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t s = st * kWave + lane;
    const bool sv = s < P.NS;
    const int64_t g_beg = g_lo + gt * kCfg;
    const int ng = (int)(min(g_beg + kCfg, g_hi + 1) - g_beg);
    if (lane < ng) cs[wv][lane] = stage_coef<kExt>(P.coef[g_beg + lane]);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

    SliceSums u;
    if (sv) u = slice_sums<kDense, kExt>(P, P.sij[s]);
    const int K = P.K;
    const int64_t NS = P.NS;
    // a tile wholly inside [first, last) with a slice for every lane stores
    // without per-candidate checks, from a per-row base
    const int64_t t0 = g_beg * NS + st * kWave;
    const bool whole = (st + 1) * kWave <= NS && t0 >= first && t0 + (int64_t)(ng - 1) * NS + (kWave - 1) < last;
    for (int t = 0; t < ng; ++t) {
        int dm;
        const double v = score_one<kDense, kExt>(cs[wv][t], u, K, sv, dm);
        if (whole) {
            const int64_t row = t0 + (int64_t)t * NS - first;
            __builtin_nontemporal_store(v, cost + row + lane);
            if (kNtDepth)
                __builtin_nontemporal_store((uint8_t)dm, dmax + row + lane);
            else
                dmax[row + lane] = (uint8_t)dm;
            continue;
        }
        const int64_t idx = (g_beg + t) * NS + s;
        if (sv && idx >= first && idx < last) {
            // streaming stores: the arrays are far larger than the caches
            __builtin_nontemporal_store(v, cost + (idx - first));
            if (kNtDepth)
                __builtin_nontemporal_store((uint8_t)dm, dmax + (idx - first));
            else
                dmax[idx - first] = (uint8_t)dm;
        }
    }
}

// ---------------------------------------------------------------------------
// scoring where slices repeat
// ---------------------------------------------------------------------------
// Slices with equal sums score alike under every config, and a model of equal
// layers has L classes among its L (L + 1) / 2 slices.  A block takes a run of
// configs, evaluates the model once per (config, class) into LDS and writes
// the run's rows, one contiguous range of candidates, by looking each slice's
// class up: the fp64 model (the general kernel issues 44 VALU instructions a
// candidate) leaves the per-candidate path, which is two LDS reads and its
// share of a 16-byte store (streaming for the costs).  The rows are written as
// one range, so every store is aligned whatever NS is: costs two to a thread, then depths
// sixteen to a thread.  Bound by HBM writes: what is left is their order.
// Consecutive runs go to one XCD and a run is kept short (kClassRun), so that
// each XCD writes a compact moving window, as a plain fill does: back to back
// on the 128-layer instance (1.10e9 candidates) runs of 66,000 candidates dealt
// round-robin over the XCDs took 1.97 ms, runs of 8,256 in XCD order 1.67 ms
// (5.9 TB/s; a kernel that only writes these bytes reaches 6.1).  Inside the
// plan search, general kernel -> this one: 128 layers 1868 -> 1673 us, 70B 109
// -> 92, extended 70B 718 -> 643, MoE 73 -> 63, uneven 61 layers 129 -> 91, 8B
// 12.4 -> 6.5 us; half and twice the run lost 13-30% and 5-15% on the 70B pair.
// A wider model's rows are cut into pieces, each written by a block of its own.
// LDS a block aims at: eight blocks of four waves fill a CU's 32 wave slots, 20
// KB each.  A row's slices that leave more are cut in pieces.
constexpr size_t kClassLds = 20 * 1024;
constexpr int kMaxClasses = 512;
constexpr int kClassCfg = 4;       // configs per block, at most
constexpr int kClassRun = 8192;    // candidates a block writes, about (1, 2 and 4 configs on 128, 80 and 48 layers)
constexpr int64_t kClassBlocks = 1024;  // blocks wanted before configs share one
// Calls the general kernel is the better for.  A block's chain (coefficients,
// classes, model, barrier, rows) is the same however little it writes: with less
// than kClassFew candidates a block (three quarters more where the space is
// extended), once there are more blocks than the machine holds at a time
// (kClassWave), general -> class: 16 islands and 16 layers (136 slices) extended 61
// -> 113 us, MoE 36 -> 40, 24 layers (300) extended 117 -> 124, MoE 46 -> 43, 28
// layers (406) extended 160 -> 128.  And a short range leaves the chain bare: a
// run of the general kernel's configs (32) is its time too, 129 layers and 12
// configs 21.1 -> 22.3, 36 configs 25.0 -> 22.7; where NS is a multiple of 64 its
// aligned rows hold out up to kClassAligned candidates (128 layers, 3.0e6 25.7 ->
// 28.6, 13.9e6 44 -> 44, 25e6 62 -> 63, 96e6 195 -> 152).
constexpr int64_t kClassFew = 900;
constexpr int64_t kClassWave = 4096;
constexpr int64_t kClassRange = 32;
constexpr int64_t kClassAligned = 32 << 20;

struct ClassTile {
    int32_t C;          // configs per block
    int32_t pieces;     // pieces of a row
    int32_t piece;      // slices per piece
    int32_t NC;         // slice classes
};

typedef double double2v __attribute__((ext_vector_type(2)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));

template <bool kDense, bool kExt>
__global__ __launch_bounds__(256) void score_class_kernel(DevProblem P, ClassTile ct, int64_t first, int64_t last,
                                                          int64_t g_lo, int64_t g_hi, double *__restrict__ cost,
                                                          uint8_t *__restrict__ dmax) {
    extern __shared__ double lds_cls[];
    __shared__ StagedCoef cs[kClassCfg];
    const int NC = ct.NC;
    double *vals = lds_cls;                                // [C][NC]
    uint16_t *cls = (uint16_t *)(vals + ct.C * NC);        // [piece]
    uint8_t *deps = (uint8_t *)(cls + ct.piece);           // [C][NC]
    const int64_t per_xcd = gridDim.x / kXcds;
    const int64_t blk = (int64_t)(blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
    const int64_t gb = blk / ct.pieces;
    const int pc = (int)(blk - gb * ct.pieces);
    if (g_lo + gb * ct.C > g_hi) return;
    const int64_t NS = P.NS;
    const int s0 = pc * ct.piece;
    const int ns = (int)min((int64_t)ct.piece, NS - s0);   // slices of this piece
    const int64_t g0 = g_lo + gb * ct.C;
    const int ng = (int)(min(g0 + ct.C, g_hi + 1) - g0);
    const int tid = threadIdx.x;
    if (tid < ng) cs[tid] = stage_coef<kExt>(P.coef[g0 + tid]);
    for (int t = tid; t < ns; t += 256) cls[t] = (uint16_t)P.cls[s0 + t];
    __syncthreads();
    // whole waves enter (the depth rule votes); lanes past the end score nothing
    for (int t0 = tid & ~(kWave - 1); t0 < NC; t0 += 256) {
        const int c = t0 + (tid & (kWave - 1));
        const bool live = c < NC;
        SliceSums u;
        if (live) u = slice_sums<kDense, kExt>(P, P.cls_ij[c]);
        for (int t = 0; t < ng; ++t) {
            int dm;
            const double v = score_one<kDense, kExt>(cs[t], u, P.K, live, dm);
            if (live) {
                vals[t * NC + c] = v;
                deps[t * NC + c] = (uint8_t)dm;
            }
        }
    }
    __syncthreads();
    // the runs of candidates this block writes: all rows at once when a piece
    // is a whole row, else one run per row
    const bool one = ct.pieces == 1;
    for (int r = 0; r < (one ? 1 : ng); ++r) {
        const int64_t run0 = (g0 + r) * NS + s0;  // candidate index of the run's first element
        const int64_t run1 = run0 + (one ? (int64_t)ng * ns : ns);
        const int64_t lo = max(run0, first), hi = min(run1, last);
        if (lo >= hi) continue;
        const int e0 = (int)(lo - run0), n = (int)(hi - lo);
        double *cp = cost + (lo - first);
        uint8_t *dp = dmax + (lo - first);
        const double *vr = vals + r * NC;
        const uint8_t *dr = deps + r * NC;
        // element e of the run: row e / ns of it, slice e % ns of the piece.
        // A thread's elements advance by a fixed step, so row and slice do too.
        auto locate = [&](int e, int &row, int &s) {
            row = e / ns;
            s = e - row * ns;
        };
        {
            const int head = (int)(((uintptr_t)cp >> 3) & 1) & (n > 0);  // to a 16-byte boundary
            const int pairs = (n - head) >> 1;
            const int srow = 512 / ns, srem = 512 - srow * ns;
            int row, s;
            locate(e0 + head + 2 * tid, row, s);
            double2v *out = (double2v *)(cp + head);
            for (int q = tid; q < pairs; q += 256) {
                const bool wrap = s + 1 == ns;
                double2v x;
                x.x = vr[row * NC + cls[s]];
                x.y = vr[(wrap ? row + 1 : row) * NC + cls[wrap ? 0 : s + 1]];
                __builtin_nontemporal_store(x, out + q);
                row += srow;
                s += srem;
                if (s >= ns) {
                    s -= ns;
                    ++row;
                }
            }
            if (tid < 2) {  // the element before the first pair, the one after the last
                const int e = tid == 0 ? 0 : n - 1;
                if (tid == 0 ? head != 0 : ((n - head) & 1) != 0) {
                    locate(e0 + e, row, s);
                    __builtin_nontemporal_store(vr[row * NC + cls[s]], cp + e);
                }
            }
        }
        {
            const int head = min(n, (int)((0 - (uintptr_t)dp) & 15));
            const int quads = (n - head) >> 4;
            const int srow = 4096 / ns, srem = 4096 - srow * ns;
            int row, s;
            locate(e0 + head + 16 * tid, row, s);
            uint4v *out = (uint4v *)(dp + head);
            for (int q = tid; q < quads; q += 256) {
                uint4v x;
                int rr = row, ss = s;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    uint32_t b = 0;
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        b |= (uint32_t)dr[rr * NC + cls[ss]] << (8 * k);
                        if (++ss == ns) {
                            ss = 0;
                            ++rr;
                        }
                    }
                    x[w] = b;
                }
                // ordinary stores: the prune reads the depths next (streaming
                // them took 701 us against 638 on the extended 70B instance)
                out[q] = x;
                row += srow;
                s += srem;
                if (s >= ns) {
                    s -= ns;
                    ++row;
                }
            }
            const int tail0 = head + 16 * quads;  // the bytes before the first quad and after the last
            const int t = tid < head ? tid : tail0 + tid - head;
            if (tid < head + (n - tail0)) {
                locate(e0 + t, row, s);
                dp[t] = dr[row * NC + cls[s]];
            }
        }
    }
}

// The class kernel's tile, or C = 0 where the general kernel is the better:
// fewer than four slices a class (the model would be evaluated nearly as often
// as there are candidates, by blocks that then wait for it), more classes than
// a block holds, blocks that write too little, or short ranges.
static ClassTile class_tile(const DevProblem &P, int64_t n_cfg) {
    ClassTile ct{};
    if (P.NC > kMaxClasses || P.NC * 4 > P.NS || n_cfg < kClassRange) return ct;
    if ((P.NS & 63) == 0 && n_cfg * P.NS < kClassAligned) return ct;
    ct.NC = (int32_t)P.NC;
    const int64_t fit1 = (int64_t)(kClassLds - sizeof(StagedCoef) * kClassCfg - 9 * (size_t)P.NC) / 2;
    ct.pieces = (int32_t)((P.NS + fit1 - 1) / fit1);
    ct.piece = (int32_t)((P.NS + ct.pieces - 1) / ct.pieces);
    const int64_t spread = n_cfg * ct.pieces / kClassBlocks;
    const int64_t fit =
        (int64_t)(kClassLds - sizeof(StagedCoef) * kClassCfg - 2 * (size_t)ct.piece) / (9 * P.NC);
    const int64_t most = std::min<int64_t>(std::min<int64_t>(kClassCfg, kClassRun / P.NS), fit);
    const int64_t C = std::max<int64_t>(1, std::min(most, spread));
    const int64_t few = P.ext ? kClassFew + kClassFew * 3 / 4 : kClassFew;
    if (C * ct.piece < few && (n_cfg + C - 1) / C * ct.pieces > kClassWave) return ct;
    ct.C = (int32_t)C;
    return ct;
}

hipError_t launch_score(const DevProblem &P, int64_t first, int64_t count, double *cost, uint8_t *dmax,
                        hipStream_t s) {
    if (count <= 0) return hipSuccess;
    const int64_t last = first + count;
    const int64_t g_lo = first / P.NS, g_hi = (last - 1) / P.NS;
    using T_ = std::true_type;
    using F_ = std::false_type;
    auto by_space = [&](auto &&go) {
        if (P.dense && !P.ext)
            go(T_{}, F_{});
        else if (!P.dense && !P.ext)
            go(F_{}, F_{});
        else if (P.dense)
            go(T_{}, T_{});
        else
            go(F_{}, T_{});
    };
    const ClassTile ct = class_tile(P, g_hi - g_lo + 1);
    if (ct.C > 0) {
        const int64_t cblocks = ((g_hi - g_lo + ct.C) / ct.C * ct.pieces + kXcds - 1) / kXcds * kXcds;
        if (cblocks > 0x7fffffffLL) return hipErrorInvalidValue;
        const size_t lds = (size_t)ct.C * P.NC * 9 + (size_t)ct.piece * 2;
        by_space([&](auto dense, auto ext) {
            score_class_kernel<decltype(dense)::value, decltype(ext)::value>
                <<<dim3((unsigned)cblocks), dim3(256), lds, s>>>(P, ct, first, last, g_lo, g_hi, cost, dmax);
        });
        return hipGetLastError();
    }
    const bool nt_depth = (P.NS & 63) == 0;
    const int cfg = score_configs(nt_depth);
    const int64_t n_gtiles = (g_hi - g_lo + cfg) / cfg;
    const int64_t n_stiles = (P.NS + kWave - 1) / kWave;
    const int64_t n_tiles = n_gtiles * n_stiles;
    int64_t blocks = (n_tiles + kScoreWaves - 1) / kScoreWaves;
    blocks = (blocks + kXcds - 1) / kXcds * kXcds;  // whole rounds over the XCDs
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    by_space([&](auto dense, auto ext) {
        constexpr bool D = decltype(dense)::value, X = decltype(ext)::value;
        if (nt_depth)
            score_kernel<D, X, true><<<dim3((unsigned)blocks), dim3(256), 0, s>>>(P, first, last, g_lo, g_hi,
                                                                                   n_stiles, n_tiles, cost, dmax);
        else
            score_kernel<D, X, false><<<dim3((unsigned)blocks), dim3(256), 0, s>>>(P, first, last, g_lo, g_hi,
                                                                                    n_stiles, n_tiles, cost, dmax);
    });
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// decoding
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void enumerate_kernel(DevProblem P, int64_t first, int64_t count, tg_pair *out) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= count) return;
    const int64_t idx = first + t;
    const int64_t g = idx / P.NS, s = idx - g * P.NS;
    const uint32_t ij = P.sij[s];
    const Coef &c = P.coef[g];
    tg_pair p;
    p.i = (int32_t)(ij & 0xFFFFu);
    p.j = (int32_t)(ij >> 16);
    p.island = c.k;
    p.tp = c.tp;
    p.cp = c.cp;
    p.dp = c.dp;
    p.ep = c.ep;
    p.zero = c.z;
    p.recompute = c.rc;
    p.offload = c.of;
    p.mb = c.mb;
    p.reserved = 0;
    out[t] = p;
}

hipError_t launch_enumerate(const DevProblem &P, int64_t first, int64_t count, tg_pair *out, hipStream_t s) {
    if (count <= 0) return hipSuccess;
    const int64_t blocks = (count + 255) / 256;
    if (blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    enumerate_kernel<<<dim3((unsigned)blocks), dim3(256), 0, s>>>(P, first, count, out);
    return hipGetLastError();
}

}  // namespace tg
