// Edge kernels on tabulated filters.  The filter w(d) = SiLU(b(d) W1) W2 of a layer is a function of the edge length alone, smooth
// on [0, rc], so its F values are kept as piecewise polynomials in LDS and an edge costs a look-up instead of a filter MLP:
// the forward and the reverse step walk the full edge lists once per layer, nothing is kept between them and no pair lists are needed.
// Part of model.hip (one translation unit): included inside namespace mlip, anonymous namespace.
#ifndef MLIP_MODEL_TABLE_H
#define MLIP_MODEL_TABLE_H

#include <utility>

// ---------------------------------------------------------------- the table
//
// kTabN intervals over [0, rc], degree 5 in the local coordinate s in [-1, 1], fp32 coefficients computed in fp64.  In units of rc /
// kTabUnits the intervals have the length 1/2 below kTabSmall (at short distances the basis functions are large and SiLU bends most), 1/4
// from kTabEnd on (at the cutoff the filter vanishes with its first three derivatives, so its error has to vanish too) and 1 between. What
// is cut off is below what the evaluation of the MLP in fp32 rounds, feature by feature (checked when the table is made, see k_filter_table);
// coefficients and evaluation round to 4e-8 (values) and 5e-8 (slopes) of the filter, the fp32 evaluation of the MLP to 1.7e-7 of both.
// kTabUnits and kTabSmall share the intervals out between short lengths and the rest: of 300 random layers with W1 of variance 1/8 all
// are represented at rc 4.5 to 5.5, 96 % at F = 64 with one and a half times that W1 or with rc 3 (the same thing: the basis goes as 1 / d), 68 %
// with twice at 4.5, 83 % at 5 (179 and 27 in their place, features pooled: 97 to 100 %, 56 %, 10 %, 21 %).
// One block of 32 features is 768 bytes per interval, [3][16][2][2]: coefficients 2 q and 2 q + 1 of features l and l + 16, 16 bytes for one lane; 162,816
// bytes of the compute unit's 160 KB.  With F = 64 every block of the grid holds the table of one half of the features.
constexpr int kTabUnits = 160, kTabSmall = 46, kTabEnd = kTabUnits - 2;
constexpr int kTabM0 = 2 * kTabSmall, kTabE0 = kTabM0 + kTabEnd - kTabSmall, kTabN = kTabE0 + 4 * (kTabUnits - kTabEnd);
constexpr int kTabStride = 32 * 6 * 4;                   // bytes of an interval
constexpr int kTabFloats = kTabN * kTabStride / 4;       // floats of one block of 32 features
constexpr int kTabLds = kTabFloats * 4 + 32;             // the table and a work counter per partition of the launch
constexpr int kTabCounters = 16;                         // counters of k_filter_table's blocks, each on a cache line of its own
constexpr int kTabHeader = 256 + 128 * kTabCounters;     // bytes in front of the first table: TabState, then those counters
constexpr int kTabNodes = 8;                             // Chebyshev nodes of an interval: coefficients 0..7, 6 and 7 measure what is cut off
static_assert(kTabLds <= 160 * 1024, "the table has to fit a compute unit's LDS");

// Whether the tables of a model represent its filters, and the handshake that tells the host.
struct TabState {
    int32_t bad;       // an interval of some layer is not represented: the edge steps may not use the tables
    int32_t done;      // counters that are through, plus kTabBad for every one with a bad interval
};

constexpr int32_t kTabBad = 1 << 16;

struct TabJob {
    const float *W1, *W2;   // [L][8][F], [L][F][F]
    float *tab;             // [L][F / 32][kTabFloats]
    TabState *state;
    int64_t *publish;       // pinned host word: generation * 2 + bad, written when the last block is through
    int64_t generation;
    double inv_h;           // kTabUnits / rc, rounded to fp32 as the edge kernels use it
    double rc;
    int p, F;
    int bf16;   // the mode with bf16 products: W2 rounded to bf16 as the forward MLP has it, scaled (the activations need no rounding here)
};

// cos(m pi / 16)
__constant__ const double kCosTab[32] = {
    1.0, 0.98078528040323044913, 0.92387953251128675613, 0.83146961230254523708, 0.70710678118654752440, 0.55557023301960222474,
    0.38268343236508977173, 0.19509032201612826785, 0.0, -0.19509032201612826785, -0.38268343236508977173, -0.55557023301960222474,
    -0.70710678118654752440, -0.83146961230254523708, -0.92387953251128675613, -0.98078528040323044913, -1.0, -0.98078528040323044913,
    -0.92387953251128675613, -0.83146961230254523708, -0.70710678118654752440, -0.55557023301960222474, -0.38268343236508977173,
    -0.19509032201612826785, 0.0, 0.19509032201612826785, 0.38268343236508977173, 0.55557023301960222474, 0.70710678118654752440,
    0.83146961230254523708, 0.92387953251128675613, 0.98078528040323044913};

// One block per interval and layer, one wavefront per Chebyshev node, lane = feature; everything in fp64.  Bound by the latency
// of one chain of loads, an exponential and 64 multiply-adds; W2 is requested before the chain and converted once, on its way to LDS
// (per use: F = 64, L = 3 19.2 us, so 15.3; with the blocks' count spread over addresses 12.9; F = 32, L = 2 12.2, 10.7 and 8.2; 13.5 and 7.9
// with every feature's own verdict).
template <int F>
__global__ void __launch_bounds__(kTabNodes * 64) k_filter_table(TabJob J)
{
    __shared__ double sv[kTabNodes][64], wv[kTabNodes][64], uv[kTabNodes][64], gv[kTabNodes][64];
    __shared__ double W2[F * F];
    const int iv = blockIdx.x, layer = blockIdx.y;
    const int node = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, f = lane & (F - 1);
    const double lo = iv < kTabM0 ? 0.5 * iv : iv < kTabE0 ? kTabSmall + (iv - kTabM0) : kTabEnd + 0.25 * (iv - kTabE0);
    const double wd = iv < kTabM0 ? 0.5 : iv < kTabE0 ? 1.0 : 0.25;
    float w1[8];
#pragma unroll
    for (int n = 0; n < 8; ++n) w1[n] = J.W1[((size_t)layer * 8 + n) * F + f];
    float w2[F * F / (kTabNodes * 64)];   // this thread's part on its way to LDS (the caller's array: no alignment assumed)
#pragma unroll
    for (int i = 0; i < F * F / (kTabNodes * 64); ++i) w2[i] = J.W2[(size_t)layer * F * F + i * kTabNodes * 64 + threadIdx.x];
    {   // t_k = sum_n b_n(d) W1[n][k], s_k = SiLU(t_k)
        const double d = (lo + wd * (0.5 + 0.5 * kCosTab[2 * node + 1])) / J.inv_h;
        const double x = fmin(d / J.rc, 1.0), y = 1.0 - x;
        double q = 0.5 * J.p * (J.p + 1);
        for (int k = J.p - 2; k >= 0; --k) q = q * x + 0.5 * (k + 1) * (k + 2);
        const double u = y * y * y * q / d;   // the envelope in its factored form, over d
        // sin((n + 1) pi x) by angle addition from the nearer end, where it is small
        const double near = x < 0.5 ? x : y, s1 = sinpi(near), c1 = x < 0.5 ? cospi(near) : -cospi(near);
        double sn = s1, cn = c1, t = 0, tt = 0;
#pragma unroll
        for (int n = 0; n < 8; ++n) {
            const double term = sn * u * (double)w1[n];
            t += term;
            tt += term * term;
            const double nx = sn * c1 + cn * s1;
            cn = cn * c1 - sn * s1;
            sn = nx;
        }
        const double sg = 1.0 / (1.0 + exp(-t)), slope = sg * (1.0 + t * (1.0 - sg));
        sv[node][lane] = t * sg;
        uv[node][lane] = tt * (slope * slope + 1.0 / 16);   // (see the verdict below)
    }
#pragma unroll
    for (int i = 0; i < F * F / (kTabNodes * 64); ++i)
        W2[i * kTabNodes * 64 + threadIdx.x] = J.bf16 ? (double)(float)(__bf16)(w2[i] * kSiluScaleInv) / kSiluScaleInv : (double)w2[i];
    __syncthreads();
    {   // w_f = sum_k s_k W2[k][f]
        double w = 0, g = 0;
#pragma unroll 16
        for (int k = 0; k < F; ++k) {
            const double v = W2[k * F + f];
            w = fma(sv[node][k], v, w);
            g = fma(uv[node][k], v * v, g);
        }
        wv[node][lane] = w;
        gv[node][lane] = g;
    }
    __syncthreads();
    double a = 0;   // Chebyshev coefficient `node` of this lane's feature
#pragma unroll
    for (int j = 0; j < kTabNodes; ++j) a += wv[j][lane] * kCosTab[node * (2 * j + 1) % 32];
    a *= node == 0 ? 1.0 / kTabNodes : 2.0 / kTabNodes;
    __syncthreads();
    sv[node][lane] = a;
    __syncthreads();
    if (node != 0) return;
    const double a0 = sv[0][lane], a1 = sv[1][lane], a2 = sv[2][lane], a3 = sv[3][lane], a4 = sv[4][lane], a5 = sv[5][lane],
                 a6 = fabs(sv[6][lane]), a7 = fabs(sv[7][lane]);
    const double c[6] = {a0 - a2 + a4, a1 - 3 * a3 + 5 * a5, 2 * a2 - 8 * a4, 4 * a3 - 20 * a5, 8 * a4, 16 * a5};
    if (lane < F) {
        float *at = J.tab + ((size_t)layer * (F / 32) + (lane >> 5)) * kTabFloats + (size_t)iv * (kTabStride / 4);
        const int l = lane & 31;
        for (int k = 0; k < 6; ++k) at[64 * (k / 2) + 4 * (l % 16) + 2 * (k % 2) + l / 16] = (float)c[k];
    }
    // What is cut off: a6 T6 + a7 T7 of the values, root mean square a6 + a7 at most, and 8 a6 + 10 a7 of the slopes (rms of T6' and T7').
    // Every feature is held to what the fp32 evaluation of the MLP rounds of it, 1e-7 of G, G^2 = sum_k W2[k][f]^2 tau_k^2 SiLU'(t_k)^2, tau_k^2 the
    // sum of the squares of t_k's eight terms, and for the slopes 1e-7 kappa G, kappa what a basis function grows by along a unit of length relative
    // to itself: 8 pi / rc from the sine, 4 / (rc - d) where it vanishes as (rc - d)^4; further to what the length's rounding to fp32, half an
    // ulp, changes on average: 2^-26 of the length times kappa.  Where SiLU' is near zero a sixteenth stands for SiLU'^2: there the feature is small
    // beside what it is elsewhere (a unit's t goes to 0 at the cutoff, so -0.28 is always passed).  G goes with the feature's column of W2:
    // scaling that against the later maps does not change the verdict.
    double g2 = 0;
#pragma unroll
    for (int j = 0; j < kTabNodes; ++j) g2 += gv[j][lane] * (1.0 / kTabNodes);
    const double mid = lo + 0.5 * wd, kappa = (8 * 3.141592653589793 / kTabUnits + 4.0 / (kTabUnits - mid)) * 0.5 * wd;   // in units of s
    const double rounding = 0x1p-26 * 2 * mid / wd * kappa;
    const double cut = fmax(a6 + a7, (8 * a6 + 10 * a7) / kappa);
    const bool feature_bad = !(cut * cut <= g2 * (1e-14 + rounding * rounding));   // (not a number: not represented)
    const bool bad = __any(feature_bad);
    if (lane == 0) {
        if (bad) J.state->bad = 1;
        // A word counts blocks and the bad ones among them, so that the last one needs no fence to know.  The blocks are spread over
        // kTabCounters of them, whose last ones go on to state->done: some 20 ns per addition to one address made up most of the launch.
        auto count = [](int32_t *word, bool is_bad) {
            const int32_t add = 1 + (is_bad ? kTabBad : 0);
            return add + __hip_atomic_fetch_add(word, add, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
        const int c = iv % kTabCounters;
        int32_t now = count(reinterpret_cast<int32_t *>(J.state) + 64 + 32 * c, bad);
        if (now % kTabBad != ((kTabN - 1 - c) / kTabCounters + 1) * (int32_t)gridDim.y) return;
        now = count(&J.state->done, now >= kTabBad);
        if (now % kTabBad == kTabCounters)
            __hip_atomic_store(J.publish, J.generation * 2 + (now >= kTabBad ? 1 : 0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// ---------------------------------------------------------------- edge steps
//
// A wavefront is four workers of 16 lanes, lane = two features of the block's 32.  A worker walks work items, each a few consecutive rows, in steps
// of 16 edges; items follow one another without a break in the pipeline (records two steps ahead, gathered rows one), and
// each worker has its own.  Lane l of a worker holds the record of edge l of its step; a DPP row broadcast hands it to the others.
//
// Measured at a million atoms in 8 slabs (F = 64, 45.8 M edges), per launch: forward 3.13 ms by MLP, 1.04 here; reverse 2.87 and 1.22 for the
// second pass over the lower edges, 1.85 here (layer 0, without gbar, 1.70).  For four edges and 32 features the forward step takes 20 vector
// instructions, 15 of them the look-up and the row sum, the reverse step 38, of which 24; broadcasts and other cross-lane instructions cost 4.4
// clocks, plain fp32 ones 2.8, so 3.2 and 3.4 on average.  By the counters (256,000 atoms) the reverse step spends 3.5 clocks of a SIMD on a vector
// instruction: the vector unit is its bound; LDS is busy 40 % of the time (24 bytes of table per edge and feature).  The forward step spends 4.3,
// with LDS busy 59 %: neither is full, a wavefront's look-ups and sums take turns.  No bank conflicts to speak of (0.2 % of the LDS cycles).
// With two workers of 32 lanes, one feature each, the broadcasts, the sums over lanes and the bookkeeping served two edges instead of four:
// 1.27 and 2.00 ms.

struct TabArgs {               // one partition
    int32_t n_rows, n_edges;   // receiver rows processed and their edges (below 2^29: 32-bit byte offsets of 8-byte sums)
    int32_t n_nodes;           // rows of g / abar
    int32_t dsum_step;         // floats from an edge's sum to the next one's
    const int64_t *row_ptr;
    const int32_t *chunk_row;  // the graph's work-item table: first row whose first edge lies at or after c * span
    int32_t span;
    const int32_t *senders, *recv;
    const float *d, *g, *abar;
    float *out;                // forward: a [n_rows][F]; reverse: gbar [n_rows][F]
    float *dsum[2];            // reverse: per edge its share of dE/dd, summed over the layers, of each block of 32 features
};
struct TabBatch {
    const float *tab;      // the layer's table
    float inv_h;
    int slots;             // blocks of an XCD for each block of 32 features; blocks beyond them have no rows
    int rows;              // rows of a work item
    int few;               // few rows for the workers: every XCD takes rows of one partition, 8 / n XCDs each
    int first;             // reverse: dsum is written, not added to
    int n;
    int64_t edge_start[kBatch + 1];
    TabArgs s[kBatch];
};
#ifndef MLIP_TAB_FWD_WAVES
#define MLIP_TAB_FWD_WAVES 12
#endif
#ifndef MLIP_TAB_BWD_WAVES
#define MLIP_TAB_BWD_WAVES 12
#endif
#ifndef MLIP_TAB_GROUP
#define MLIP_TAB_GROUP 4
#endif
#ifndef MLIP_TAB_ROWS
#define MLIP_TAB_ROWS 2
#endif
constexpr int kTabRows = MLIP_TAB_ROWS;     // most rows of a work item
constexpr int kTabGroup = MLIP_TAB_GROUP;   // edges whose values are computed together (8: the reverse step spills, 4 % slower; 2: 4 % slower)
constexpr int kTabFwdWaves = MLIP_TAB_FWD_WAVES, kTabBwdWaves = MLIP_TAB_BWD_WAVES;

template <int K> __device__ inline int row_bcast(int v) { return __builtin_amdgcn_mov_dpp(v, 0x150 + K, 0xf, 0xf, true); }
template <int K> __device__ inline float row_bcast(float v)
{
    return __builtin_bit_cast(float, row_bcast<K>(__builtin_bit_cast(int, v)));
}
__device__ inline void pin(float &v) { asm volatile("" : "+v"(v)); }   // v is computed by here, not where it is used
template <class Fn, int... K> __device__ __forceinline__ void unrolled(std::integer_sequence<int, K...>, Fn fn)
{
    (fn(std::integral_constant<int, K>{}), ...);
}

struct TabRec {      // as loaded
    int32_t sj, rk;
    float d, before; // before: reverse, the sum of the later layers at edge tb + k_out
};
struct TabStep {     // one step of a worker
    int32_t tb, last;   // first edge, the item's last edge
    int32_t r1;         // the row after the item's
    int32_t r0;         // the item's first row if this is its first step, or 2^31 - 1
};
struct TabEdge {     // what the lanes of the worker need of an edge
    int32_t goff;    // byte offset of the sender's row; past the end of the array for an edge past the item's last: its row reads 0
    int32_t loff;    // byte offset of the interval in the table
    float s, slope;  // place in the interval, ds / dd
    int32_t rk, raw; // receiver; r1 for an edge past the end / the clamped record's
};
__device__ inline TabEdge tab_edge(const TabRec &R, const TabStep &S, float inv_h, int l16, int row_bytes)
{
    TabEdge E;
    const float v = R.d * inv_h;
    const bool small = v < (float)kTabSmall, end = v >= (float)kTabEnd, valid = S.tb + l16 <= S.last;
    const float sc = small ? 2.f : end ? 4.f : 1.f;
    const float b = small ? 0.f : end ? (float)(kTabE0 - 4 * kTabEnd) : (float)(kTabM0 - kTabSmall);
    const int iv = min((int)fmaf(v, sc, b), kTabN - 1);
    E.slope = (2.f * inv_h) * sc;
    E.s = fmaf(R.d, E.slope, fmaf(2.f, b - (float)iv, -1.f));
    E.loff = __mul24(iv, kTabStride);
    E.goff = valid ? R.sj * row_bytes : (int32_t)0x80000000;
    E.rk = valid ? R.rk : S.r1;
    E.raw = R.rk;
    return E;
}

// the six coefficients of the lane's two features
struct TabCoeff { f32x4 q0, q1, q2; };
__device__ inline TabCoeff tab_read(const char *at)
{
    return TabCoeff{*reinterpret_cast<const f32x4 *>(at), *reinterpret_cast<const f32x4 *>(at + 256), *reinterpret_cast<const f32x4 *>(at + 512)};
}

// bit 16 w + k: edge k of worker w is the last one of its row; rnext: receiver of the following edge, r1 after the last
__device__ inline uint64_t tab_ends(const TabEdge &E, const TabStep &S, int32_t next_first, int l16, int32_t &rnext)
{
    const int32_t up = __builtin_amdgcn_mov_dpp(E.rk, 0x101, 0xf, 0xf, true);   // row_shl:1, the next lane's
    rnext = l16 == 15 ? (S.tb + 16 <= S.last ? next_first : S.r1) : up;
    return __ballot(rnext != E.rk);   // (past the end both are r1)
}

// a buffer of n bytes from p on, as 32-bit accesses see it (beyond n they read 0 and write nothing)
__device__ inline __amdgpu_buffer_rsrc_t tab_buffer(const void *p, uint32_t n)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)n, kBufferFlags);
}
// The lane's two features, l and l + 16: 64 bytes of 16 lanes at a time.  (Features 2 l and 2 l + 1 as 8 bytes of a lane: twice the cache
// accesses for the same rows, and the address unit busy for 82 % of the forward step.)
__device__ inline f32x2 buffer_load_2(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return f32x2{buffer_load_f32(r, off, 0, 0), buffer_load_f32(r, off + 64, 0, 0)};
}
__device__ inline void buffer_store_2(f32x2 v, __amdgpu_buffer_rsrc_t r, uint32_t off)
{
    buffer_store_f32(v[0], r, off, 0, 0);
    buffer_store_f32(v[1], r, off + 64, 0, 0);
}
__device__ inline int32_t buffer_load_i32(__amdgpu_buffer_rsrc_t r, uint32_t off) { return (int32_t)__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0); }

// Work items.  Every XCD takes a contiguous eighth of the launch's edges, cut at the rows where the graph's work-item tables (chunk_row)
// have an entry (of a launch with about a row for a worker, where one partition after the other and a look at those tables would be most of
// its time, 21 us for 8 x 192 rows, rows of one partition); the F / 32 blocks of features each go through all of it, on the same XCD.  The
// XCD's rows are dealt to its blocks in turn, kTabDeal items at a time, so that at any moment they work on a short run of rows whose
// neighbourhoods share the L2; within its block's share every worker starts at its own item and then draws from a counter in LDS.  (Draws
// from one counter per XCD in memory: one per 35 ns, 140 us a launch at 32,000 rows.)
constexpr int kTabDeal = 8;
static_assert(kTabDeal == 8, "tab_walk shifts by three");
__device__ inline int32_t tab_cut(const TabArgs &A, int64_t edge)   // the row at which the partition is cut for its edge `edge`
{
    return edge <= 0 ? 0 : edge >= A.n_edges ? A.n_rows : min(A.chunk_row[edge / A.span], A.n_rows);
}

// What both kernels share: the walk over partitions, items and steps.  Per partition open(A); per step load(step) -> TabRec two steps ahead,
// gather(edge, rows) one step ahead and compute(step, edge, before, rows, next_first); zero_rows(r0, r1) for rows without edges.
template <int F, int NW, class Rows, class Open, class Load, class Gather, class Compute, class Zero>
__device__ __forceinline__ void tab_walk(const TabBatch &B, float *lds, int hb, Open open, Load load, Gather gather, Compute compute, Zero zero_rows)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, l16 = lane & 15;
    constexpr int NH = F / 32;
    const int32_t n_slots = B.slots, xcd = blockIdx.x & 7, slot = (int32_t)(blockIdx.x >> 3) / NH;
    const int64_t total = B.edge_start[B.n], share = (total + 7) >> 3;
    const int64_t from = xcd * share, to = xcd == 7 ? total + 1 : from + share;   // the XCD's edges
    const int32_t mine = xcd * B.n >> 3, mine_from = (8 * mine + B.n - 1) / B.n, mine_n = (8 * mine + 8 + B.n - 1) / B.n - mine_from;   // B.few
    int32_t *counter = reinterpret_cast<int32_t *>(lds) + kTabFloats;   // items drawn, per partition
    if (threadIdx.x < kBatch) counter[threadIdx.x] = 4 * NW;
    const int32_t rows = B.rows;
    int32_t r0 = 0, r1 = 0, e0 = 0, e1 = 0;   // rows and edges of the worker's next item
    int32_t drawn = 0;                        // the item after it, as the worker's first lane drew it
    int part = 0;
    bool have = false;                        // whether there is a next item
    int32_t lo = 0, hi = 0;                   // the XCD's rows; lo: the first one dealt to this block
    __amdgpu_buffer_rsrc_t ptr;
    const int32_t turn = n_slots * kTabDeal * rows;   // rows from one of the block's turns to the next
    auto fetch = [&](int32_t item) {
        r0 = lo + __mul24(item >> 3, turn) + __mul24(item & (kTabDeal - 1), rows);
        r1 = min(r0 + rows, hi);
        have = r0 < hi;
        e0 = buffer_load_i32(ptr, (uint32_t)r0 * 8u);   // (past the last row: reads 0)
        e1 = buffer_load_i32(ptr, (uint32_t)r1 * 8u);
    };
    auto draw = [&]() {
        int zero = 0;
        asm("" : "+v"(zero));   // (an address that looks uniform would be combined over the lanes, and the result waited for at once)
        if (l16 == 0) drawn = __hip_atomic_fetch_add(counter + part + zero, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    auto next_part = [&]() {   // the first partition from `part` on in which the wavefront has an item
        for (; part < B.n; ++part) {
            const TabArgs &A = B.s[part];
            if (B.few) {
                if (part != mine) continue;
                lo = (int32_t)((int64_t)A.n_rows * (xcd - mine_from) / mine_n);
                hi = (int32_t)((int64_t)A.n_rows * (xcd - mine_from + 1) / mine_n);
            } else {
                // decided from the arguments alone, without a look at every partition's arrays; one without edges goes to the XCD of the
                // edge behind it
                const int64_t at = B.edge_start[part], end = B.edge_start[part + 1];
                if (at < end ? at >= to || end <= from : at < from || at >= to) continue;
                lo = tab_cut(A, from - at);
                hi = to > total ? A.n_rows : tab_cut(A, to - at);
            }
            lo += slot * kTabDeal * rows;
            ptr = tab_buffer(A.row_ptr, ((uint32_t)A.n_rows + 1u) * 8u);
            fetch(4 * wave + (lane >> 4));
            if (__any(have)) {
                open(A);
                break;
            }
        }
    };
    TabStep front, SA, SB;
    TabRec RA, RB;
    TabEdge EA, EB;
    float before_a = 0.f, before_b;
    Rows ga, gb;
    auto advance = [&]() {
        front.tb += 16;
        front.r0 = 0x7fffffff;
        const bool pop = front.tb > front.last;
        if (__any(pop)) {
            if (pop) {
                const bool edges = have && e0 < e1;
                front = TabStep{edges ? e0 : 1, edges ? e1 - 1 : 0, r1, edges ? r0 : 0x7fffffff};
                if (have && e0 == e1) zero_rows(r0, r1);
                fetch(row_bcast<0>(drawn));
                draw();
            }
        }
    };
    next_part();
    {
        LdsFill<kTabFloats / 4, NW * 64> fill;
        fill.load(B.tab + (size_t)hb * kTabFloats);
        fill.store(lds);
    }
    __syncthreads();
    for (; part < B.n; ++part, next_part()) {
        draw();
        front = TabStep{1, 0, 0, 0x7fffffff};   // no edges
        advance();
        SA = front;
        RA = load(SA);
        advance();
        SB = front;
        RB = load(SB);
        EA = tab_edge(RA, SA, B.inv_h, l16, F * 4);
        before_a = RA.before;
        gather(EA, ga);
        while (__any(have || SA.tb <= SA.last || SB.tb <= SB.last)) {
            advance();
            const TabStep SC = front;
            RA = load(SC);
            EB = tab_edge(RB, SB, B.inv_h, l16, F * 4);
            before_b = RB.before;
            gather(EB, gb);
            __builtin_amdgcn_sched_barrier(0);
            compute(SA, EA, before_a, ga, row_bcast<0>(EB.rk));
            advance();
            SA = SC;
            const TabStep SD = front;
            RB = load(SD);
            EA = tab_edge(RA, SA, B.inv_h, l16, F * 4);
            before_a = RA.before;
            gather(EA, ga);
            __builtin_amdgcn_sched_barrier(0);
            compute(SB, EB, before_b, gb, row_bcast<0>(EA.rk));
            SB = SD;
        }
    }
}

// Forward step over the owned rows: a_i = sum_e w_e * g_send(e).
template <int F, int NW> __device__ __forceinline__ void edge_fwd_tab(const TabBatch &B, float *lds)
{
    constexpr int kRow = F * 4;
    const int lane = threadIdx.x & 63, l16 = lane & 15, at_f = l16 * 4;   // byte offset of the lane's first feature in a block of 32
    const int hb = (blockIdx.x >> 3) & (F / 32 - 1);
    const char *tab = reinterpret_cast<const char *>(lds) + l16 * 16;
    struct Rows { f32x2 g[16]; };
    __amdgpu_buffer_rsrc_t send, recv, dist, g, out;
    f32x2 acc = {0.f, 0.f};
    auto zero_rows = [&](int32_t r, int32_t end) {
        for (; r < end; ++r) buffer_store_2(f32x2{0.f, 0.f}, out, r * kRow + at_f);
    };
    tab_walk<F, NW, Rows>(B, lds, hb,
        [&](const TabArgs &A) {
            const uint32_t n_rec = (uint32_t)A.n_edges * 4u;
            send = tab_buffer(A.senders, n_rec);
            recv = tab_buffer(A.recv, n_rec);
            dist = tab_buffer(A.d, n_rec);
            g = tab_buffer(A.g + 32 * hb, (uint32_t)A.n_nodes * kRow - 128u * hb);
            out = tab_buffer(A.out + 32 * hb, (uint32_t)A.n_rows * kRow - 128u * hb);
        },
        [&](const TabStep &S) {
            const uint32_t at = (uint32_t)min(S.tb + l16, S.last) * 4u;
            return TabRec{buffer_load_i32(send, at), buffer_load_i32(recv, at), buffer_load_f32(dist, at, 0, 0), 0.f};
        },
        [&](const TabEdge &E, Rows &R) {
            unrolled(std::make_integer_sequence<int, 16>{}, [&](auto k) { R.g[k] = buffer_load_2(g, row_bcast<k>(E.goff) + at_f); });
        },
        [&](const TabStep &S, const TabEdge &E, float, const Rows &R, int32_t next_first) {
            int32_t rnext;
            const uint64_t ends = tab_ends(E, S, next_first, l16, rnext);
            const uint32_t two = (uint32_t)ends | (uint32_t)(ends >> 32), any = two | two >> 16;
            const uint32_t mine = (uint32_t)(ends >> (lane & 48));
            const int32_t first = row_bcast<0>(E.raw);
            if (__any(S.r0 < first)) zero_rows(S.r0, first);   // rows of the item before its first edge are empty
            // values first, kTabGroup edges together with nothing in between that could stop their reads and chains from overlapping;
            // then the row sums with their branches
            unrolled(std::make_integer_sequence<int, 16 / kTabGroup>{}, [&](auto grp) {
                constexpr int k0 = grp * kTabGroup;
                __builtin_amdgcn_sched_barrier(0);
                float p[kTabGroup][2];
                unrolled(std::make_integer_sequence<int, kTabGroup>{}, [&](auto t) {
                    const TabCoeff c = tab_read(tab + row_bcast<k0 + t>(E.loff));
                    const float s = row_bcast<k0 + t>(E.s);
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        p[t][i] = fmaf(s, fmaf(s, fmaf(s, fmaf(s, fmaf(s, c.q2[2 + i], c.q2[i]), c.q1[2 + i]), c.q1[i]), c.q0[2 + i]), c.q0[i]);
                });
#pragma unroll
                for (int t = 0; t < kTabGroup; ++t) {
                    pin(p[t][0]);
                    pin(p[t][1]);
                }
                unrolled(std::make_integer_sequence<int, kTabGroup>{}, [&](auto t) {
                    constexpr int k = k0 + t;
                    acc[0] = fmaf(p[t][0], R.g[k][0], acc[0]);
                    acc[1] = fmaf(p[t][1], R.g[k][1], acc[1]);
                    if (__builtin_expect((any & (1u << k)) != 0, 0)) {
                        const int32_t row = row_bcast<k>(E.rk), nrow = row_bcast<k>(rnext);
                        if (mine & (1u << k)) {
                            buffer_store_2(acc, out, row * kRow + at_f);
                            acc = f32x2{0.f, 0.f};
                            zero_rows(row + 1, nrow);   // empty rows in between
                        }
                    }
                });
            });
        },
        zero_rows);
}
template <int F>
__global__ void __launch_bounds__(kTabFwdWaves * 64, kTabFwdWaves / 4) k_edge_fwd_tab(TabBatch B)
{
    extern __shared__ float lds[];
    edge_fwd_tab<F, kTabFwdWaves>(B, lds);
}

// Sums of q[0..15] over the 16 lanes of each row: lane l returns the sum of q[tab_edge_of(l)].  Each step adds lanes across one bit of the lane
// number and lets the lanes on either side go on with one of two edges.
__device__ inline int tab_edge_of(int lane) { return ((lane & 8) ? 0 : 8) + ((lane & 4) ? 0 : 4) + (lane & 3); }
template <int CTRL> __device__ inline float add_dpp(float v)   // v plus what the pattern brings of it
{
    return v + __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
template <int BANKS> __device__ inline float keep_banks(float v, float w)   // w in the named quads of every row of 16 lanes, v in the others
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, v), __builtin_bit_cast(int, w), 0xe4, 0xf, BANKS, false));
}
__device__ inline float tab_reduce(const float (&q)[16], int lane)
{
    float z[8], y[4], x[2];
#pragma unroll
    for (int k = 0; k < 8; ++k)     // row_ror:8; lanes 0-7 of a row keep edge k + 8, lanes 8-15 edge k
        z[k] = keep_banks<0xc>(add_dpp<0x128>(q[k + 8]), add_dpp<0x128>(q[k]));
#pragma unroll
    for (int k = 0; k < 4; ++k)     // row_half_mirror; even quads keep edge k + 4, odd ones edge k
        y[k] = keep_banks<0xa>(add_dpp<0x141>(z[k + 4]), add_dpp<0x141>(z[k]));
    const unsigned bit1 = (lane & 2) ? ~0u : 0u, bit0 = (lane & 1) ? ~0u : 0u;
    auto keep = [](unsigned mask, float v, float w) {   // w where the mask is set
        return __builtin_bit_cast(float, (__builtin_bit_cast(unsigned, w) & mask) | (__builtin_bit_cast(unsigned, v) & ~mask));
    };
#pragma unroll
    for (int k = 0; k < 2; ++k)     // quad_perm 2,3,0,1
        x[k] = keep(bit1, add_dpp<0x4e>(y[k]), add_dpp<0x4e>(y[k + 2]));
    return keep(bit0, add_dpp<0xb1>(x[0]), add_dpp<0xb1>(x[1]));   // quad_perm 1,0,3,2
}

// Reverse step over all local rows, owned and ghost: gbar_i = sum_e w_e * abar_send(e) and, added up over the layers, for every edge
// its share sum_f w'_f (abar_j g_i)_f of dE/dd.  The share with abar_i g_j is the reverse edge's, whose row gathers abar_i: the forces
// take both (k_force_rows), and the step gathers one row per edge instead of two.  (In a partition an owned row's edges from
// ghosts have no share, abar of a ghost being zero, and the ghosts' rows hold the other ones.)
template <int F, bool GBAR, int NW> __device__ __forceinline__ void edge_bwd_tab(const TabBatch &B, float *lds)
{
    constexpr int kRow = F * 4;
    const int lane = threadIdx.x & 63, l16 = lane & 15, at_f = l16 * 4;   // byte offset of the lane's first feature in a block of 32
    const int hb = (blockIdx.x >> 3) & (F / 32 - 1);
    const char *tab = reinterpret_cast<const char *>(lds) + l16 * 16;
    const int k_out = tab_edge_of(lane);                 // the edge of a step whose sum this lane gets
    const int slope_from = ((lane & 48) | k_out) * 4;    // and the lane that has its record
    struct Rows { f32x2 a[16], gi0, gi1; };              // the senders' rows of abar, and g of the first and the last receiver
    __amdgpu_buffer_rsrc_t send, recv, dist, g, abar, out, sums;
    int sum_shift = 2;
    f32x2 acc = {0.f, 0.f};
    auto zero_rows = [&](int32_t r, int32_t end) {
        if (GBAR)
            for (; r < end; ++r) buffer_store_2(f32x2{0.f, 0.f}, out, r * kRow + at_f);
    };
    tab_walk<F, NW, Rows>(B, lds, hb,
        [&](const TabArgs &A) {
            const uint32_t n_rec = (uint32_t)A.n_edges * 4u;
            send = tab_buffer(A.senders, n_rec);
            recv = tab_buffer(A.recv, n_rec);
            dist = tab_buffer(A.d, n_rec);
            g = tab_buffer(A.g + 32 * hb, (uint32_t)A.n_nodes * kRow - 128u * hb);
            abar = tab_buffer(A.abar + 32 * hb, (uint32_t)A.n_nodes * kRow - 128u * hb);
            out = tab_buffer(A.out + 32 * hb, (uint32_t)A.n_rows * kRow - 128u * hb);
            sum_shift = A.dsum_step == 2 ? 3 : 2;
            sums = tab_buffer(hb ? A.dsum[1] : A.dsum[0], ((uint32_t)A.n_edges << sum_shift) - (sum_shift == 3 ? 4u * hb : 0u));
        },
        [&](const TabStep &S) {
            const uint32_t at = (uint32_t)min(S.tb + l16, S.last) * 4u;
            return TabRec{buffer_load_i32(send, at), buffer_load_i32(recv, at), buffer_load_f32(dist, at, 0, 0),
                          B.first ? 0.f : buffer_load_f32(sums, (uint32_t)min(S.tb + k_out, S.last) << sum_shift, 0, 0)};
        },
        [&](const TabEdge &E, Rows &R) {
            R.gi0 = buffer_load_2(g, row_bcast<0>(E.raw) * kRow + at_f);
            R.gi1 = buffer_load_2(g, row_bcast<15>(E.raw) * kRow + at_f);
            unrolled(std::make_integer_sequence<int, 16>{}, [&](auto k) { R.a[k] = buffer_load_2(abar, row_bcast<k>(E.goff) + at_f); });
        },
        [&](const TabStep &S, const TabEdge &E, float before, const Rows &R, int32_t next_first) {
            int32_t rnext;
            const uint64_t ends = tab_ends(E, S, next_first, l16, rnext);
            const uint32_t two = (uint32_t)ends | (uint32_t)(ends >> 32), any = two | two >> 16;
            const uint32_t mine = (uint32_t)(ends >> (lane & 48));
            if (GBAR) {
                const int32_t first = row_bcast<0>(E.raw);
                if (__any(S.r0 < first)) zero_rows(S.r0, first);   // rows of the item before its first edge are empty
            }
            const int32_t row_last = row_bcast<15>(E.raw);
            f32x2 gi = R.gi0;
            float q[16];
            unrolled(std::make_integer_sequence<int, 16 / kTabGroup>{}, [&](auto grp) {
                constexpr int k0 = grp * kTabGroup;
                __builtin_amdgcn_sched_barrier(0);
                float p[kTabGroup][2], dp[kTabGroup][2];
                unrolled(std::make_integer_sequence<int, kTabGroup>{}, [&](auto t) {   // value and slope
                    const TabCoeff c = tab_read(tab + row_bcast<k0 + t>(E.loff));
                    const float s = row_bcast<k0 + t>(E.s);
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const float p4 = fmaf(s, c.q2[2 + i], c.q2[i]), p3 = fmaf(s, p4, c.q1[2 + i]), p2 = fmaf(s, p3, c.q1[i]),
                                    p1 = fmaf(s, p2, c.q0[2 + i]);
                        dp[t][i] = fmaf(s, fmaf(s, fmaf(s, fmaf(s, c.q2[2 + i], p4), p3), p2), p1);
                        p[t][i] = GBAR ? fmaf(s, p1, c.q0[i]) : 0.f;
                    }
                });
#pragma unroll
                for (int t = 0; t < kTabGroup; ++t)
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        if (GBAR) pin(p[t][i]);
                        pin(dp[t][i]);
                    }
                unrolled(std::make_integer_sequence<int, kTabGroup>{}, [&](auto t) {
                    constexpr int k = k0 + t;
                    if (GBAR) {
                        acc[0] = fmaf(p[t][0], R.a[k][0], acc[0]);
                        acc[1] = fmaf(p[t][1], R.a[k][1], acc[1]);
                    }
                    q[k] = fmaf(dp[t][0], R.a[k][0] * gi[0], dp[t][1] * (R.a[k][1] * gi[1]));
                    pin(q[k]);
                    if (__builtin_expect((any & (1u << k)) != 0, 0)) {
                        const int32_t row = row_bcast<k>(E.rk), nrow = row_bcast<k>(rnext);
                        if (mine & (1u << k)) {
                            if (GBAR) buffer_store_2(acc, out, row * kRow + at_f);
                            acc = f32x2{0.f, 0.f};
                            zero_rows(row + 1, nrow);   // empty rows in between
                            if (k < 15 && S.tb + k < S.last) {   // the next row starts inside this step
                                gi = R.gi1;
                                if (nrow != row_last) {   // a third row inside one step (short rows): fetch it now
                                    const f32x2 third = buffer_load_2(g, nrow * kRow + at_f);
                                    float a0 = third[0], a1 = third[1];
                                    pin(a0);
                                    pin(a1);
                                    gi = f32x2{a0, a1};   // (completed here: left pending, every later use would wait)
                                }
                            }
                        }
                    }
                });
            });
            __builtin_amdgcn_sched_barrier(0);
            const float sum = tab_reduce(q, lane);
            const float slope = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(slope_from, __builtin_bit_cast(int, E.slope)));
            if (S.tb + k_out <= S.last)
                buffer_store_f32(fmaf(sum, slope, before), sums, (uint32_t)(S.tb + k_out) << sum_shift, 0, 0);
        },
        zero_rows);
}
template <int F, bool GBAR>
__global__ void __launch_bounds__(kTabBwdWaves * 64, kTabBwdWaves / 4) k_edge_bwd_tab(TabBatch B)
{
    extern __shared__ float lds[];
    edge_bwd_tab<F, GBAR, kTabBwdWaves>(B, lds);
}

// ---------------------------------------------------------------- either way
//
// The edge steps of a call whose host has not heard yet whether the tables represent the filters: one launch that goes by *bad, so that
// the way and every bit of the result follow from the weights alone, whatever the handle has seen before.  A row's or an edge's sum does
// not depend on the wavefronts of a block, so either way gives what its own kernel gives; the reverse step takes 8 of them, the most that
// leave the way by MLP the registers it needs.  Per launch on tables 20.0 us forward (20.1 in k_edge_fwd_tab), 25.8 and 24.9 reverse (24.4,
// 24.5) at 15,600 rows and F = 32.  With a launch for each way, the other one's ending at once, a pass of four models took 691 us there, here
// 669; 500 atoms in the fixed workspace 248 and 240.  (The lower edges' terms added by the reverse kernel itself, which spares on tables a
// launch that ends at once: 653 and 228, but by MLP 122 us a launch, 103 with 32 of their rows in flight, for 47 and 16 apart.)
constexpr int kBothBwdWaves = 8;
static_assert(kTabFwdWaves == kFwdWaves, "the forward step has one block size for both ways");
struct BothBatch {
    TabBatch tab;
    EdgeBatch mlp;
    const int32_t *bad;
};
template <int F, int PREC>
__global__ void __launch_bounds__(kFwdWaves * 64, kFwdWaves / 4) k_edge_fwd_both(BothBatch B)
{
    extern __shared__ float lds[];
    if (*B.bad != 0)
        edge_fwd<F, PREC>(B.mlp, lds);
    else if ((int)(blockIdx.x >> 3) < B.tab.slots * (F / 32))
        edge_fwd_tab<F, kFwdWaves>(B.tab, lds);
}
template <int F, int PREC, bool GBAR>
__global__ void __launch_bounds__(kBothBwdWaves * 64, kBothBwdWaves / 4) k_edge_bwd_both(BothBatch B)
{
    extern __shared__ float lds[];
    if (*B.bad != 0)
        edge_bwd<F, PREC, kBothBwdWaves>(B.mlp, lds);
    else if ((int)(blockIdx.x >> 3) < B.tab.slots * (F / 32))
        edge_bwd_tab<F, GBAR, kBothBwdWaves>(B.tab, lds);
}

#endif  // MLIP_MODEL_TABLE_H
