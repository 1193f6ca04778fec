// Edge kernels on tabulated filters.  The filter w(d) = SiLU(b(d) W1) W2 of a layer is a function of the edge length alone, smooth
// on [0, rc], so its F values and their slopes are kept as piecewise polynomials and an edge costs a look-up in LDS instead of a filter
// MLP: the forward and the reverse step walk the edge lists, nothing is kept between them and no pair lists are needed.
// Part of model.hip (one translation unit): included inside namespace mlip, anonymous namespace.
#ifndef MLIP_MODEL_TABLE_H
#define MLIP_MODEL_TABLE_H

#include <utility>

// ---------------------------------------------------------------- the table
//
// Polynomials of degree 5 in the local coordinate s in [-1, 1] on intervals of [0, rc], fp32 coefficients computed in fp64.  [0, rc] is cut
// into 60 units of one length, a unit into 1 to 11 intervals (kTabPer): many where the filters of ordinary weights bend most (from rc/15 to
// rc/5) and at the cutoff, where the filter vanishes with its first three derivatives, so that its error has to vanish too.  They are shared out
// so that few models are refused, sampled at W1 of twice and two and a half times the usual size, where the slopes are the first to be: of those at
// two and a half times, F = 64, 43 %; 60 % with 64 units and the intervals beyond 2/5 rc one to a unit, 57 % with one table of 212 intervals
// and 32 features for values and slopes.  (48 units refuse as few, and the slopes are off by a third more from rc/2 on.)  Three tables a
// layer, for the three kinds of steps:
//   values  w, kTabN intervals, for all F features: the forward step needs nothing else;
//   slopes  dw/dd, the same intervals, for all F features: the last reverse step (layer 0), which needs no sums over rows;
//   both    w on intervals half as long, 32 features at a time: the other reverse steps take w and, as the polynomial's derivative, dw/dd.
// A derivative is as good as a polynomial of its own only on intervals 0.55 times as long, and the table has to fit LDS: one that serves for
// both holds 32 features, the other two all 64, which spares an edge's second look at its record and its broadcasts (20 vector instructions
// for four edges and 32 features, 17 with 64 at a time).  What is cut off is below what the evaluation of the MLP in fp32 rounds, feature by
// feature, of the slopes in root mean square over an interval (checked when the tables are made, see k_filter_table); coefficients and
// evaluation round to 3.6e-8 of values and slopes (5e-8 of the slopes as a derivative), the fp32 evaluation of the MLP to 1.7e-7 of both.
// An interval is, for 64 features, [6 coefficients][64], for 32 features [3][16 lanes][2 coefficients][2 features]: 16 bytes of a lane at a
// time, 16 lanes 256 bytes of a row.  Values or slopes of F = 64 and both of 32 features take 162,816 bytes of the compute unit's 160 KB.
constexpr int kTabUnits = 60, kTabN = 106;
constexpr int kTabPer[kTabUnits] = {1, 1, 2, 2, 3, 3, 4, 4, 4, 4, 3, 2, 2, 2, 2, 2, 2, 2, 2, 2, 2, 2, 2, 2, 2, 2, 1, 1, 1, 1,
                                    1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 1, 2, 11};
struct TabGrid {
    struct Unit { float n, at; } unit[kTabUnits];   // its intervals and the first one's number
    int unit_of[kTabN];
};
constexpr TabGrid make_tab_grid()
{
    TabGrid G{};
    int at = 0;
    for (int j = 0; j < kTabUnits; ++j) {
        G.unit[j].n = (float)kTabPer[j];
        G.unit[j].at = (float)at;
        for (int i = 0; i < kTabPer[j]; ++i) G.unit_of[at++] = j;
    }
    return G;
}
constexpr int tab_intervals()
{
    int n = 0;
    for (int j = 0; j < kTabUnits; ++j) n += kTabPer[j];
    return n;
}
static_assert(tab_intervals() == kTabN, "the units' intervals");
__constant__ const TabGrid kTabGrid = make_tab_grid();
constexpr int tab_floats(int F) { return kTabN * F * 6; }               // of the values or the slopes
constexpr int tab_layer(int F) { return 4 * tab_floats(F); }            // of a layer: values, slopes, both
constexpr int kTabLut = kTabUnits * (int)sizeof(TabGrid::Unit);         // the units, behind the table in LDS
constexpr int kTabBothFloats = 2 * kTabN * 32 * 6;                      // of both for 32 features
constexpr int tab_lds(int floats) { return floats * 4 + kTabLut + 32; } // and a work counter per partition of the launch
constexpr int kTabCounters = 16;                         // counters of k_filter_table's blocks, each on a cache line of its own
constexpr int kTabHeader = 256 + 128 * kTabCounters;     // bytes in front of the first table: TabState, then those counters
constexpr int kTabNodes = 8;                             // Chebyshev nodes of an interval: coefficients 0..7, 6 and 7 measure what is cut off
static_assert(tab_lds(tab_floats(64)) <= 160 * 1024 && tab_lds(kTabBothFloats) <= 160 * 1024, "the table has to fit a compute unit's LDS");

// Whether the tables of a model represent its filters, and the handshake that tells the host.
struct TabState {
    int32_t bad;       // an interval of some layer is not represented: the edge steps may not use the tables
    int32_t done;      // counters that are through, plus kTabBad for every one with a bad interval
};

constexpr int32_t kTabBad = 1 << 16;

struct TabJob {
    const float *W1, *W2;   // [L][8][F], [L][F][F]
    float *tab;             // [L][tab_layer(F)]: values, slopes, both
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
// of one chain of loads, an exponential and 64 multiply-adds; W2 is requested before the chain and converted once, on its way to LDS.
template <int F>
__global__ void __launch_bounds__(kTabNodes * 64) k_filter_table(TabJob J)
{
    __shared__ double sv[kTabNodes][64], wv[kTabNodes][64], uv[kTabNodes][64], gv[kTabNodes][64], slope_g[kTabNodes];
    __shared__ double W2[F * F], half[2][kTabNodes][64];
    __shared__ int any_bad;
    const int iv = blockIdx.x, layer = blockIdx.y;
    const int node = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, f = lane & (F - 1);
    // The place s of the interval as the edge kernels compute it from a length d: d * per_d - at, the product's factor rounded to fp32.
    const TabGrid::Unit unit = kTabGrid.unit[kTabGrid.unit_of[iv]];
    if (threadIdx.x == 0) any_bad = 0;
    const double per_d = (double)(2.0f * (float)J.inv_h * unit.n), at = 2.0 * (kTabGrid.unit_of[iv] * (double)unit.n + iv - (double)unit.at) + 1.0;
    auto length = [&](double s) { return fmin((s + at) / per_d, J.rc); };
    auto kappa = [&](double d) { return 8 * 3.141592653589793 / J.rc + 4.0 / (J.rc - d); };   // (see the verdict below)
    float w1[8];
#pragma unroll
    for (int n = 0; n < 8; ++n) w1[n] = J.W1[((size_t)layer * 8 + n) * F + f];
    float w2[F * F / (kTabNodes * 64)];   // this thread's part on its way to LDS (the caller's array: no alignment assumed)
#pragma unroll
    for (int i = 0; i < F * F / (kTabNodes * 64); ++i) w2[i] = J.W2[(size_t)layer * F * F + i * kTabNodes * 64 + threadIdx.x];
    {   // t_k = sum_n b_n(d) W1[n][k], s_k = SiLU(t_k), and their slopes along d
        const double d = length(kCosTab[2 * node + 1]);
        const double x = d / J.rc, y = 1.0 - x;
        double q = 0.5 * J.p * (J.p + 1), power = 1;
        for (int k = J.p - 2; k >= 0; --k) {
            q = q * x + 0.5 * (k + 1) * (k + 2);
            power *= x;
        }
        // the envelope in its factored form, over d
        const double u = y * y * y * q / d, du = (-0.5 * J.p * (J.p + 1) * (J.p + 2) * power * y * y / J.rc - u) / d, per_x = 3.141592653589793 / J.rc;
        // sin((n + 1) pi x) by angle addition from the nearer end, where it is small
        const double near = x < 0.5 ? x : y, s1 = sinpi(near), c1 = x < 0.5 ? cospi(near) : -cospi(near);
        double sn = s1, cn = c1, t = 0, tt = 0, dt = 0;
#pragma unroll
        for (int n = 0; n < 8; ++n) {
            const double term = sn * u * (double)w1[n];
            t += term;
            tt += term * term;
            dt += (cn * u * (per_x * (n + 1)) + sn * du) * (double)w1[n];
            const double nx = sn * c1 + cn * s1;
            cn = cn * c1 - sn * s1;
            sn = nx;
        }
        const double sg = 1.0 / (1.0 + exp(-t)), slope = sg * (1.0 + t * (1.0 - sg));
        sv[node][lane] = t * sg;
        half[0][node][lane] = dt * slope;
        uv[node][lane] = tt * (slope * slope + 1.0 / 16);   // (see the verdict below)
        if (lane == 0) slope_g[node] = kappa(d) * kappa(d);
    }
#pragma unroll
    for (int i = 0; i < F * F / (kTabNodes * 64); ++i)
        W2[i * kTabNodes * 64 + threadIdx.x] = J.bf16 ? (double)(float)(__bf16)(w2[i] * kSiluScaleInv) / kSiluScaleInv : (double)w2[i];
    __syncthreads();
    {   // w_f = sum_k s_k W2[k][f]
        double w = 0, dw = 0, g = 0;
#pragma unroll 16
        for (int k = 0; k < F; ++k) {
            const double v = W2[k * F + f];
            w = fma(sv[node][k], v, w);
            dw = fma(half[0][node][k], v, dw);
            g = fma(uv[node][k], v * v, g);
        }
        wv[node][lane] = w;
        gv[node][lane] = g;
        __syncthreads();
        uv[node][lane] = dw;
    }
    __syncthreads();
    auto coefficient = [&](const double (&v)[kTabNodes][64]) {   // Chebyshev coefficient `node` of this lane's feature, of the values at the nodes
        double a = 0;
#pragma unroll
        for (int j = 0; j < kTabNodes; ++j) a += v[j][lane] * kCosTab[node * (2 * j + 1) % 32];
        return a * (node == 0 ? 1.0 / kTabNodes : 2.0 / kTabNodes);
    };
    const double value = coefficient(wv), slope = coefficient(uv);
    __syncthreads();
    sv[node][lane] = value;
    uv[node][lane] = slope;
    __syncthreads();
    {   // w at the nodes of the interval's halves
        double h0 = 0, h1 = 0, hp0 = 0, hp1 = 0;
        const double x0 = 0.5 * (kCosTab[2 * node + 1] - 1.0), x1 = x0 + 1.0;
#pragma unroll
        for (int m = kTabNodes - 1; m >= 0; --m) {   // Clenshaw, one step late: (h, its predecessor) in hp
            const double a = sv[m][lane], n0 = a + 2.0 * x0 * h0 - hp0, n1 = a + 2.0 * x1 * h1 - hp1;
            hp0 = h0;
            hp1 = h1;
            h0 = n0;
            h1 = n1;
        }
        half[0][node][lane] = h0 - x0 * hp0;
        half[1][node][lane] = h1 - x1 * hp1;
    }
    __syncthreads();
    const double half0 = coefficient(half[0]), half1 = coefficient(half[1]);
    __syncthreads();
    half[0][node][lane] = half0;
    half[1][node][lane] = half1;
    __syncthreads();
    // What is cut off: a6 T6 + a7 T7 of the values, a6 + a7 at most; of the slopes root mean squares over an interval, 0.71 (a6 + a7) of polynomials
    // of their own and 8 a6 + 10 a7 of derivatives (those of T6' and T7'), which an interval's ends exceed by 1.4 and by 5.  The halves'
    // polynomials come from the whole one of degree 7: the first term that this leaves out, a8 T8, is known from the slopes, whose a7 is 16 times that,
    // and its derivative, 12 a8, added.  Every feature is held to what the fp32 evaluation of the MLP rounds of it, 1e-7 of G,
    // G^2 = sum_k W2[k][f]^2 tau_k^2 SiLU'(t_k)^2, tau_k^2 the sum of the squares of t_k's eight terms, and for the slopes 1e-7 kappa G, kappa
    // what a basis function grows by along a unit of length relative to itself: 8 pi / rc from the sine, 4 / (rc - d) where it vanishes as
    // (rc - d)^4; further to what the length's rounding to fp32, half an ulp, changes on average: 2^-26 of the length times kappa.  Where SiLU' is
    // near zero a sixteenth stands for SiLU'^2: there the feature is small beside what it is elsewhere (a unit's t goes to 0 at the cutoff,
    // so -0.28 is always passed).  G goes with the feature's column of W2: scaling that against the later maps does not change the verdict.
    if (node < 4) {   // the wavefronts' tables: values, slopes, both on either half
        const double(&a)[kTabNodes][64] = node == 0 ? sv : node == 1 ? uv : half[node - 2];
        const double a0 = a[0][lane], a1 = a[1][lane], a2 = a[2][lane], a3 = a[3][lane], a4 = a[4][lane], a5 = a[5][lane];
        const double c[6] = {a0 - a2 + a4, a1 - 3 * a3 + 5 * a5, 2 * a2 - 8 * a4, 4 * a3 - 20 * a5, 8 * a4, 16 * a5};
        if (lane < F) {
            float *to = J.tab + (size_t)layer * tab_layer(F);
            const int of_lane = 4 * (lane % 32 / 2) + lane % 2;   // 32 features: where the lane's lie in [16][2][2]
            to += node >= 2 ? 2 * tab_floats(F) + lane / 32 * kTabBothFloats + (2 * iv + node - 2) * 192 + of_lane
                            : node * tab_floats(F) + iv * (F * 6) + (F == 64 ? lane : of_lane);
            const bool wide = F == 64 && node < 2;
#pragma unroll
            for (int k = 0; k < 6; ++k) to[wide ? 64 * k : 64 * (k / 2) + 2 * (k % 2)] = (float)c[k];
        }
        double g2 = 0;
#pragma unroll
        for (int j = 0; j < kTabNodes; ++j) g2 += gv[j][lane] * (node == 1 ? slope_g[j] : 1.0) * (1.0 / kTabNodes);
        const double mid = length(node == 2 ? -0.5 : node == 3 ? 0.5 : 0.0), rounding = 0x1p-26 * mid * kappa(mid);
        const double a6 = fabs(a[6][lane]), a7 = fabs(a[7][lane]);
        // (a place grows by 2 per_d along a unit of length in a half)
        const double cut = node == 0   ? a6 + a7
                           : node == 1 ? 0.71 * (a6 + a7)
                                       : fmax(a6 + a7, ((8 * a6 + 10 * a7) * 2 * per_d + 0.75 * fabs(uv[7][lane])) / kappa(mid));
        const bool feature_bad = !(cut * cut <= g2 * (1e-14 + rounding * rounding));   // (not a number: not represented)
        if (__any(feature_bad) && lane == 0) any_bad = 1;
    }
    __syncthreads();
    if (node != 0) return;
    const bool bad = any_bad != 0;
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
// A wavefront is four workers of 16 lanes, lane = neighbouring features.  A worker walks work items, each one or two rows, in steps of 16 edges;
// items follow one another without a break in the pipeline (records two steps ahead, gathered rows a few edges), and each worker has its
// own.  Lane l of a worker holds the record of edge l of its step; a DPP row broadcast hands it to the others.
//
// What a step costs (measured one thing at a time): a wavefront issues a vector instruction every 5 clocks, one that takes its
// predecessor's result every 8.25, a DPP one every 8, and a SIMD issues two of them at a time, whatever the number of wavefronts; LDS reads 256
// bytes a clock with 16-byte reads, less than half of that with 8-byte ones; a row of 256 bytes takes the vector-memory path 4.2
// clocks where it lies in the L2, whatever the width of the load, and a store of 4 bytes a lane as much as one of 16.
//
// Bounds and times, 256,000 atoms, F = 64, us a launch (with one table for values and slopes, 32 features a block, in brackets): forward, LDS 83 %
// busy, 214 (260); reverse, the vector unit, 3.4 clocks an instruction, 381 (383); layer 0, LDS 62 %, address unit 73 %, 259 (357).  A
// million atoms in 8 slabs: 867, 1767, 1175 (1052, 1764, 1654).  Of these the forward and layer 0's steps fetch 4.3 and 6.4 GB, rows gathered
// again from beyond the L2 (half a plane of the lattice under way in an XCD), layer 0's at 5.9 TB/s.

struct TabArgs {               // one partition
    int32_t n_rows, n_edges;   // receiver rows processed and their edges (below 2^29: byte offsets below 2^31)
    int32_t n_nodes;           // rows of g / abar
    const int64_t *row_ptr;
    const int32_t *chunk_row;  // the graph's work-item table: first row whose first edge lies at or after c * span
    int32_t span;
    const int32_t *senders;
    const float *d, *g, *abar;
    float *out;                // forward: a [n_rows][F]; reverse: gbar [n_rows][F]
    float *dsum[2];            // reverse: per edge its share of dE/dd, summed over the layers, of each block of 32 features; layer 0's step adds
                               // up the blocks' sums and its own share in the first
};
struct TabBatch {
    const float *tab;      // the layer's table of the step's kind
    float inv_h;
    int slots;             // blocks of an XCD for each block of features; blocks beyond them have no rows
    int rows;              // rows of a work item
    int few;               // few rows for the workers: every XCD takes rows of one partition, 8 / n XCDs each
    int together;          // fewer still: a wavefront's four workers take a row together
    int first;             // reverse: dsum is written, not added to
    int n;
    int64_t edge_start[kBatch + 1];
    TabArgs s[kBatch];
};
// Wavefronts per block, values that are computed together (of one edge or of several), and edges whose rows are on their way.
#ifndef MLIP_TAB_FWD
#define MLIP_TAB_FWD 16, 8, 4
#endif
#ifndef MLIP_TAB_BWD
#define MLIP_TAB_BWD 16, 4, 4
#endif
#ifndef MLIP_TAB_LAST
#define MLIP_TAB_LAST 12, 8, 8
#endif
struct TabShape { int waves, values, ring; };
constexpr TabShape kTabFwd = {MLIP_TAB_FWD}, kTabBwd = {MLIP_TAB_BWD}, kTabLast = {MLIP_TAB_LAST};
constexpr int kTabRows = 2;     // most rows of a work item
enum { TAB_FWD, TAB_BWD, TAB_LAST };   // the forward step, a reverse step, the reverse step of layer 0 (no sums over rows)
template <int F, int KIND> struct TabKind {
    static constexpr int kI = KIND == TAB_BWD ? 2 : F / 16;              // features of a lane
    static constexpr int kBlocks = F / (16 * kI);                        // blocks of features, each with a table of its own
    static constexpr int kFloats = KIND == TAB_BWD ? kTabBothFloats : tab_floats(F);
    static constexpr int kPerUnit = KIND == TAB_BWD ? 2 : 1;             // its intervals to one of the grid
    static constexpr int kOffset = KIND == TAB_FWD ? 0 : KIND == TAB_LAST ? tab_floats(F) : 2 * tab_floats(F);   // in the layer's tables
};

template <int K> __device__ inline int row_bcast(int v) { return __builtin_amdgcn_mov_dpp(v, 0x150 + K, 0xf, 0xf, true); }
template <int K> __device__ inline float row_bcast(float v)
{
    return __builtin_bit_cast(float, row_bcast<K>(__builtin_bit_cast(int, v)));
}
template <class Fn, int... K> __device__ __forceinline__ void unrolled(std::integer_sequence<int, K...>, Fn fn)
{
    (fn(std::integral_constant<int, K>{}), ...);
}
template <int N, class Fn> __device__ __forceinline__ void unrolled(Fn fn) { unrolled(std::make_integer_sequence<int, N>{}, fn); }
// All N values are computed by here, and nothing is done with one of them before: what is done step by step for N values stays so (left alone,
// the compiler puts the steps for one value behind one another).
template <int N> __device__ __forceinline__ void fence(float *v)
{
    static_assert(N == 1 || N % 2 == 0);
    if constexpr (N == 1) asm volatile("" : "+v"(v[0]));
    else if constexpr (N == 2) asm volatile("" : "+v"(v[0]), "+v"(v[1]));
    else if constexpr (N == 4) asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]));
    else {
        asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]), "+v"(v[7]));
        if constexpr (N > 8) fence<N - 8>(v + 8);
    }
}

// I neighbouring features of a row, the lane's, at byte offset off
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
template <int I> struct TabRow {
    typedef float vec __attribute__((ext_vector_type(I)));
    float v[I];
    __device__ __forceinline__ void load(__amdgpu_buffer_rsrc_t r, uint32_t off)
    {
        vec x;
        if constexpr (I == 4) x = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
        else x = __builtin_bit_cast(vec, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
#pragma unroll
        for (int i = 0; i < I; ++i) v[i] = x[i];
    }
    __device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t r, uint32_t off) const
    {
        vec x;
#pragma unroll
        for (int i = 0; i < I; ++i) x[i] = v[i];
        if constexpr (I == 4) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, x), r, off, 0, 0);
        else __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, x), r, off, 0, 0);
    }
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int i = 0; i < I; ++i) v[i] = 0.f;
    }
};
// the six coefficients of the lane's I features in an interval
template <int I> struct TabCoeff {
    f32x4 q[I * 6 / 4];
    __device__ __forceinline__ void read(const char *at)
    {
#pragma unroll
        for (int i = 0; i < I * 6 / 4; ++i) q[i] = *reinterpret_cast<const f32x4 *>(at + 256 * i);
    }
    __device__ __forceinline__ float c(int k, int i) const { return I == 4 ? q[k][i] : q[k / 2][2 * (k % 2) + i]; }
};
// The polynomials of G edges at their places s, p[t][i] of the lane's i-th feature, and with DERIVE their derivatives dp, step by step for all
// of them.
template <bool DERIVE, int G, int I>
__device__ __forceinline__ void tab_values(const TabCoeff<I> (&c)[G], const float (&s)[G], float (&p)[G][I], float (&dp)[G][I])
{
#pragma unroll
    for (int t = 0; t < G; ++t)
#pragma unroll
        for (int i = 0; i < I; ++i) p[t][i] = dp[t][i] = c[t].c(5, i);
#pragma unroll
    for (int k = 4; k >= 0; --k) {
        if (DERIVE && k < 4) {
#pragma unroll
            for (int t = 0; t < G; ++t)
#pragma unroll
                for (int i = 0; i < I; ++i) dp[t][i] = fmaf(s[t], dp[t][i], p[t][i]);
            fence<G * I>(&dp[0][0]);
        }
#pragma unroll
        for (int t = 0; t < G; ++t)
#pragma unroll
            for (int i = 0; i < I; ++i) p[t][i] = fmaf(s[t], p[t][i], c[t].c(k, i));
        fence<G * I>(&p[0][0]);
    }
}

struct TabItem {     // a work item: row r0 and, if there is one, row r0 + 1
    int32_t r0, e0;  // and the first edge
    int32_t n0, n;   // edges of the first row, of both
};
struct TabStep {     // one step of a worker: edges tb to tb + 15 of an item, as far as they go
    int32_t tb;
    TabItem item;
};
struct TabRec {      // as loaded
    int32_t sj;
    float d, before, before1; // reverse: the sums of the later layers at the lane's edge
};
struct TabEdge {     // what the lanes of the worker need of an edge
    int32_t goff;    // byte offset of the sender's row; past the end of the array for an edge past the item's last: its row reads 0
    int32_t loff;    // byte offset of the interval in the table
    float s, slope;  // place in the interval; of the lane's own edge ds / dd
};
// bit 16 w + k where a worker w's lane k has it: the workers' bits together, and the lane's own worker's
struct TabBits {
    uint32_t any, mine;
    __device__ __forceinline__ TabBits(bool bit, int lane)
    {
        const uint64_t b = __ballot(bit);
        const uint32_t two = (uint32_t)b | (uint32_t)(b >> 32);
        any = two | two >> 16;
        mine = (uint32_t)(b >> (lane & 48));
    }
};

// a buffer of n bytes from p on, as 32-bit accesses see it (beyond n they read 0 and write nothing)
__device__ inline __amdgpu_buffer_rsrc_t tab_buffer(const void *p, uint32_t n)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, (int)n, kBufferFlags);
}
__device__ inline int32_t buffer_load_i32(__amdgpu_buffer_rsrc_t r, uint32_t off) { return (int32_t)__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0); }

// Work items.  Every XCD takes a contiguous eighth of the launch's edges, cut at the rows where the graph's work-item tables (chunk_row)
// have an entry (of a launch with about a row for a worker, where one partition after the other and a look at those tables would be most of
// its time, 21 us for 8 x 192 rows, rows of one partition); the blocks of features each go through all of it, on the same XCD.  The
// XCD's rows are dealt to its blocks in turn, kTabDeal items at a time, so that at any moment they work on a short run of rows whose
// neighbourhoods share the L2; within its block's share every worker starts at its own item and then draws from a counter in LDS.  (Draws
// from one counter per XCD in memory: one per 35 ns, 140 us a launch at 32,000 rows.)
constexpr int kTabDeal = 8;
static_assert(kTabDeal == 8, "edge_tab shifts by three");
__device__ inline int32_t tab_cut(const TabArgs &A, int64_t edge)   // the row at which the partition is cut for its edge `edge`
{
    return edge <= 0 ? 0 : edge >= A.n_edges ? A.n_rows : min(A.chunk_row[edge / A.span], A.n_rows);
}

// Sums of q[0..15] over the 16 lanes of each row of lanes: lane l returns the sum of q[l].  Each step adds lanes across one bit of the
// lane number and lets the lanes on either side go on with one of two edges.
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
    for (int k = 0; k < 8; ++k)     // row_ror:8; lanes 8-15 of a row keep edge k + 8, lanes 0-7 edge k
        z[k] = keep_banks<0xc>(add_dpp<0x128>(q[k]), add_dpp<0x128>(q[k + 8]));
#pragma unroll
    for (int k = 0; k < 4; ++k)     // row_half_mirror; odd quads keep edge k + 4, even ones edge k
        y[k] = keep_banks<0xa>(add_dpp<0x141>(z[k]), add_dpp<0x141>(z[k + 4]));
    const unsigned bit1 = (lane & 2) ? ~0u : 0u, bit0 = (lane & 1) ? ~0u : 0u;
    auto keep = [](unsigned mask, float v, float w) {   // w where the mask is set
        return __builtin_bit_cast(float, (__builtin_bit_cast(unsigned, w) & mask) | (__builtin_bit_cast(unsigned, v) & ~mask));
    };
#pragma unroll
    for (int k = 0; k < 2; ++k)     // quad_perm 2,3,0,1
        x[k] = keep(bit1, add_dpp<0x4e>(y[k]), add_dpp<0x4e>(y[k + 2]));
    return keep(bit0, add_dpp<0xb1>(x[0]), add_dpp<0xb1>(x[1]));   // quad_perm 1,0,3,2
}

// TAB_FWD over the owned rows: a_i = sum_e w_e * g_send(e).
// TAB_BWD over all local rows, owned and ghost: gbar_i = sum_e w_e * abar_send(e) and, added up over the layers, for every edge its share
// sum_f w'_f (abar_j g_i)_f of dE/dd.  The share with abar_i g_j is the reverse edge's, whose row gathers abar_i: the forces take both
// (k_force_rows), and the step gathers one row per edge instead of two.  (In a partition an owned row's edges from ghosts have no share,
// abar of a ghost being zero, and the ghosts' rows hold the other ones.)  TAB_LAST: the shares alone.
template <int F, int KIND, int NW, int VALUES, int RING, bool TOGETHER> __device__ __forceinline__ void edge_tab_walk(const TabBatch &B, char *lds)
{
    using K = TabKind<F, KIND>;
    constexpr int kRow = F * 4, kI = K::kI, GROUP = VALUES / kI;   // edges that are computed together
    constexpr bool SUMS = KIND != TAB_LAST, SHARES = KIND != TAB_FWD;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, l16 = lane & 15, at_f = l16 * (4 * kI);
    const int hb = K::kBlocks > 1 ? (blockIdx.x >> 3) & (K::kBlocks - 1) : 0;   // the block of features
    const char *tab = lds + l16 * 16, *lut = lds + K::kFloats * 4;
    const int32_t n_slots = B.slots, xcd = blockIdx.x & 7, slot = (int32_t)(blockIdx.x >> 3) / K::kBlocks;
    const int64_t total = B.edge_start[B.n], share = (total + 7) >> 3;
    const int64_t from = xcd * share, to = xcd == 7 ? total + 1 : from + share;   // the XCD's edges
    const int32_t mine = xcd * B.n >> 3, mine_from = (8 * mine + B.n - 1) / B.n, mine_n = (8 * mine + 8 + B.n - 1) / B.n - mine_from;   // B.few
    int32_t *counter = reinterpret_cast<int32_t *>(lds + K::kFloats * 4 + kTabLut);   // items drawn, per partition
    // A wavefront's workers take items of their own or, where there are few rows for them (plan_edge_tab), one row together, every fourth
    // step of it each.
    constexpr int stride = TOGETHER ? 64 : 16;            // from a worker's step to its next one
    const int offset = TOGETHER ? lane & 48 : 0;          // its first one
    if (threadIdx.x < kBatch) counter[threadIdx.x] = TOGETHER ? NW : 4 * NW;
    if (threadIdx.x < kTabUnits) {
        const TabGrid::Unit unit = kTabGrid.unit[threadIdx.x];
        reinterpret_cast<TabGrid::Unit *>(lds + K::kFloats * 4)[threadIdx.x] = TabGrid::Unit{unit.n * K::kPerUnit, unit.at * K::kPerUnit};
    }
    const int32_t rows = B.rows;
    int32_t r0 = 0, r1 = 0;                   // rows of the worker's next item
    int32_t p0 = 0, p1 = 0, p2 = 0;           // row_ptr from r0 on
    int32_t drawn = 0;                        // the item after it, as the worker's first lane drew it
    int part = 0;
    bool have = false;                        // whether there is a next item
    int32_t lo = 0, hi = 0;                   // the XCD's rows; lo: the first one dealt to this block
    __amdgpu_buffer_rsrc_t ptr, send, dist, g, abar, out, sums, sums1;
    const int32_t turn = n_slots * kTabDeal * rows;   // rows from one of the block's turns to the next
    auto choose = [&](int32_t k) {
        r0 = lo + __mul24(k >> 3, turn) + __mul24(k & (kTabDeal - 1), rows);
        r1 = min(r0 + rows, hi);
        have = r0 < hi;
    };
    // Where the next item's edges lie: asked for at every step, whether or not the item is a new one, so that the answer has its registers
    // to itself (in the branch of those workers that take an item the compiler moves it, and waits for every load under way).
    auto fetch = [&]() {   // (past the last row: reads 0)
        p0 = buffer_load_i32(ptr, (uint32_t)r0 * 8u);
        p1 = buffer_load_i32(ptr, (uint32_t)r0 * 8u + 8u);
        p2 = buffer_load_i32(ptr, (uint32_t)r1 * 8u);
    };
    auto draw = [&]() {
        int zero = 0;
        asm("" : "+v"(zero));   // (an address that looks uniform would be combined over the lanes, and the result waited for at once)
        if (TOGETHER ? lane == 0 : l16 == 0) drawn = __hip_atomic_fetch_add(counter + part + zero, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
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
            choose(TOGETHER ? wave : 4 * wave + (lane >> 4));
            if (__any(have)) {
                fetch();
                const uint32_t n_rec = (uint32_t)A.n_edges * 4u, n_nodes = (uint32_t)A.n_nodes * kRow - 128u * hb;
                send = tab_buffer(A.senders, n_rec);
                dist = tab_buffer(A.d, n_rec);
                g = tab_buffer(A.g + 32 * hb, n_nodes);
                if (SHARES) {
                    abar = tab_buffer(A.abar + 32 * hb, n_nodes);
                    sums = tab_buffer(hb ? A.dsum[1] : A.dsum[0], n_rec);
                    if (KIND == TAB_LAST && F == 64) sums1 = tab_buffer(A.dsum[1], B.first ? 0 : n_rec);
                }
                if (SUMS) out = tab_buffer(A.out + 32 * hb, (uint32_t)A.n_rows * kRow - 128u * hb);
                break;
            }
        }
    };

    TabRow<kI> ring[RING], acc, none;
    acc.clear();
    none.clear();
    struct Heads { TabRow<kI> first, second; };   // g of the receivers of a step's first edge and of its item's second row
    TabStep front, SA, SB;
    TabRec RA, RB;
    TabEdge EA, EB;
    Heads HA, HB;
    auto load = [&](const TabStep &S) {   // (past the item's last edge another item's, or nothing: not counted)
        const int32_t e = S.item.e0 + S.tb + l16;
        const float before1 = KIND == TAB_LAST && F == 64 ? buffer_load_f32(sums1, (uint32_t)e * 4u, 0, 0) : 0.f;
        return TabRec{buffer_load_i32(send, (uint32_t)e * 4u), buffer_load_f32(dist, (uint32_t)e * 4u, 0, 0),
                      SHARES && !B.first ? buffer_load_f32(sums, (uint32_t)e * 4u, 0, 0) : 0.f, before1};
    };
    auto edge = [&](const TabRec &R, const TabStep &S) {
        TabEdge E;
        const float v = R.d * B.inv_h;
        const int j = min((int)v, kTabUnits - 1);
        const f32x2 unit = *reinterpret_cast<const f32x2 *>(lut + 8 * j);
        // the interval within the unit; the last one of its own at most, as the place and the slope are in this unit's measure.  (Products and sums
        // that decide about it are spelled out: left to the compiler, one copy of the loop rounds v and another does not, and a length at an
        // interval's end takes one or the other with the step that its worker happens to be at.)
        const float k = fminf(truncf(fmaf(R.d, B.inv_h, -(float)j) * unit[0]), unit[0] - 1.f);
        E.slope = (2.f * B.inv_h) * unit[0];
        E.s = fmaf(R.d, E.slope, fmaf(-2.f, fmaf((float)j, unit[0], k), -1.f));
        E.loff = __mul24((int)(unit[1] + k), 16 * kI * 24);
        E.goff = S.tb + l16 < S.item.n ? R.sj * kRow : (int32_t)0x80000000;
        return E;
    };
    auto heads = [&](const TabStep &S, Heads &H) {
        if (SHARES) {
            H.first.load(g, (S.item.r0 + (S.tb >= S.item.n0 ? 1 : 0)) * kRow + at_f);
            H.second.load(g, (S.item.r0 + 1) * kRow + at_f);
        }
    };
    auto gather = [&](const TabEdge &E, auto k) { ring[k % RING].load(SHARES ? abar : g, row_bcast<k>(E.goff) + at_f); };
    auto compute = [&](const TabStep &S, const TabEdge &E, float before, const Heads &H, const TabEdge &next) {
        const int32_t u = S.tb + l16 + 1;
        const TabBits ends(!TOGETHER && (u == S.item.n0 || u == S.item.n) && u <= S.item.n, lane);   // an edge that is its row's last
        TabRow<kI> gi = H.first;
        float q[16];
        unrolled<16 / GROUP>([&](auto grp) {
            constexpr int k0 = grp * GROUP;
            __builtin_amdgcn_sched_barrier(0);
            TabCoeff<kI> c[GROUP];
            float s[GROUP], p[GROUP][kI], dp[GROUP][kI];
            unrolled<GROUP>([&](auto t) { c[t].read(tab + row_bcast<k0 + t>(E.loff)); });
            unrolled<GROUP>([&](auto t) { s[t] = row_bcast<k0 + t>(E.s); });
            tab_values<KIND == TAB_BWD>(c, s, p, dp);
            unrolled<GROUP>([&](auto t) {
                constexpr int k = k0 + t;
                const TabRow<kI> &x = ring[k % RING];
                if (SUMS) {
#pragma unroll
                    for (int i = 0; i < kI; ++i) acc.v[i] = fmaf(p[t][i], x.v[i], acc.v[i]);
                }
                if (SHARES) {
                    float a[kI];
#pragma unroll
                    for (int i = 0; i < kI; ++i) a[i] = x.v[i] * gi.v[i];
                    const float(&w)[kI] = KIND == TAB_BWD ? dp[t] : p[t];
                    q[k] = w[0] * a[0];
#pragma unroll
                    for (int i = 1; i < kI; ++i) q[k] = fmaf(w[i], a[i], q[k]);
                    fence<1>(q + k);
                }
                if (__builtin_expect((ends.any & (1u << k)) != 0, 0)) {
                    if (ends.mine & (1u << k)) {
                        if (SUMS) {
                            acc.store(out, (S.item.r0 + (S.tb + k >= S.item.n0 ? 1 : 0)) * kRow + at_f);
                            acc.clear();
                        }
                        if (SHARES) gi = H.second;
                    }
                }
            });
            unrolled<GROUP>([&](auto t) {
                constexpr int k = k0 + t + RING;
                if constexpr (k < 16) gather(E, std::integral_constant<int, k>{});
                else gather(next, std::integral_constant<int, k - 16>{});
            });
        });
        if (SUMS && TOGETHER && __any(S.item.n > 0 && S.tb - offset + 64 >= S.item.n)) {   // the row's last step: the workers' sums together
#pragma unroll
            for (int i = 0; i < kI; ++i) acc.v[i] += __shfl_xor(acc.v[i], 16, 64);
#pragma unroll
            for (int i = 0; i < kI; ++i) acc.v[i] += __shfl_xor(acc.v[i], 32, 64);
            if (lane < 16) acc.store(out, S.item.r0 * kRow + at_f);
            acc.clear();
        }
        if (SHARES) {
            __builtin_amdgcn_sched_barrier(0);
            const float sum = tab_reduce(q, lane);
            if (S.tb + l16 < S.item.n)
                buffer_store_f32(KIND == TAB_BWD ? fmaf(sum, E.slope, before) : sum + before, sums, (uint32_t)(S.item.e0 + S.tb + l16) * 4u, 0, 0);
        }
    };
    auto advance = [&]() {
        front.tb += stride;
        const bool pop = front.tb - offset >= front.item.n;
        if (__any(pop)) {
            if (pop) {
                front = TabStep{offset, TabItem{r0, p0, (r1 - r0 == 2 ? p1 : p2) - p0, have ? p2 - p0 : 0}};
                if (SUMS) {
                    const bool none0 = have && front.item.n0 == 0, none1 = have && r1 - r0 == 2 && front.item.n == front.item.n0;
                    if (__builtin_expect(__any(none0 || none1), 0)) {   // rows without edges
                        if (none0) none.store(out, r0 * kRow + at_f);
                        if (none1) none.store(out, (r0 + 1) * kRow + at_f);
                    }
                }
                choose(TOGETHER ? __builtin_amdgcn_readfirstlane(drawn) : row_bcast<0>(drawn));
                draw();
            }
        }
        fetch();
    };
    auto begin = [&]() {   // the records of a partition's first two steps
        draw();
        front = TabStep{offset, TabItem{0, 0, 0, 0}};   // no edges
        advance();
        SA = front;
        RA = load(SA);
        advance();
        SB = front;
        RB = load(SB);
    };
    next_part();
    {
        LdsFill<K::kFloats / 4, NW * 64> fill;
        fill.load(B.tab + (size_t)hb * K::kFloats);
        fill.store(lds);
    }
    __syncthreads();
    for (; part < B.n; ++part, next_part()) {
        float before_a, before_b;
        begin();
        EA = edge(RA, SA);
        before_a = RA.before + RA.before1;
        heads(SA, HA);
        unrolled<RING>([&](auto k) { gather(EA, k); });
        while (__any(have || SA.tb - offset < SA.item.n || SB.tb - offset < SB.item.n)) {
            advance();
            const TabStep SC = front;
            RA = load(SC);
            EB = edge(RB, SB);
            before_b = RB.before + RB.before1;
            heads(SB, HB);
            __builtin_amdgcn_sched_barrier(0);
            compute(SA, EA, before_a, HA, EB);
            // Few rows: where the second step would be empty it is most of what is left of the launch (108 atoms, a row a wavefront: 8.0 us forward,
            // 6.2 without; 4,000 atoms, a row a worker: 13.5 and 12.3).  Layer 0's step, a row a worker, has no registers for the way out.
            if ((TOGETHER || KIND != TAB_LAST) && B.few && !__any(have || SB.tb - offset < SB.item.n || SC.tb - offset < SC.item.n)) break;
            advance();
            SA = SC;
            const TabStep SD = front;
            RB = load(SD);
            EA = edge(RA, SA);
            before_a = RA.before + RA.before1;
            heads(SA, HA);
            __builtin_amdgcn_sched_barrier(0);
            compute(SB, EB, before_b, HB, EA);
            SB = SD;
        }
    }
}
template <int F, int KIND, int NW> __device__ __forceinline__ void edge_tab(const TabBatch &B, char *lds)
{
    constexpr TabShape shape = KIND == TAB_FWD ? kTabFwd : KIND == TAB_BWD ? kTabBwd : kTabLast;
    if (B.together) edge_tab_walk<F, KIND, NW, shape.values, shape.ring, true>(B, lds);
    else edge_tab_walk<F, KIND, NW, shape.values, shape.ring, false>(B, lds);
}
template <int F>
__global__ void __launch_bounds__(kTabFwd.waves * 64, kTabFwd.waves / 4) k_edge_fwd_tab(TabBatch B)
{
    extern __shared__ __align__(16) char tab_mem[];
    edge_tab<F, TAB_FWD, kTabFwd.waves>(B, tab_mem);
}
template <int F>
__global__ void __launch_bounds__(kTabBwd.waves * 64, kTabBwd.waves / 4) k_edge_bwd_tab(TabBatch B)
{
    extern __shared__ __align__(16) char tab_mem[];
    edge_tab<F, TAB_BWD, kTabBwd.waves>(B, tab_mem);
}
template <int F>
__global__ void __launch_bounds__(kTabLast.waves * 64, kTabLast.waves / 4) k_edge_last_tab(TabBatch B)
{
    extern __shared__ __align__(16) char tab_mem[];
    edge_tab<F, TAB_LAST, kTabLast.waves>(B, tab_mem);
}

// ---------------------------------------------------------------- either way
//
// The edge steps of a call whose host has not heard yet whether the tables represent the filters: one launch that goes by *bad, so that
// the way and every bit of the result follow from the weights alone, whatever the handle has seen before.  A row's or an edge's sum does
// not depend on the wavefronts of a block, so either way gives what its own kernel gives; the reverse step takes 8 of them, the most that
// leave the way by MLP the registers it needs.
constexpr int kBothBwdWaves = 8;
struct BothBatch {
    TabBatch tab;
    EdgeBatch mlp;
    const int32_t *bad;
};
static_assert(sizeof(BothBatch) <= 4096, "kernel arguments");
template <int F, int PREC>
__global__ void __launch_bounds__(kFwdWaves * 64, kFwdWaves / 4) k_edge_fwd_both(BothBatch B)
{
    extern __shared__ __align__(16) float lds[];
    if (*B.bad != 0)
        edge_fwd<F, PREC>(B.mlp, lds);
    else if ((int)(blockIdx.x >> 3) < B.tab.slots)
        edge_tab<F, TAB_FWD, kFwdWaves>(B.tab, reinterpret_cast<char *>(lds));
}
template <int F, int PREC, int KIND>
__global__ void __launch_bounds__(kBothBwdWaves * 64, kBothBwdWaves / 4) k_edge_bwd_both(BothBatch B)
{
    extern __shared__ __align__(16) float lds[];
    if (*B.bad != 0)
        edge_bwd<F, PREC, kBothBwdWaves>(B.mlp, lds);
    else if ((int)(blockIdx.x >> 3) < B.tab.slots * TabKind<F, KIND>::kBlocks)
        edge_tab<F, KIND, kBothBwdWaves>(B.tab, reinterpret_cast<char *>(lds));
}

#endif  // MLIP_MODEL_TABLE_H
