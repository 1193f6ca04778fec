// Radial message-passing potential on gfx950: forward, hand-written reverse pass, forces.
//
// Model (benchmark configuration 0):  h0 = Emb[z];  per layer  g = h Wm,
//   a_i = sum_{e: recv=i} (SiLU(b_e W1) W2) * g_send(e),  h += SiLU(a Wo);
//   eps_i = SiLU(h Wr1) . wr2,  E = sum eps,  F = -dE/dr.
// Partitioned execution follows the paper's scheme (Graph-Parallel Message
// Passing; Distributing Atom Graphs): every partition computes the edges whose
// receiver it owns, ghost rows of g are refreshed from their owners before each
// layer's edge step and ghost-row gradients are added back to the owners in the
// reverse pass.
//
// Kernel design
//  * Every edge's filter is a function of its length: where the weights allow it (decided on the device), the layers run on tables of
//    it (model_table.h), and what follows on pair lists, kept filter values and the edge kernels is the way without.
//  * All dense contractions (filter MLP per edge, F x F maps per node and per bond) run on the 16-bit matrix
//    pipeline: fp32 products as exact three-part bf16 sums with fp32 accumulation, with items (edges, nodes or
//    bonds) as the 32 MFMA columns and features as rows.  In that orientation the accumulator layout of one
//    product is directly the B operand of the next one if the contraction index is visited in the order the
//    accumulator registers hold it; the weight (A) operands are pre-packed in that order, so chained products
//    need no transposition or lane exchange.
//  * The per-receiver reduction is LDS-staged: a 32-edge tile of filter outputs
//    is written to LDS edge-major, then each lane owns one feature, reads the
//    tile row by row, multiplies with the gathered sender row (one coalesced
//    256-byte load per edge) and keeps a running sum that is flushed when the
//    receiver changes.  No atomics; the summation order is the canonical edge order.
//  * Reverse pass without scatter: the edge set is symmetric (i<-j,S) <-> (j<-i,-S)
//    with bitwise equal length, hence equal filter value w.  So
//      gbar_i = sum_{e in row i} w_e * abar_send(e)
//      dE/dd summed over an edge and its mirror = dw/dd . (abar_i*g_j + abar_j*g_i)
//    are both receiver-side gathers.  In a partition, abar of ghost rows is zero
//    and ghost rows carry the sub-row of neighbours owned by the partition, which
//    yields exactly the ghost-row gradients the owner must receive.
#include "mlip_internal.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <type_traits>

namespace mlip {

namespace {

#include "model_tiles.h"
#include "model_edge.h"
#include "model_node.h"
#include "model_bond.h"
#include "model_table.h"

inline unsigned blocks_for(int64_t n, int threads) { return (unsigned)((n + threads - 1) / threads); }

// ---------------------------------------------------------------- host driver

struct Packs {  // offsets (floats) into the packed-weight buffer
    size_t per_layer, A1, A1s, W2t, W2n, Wmt, Wmn, Wot, Won, readout_t, readout_n, total;
};

Packs pack_layout(int F, int L)
{
    Packs p;
    const size_t ff = (size_t)F * F * 3 / 2, p1 = (size_t)(F / 32) * 3 * 64 * 2;   // three bf16 parts
    p.A1 = 0;
    p.A1s = p1;
    p.W2t = 2 * p1;
    p.W2n = p.W2t + ff;
    p.Wmt = p.W2n + ff;
    p.Wmn = p.Wmt + ff;
    p.Wot = p.Wmn + ff;
    p.Won = p.Wot + ff;
    p.per_layer = p.Won + ff;
    p.readout_t = p.per_layer * (size_t)L;
    p.readout_n = p.readout_t + ff;
    p.total = p.readout_n + ff;
    return p;
}

constexpr int kNodeBlocks = 256;   // one per compute unit (512: 38 us against 27 for the largest of them at 32,000 atoms, 4 % slower at a million)

template <int F> struct Lds {
    using D = Dims<F>;
    static constexpr size_t edge_fwd(int prec) { return sizeof(float) * (pack_floats<F>(prec) + D::PACK1 + kFwdWaves * D::TILE); }
    static constexpr size_t edge_bwd(int prec, int waves) { return sizeof(float) * (pack_floats<F>(prec) + D::PACK1 + waves * kQueue * D::FS); }
};

// Dynamic LDS size of a kernel, set once per handle (a handle lives on one device and is used by one thread at a
// time, so this state needs no lock and is right for the device the handle's memory is on).  Returns the slot of
// the kernel in g->fn_occ, whose second member caches the resident blocks per compute unit (0: not queried).
int configure_kernel(mlip_graph *g, const void *fn, size_t lds, int *slot)
{
    for (size_t k = 0; k < g->fn_occ.size(); ++k)
        if (g->fn_occ[k].first == fn) { *slot = (int)k; return MLIP_OK; }
    MLIP_HIP(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    g->fn_occ.emplace_back(fn, 0);
    *slot = (int)g->fn_occ.size() - 1;
    return MLIP_OK;
}

template <int F, int OP> int launch_node(mlip_graph *g, NodeBatch &b)
{
    using N = NodeOp<OP>;
    const size_t lds = sizeof(float) * N::NPACK * Dims<F>::PACK3;
    int slot = 0;
    MLIP_TRY(configure_kernel(g, reinterpret_cast<const void *>(&k_node<F, OP>), lds, &slot));
    b.tile_start[0] = 0;
    for (int q = 0; q < b.n; ++q) b.tile_start[q + 1] = b.tile_start[q] + (std::max<int64_t>(b.s[q].n_rows, 0) + 31) / 32;
    for (int q = b.n; q < kBatch; ++q) b.tile_start[q + 1] = b.tile_start[b.n];
    const int64_t n_tiles = b.tile_start[b.n];
    if (n_tiles <= 0) return MLIP_OK;
    // every block keeps the weights in LDS and walks several tiles
    const unsigned blocks = (unsigned)std::min<int64_t>(n_tiles, kNodeBlocks);
    k_node<F, OP><<<blocks, N::NW * 64, lds, g->stream>>>(b);
    MLIP_HIP(hipGetLastError());
    return MLIP_OK;
}

template <int F, int STAGE, int PREC> int launch_bond_mlp(mlip_graph *g, const BondArgs &a)
{
    constexpr int NW = BondStage<STAGE>::NW;
    constexpr size_t lds = sizeof(float) * (BondStage<STAGE>::NPACK * pack_floats<F>(PREC) + NW * BondStage<STAGE>::TILE);
    int slot = 0;
    MLIP_TRY(configure_kernel(g, reinterpret_cast<const void *>(&k_bond_mlp<F, STAGE, PREC>), lds, &slot));
    if (a.n <= 0) return MLIP_OK;
    // every block keeps its operand packs in LDS and walks several tiles
    const unsigned blocks = (unsigned)std::min<int64_t>((a.n + 31) / 32, BondStage<STAGE>::BLOCKS);
    k_bond_mlp<F, STAGE, PREC><<<blocks, NW * 64, lds, g->stream>>>(a);
    MLIP_HIP(hipGetLastError());
    return MLIP_OK;
}

// Runs one node operation over all partitions, kBatch per launch; common holds what they share, fill(view, args) sets the rows.
template <int F, int OP, class Fill> int node_pass(mlip_graph *g, SlabView *views, int P, const NodeBatch &common, Fill fill)
{
    int n_clear = common.n_clear;   // by the first launch that has rows
    for (int p0 = 0; p0 < P; p0 += kBatch) {
        NodeBatch nb = common;
        nb.n_clear = n_clear;
        nb.n = std::min(kBatch, P - p0);
        for (int q = 0; q < nb.n; ++q) {
            SlabView &v = views[p0 + q];
            NodeArgs &na = nb.s[q];
            na = NodeArgs{};
            na.n_rows = v.n_owned;
            na.n_pure = v.n_pure;
            na.nodes = v.nodes;
            fill(v, na);
        }
        MLIP_TRY((launch_node<F, OP>(g, nb)));
        if (nb.tile_start[nb.n] > 0) n_clear = 0;
    }
    return MLIP_OK;
}

// Edge-kernel launches of one call: two per layer and batch of partitions (L <= 8, at most 64 / kBatch batches).
constexpr int kWorkLaunches = 2 * 8 * (64 / kBatch);

int count_compute_units(mlip_graph *g)   // once per handle
{
    if (g->n_cu != 0) return MLIP_OK;
    int dev = 0, n = 0;
    MLIP_HIP(hipGetDevice(&dev));
    MLIP_HIP(hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev));
    if (n < 8) { set_error("%d compute units: the edge kernels take eighths of the device", n); return MLIP_EHIP; }
    g->n_cu = n;
    return MLIP_OK;
}

// Work items and counters of an edge step by MLP.
int plan_edge(mlip_graph *g, EdgeBatch &b)
{
    MLIP_TRY(count_compute_units(g));
    if (g->work_next >= kWorkLaunches) {
        set_error("more than %d edge-kernel launches in one call", kWorkLaunches);
        return MLIP_ESTATE;
    }
    b.work = g->work_ptr + (size_t)g->work_next * (8 * kWorkCounterStride);
    b.chunk_start[0] = 0;
    for (int q = 0; q < b.n; ++q) b.chunk_start[q + 1] = b.chunk_start[q] + (b.s[q].n_rows > 0 ? b.s[q].n_chunks : 0);
    for (int q = b.n; q < kBatch; ++q) b.chunk_start[q + 1] = b.chunk_start[b.n];
    return MLIP_OK;
}

// Blocks of a persistent launch on an XCD: what is resident at once, no more than the work needs (few items: one per block, so that they
// spread over the compute units).
int64_t edge_slots(const mlip_graph *g, const EdgeBatch &b, int occ)
{
    return std::min<int64_t>((int64_t)(g->n_cu / 8) * occ, (b.chunk_start[b.n] + 7) / 8);
}

template <int F, int PREC> int launch_edge(mlip_graph *g, EdgeBatch &b, bool backward)
{
    const size_t lds = backward ? Lds<F>::edge_bwd(PREC, kBwdWaves) : Lds<F>::edge_fwd(PREC);
    const int threads = (backward ? kBwdWaves : kFwdWaves) * 64;
    // resident blocks per compute unit, queried once per kernel and handle
    const void *fn = backward ? reinterpret_cast<const void *>(&k_edge_bwd<F, PREC>) : reinterpret_cast<const void *>(&k_edge_fwd<F, PREC>);
    int slot = 0;
    MLIP_TRY(configure_kernel(g, fn, lds, &slot));
    int occ = g->fn_occ[slot].second;
    if (occ == 0) {
        MLIP_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, fn, threads, lds));
        if (occ < 1) { set_error("edge kernel does not fit the device"); return MLIP_EHIP; }
        g->fn_occ[slot].second = occ;
    }
    MLIP_TRY(plan_edge(g, b));
    const unsigned blocks = (unsigned)(8 * edge_slots(g, b, occ));
    if (blocks == 0) return MLIP_OK;
    if (backward)
        k_edge_bwd<F, PREC><<<blocks, threads, lds, g->stream>>>(b);
    else
        k_edge_fwd<F, PREC><<<blocks, threads, lds, g->stream>>>(b);
    MLIP_HIP(hipGetLastError());
    return MLIP_OK;
}

// Upper edges of a view: every pair of two owned-row edges has one, and an owned-row edge from a ghost sender is one, whose
// reverse edge is in a ghost row (as build_pairs_impl counts them).
int64_t upper_edges(const SlabView &v)
{
    const int64_t n_ghost_edges = v.n_edges - v.n_edges_owned;
    return (v.n_edges_owned - n_ghost_edges) / 2 + n_ghost_edges;
}

// Rows for a compute unit up to which the four workers of a wavefront take a row together: a launch of so few rows takes as long as one
// row's chain, `one` steps of 64 edges instead of `four` of 16 (108 atoms, F = 32: forward 10.6 us, so 6.2).  With more rows the launch takes the
// sum of the steps, of which the row alone is `four` and together 4 `one`: the line lies where what the chain gains is what the empty workers cost, 16
// measured.  Energy and forces, three layers, us a call with rows for workers and taken together, at 6 edges a row never the faster (F = 64, 1,536 atoms 93
// and 97, 8,192 111 and 134); 20 edges: F = 32, 2,048 atoms (8 rows for a compute unit) 85 and 80, 4,096 87 and 90, 8,192 96 and 107; 42: F = 64, 2,048
// 123 and 102, 4,096 134 and 119, 8,192 154 and 154, F = 32 115 and 110; 70: F = 32, 4,096 117 and 106, 8,192 132 and 152, F = 64, 4,096 154 and
// 147, 8,192 185 and 207.  (At 34 to 40 edges and F = 64 the last fifth below the limit of 32 is 3 % the slower.)
int64_t tab_together(int64_t rows, int64_t edges)
{
    const int64_t mean = (edges + rows - 1) / rows;   // (a row in two has more)
    const int64_t four = (mean + 1 + 15) / 16, one = (mean + 1 + 63) / 64, empty = 4 * one - four;
    constexpr int64_t kMost = 32;
    return empty > 0 ? std::min(kMost, 16 * (four - one) / empty) : kMost;
}

// Rows of an edge step on tables, split over the chip; blocks of `waves` wavefronts, `blocks` of them for the blocks of features.
int plan_edge_tab(mlip_graph *g, TabBatch &b, int blocks, int waves)
{
    MLIP_TRY(count_compute_units(g));
    // A few rows at a time, so that the rows all workers of an XCD are at stay close together (a million atoms, forward, 32 features in a
    // block: 1.6 GB fetched with two, 8.2 with 22; 1.10 ms with two, 1.12 with one or three, 1.22 with six.  64 features in a block: 4.3 GB;
    // 0.83 to 0.87 ms with one or two, the reverse steps 2 % slower with one); one where there are not even eight items for every worker.
    int64_t rows = 0, edges = 0;
    for (int q = 0; q < b.n; ++q) {
        rows += b.s[q].n_rows;
        edges += b.s[q].n_edges;
    }
    const int64_t workers = (int64_t)(g->n_cu / blocks) * waves * 4;
    b.rows = (int)std::min<int64_t>(kTabRows, std::max<int64_t>(1, rows / (8 * workers)));
    b.few = rows <= workers;
    b.together = rows > 0 && rows <= (g->n_cu / blocks) * tab_together(rows, edges);
    if (b.together) b.rows = 1;
    b.edge_start[0] = 0;
    for (int q = 0; q < kBatch; ++q) b.edge_start[q + 1] = b.edge_start[q] + (q < b.n ? b.s[q].n_edges : 0);
    // persistent grid: one block per compute unit (the table fills its LDS), fewer where there are not even kTabDeal items for each
    const int64_t items = (rows + b.rows - 1) / b.rows;
    b.slots = (int)std::max<int64_t>(rows > 0, std::min<int64_t>(g->n_cu / 8 / blocks, (items + 8 * kTabDeal - 1) / (8 * kTabDeal)));
    return MLIP_OK;
}

// Edge steps on tables, one launch for up to kBatch partitions.
template <int F, int KIND> int launch_edge_tab(mlip_graph *g, TabBatch &b)
{
    using K = TabKind<F, KIND>;
    void (*kernel)(TabBatch) = KIND == TAB_FWD ? &k_edge_fwd_tab<F> : KIND == TAB_BWD ? &k_edge_bwd_tab<F> : &k_edge_last_tab<F>;
    constexpr int waves = (KIND == TAB_FWD ? kTabFwd : KIND == TAB_BWD ? kTabBwd : kTabLast).waves, lds = tab_lds(K::kFloats);
    int slot = 0;
    MLIP_TRY(configure_kernel(g, reinterpret_cast<const void *>(kernel), lds, &slot));
    b.tab += K::kOffset;
    MLIP_TRY(plan_edge_tab(g, b, K::kBlocks, waves));
    if (b.slots == 0) return MLIP_OK;
    kernel<<<(unsigned)(8 * K::kBlocks * b.slots), waves * 64, lds, g->stream>>>(b);
    MLIP_HIP(hipGetLastError());
    return MLIP_OK;
}

// The same with the way left to the device: *bad != 0 by MLP.
template <int F, int PREC, int KIND> int launch_edge_both(mlip_graph *g, TabBatch &tab, EdgeBatch &mlp, const int32_t *bad)
{
    using K = TabKind<F, KIND>;
    void (*kernel)(BothBatch);
    if constexpr (KIND == TAB_FWD) kernel = &k_edge_fwd_both<F, PREC>;
    else kernel = &k_edge_bwd_both<F, PREC, KIND>;
    constexpr int waves = KIND == TAB_FWD ? kFwdWaves : kBothBwdWaves;
    const size_t lds = std::max<size_t>(tab_lds(K::kFloats), KIND == TAB_FWD ? Lds<F>::edge_fwd(PREC) : Lds<F>::edge_bwd(PREC, waves));
    int slot = 0;
    MLIP_TRY(configure_kernel(g, reinterpret_cast<const void *>(kernel), lds, &slot));
    tab.tab += K::kOffset;
    MLIP_TRY(plan_edge_tab(g, tab, K::kBlocks, waves));
    MLIP_TRY(plan_edge(g, mlp));
    const int64_t slots = std::max<int64_t>(K::kBlocks * tab.slots, edge_slots(g, mlp, 1));
    if (slots == 0) return MLIP_OK;
    BothBatch b;
    b.tab = tab;
    b.mlp = mlp;
    b.bad = bad;
    kernel<<<(unsigned)(8 * slots), waves * 64, lds, g->stream>>>(b);
    MLIP_HIP(hipGetLastError());
    return MLIP_OK;
}

// bw != nullptr: the three-body variant
template <int F>
int forward_t(mlip_graph *g, const mlip_weights_t *w, const mlip_bond_weights_t *bw, int32_t mode, double *energy,
              float *forces, float *atom_energy, Carver *scratch)
{
    hipStream_t s = g->stream;
    const int L = w->L;
    const int prec = (w->precision == MLIP_PRECISION_BF16) ? kPrecBf16
                     : (w->precision == MLIP_PRECISION_FP32_SPLIT) ? kPrecF16x3 : kPrecF32;
    const bool slabs = (mode == MLIP_MODE_SLABS);
    const int P = slabs ? g->P : 1;
    SlabView *views = slabs ? g->slabs.data() : &g->whole;
    const size_t rowb = (size_t)F * sizeof(float);

    // ---- workspace
    for (int p = 0; p < P; ++p)
        if (views[p].n_local * (int64_t)F * 4 >= ((int64_t)1 << 31)) {
            set_error("a partition holds more than 2^31 bytes of node features; use more slabs");
            return MLIP_EINVAL;
        }
    // every array of the call either lives in the view's own grow-only buffer or is carved from the fixed block
    auto place = [&](DevBuf &buf, size_t bytes, float *&ptr) -> int {
        if (scratch) {
            ptr = static_cast<float *>(scratch->take(bytes));
            return MLIP_OK;   // a failed carve is reported once, below
        }
        MLIP_TRY(buf.ensure(bytes));
        ptr = buf.as<float>();
        return MLIP_OK;
    };
    // ---- packed weights and filter tables: kept in the handle until a call comes with a different weight struct or cutoff; the
    // fixed block of the static variant is shared by all handles, so there they are made on every call
    const Packs pk = pack_layout(F, L);
    float *wp = nullptr;
    MLIP_TRY(place(g->wpack, pk.total * sizeof(float), wp));
    char *tables = nullptr;
    if (L > 0) {
        if (!scratch) MLIP_TRY(g->tables.ensure(table_bytes(F, L)));
        tables = static_cast<char *>(scratch ? scratch->tables : g->tables.p);
    }
    TabState *tab_state = reinterpret_cast<TabState *>(tables);
    float *tab0 = reinterpret_cast<float *>(tables + kTabHeader);
    auto layer_table = [&](int l) { return tab0 + (size_t)l * tab_layer(F); };
    const float tab_inv_h = (float)(kTabUnits / g->r_cut);
    const bool repack = scratch != nullptr || !g->packed_w_valid || std::memcmp(&g->packed_w, w, sizeof(*w)) != 0 || g->table_rcut != g->r_cut;
    const int w2_kind = prec == kPrecBf16 ? PACK_FF_BF16 : prec == kPrecF16x3 ? PACK_FF_F16X2 : PACK_FF_BF16X3;
    int64_t *verdict = static_cast<int64_t *>(g->pinned) + kPinnedTableWord;
    if (repack && !(scratch && scratch->failed())) {
        prof_begin(g, MLIP_PROF_NODE);
        g->packed_w_valid = false;
        PackBatch pb{};
        pb.F = F;
        if (L > 0) {
            pb.clear = &tab_state->bad;
            pb.n_clear = kTabHeader / 4;
        }
        const size_t ff = (size_t)F * F;   // floats of a weight matrix
        for (int l = 0; l < L; ++l) {
            float *base = wp + pk.per_layer * l;
            pb.add(w->W1 + (size_t)l * 8 * F, base + pk.A1, PACK_W1, 0, 1.0f);
            pb.add(w->W1 + (size_t)l * 8 * F, base + pk.A1s, PACK_W1, 0, kSiluScale);
            pb.add(w->W2 + l * ff, base + pk.W2t, w2_kind, 1, kSiluScaleInv);
            pb.add(w->W2 + l * ff, base + pk.W2n, w2_kind, 0, 1.0f);
            pb.add(w->Wm + l * ff, base + pk.Wmt, PACK_FF_BF16X3, 1, 1.0f);
            pb.add(w->Wm + l * ff, base + pk.Wmn, PACK_FF_BF16X3, 0, 1.0f);
            pb.add(w->Wo + l * ff, base + pk.Wot, PACK_FF_BF16X3, 1, 1.0f);
            pb.add(w->Wo + l * ff, base + pk.Won, PACK_FF_BF16X3, 0, 1.0f);
        }
        pb.add(w->Wr1, wp + pk.readout_t, PACK_FF_BF16X3_ALT, 1, 1.0f);
        pb.add(w->Wr1, wp + pk.readout_n, PACK_FF_BF16X3, 0, 1.0f);
        k_pack<<<dim3(blocks_for((int64_t)F * F, 256), pb.n), 256, 0, s>>>(pb);
        if (L > 0) {
            TabJob job{};
            job.W1 = w->W1;
            job.W2 = w->W2;
            job.tab = tab0;
            job.state = tab_state;
            job.publish = verdict;
            job.generation = ++g->table_generation;
            job.inv_h = (double)tab_inv_h;
            job.rc = g->r_cut;
            job.p = w->p;
            job.F = F;
            job.bf16 = prec == kPrecBf16;
            k_filter_table<F><<<dim3(kTabN, L), kTabNodes * 64, 0, s>>>(job);
        }
        MLIP_HIP(hipGetLastError());
        if (!scratch) {
            g->packed_w = *w;
            g->packed_w_valid = true;
            g->table_rcut = g->r_cut;
            g->kept_generation = g->table_generation;
        }
        prof_end(g);
    }
    // Whether the tables represent this model's filters is decided on the device when they are made.  Until the host has seen the word, the
    // launches go by the device's: the way depends on the weights alone, not on what the handle has seen before or on when the host looks.
    enum { BY_TABLE, BY_MLP, BOTH_WAYS };
    int by = BOTH_WAYS;
    int64_t most_edges = 0;
    for (int p = 0; p < P; ++p) most_edges = std::max(most_edges, views[p].n_edges);
    if (L == 0 || most_edges >= (int64_t)1 << 29) {   // the steps on tables address an edge's records and sums, 4 bytes each, by offsets below 2^31
        by = BY_MLP;
    } else if (!repack) {
        const int64_t word = __atomic_load_n(verdict, __ATOMIC_RELAXED);
        if (word >> 1 == g->kept_generation) by = (word & 1) ? BY_MLP : BY_TABLE;
    }
    const int32_t *gate = by == BOTH_WAYS ? &tab_state->bad : nullptr;   // != null: the launches look at it


    // By MLP: both edges of an edge / reverse-edge pair have the same length, hence bit for bit the same filter values: the
    // forward kernel keeps those of the upper edges, the reverse kernel runs on the partitions' upper-edge graphs and a
    // row-wise kernel adds the lower edges' terms.
    if (L > 0 && (by != BY_TABLE || scratch)) {   // (the fixed block has their place in any case: its limit does not depend on the way)
        prof_begin(g, MLIP_PROF_GRAPH);
        // Undecided calls make the lists only if the device says that they are needed where they are carved or long (4.2 M edges, 80 us; four
        // launches that end at once take 9), and keep those of a smaller graph for the next model of a committee (700,000 edges, 28 us).
        int64_t edges = 0;
        for (int p = 0; p < P; ++p) edges += views[p].n_edges;
        MLIP_TRY(build_pairs_impl(g, views, P, scratch, scratch || edges >= (int64_t)1 << 22 ? gate : nullptr, by != BY_TABLE));
        prof_end(g);
    }
    int64_t n_parts = 0;
    for (int p = 0; p < P; ++p) {
        SlabView &v = views[p];
        const size_t no = (size_t)std::max<int64_t>(v.n_owned, 1), nl = (size_t)std::max<int64_t>(v.n_local, 1);
        MLIP_TRY(place(v.h, no * rowb, v.ws.h));
        MLIP_TRY(place(v.hbar, no * rowb, v.ws.hbar));
        if (bw) {   // every layer's is kept for the bonds' own reverse step
            MLIP_TRY(v.bonds.abar_keep.ensure(nl * rowb * (size_t)std::max(L, 1)));
            v.ws.abar = v.bonds.abar_keep.as<float>();
        } else {
            MLIP_TRY(place(v.abar, nl * rowb, v.ws.abar));
        }
        MLIP_TRY(place(v.gbar, nl * rowb, v.ws.gbar));
        MLIP_TRY(place(v.eps, no * sizeof(float), v.ws.eps));
        const size_t ne = (size_t)std::max<int64_t>(v.n_edges, 1);
        MLIP_TRY(place(v.dsum, ne * sizeof(float) * (scratch ? 1 : F / 32), v.ws.dsum));
        MLIP_TRY(place(v.floc, nl * 3 * sizeof(float), v.ws.floc));
        MLIP_TRY(place(v.g, nl * rowb * (size_t)std::max(L, 1), v.ws.g));
        MLIP_TRY(place(v.a, no * rowb * (size_t)std::max(L, 1), v.ws.a));
        v.ws.wst = nullptr;
        if (L > 0)   // kept filter values, a slice per layer (layer 0's reverse step needs none: its slice stays empty, and
                     // the fixed block holds none for it)
            MLIP_TRY(place(v.wst, (size_t)std::max<int64_t>(upper_edges(v), 1) * rowb * (size_t)(scratch ? L - 1 : L), v.ws.wst));
        v.ws.dsum2 = nullptr;
        if (F == 64 && L > 1 && by != BY_MLP)   // on tables every block of 32 features has its own sums (the one step of a model of one layer takes all
                                                // 64 at a time); in the fixed block, whose limit does not depend on the way, the second ones
                                                // lie where the way by MLP has its kept filter values (F per pair, at least one per edge)
            v.ws.dsum2 = scratch ? v.ws.wst : v.ws.dsum + ne;
        n_parts += (v.n_owned + 31) / 32;
    }
    float *energy_part_f = nullptr;
    MLIP_TRY(place(g->energy_part, (size_t)std::max<int64_t>(n_parts, 1) * sizeof(double), energy_part_f));
    float *work_f = nullptr;
    // one set of counters per edge-kernel launch: two per layer and batch of partitions
    const size_t work_n = (size_t)std::max(1, 2 * L * ((P + kBatch - 1) / kBatch)) * 8 * kWorkCounterStride;
    MLIP_TRY(place(g->work, work_n * sizeof(int32_t), work_f));
    if (scratch && scratch->failed()) {
        set_error("this graph and model need more than the %zu bytes of static workspace", scratch->size);
        return MLIP_EINVAL;
    }
    double *energy_part = reinterpret_cast<double *>(energy_part_f);
    g->work_ptr = reinterpret_cast<int32_t *>(work_f);
    g->work_next = 0;
    auto wslice = [&](SlabView &v, int l) { return v.ws.wst + (size_t)(scratch ? l - 1 : l) * (size_t)upper_edges(v) * F; };   // l >= 1
    // dE/da of a layer: one array for all layers in turn, or one per layer where the three-body variant keeps them
    auto abarslice = [&](SlabView &v, int l) { return v.ws.abar + (bw ? (size_t)l * (size_t)v.n_local * F : 0); };

    // ---- batches for the small kernels (embedding, ghost transfers, forces, energy): up to kBatch partitions per launch
    enum { U_OWNED, U_GHOST, U_LOCAL };
    auto small_batch = [&](int p0, int unit, int layer) {
        SmallBatch sb{};
        sb.tables = by == BY_TABLE;
        sb.gate = gate;
        sb.n = std::min(kBatch, P - p0);
        sb.start[0] = 0;
        for (int q = 0; q < kBatch; ++q) {
            if (q >= sb.n) { sb.start[q + 1] = sb.start[q]; continue; }
            SlabView &v = views[p0 + q];
            SmallArgs &a = sb.s[q];
            a.n_owned = v.n_owned;
            a.n_pure = v.n_pure;
            a.n_local = v.n_local;
            a.nodes = v.nodes;
            a.row_ptr = v.row_ptr;
            a.senders = v.senders;
            a.mirror = v.mirror;
            a.shiftp = v.shiftp;
            a.gbar = v.ws.gbar;
            a.abar = abarslice(v, std::max(layer, 0));
            a.floc = v.ws.floc;
            a.eps = v.ws.eps;
            a.dsum = v.ws.dsum;
            a.d = v.d;
            a.wstore = layer >= 1 ? wslice(v, layer) : nullptr;
            a.uslot = v.pairs.uslot;
            a.l_row_ptr = v.pairs.l_row_ptr;
            a.l_senders = v.pairs.l_senders;
            a.l_slot = v.pairs.l_slot;
            const bool bonds = bw && v.bonds.n > 0;
            sb.bonds |= bonds;
            a.bond_of_edge = bonds ? v.bonds.of_edge.as<int32_t>() : nullptr;
            a.wb_bf16 = (prec == kPrecBf16);
            a.wb = (bonds && layer >= 0)
                       ? static_cast<char *>(v.bonds.wb.p) + (size_t)layer * (size_t)std::max<int64_t>(v.bonds.n, 1) * F *
                                                                   (a.wb_bf16 ? sizeof(__bf16) : sizeof(float))
                       : nullptr;
            const int64_t items = unit == U_OWNED ? v.n_owned : unit == U_GHOST ? v.n_ghost : v.n_local;
            sb.start[q + 1] = sb.start[q] + std::max<int64_t>(items, 0);
        }
        return sb;
    };
    GhostIndex gidx{};
    if (slabs) {
        gidx.needed_by = g->needed_by;
        gidx.gbase = g->part.gbase.as<int32_t>();
        gidx.ghost_local = g->part.ghost_local.as<int32_t>();
    }

    BasisParams bp;
    bp.rc = (float)g->r_cut;
    bp.inv_rc = (float)(1.0 / g->r_cut);
    bp.p = w->p;
    const double pd = (double)w->p;
    bp.pc0 = (float)(pd * (pd + 1) * (pd + 2) / 2);

    // ---- three-body variant: bond lists, bond embedding, triplet update, bond terms of the layers' filters.
    // All bonds and triplets of an owned centre are local to its partition, so this part needs no transfer.
    float *bpk = nullptr;        // packed F x F operands of the bond part
    const size_t ffp = (size_t)Dims<F>::PACK3;   // floats of an operand slot
    // operand slots: 0 Wta (y = x W), 1 Wtb, 2 Wt2, 3 Wta^T, 4 Wtb^T, 5 Wt2^T, 6 + l Wb_l, 6 + L + l Wb_l^T; after them We0
    // and Wtc packed for the K = 8 products
    BasisParams bpb = bp;
    auto bstride = [&](SlabView &v) { return (size_t)std::max<int64_t>(v.bonds.n, 1) * F; };   // elements per [n][F] array
    // the [bonds x F] arrays are bf16 in the bf16 mode, fp32 otherwise
    const bool bond_bf16 = (prec == kPrecBf16);
    const size_t belem = bond_bf16 ? sizeof(__bf16) : sizeof(float);
    auto bond_elem = [&](auto &&launch) {   // calls launch with a value of the arrays' element type
        if (bond_bf16) launch((__bf16)0.0f);
        else launch(0.0f);
    };
    auto wbslice = [&](SlabView &v, int l) -> void * {
        return static_cast<char *>(v.bonds.wb.p) + (size_t)l * bstride(v) * belem;
    };
    auto bond_args = [&](SlabView &v) {   // everything a stage of k_bond_mlp may touch; the stage's operands are set by the caller
        BondGraph &BG = v.bonds;
        BondArgs a{};
        a.n = BG.n;
        a.d = BG.d.as<float>();
        a.u = BG.u.as<float>();
        a.du = BG.du.as<float>();
        a.edge = BG.edge.as<int32_t>();
        a.sender = BG.sender.as<int32_t>();
        a.recv = v.recv;
        a.We0p = bpk + (size_t)(6 + 2 * L) * ffp;
        a.bp = bpb;
        a.wb_stride = bstride(v);
        a.P = BG.P.p;
        a.Q = BG.Q.p;
        a.S = BG.S.p;
        a.m = BG.m.p;
        a.wb = BG.wb.p;
        a.abar = BG.abar_keep.as<float>();
        a.abar_stride = (size_t)v.n_local * F;
        a.g = v.ws.g;
        a.g_stride = (size_t)v.n_local * F;
        a.e1bar = BG.e1bar.p;
        a.ubar = BG.ubar.as<float>();
        a.Sbar = BG.Sbar.p;
        a.Pbar = BG.Pbar.p;
        a.Qbar = BG.Qbar.p;
        a.dbond = BG.dbond.as<float>();
        return a;
    };
    bool any_bonds = false;
    if (bw) {
        bpb.rc = bw->r_bond;
        bpb.inv_rc = 1.0f / bw->r_bond;
        prof_begin(g, MLIP_PROF_BOND);
        for (int p = 0; p < P; ++p) MLIP_TRY(build_bonds_impl(g, views[p], (double)bw->r_bond, w->p));
        prof_end(g);
        for (int p = 0; p < P; ++p) {
            BondGraph &BG = views[p].bonds;
            const size_t bs = bstride(views[p]), nb1 = (size_t)std::max<int64_t>(BG.n, 1);
            DevBuf *fb[] = {&BG.P, &BG.Q, &BG.S, &BG.m, &BG.e1bar, &BG.Sbar, &BG.Pbar, &BG.Qbar};
            for (DevBuf *b : fb) MLIP_TRY(b->ensure(bs * belem));
            MLIP_TRY(BG.wb.ensure(bs * belem * (size_t)std::max(L, 1)));
            MLIP_TRY(BG.ubar.ensure(nb1 * sizeof(float)));
            MLIP_TRY(BG.dbond.ensure(nb1 * sizeof(float)));
            MLIP_TRY(BG.rbar.ensure(nb1 * 3 * sizeof(float)));
            any_bonds = any_bonds || BG.n > 0;
        }
        MLIP_TRY(g->bond_wpack.ensure(((size_t)(6 + 2 * L) * ffp + 2 * Dims<F>::PACK1) * sizeof(float)));
        bpk = g->bond_wpack.as<float>();
        prof_begin(g, MLIP_PROF_BOND);
        const size_t ff = (size_t)F * F;   // floats of a weight matrix
        const float *Wta = bw->Wt1, *Wtb = bw->Wt1 + ff, *Wtc = bw->Wt1 + 2 * ff;
        const bool repack_b = !g->packed_bw_valid || std::memcmp(&g->packed_bw, bw, sizeof(*bw)) != 0 ||
                              std::memcmp(&g->packed_bw_w, w, sizeof(*w)) != 0;
        g->packed_bw_valid = false;
        if (repack_b) {   // the bond MLPs' F x F products follow the filter MLP's precision mode
            PackBatch pb{};
            pb.F = F;
            auto pack_bond = [&](const float *Wsrc, int trans, int slot) { pb.add(Wsrc, bpk + (size_t)slot * ffp, w2_kind, trans, 1.0f); };
            pack_bond(Wta, 1, 0);
            pack_bond(Wtb, 1, 1);
            pack_bond(bw->Wt2, 1, 2);
            pack_bond(Wta, 0, 3);
            pack_bond(Wtb, 0, 4);
            pack_bond(bw->Wt2, 0, 5);
            for (int l = 0; l < L; ++l) {
                pack_bond(bw->Wb + l * ff, 1, 6 + l);
                pack_bond(bw->Wb + l * ff, 0, 6 + L + l);
            }
            pb.add(bw->We0, bpk + (size_t)(6 + 2 * L) * ffp, PACK_W1, 0, 1.0f);
            pb.add(Wtc, bpk + (size_t)(6 + 2 * L) * ffp + Dims<F>::PACK1, PACK_W1, 0, 1.0f);
            k_pack<<<dim3(blocks_for((int64_t)F * F, 256), pb.n), 256, 0, s>>>(pb);
        }
        MLIP_HIP(hipGetLastError());
        g->packed_bw = *bw;
        g->packed_bw_w = *w;
        g->packed_bw_valid = true;
        for (int p = 0; p < P; ++p) {   // P = e0 Wta, Q = e0 Wtb with e0 = bbond(d) We0
            BondArgs a = bond_args(views[p]);
            a.W[0] = bpk + 0 * ffp;
            a.W[1] = bpk + 1 * ffp;
            MLIP_TRY(prec == kPrecBf16 ? (launch_bond_mlp<F, BOND_HEAD, kPrecBf16>(g, a))
                     : prec == kPrecF16x3 ? (launch_bond_mlp<F, BOND_HEAD, kPrecF16x3>(g, a)) : (launch_bond_mlp<F, BOND_HEAD, kPrecF32>(g, a)));
        }
        prof_end(g);
        prof_begin(g, MLIP_PROF_TRIPLET_FWD);
        for (int p = 0; p < P; ++p) {
            SlabView &v = views[p];
            BondGraph &BG = v.bonds;
            if (BG.n > 0)
                bond_elem([&](auto zero) {
                    using BT = decltype(zero);
                    k_triplet_fwd<F, BT><<<blocks_for(v.n_owned, 4), 256, 0, s>>>(
                        v.n_owned, BG.ptr.as<int64_t>(), BG.rhat.as<float>(), BG.u.as<float>(), BG.P.as<BT>(), BG.Q.as<BT>(), Wtc,
                        bpk + (size_t)(6 + 2 * L) * ffp + Dims<F>::PACK1, BG.S.as<BT>());
                });
        }
        MLIP_HIP(hipGetLastError());
        prof_end(g);
        prof_begin(g, MLIP_PROF_BOND);
        for (int p = 0; p < P; ++p) {   // m = S Wt2, e1 = e0 + u SiLU(m), wb_l = e1 Wb_l
            BondArgs a = bond_args(views[p]);
            a.W[0] = bpk + 2 * ffp;
            for (int l = 0; l < std::min(L, 3); ++l) a.W[1 + l] = bpk + (6 + l) * ffp;
            a.Wx = bpk + (6 + 3) * ffp;
            a.n_layers = L;
            MLIP_TRY(prec == kPrecBf16 ? (launch_bond_mlp<F, BOND_TAIL, kPrecBf16>(g, a))
                     : prec == kPrecF16x3 ? (launch_bond_mlp<F, BOND_TAIL, kPrecF16x3>(g, a)) : (launch_bond_mlp<F, BOND_TAIL, kPrecF32>(g, a)));
        }
        prof_end(g);
    }

    auto gslice = [&](SlabView &v, int l) { return v.ws.g + (size_t)l * (size_t)v.n_local * F; };
    auto aslice = [&](SlabView &v, int l) { return v.ws.a + (size_t)l * (size_t)v.n_owned * F; };

    // what the node launches share; the ghost rows' addresses are set per launch
    NodeBatch common{};
    common.wr2 = w->wr2;
    common.emb = w->emb;
    common.species = g->species.as<int32_t>();
    common.ghosts = gidx;
    auto ghost_tab = [&](auto &&array_of) {
        if (slabs)
            for (int q = 0; q < P; ++q) common.tab.p[q] = array_of(views[q]);
    };
    auto layer_pack = [&](int l) { return wp + pk.per_layer * l; };
    auto tab_batch = [&](int p0, int l, bool backward) {   // the edge steps on tables: forward over the owned rows, reverse over the ghost rows
        TabBatch b{};                                      // too, as what they get goes back to their owners
        b.n = std::min(kBatch, P - p0);
        b.tab = layer_table(l);
        b.inv_h = tab_inv_h;
        b.first = l == L - 1;
        for (int q = 0; q < b.n; ++q) {
            SlabView &v = views[p0 + q];
            TabArgs &a = b.s[q];
            a.n_rows = (int32_t)(backward ? v.n_local : v.n_owned);
            a.n_edges = (int32_t)(backward ? v.n_edges : v.n_edges_owned);
            a.n_nodes = (int32_t)v.n_local;
            a.row_ptr = v.row_ptr;
            a.chunk_row = v.chunk_row;
            a.span = v.span;
            a.senders = v.senders;
            a.d = v.d;
            a.g = gslice(v, l);
            a.abar = backward ? abarslice(v, l) : nullptr;
            a.out = backward ? v.ws.gbar : aslice(v, l);
            a.dsum[0] = v.ws.dsum;
            a.dsum[1] = v.ws.dsum2;
        }
        return b;
    };
    auto edge_batch = [&](int p0, int l, bool backward) {   // by MLP: forward over the owned rows, reverse over their upper edges
        EdgeBatch b{};
        const float *base = layer_pack(l);
        b.n = std::min(kBatch, P - p0);
        b.c.A1 = base + pk.A1;
        b.c.A1s = base + pk.A1s;
        b.c.A2t = base + pk.W2t;
        b.c.A2n = base + pk.W2n;
        b.c.bp = bp;
        b.c.need_gbar = backward && l > 0;   // dE/dh0 is never used: the embedding does not depend on positions
        b.c.first = l == L - 1;
        for (int q = 0; q < b.n; ++q) {
            SlabView &v = views[p0 + q];
            EdgeArgs &a = b.s[q];
            const PairGraph &Q = v.pairs;
            a.n_rows = v.n_owned;
            a.n_nodes = v.n_local;
            a.g = gslice(v, l);
            a.wstore = l >= 1 ? wslice(v, l) : nullptr;
            if (backward) {
                a.n_chunks = chunks_of(Q.n_upper, Q.span);
                a.chunk_row = Q.u_chunk_row;
                a.row_ptr = Q.u_row_ptr;
                a.senders = Q.u_senders;
                a.recv = Q.u_recv;
                a.d = Q.u_d;
                a.mirror = Q.u_mirror;
                a.eid = Q.u_eid;
                a.abar = abarslice(v, l);
                a.out = v.ws.gbar;
                a.dsum = v.ws.dsum;
            } else {
                a.n_chunks = chunks_of(v.n_edges_owned, v.span);
                a.chunk_row = v.chunk_row;
                a.row_ptr = v.row_ptr;
                a.senders = v.senders;
                a.recv = v.recv;
                a.d = v.d;
                a.out = aslice(v, l);
                a.uslot = Q.uslot;
            }
        }
        return b;
    };
    auto edge_step_at = [&](auto precision, int p0, int l, bool backward) -> int {
        constexpr int PREC = decltype(precision)::value;
        TabBatch tab{};
        EdgeBatch mlp{};
        if (by != BY_MLP) tab = tab_batch(p0, l, backward);
        if (by != BY_TABLE) mlp = edge_batch(p0, l, backward);
        if (by == BY_MLP) return launch_edge<F, PREC>(g, mlp, backward);
        auto on_tables = [&](auto kind) {
            constexpr int KIND = decltype(kind)::value;
            return by == BOTH_WAYS ? launch_edge_both<F, PREC, KIND>(g, tab, mlp, gate) : launch_edge_tab<F, KIND>(g, tab);
        };
        if (!backward) return on_tables(std::integral_constant<int, TAB_FWD>{});
        if (l > 0) return on_tables(std::integral_constant<int, TAB_BWD>{});
        return on_tables(std::integral_constant<int, TAB_LAST>{});
    };
    auto edge_step = [&](int p0, int l, bool backward) -> int {   // of up to kBatch partitions from p0 on
        prof_begin(g, backward ? MLIP_PROF_EDGE_BWD : MLIP_PROF_EDGE_FWD);
        MLIP_TRY(prec == kPrecBf16    ? edge_step_at(std::integral_constant<int, kPrecBf16>{}, p0, l, backward)
                 : prec == kPrecF16x3 ? edge_step_at(std::integral_constant<int, kPrecF16x3>{}, p0, l, backward)
                                      : edge_step_at(std::integral_constant<int, kPrecF32>{}, p0, l, backward));
        ++g->work_next;
        prof_end(g);
        return MLIP_OK;
    };
    auto bond_sum = [&](int p0, int l, bool backward) -> int {   // the bonds' terms of the rows that edge_step has summed
        prof_begin(g, MLIP_PROF_BOND);
        BondSumBatch b{};
        b.n = std::min(kBatch, P - p0);
        for (int q = 0; q < b.n; ++q) {
            SlabView &v = views[p0 + q];
            b.start[q + 1] = b.start[q] + v.n_owned;
            if (v.bonds.n > 0)
                b.s[q] = BondSumArgs{v.bonds.ptr.as<int64_t>(), v.bonds.sender.as<int32_t>(), backward ? v.bonds.mirror.as<int32_t>() : nullptr,
                                     wbslice(v, l), backward ? abarslice(v, l) : gslice(v, l), backward ? v.ws.gbar : aslice(v, l)};
        }
        if (b.start[b.n] > 0)
            bond_elem([&](auto zero) { k_bond_sum<F, decltype(zero)><<<grid8((b.start[b.n] + 3) / 4), 256, 0, s>>>(b); });
        MLIP_HIP(hipGetLastError());
        prof_end(g);
        return MLIP_OK;
    };
    int64_t tiles_before = 0;
    auto tile_sums = [&](SlabView &v) {
        double *at = energy_part + tiles_before;
        tiles_before += (v.n_owned + 31) / 32;
        return at;
    };

    // ---- forward layers
    for (int l = 0; l < L; ++l) {
        const float *base = layer_pack(l);
        prof_begin(g, MLIP_PROF_NODE);
        ghost_tab([&](SlabView &v) { return gslice(v, l); });
        if (l == 0) {
            common.P[0] = base + pk.Wmt;
            common.clear = g->work_ptr;
            common.n_clear = (int)work_n;
            MLIP_TRY((node_pass<F, OP_EMBED>(g, views, P, common, [&](SlabView &v, NodeArgs &na) {
                na.Z = v.ws.h;
                na.Y = gslice(v, 0);
            })));
            common.n_clear = 0;
        } else {
            common.P[0] = layer_pack(l - 1) + pk.Wot;
            common.P[1] = base + pk.Wmt;
            MLIP_TRY((node_pass<F, OP_UPDATE>(g, views, P, common, [&](SlabView &v, NodeArgs &na) {
                na.X = aslice(v, l - 1);
                na.Z = v.ws.h;
                na.Y = gslice(v, l);
            })));
        }
        prof_end(g);
        for (int p0 = 0; p0 < P; p0 += kBatch) {   // the partitions in order, up to kBatch per launch
            MLIP_TRY(edge_step(p0, l, false));
            if (any_bonds) MLIP_TRY(bond_sum(p0, l, false));
        }
    }

    // ---- the last layer's update, the readout and the first step back
    prof_begin(g, MLIP_PROF_NODE);
    if (L > 0) {
        common.P[0] = layer_pack(L - 1) + pk.Wot;
        common.P[1] = wp + pk.readout_t;
        common.P[2] = wp + pk.readout_n;
        common.P[3] = layer_pack(L - 1) + pk.Won;
        MLIP_TRY((node_pass<F, OP_TURN>(g, views, P, common, [&](SlabView &v, NodeArgs &na) {
            na.X = aslice(v, L - 1);
            na.Z = v.ws.h;
            na.hbar = L > 1 ? v.ws.hbar : nullptr;   // (layer 0's step back is the last one)
            na.Y = abarslice(v, L - 1);
            na.eps = v.ws.eps;
            na.tile_sum = tile_sums(v);
        })));
    } else {
        common.P[0] = wp + pk.readout_t;
        MLIP_TRY((node_pass<F, OP_READ>(g, views, P, common, [&](SlabView &v, NodeArgs &na) {
            na.eps = v.ws.eps;
            na.tile_sum = tile_sums(v);
        })));
    }
    prof_end(g);
    const EnergySum energy_sum{tiles_before, energy_part, energy};

    // ---- reverse pass
    if (L > 0)   // ghost rows carry no dE/da: zero once, no kernel ever writes them
        for (int p0 = 0; p0 < P; p0 += kBatch) {
            const SmallBatch sb = small_batch(p0, U_GHOST, -1);
            if (sb.start[sb.n] > 0)
                k_zero_ghost_rows<<<dim3(blocks_for(sb.start[sb.n] * (F / 4), 256), bw ? L : 1), 256, 0, s>>>(sb, F);
        }
    MLIP_HIP(hipGetLastError());
    for (int l = L - 1; l >= 0; --l) {
        const float *base = wp + pk.per_layer * l;
        const bool need_gbar = l > 0;  // (as in edge_batch)
        for (int p0 = 0; p0 < P; p0 += kBatch) {
            MLIP_TRY(edge_step(p0, l, true));
            if (need_gbar && by != BY_TABLE) {   // second pass: the lower edges' terms of the rows' sums
                prof_begin(g, MLIP_PROF_EDGE_BWD_LOWER);
                const SmallBatch sb = small_batch(p0, U_OWNED, l);
                if (sb.start[sb.n] > 0)
                    k_edge_lower<F><<<blocks_for(sb.start[sb.n], 4), 256, 0, s>>>(sb);
                MLIP_HIP(hipGetLastError());
                prof_end(g);
            }
            if (need_gbar && any_bonds) MLIP_TRY(bond_sum(p0, l, true));
        }
        if (need_gbar) {
            if (slabs && (by != BY_TABLE || any_bonds)) {
                prof_begin(g, MLIP_PROF_GHOST);
                for (int p0 = 0; p0 < P; p0 += kBatch) {   // the ghost rows' gradients; the owners collect them below
                    const SmallBatch sb = small_batch(p0, U_GHOST, l);
                    if (sb.start[sb.n] > 0)
                        k_ghost_gbar<F><<<blocks_for(sb.start[sb.n], 4), 256, 0, s>>>(sb);
                }
                MLIP_HIP(hipGetLastError());
                prof_end(g);
            }
            prof_begin(g, MLIP_PROF_NODE);
            common.P[0] = base + pk.Wmn;
            common.P[1] = layer_pack(l - 1) + pk.Wot;
            common.P[2] = layer_pack(l - 1) + pk.Won;
            ghost_tab([&](SlabView &v) { return v.ws.gbar; });
            MLIP_TRY((node_pass<F, OP_BACK>(g, views, P, common, [&](SlabView &v, NodeArgs &na) {
                na.X = v.ws.gbar;
                na.X2 = aslice(v, l - 1);
                na.Z = v.ws.hbar;
                na.hbar = l > 1 ? v.ws.hbar : nullptr;   // (layer 0's step back is the last one)
                na.Y = abarslice(v, l - 1);
            })));
            prof_end(g);
        }
    }

    // ---- reverse of the bond update: e1 = e0 + u SiLU(m), m = S Wt2, S = triplet sum, e0 = bbond(d) We0
    if (any_bonds) {
        prof_begin(g, MLIP_PROF_BOND);
        const float *Wtc = bw->Wt1 + 2 * (size_t)F * F;
        for (int p = 0; p < P; ++p) {   // e1bar = sum_l dE/dwb_l Wb_l^T, ubar, Sbar = (e1bar u SiLU'(m)) Wt2^T
            BondArgs a = bond_args(views[p]);
            a.W[0] = bpk + 5 * ffp;
            for (int l = 0; l < std::min(L, 3); ++l) a.W[1 + l] = bpk + (6 + L + l) * ffp;
            a.Wx = bpk + (6 + L + 3) * ffp;
            a.n_layers = L;
            MLIP_TRY(prec == kPrecBf16 ? (launch_bond_mlp<F, BOND_EBAR, kPrecBf16>(g, a))
                     : prec == kPrecF16x3 ? (launch_bond_mlp<F, BOND_EBAR, kPrecF16x3>(g, a)) : (launch_bond_mlp<F, BOND_EBAR, kPrecF32>(g, a)));
        }
        prof_end(g);
        prof_begin(g, MLIP_PROF_TRIPLET_BWD);
        for (int p = 0; p < P; ++p) {
            SlabView &v = views[p];
            BondGraph &BG = v.bonds;
            if (BG.n > 0)
                bond_elem([&](auto zero) {
                    using BT = decltype(zero);
                    k_triplet_bwd<F, BT><<<blocks_for(v.n_owned, 4), 256, 0, s>>>(
                        v.n_owned, BG.ptr.as<int64_t>(), BG.rhat.as<float>(), BG.u.as<float>(), BG.P.as<BT>(), BG.Q.as<BT>(), Wtc,
                        bpk + (size_t)(6 + 2 * L) * ffp + Dims<F>::PACK1, BG.Sbar.as<BT>(), BG.Pbar.as<BT>(), BG.Qbar.as<BT>(),
                        BG.ubar.as<float>(), BG.rbar.as<float>());
                });
        }
        MLIP_HIP(hipGetLastError());
        prof_end(g);
        prof_begin(g, MLIP_PROF_BOND);
        for (int p = 0; p < P; ++p) {   // e0bar = e1bar + Pbar Wta^T + Qbar Wtb^T, and dE/dd of the bonds from it
            BondArgs a = bond_args(views[p]);
            a.W[0] = bpk + 3 * ffp;
            a.W[1] = bpk + 4 * ffp;
            MLIP_TRY(prec == kPrecBf16 ? (launch_bond_mlp<F, BOND_E0BAR, kPrecBf16>(g, a))
                     : prec == kPrecF16x3 ? (launch_bond_mlp<F, BOND_E0BAR, kPrecF16x3>(g, a)) : (launch_bond_mlp<F, BOND_E0BAR, kPrecF32>(g, a)));
        }
        prof_end(g);
    }

    // ---- forces: the bonds' part first, the radial rows add theirs
    prof_begin(g, MLIP_PROF_FORCE);
    const double *pos = g->pos.as<double>();
    if (any_bonds && L > 0)
        for (int p = 0; p < P; ++p) {
            SlabView &v = views[p];
            if (v.bonds.n <= 0) continue;
            BondGraph &BG = v.bonds;
            k_bond_force<<<blocks_for(v.n_owned, 16), 256, 0, s>>>(v.n_owned, BG.ptr.as<int64_t>(), BG.mirror.as<int32_t>(),
                                                                    BG.dbond.as<float>(), BG.rbar.as<float>(),
                                                                    BG.rhat.as<float>(), BG.d.as<float>(), v.ws.floc);
            if (v.n_ghost > 0)
                k_bond_force_ghost<<<blocks_for(v.n_ghost, 16), 256, 0, s>>>(
                    v.n_ghost, v.n_owned, v.row_ptr, v.mirror, BG.of_edge.as<int32_t>(), BG.dbond.as<float>(),
                    BG.rbar.as<float>(), BG.rhat.as<float>(), BG.d.as<float>(), v.ws.floc);
        }
    const bool direct = !slabs && L > 0;   // no ghost rows: the rows' sums are the forces
    for (int p0 = 0; p0 < P; p0 += kBatch) {
        const SmallBatch sb = small_batch(p0, U_LOCAL, -1);
        EnergySum es = energy_sum;
        if (p0 > 0) es.energy = nullptr;
        const int64_t force_blocks = (sb.start[sb.n] + 15) / 16 + (es.energy ? 1 : 0);
        if (L > 0 && force_blocks > 0)
            k_force_rows<<<grid8(force_blocks), 256, 0, s>>>(sb, pos, g->cell, direct ? forces : nullptr, atom_energy, es);
        else if (L == 0 && sb.start[sb.n] > 0)
            k_zero_floc<<<blocks_for(sb.start[sb.n], 256), 256, 0, s>>>(sb);
        MLIP_HIP(hipGetLastError());
    }
    if (L == 0) k_energy_total<<<1, 256, 0, s>>>(energy_sum);
    if (!direct) {   // owned rows to the caller's arrays; a border atom also collects what its ghost rows gathered elsewhere
        PtrTable tab{};
        for (int q = 0; q < P; ++q) tab.p[q] = views[q].ws.floc;
        for (int p0 = 0; p0 < P; p0 += kBatch) {
            const SmallBatch sb = small_batch(p0, U_OWNED, -1);
            if (sb.start[sb.n] > 0)
                k_store_owned<<<blocks_for(sb.start[sb.n], 256), 256, 0, s>>>(sb, tab, gidx, forces, atom_energy);
        }
    }
    MLIP_HIP(hipGetLastError());
    prof_end(g);
    return MLIP_OK;
}

}  // namespace

size_t table_bytes(int F, int L) { return kTabHeader + (size_t)L * tab_layer(F) * sizeof(float); }
static_assert(kStaticTableBytes == kTabHeader + (size_t)8 * tab_layer(64) * sizeof(float), "the largest model's tables");

int forward_impl(mlip_graph *g, const mlip_weights_t *w, int32_t mode, double *energy, float *forces, float *atom_energy,
                 Carver *scratch)
{
    if (w->F == 32) return forward_t<32>(g, w, nullptr, mode, energy, forces, atom_energy, scratch);
    return forward_t<64>(g, w, nullptr, mode, energy, forces, atom_energy, scratch);
}

int forward_bonds_impl(mlip_graph *g, const mlip_weights_t *w, const mlip_bond_weights_t *bw, int32_t mode,
                       double *energy, float *forces, float *atom_energy)
{
    if (w->F == 32) return forward_t<32>(g, w, bw, mode, energy, forces, atom_energy, nullptr);
    return forward_t<64>(g, w, bw, mode, energy, forces, atom_energy, nullptr);
}

}  // namespace mlip
