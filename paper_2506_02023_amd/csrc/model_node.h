// Node kernels (F x F products over atoms) and the small kernels: embedding, ghost transfers, forces, energy.
// Part of model.hip (one translation unit): included inside namespace mlip, anonymous namespace.
#ifndef MLIP_MODEL_NODE_H
#define MLIP_MODEL_NODE_H

// ---------------------------------------------------------------- node kernels

// One launch between two edge steps, over all atoms of all partitions: everything a row needs there is done while the row is
// in registers.
//   EMBED     h = Emb[z];  g_0 = h Wm_0
//   UPDATE    h += SiLU(a Wo);  g of the next layer = h Wm
//   TURN      the last layer's update, the readout and the first step back: h' = h + SiLU(q), q = a Wo;  x = h' Wr1;
//             eps = SiLU(x) . wr2;  hbar = (wr2 SiLU'(x)) Wr1^T;  abar = (hbar SiLU'(q)) Wo^T
//   BACK      hbar += gbar Wm^T;  q = a Wo of the layer before;  abar = (hbar SiLU'(q)) Wo^T
//   READ      a model without layers: eps of h = Emb[z] only
// A wavefront takes 32 rows.  Rows are loaded in the accumulator layout of the MFMAs (lane (c, h) holds features 8 i + 4 h + 0..3
// of row c), which is the layout of a product's other operand as well, so the products chain in registers with no transposition
// and no LDS but for the packed weights.  The next tile's rows are requested before this one's products.  Bound by memory at a
// million atoms, where the step takes 1.7 ms in them (2.3 ms in 13 launches of one fp32 MFMA product each and separate
// ghost copies, whose rows were read and written again in between), by the launches' own length below ten thousand:
// 61 us a step at 4,000 atoms against 134.
enum { OP_EMBED = 0, OP_UPDATE = 1, OP_TURN = 2, OP_BACK = 3, OP_READ = 4 };

struct NodeArgs {      // one partition
    int64_t n_rows;
    const float *X;    // a (UPDATE, TURN), gbar (BACK); EMBED and READ take the atoms' rows of the embedding table
    const float *X2;   // BACK: a of the layer before
    float *Z;          // h (EMBED: out, UPDATE: in and out, TURN: in); hbar (BACK: in and out)
    float *Y;          // g (EMBED, UPDATE); abar (TURN, BACK)
    float *hbar;       // TURN: out (or null); BACK: Z is written back unless null
    float *eps;        // TURN, READ
    double *tile_sum;  // TURN, READ: energy of every 32-row tile of this launch
    int64_t n_pure;    // border rows (n_pure .. n_rows) have ghost rows in other partitions
    const int32_t *nodes;
};

// What a border atom's owner needs to reach the atom's ghost rows in the other partitions: the partitions that
// hold it as a ghost (bits of needed_by) and its row in each of them (ghost_local, starting at gbase[atom]).
struct GhostIndex {
    const unsigned long long *needed_by;
    const int32_t *gbase, *ghost_local;
};
struct PtrTable { float *p[kMaxSlabs]; };

struct NodeBatch {     // up to kBatch partitions per launch, 32-row tiles numbered across them
    const float *P[4]; // packed weights, in the order of the products
    const float *wr2, *emb;
    const int32_t *species;
    int32_t *clear;    // EMBED: words to clear (the edge kernels' work counters)
    int n_clear;
    int n;
    int64_t tile_start[kBatch + 1];
    NodeArgs s[kBatch];
    GhostIndex ghosts;
    PtrTable tab;      // EMBED, UPDATE: the g arrays of all partitions; BACK: their gbar arrays (slab mode)
};

template <int OP> struct NodeOp {
    static constexpr int NPACK = OP == OP_EMBED ? 1 : OP == OP_UPDATE ? 2 : OP == OP_TURN ? 4 : OP == OP_BACK ? 3 : 1;
    static constexpr int NW = OP == OP_TURN ? 4 : 8;   // wavefronts per block (TURN needs more than 256 registers: 394 us against 520 with 8)
};

template <int F, int OP>
__global__ void __launch_bounds__(NodeOp<OP>::NW * 64) k_node(NodeBatch B)
{
    constexpr int NB = Dims<F>::NB, NP = NodeOp<OP>::NPACK, NW = NodeOp<OP>::NW, PACK = Dims<F>::PACK3;
    extern __shared__ float lds[];
    LdsFill<PACK / 4, NW * 64> fill[NP];   // all packs requested at once, and the first tile's rows with them
#pragma unroll
    for (int q = 0; q < NP; ++q) fill[q].load(B.P[q]);
    if (OP == OP_EMBED)
        for (int64_t i = (int64_t)blockIdx.x * (NW * 64) + threadIdx.x; i < B.n_clear; i += (int64_t)gridDim.x * (NW * 64)) B.clear[i] = 0;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int c32 = lane & 31, h4 = 4 * (lane >> 5);
    auto pack = [&](int q) { return reinterpret_cast<const __bf16 *>(lds + q * PACK); };
    auto load = [&](f32x16 (&v)[NB], const float *Y, int64_t row, bool ok) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                f32x4 x = {0.f, 0.f, 0.f, 0.f};
                if (ok) x = *reinterpret_cast<const f32x4 *>(Y + row * F + 32 * b + 8 * a + h4);
#pragma unroll
                for (int c = 0; c < 4; ++c) v[b][4 * a + c] = x[c];
            }
    };
    auto store = [&](const f32x16 (&v)[NB], float *Y, int64_t row, bool ok) {
        if (ok)
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int a = 0; a < 4; ++a)
                    *reinterpret_cast<f32x4 *>(Y + row * F + 32 * b + 8 * a + h4) =
                        f32x4{v[b][4 * a], v[b][4 * a + 1], v[b][4 * a + 2], v[b][4 * a + 3]};
    };
    const int64_t n_tiles = B.tile_start[B.n];
    const int64_t stride = (int64_t)gridDim.x * NW;
    int64_t ti = (int64_t)wave * gridDim.x + blockIdx.x;   // few tiles: one per block
    f32x16 x[NB], z[NB];   // X and Z rows of the tile at hand
    auto fetch = [&](int64_t t) {
        const int part = batch_find(B.tile_start, B.n, t);
        const NodeArgs &A = B.s[part];
        const int64_t row = (t - B.tile_start[part]) * 32 + c32;
        const bool ok = row < A.n_rows;
        if (OP == OP_EMBED || OP == OP_READ) {
            const float *e = B.emb;   // the caller's table: no alignment assumed
            if (ok) e += (int64_t)B.species[A.nodes ? A.nodes[row] : row] * F;
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int a = 0; a < 4; ++a)
#pragma unroll
                    for (int c = 0; c < 4; ++c) x[b][4 * a + c] = e[32 * b + 8 * a + h4 + c];
            return;
        }
        load(x, A.X, row, ok);
        if (OP == OP_UPDATE || OP == OP_TURN || OP == OP_BACK) load(z, A.Z, row, ok);
    };
    if (ti < n_tiles) fetch(ti);
#pragma unroll
    for (int q = 0; q < NP; ++q) fill[q].store(lds + q * PACK);
    __syncthreads();
    for (; ti < n_tiles; ti += stride) {
        const int part = batch_find(B.tile_start, B.n, ti);
        const NodeArgs &A = B.s[part];
        const int64_t row = (ti - B.tile_start[part]) * 32 + c32;
        const bool ok = row < A.n_rows;
        const bool border = ok && row >= A.n_pure;
        f32x16 y[NB];
        // rows of g also go to the atom's ghost rows in the other partitions (the border-node transfer)
        auto store_g = [&](const f32x16 (&v)[NB]) {
            store(v, A.Y, row, ok);
            if (border) {
                const int32_t u = A.nodes[row];
                unsigned long long nb = B.ghosts.needed_by[u];
                const int32_t *loc = B.ghosts.ghost_local + B.ghosts.gbase[u];
                while (nb) {
                    const int qq = __builtin_ctzll(nb);
                    nb &= nb - 1;
                    store(v, B.tab.p[qq], *loc++, true);
                }
            }
        };
        if (OP == OP_EMBED) {
            store(x, A.Z, row, ok);
            gemm_rl_bf16x3<F>(pack(0), x, y, lane);
            if (ti + stride < n_tiles) fetch(ti + stride);
            store_g(y);
        } else if (OP == OP_UPDATE) {
            f32x16 hn[NB];
            gemm_rl_bf16x3<F>(pack(0), x, y, lane);
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) hn[b][r] = z[b][r] + y[b][r] * sigmoidf_fast(y[b][r]);
            if (ti + stride < n_tiles) fetch(ti + stride);   // in flight during the second product
            store(hn, A.Z, row, ok);
            gemm_rl_bf16x3<F>(pack(1), hn, y, lane);
            store_g(y);
        } else if (OP == OP_TURN || OP == OP_READ) {
            f32x16 q[NB];
            if (OP == OP_TURN) {
                gemm_rl_bf16x3<F>(pack(0), x, q, lane);
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const float sg = sigmoidf_fast(q[b][r]);
                        z[b][r] = z[b][r] + q[b][r] * sg;
                        q[b][r] = sg * (1.0f + q[b][r] * (1.0f - sg));   // SiLU'(q)
                    }
                gemm_rl_bf16x3<F>(pack(1), z, y, lane);
            } else {
                gemm_rl_bf16x3<F>(pack(0), x, y, lane);
            }
            if (ti + stride < n_tiles) fetch(ti + stride);
            float part_eps = 0.f;
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int a = 0; a < 4; ++a)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const float wv = B.wr2[32 * b + 8 * a + h4 + c], v = c & 1 ? -y[b][4 * a + c] : y[b][4 * a + c];
                        const float sg = sigmoidf_fast(v);
                        part_eps += v * sg * wv;
                        y[b][4 * a + c] = wv * sg * (1.0f + v * (1.0f - sg));
                    }
            part_eps += __shfl_xor(part_eps, 32, 64);
            if (ok && h4 == 0) A.eps[row] = part_eps;
            double e = ok ? (double)part_eps : 0.0;   // the tile's energy, in a fixed order
#pragma unroll
            for (int off = 16; off > 0; off >>= 1) e += __shfl_xor(e, off, 64);
            if (lane == 0) A.tile_sum[ti - B.tile_start[part]] = e;
            if (OP == OP_TURN) {
                f32x16 hb[NB];
                gemm_rl_bf16x3<F>(pack(2), y, hb, lane);
                if (A.hbar) store(hb, A.hbar, row, ok);
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int r = 0; r < 16; ++r) hb[b][r] *= q[b][r];
                gemm_rl_bf16x3<F>(pack(3), hb, y, lane);
                store(y, A.Y, row, ok);
            }
        } else {   // OP_BACK
            f32x16 a2[NB];
            load(a2, A.X2, row, ok);
            if (border) {   // what the atom's ghost rows gathered comes back, in ascending partition order
                const int32_t u = A.nodes[row];
                unsigned long long nb = B.ghosts.needed_by[u];
                const int32_t *loc = B.ghosts.ghost_local + B.ghosts.gbase[u];
                while (nb) {
                    const int qq = __builtin_ctzll(nb);
                    nb &= nb - 1;
                    f32x16 gq[NB];
                    load(gq, B.tab.p[qq], *loc++, true);
#pragma unroll
                    for (int b = 0; b < NB; ++b) x[b] += gq[b];
                }
            }
            f32x16 hb[NB];
            gemm_rl_bf16x3<F>(pack(0), x, hb, lane);
#pragma unroll
            for (int b = 0; b < NB; ++b) hb[b] += z[b];
            if (ti + stride < n_tiles) fetch(ti + stride);
            if (A.hbar) store(hb, A.hbar, row, ok);
            gemm_rl_bf16x3<F>(pack(1), a2, y, lane);
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const float sg = sigmoidf_fast(y[b][r]);
                    hb[b][r] *= sg * (1.0f + y[b][r] * (1.0f - sg));
                }
            gemm_rl_bf16x3<F>(pack(2), hb, y, lane);
            store(y, A.Y, row, ok);
        }
    }
}

// ---------------------------------------------------------------- small kernels
//
// Embedding, ghost transfers, force assembly and the energy partial sums run over all partitions in one launch
// (up to kBatch partitions per launch, like the edge and node kernels): items are numbered across the
// partitions, start[q] is the first item of partition q.

struct SmallArgs {   // one partition
    int64_t n_owned, n_pure, n_local;
    const int32_t *nodes;          // local -> global (nullptr: identity)
    const int64_t *row_ptr;
    const int32_t *senders, *mirror;
    const uint32_t *shiftp;
    float *gbar, *abar, *floc, *eps;
    // upper / lower split of the owned rows' edges
    const int32_t *uslot;          // [E_owned] upper edges: their index in the upper-edge graph, where their filter values are kept
    const int64_t *l_row_ptr;      // the owned rows' lower edges: CSR, sender row, where the pair's filter values are kept
    const int32_t *l_senders, *l_slot;
    const float *dsum, *wstore, *d;
    const int32_t *bond_of_edge;   // three-body variant (or nullptr): bond of an edge
    const void *wb;                // bond filter rows of the layer: fp32, or bf16 if wb_bf16
    int wb_bf16;
};

struct SmallBatch {
    int n;
    int tables;            // whether the edge steps run on tables; if not, the filter values are kept, edge by edge
    int bonds;             // whether a partition has bonds
    const int32_t *gate;   // != null: not known when this is launched, *gate == 0 says that they did
    __device__ bool on_tables() const { return gate ? *gate == 0 : tables != 0; }
    int64_t start[kBatch + 1];
    SmallArgs s[kBatch];
};

// ghost rows of abar are zero (ghost rows carry no dE/da); blockIdx.y: the layer, where every layer's abar is kept
__global__ void k_zero_ghost_rows(SmallBatch B, int F)
{
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int F4 = F / 4;
    const int64_t gk = idx / F4;
    if (gk >= B.start[B.n]) return;
    const int part = batch_find(B.start, B.n, gk);
    const SmallArgs &A = B.s[part];
    const int64_t k = gk - B.start[part];
    *reinterpret_cast<f32x4 *>(A.abar + ((int64_t)blockIdx.y * A.n_local + A.n_owned + k) * F + (idx % F4) * 4) = f32x4{0.f, 0.f, 0.f, 0.f};
}

// Second pass of the reverse edge step: the lower edges' terms of the row sums, with the filter values w read from the
// row of the edge's pair, which the forward kernel kept: gbar_i += sum over the lower edges e = (i <- j) of row i of
// w * abar_j.  One wavefront per row, lane = feature; the lower edges of 64 edges at a time are taken kLowerChunk at a
// time, all their rows in flight together.  Bound by the kept rows' bytes: 1.21 ms at a million atoms for 5.9 GB of them, 8.0 GB
// with the gathered rows as measured, 6.6 TB/s (a large copy reaches 4.67 TB/s on this card, a large read 6 to 7).
constexpr int kLowerChunk = 16;   // lower edges whose rows are in flight together (32 measured no faster)

template <int F>
__global__ void __launch_bounds__(256) k_edge_lower(SmallBatch B)
{
    if (B.on_tables()) return;   // the reverse step has the lower edges already
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t gk = (int64_t)blockIdx.x * 4 + wave;
    if (gk >= B.start[B.n]) return;
    const int part = batch_find(B.start, B.n, gk);
    const SmallArgs &A = B.s[part];
    const int64_t r = gk - B.start[part];
    const unsigned f = lane & (F - 1);
    // the row's lower edges (wave-uniform, kept scalar; edge indices fit 32 bits)
    const int64_t e0 = __builtin_amdgcn_readfirstlane((int32_t)A.l_row_ptr[r]);
    const int64_t e1 = __builtin_amdgcn_readfirstlane((int32_t)A.l_row_ptr[r + 1]);
    const float before = A.gbar[r * F + f];   // (requested with the indices)
    float acc = 0.f;
    for (int64_t eb = e0; eb < e1; eb += 64) {
        const int n = (int)min((int64_t)64, e1 - eb);
        const int64_t el = min(eb + lane, e1 - 1);
        const int32_t jl = A.l_senders[el];
        const int32_t sl = A.l_slot[el];   // where the pair's filter values are kept
        for (int c = 0; c < n; c += kLowerChunk) {
            float wv[kLowerChunk], gv[kLowerChunk];
#pragma unroll
            for (int t = 0; t < kLowerChunk; ++t) {
                wv[t] = gv[t] = 0.f;
                if (c + t < n) {   // wave-uniform: no load is issued for an edge that is not there
                    const int64_t j = __builtin_amdgcn_readlane(jl, c + t), m = __builtin_amdgcn_readlane(sl, c + t);
                    wv[t] = __builtin_nontemporal_load(A.wstore + m * F + f);
                    gv[t] = A.abar[j * F + f];
                }
            }
#pragma unroll
            for (int t = 0; t < kLowerChunk; ++t) acc = fmaf(wv[t], gv[t], acc);
        }
    }
    if (F == 64 || lane < F) A.gbar[r * F + f] = before + acc;
}

// gbar of the ghost rows: gbar_i = sum over the ghost's sub-row (its neighbours owned by this partition) of
// w_e * abar_send(e).  w_e is the reverse edge's, which the forward pass kept (both edges of a pair have the
// same length, hence the same filter value).  One wavefront per row, lane = feature, edges in row order.
template <int F>
__global__ void __launch_bounds__(256) k_ghost_gbar(SmallBatch B)
{
    const bool kept = !B.on_tables();
    if (!kept && !B.bonds) return;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t gk = (int64_t)blockIdx.x * 4 + wave;
    if (gk >= B.start[B.n]) return;
    const int part = batch_find(B.start, B.n, gk);
    const SmallArgs &A = B.s[part];
    const int64_t r = A.n_owned + (gk - B.start[part]);
    const unsigned f = lane & (F - 1);
    if (!kept && !A.bond_of_edge) return;
    const int64_t e0 = A.row_ptr[r], e1 = A.row_ptr[r + 1];
    float acc = kept ? 0.f : A.gbar[r * F + f];   // on tables the reverse step has summed the edges' terms: the bonds' are added
    for (int64_t eb = e0; eb < e1; eb += 16) {   // 16 edges at a time: ids by lane, then all rows in flight together
        const int n = (int)min((int64_t)16, e1 - eb);
        const int64_t el = min(eb + (lane & 15), e1 - 1);
        const int32_t jl = A.senders[el], ml = A.mirror[el];
        const int32_t bl = A.bond_of_edge ? A.bond_of_edge[ml] : -1;   // three-body variant: the reverse edge's bond
        const int32_t sl = kept ? A.uslot[ml] : 0;   // where the reverse edge (an upper one: its sender is a ghost) keeps its filter values
        float wv[16], av[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int64_t j = __builtin_amdgcn_readlane(jl, k), m = __builtin_amdgcn_readlane(sl, k);
            const int64_t b = __builtin_amdgcn_readlane(bl, k);
            wv[k] = kept ? A.wstore[m * F + f] : 0.f;
            if (b >= 0)
                wv[k] += A.wb_bf16 ? Elem<__bf16>::load(static_cast<const __bf16 *>(A.wb) + b * F + f)
                                   : static_cast<const float *>(A.wb)[b * F + f];
            av[k] = A.abar[j * F + f];
        }
#pragma unroll
        for (int k = 0; k < 16; ++k)
            if (k < n) acc = fmaf(wv[k], av[k], acc);
    }
    if (F == 64 || lane < F) A.gbar[r * F + f] = acc;
}

__device__ inline void unpack_shift(uint32_t p, int &a, int &b, int &c)
{
    a = (int)(p >> 20) - 512;
    b = (int)((p >> 10) & 1023u) - 512;
    c = (int)(p & 1023u) - 512;
}

// total energy: the tiles' fp64 sums in a fixed order, by one block
__device__ inline void energy_total(int64_t n, const double *__restrict__ part, double *__restrict__ energy)
{
    __shared__ double sh[4];
    double s = 0;
    for (int64_t k = threadIdx.x; k < n; k += 256) s += part[k];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) *energy = (sh[0] + sh[1]) + (sh[2] + sh[3]);
}

struct EnergySum { int64_t n; const double *part; double *energy; };   // energy == nullptr: not in this launch

// F_loc[r] = sum_{e in local row r} dsum_e * rhat_e (plus the bond part's F_loc, if any), edge vectors from fp64 positions;
// 16 lanes per row, 16 rows per block.  Without ghost rows a row's sum is the atom's force and goes to the caller's arrays
// (forces != nullptr), the atom's energy with it.  The block behind those of the rows adds up the energy.
__global__ void __launch_bounds__(256)
k_force_rows(SmallBatch B, const double *__restrict__ pos, CellParams cp, float *__restrict__ forces,
             float *__restrict__ atom_energy, EnergySum E)
{
    const int64_t block = xcd_block();   // neighbouring rows gather the same atoms and, on tables, one another's sums
    if (block * 16 >= B.start[B.n]) {
        if (E.energy && block * 16 < B.start[B.n] + 16) energy_total(E.n, E.part, E.energy);
        return;
    }
    const int64_t gr = block * 16 + (threadIdx.x >> 4);
    if (gr >= B.start[B.n]) return;   // whole groups of 16 lanes leave together; the shuffles below stay inside a group
    const int part = batch_find(B.start, B.n, gr);
    const SmallArgs &A = B.s[part];
    const int64_t r = gr - B.start[part];
    const int32_t *nodes = A.nodes;
    const int64_t ig = nodes ? nodes[r] : r;
    const double xi = pos[3 * ig], yi = pos[3 * ig + 1], zi = pos[3 * ig + 2];
    double fx = 0, fy = 0, fz = 0;
    const int64_t e1 = A.row_ptr[r + 1];
    const bool tables = B.on_tables();
    for (int64_t e = A.row_ptr[r] + (threadIdx.x & 15); e < e1; e += 16) {
        const int64_t jl = A.senders[e];
        const int64_t jg = nodes ? nodes[jl] : jl;
        int S0, S1, S2;
        unpack_shift(A.shiftp[e], S0, S1, S2);
        const double t0 = (pos[3 * jg] - xi) + (((double)S0 * cp.C[0] + (double)S1 * cp.C[3]) + (double)S2 * cp.C[6]);
        const double t1 = (pos[3 * jg + 1] - yi) + (((double)S0 * cp.C[1] + (double)S1 * cp.C[4]) + (double)S2 * cp.C[7]);
        const double t2 = (pos[3 * jg + 2] - zi) + (((double)S0 * cp.C[2] + (double)S1 * cp.C[5]) + (double)S2 * cp.C[8]);
        // dE/dd times the unit vector: the edge's stored length (the fp64 length rounded once to fp32) is accurate
        // to 6e-8, far inside the force bound, and spares an fp64 square root and division per edge
        float dd = A.dsum[e];
        if (tables) dd += A.dsum[A.mirror[e]];   // an edge holds the share in which its receiver's row of g took part: the reverse edge has the other one
        const double s = (double)(dd * __builtin_amdgcn_rcpf(A.d[e]));
        fx += s * t0;
        fy += s * t1;
        fz += s * t2;
    }
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) {
        fx += __shfl_xor(fx, off, 64);
        fy += __shfl_xor(fy, off, 64);
        fz += __shfl_xor(fz, off, 64);
    }
    if ((threadIdx.x & 15) == 0) {
        float *fl = A.floc + 3 * r;
        float x = (float)fx, y = (float)fy, z = (float)fz;
        if (A.bond_of_edge) {   // three-body variant: the bonds' part is there already
            x += fl[0];
            y += fl[1];
            z += fl[2];
        }
        float *to = forces ? forces + 3 * ig : fl;
        to[0] = x;
        to[1] = y;
        to[2] = z;
        if (forces && atom_energy) atom_energy[ig] = A.eps[r];
    }
}

__global__ void k_zero_floc(SmallBatch B)
{
    const int64_t gr = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gr >= B.start[B.n]) return;
    const int part = batch_find(B.start, B.n, gr);
    const int64_t r = gr - B.start[part];
    float *f = B.s[part].floc + 3 * r;
    f[0] = 0.f;
    f[1] = 0.f;
    f[2] = 0.f;
}

// owned rows: forces[global] = F_loc (+ for a border atom, in ascending partition order, the position gradients its
// ghost rows collected in the other partitions: gathered by the owner, one writer per atom); atom_energy[global] = eps
// (tab: the floc arrays of all partitions)
__global__ void k_store_owned(SmallBatch B, PtrTable tab, GhostIndex G, float *__restrict__ forces,
                              float *__restrict__ atom_energy)
{
    const int64_t gr = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gr >= B.start[B.n]) return;
    const int part = batch_find(B.start, B.n, gr);
    const SmallArgs &A = B.s[part];
    const int64_t r = gr - B.start[part];
    const int64_t u = A.nodes ? A.nodes[r] : r;
    float fx = A.floc[3 * r], fy = A.floc[3 * r + 1], fz = A.floc[3 * r + 2];
    if (r >= A.n_pure) {
        unsigned long long nb = G.needed_by[u];
        const int32_t *loc = G.ghost_local + G.gbase[u];
        while (nb) {
            const int qq = __builtin_ctzll(nb);
            nb &= nb - 1;
            const float *fg = tab.p[qq] + 3 * (int64_t)(*loc++);
            fx += fg[0];
            fy += fg[1];
            fz += fg[2];
        }
    }
    forces[3 * u] = fx;
    forces[3 * u + 1] = fy;
    forces[3 * u + 2] = fz;
    if (atom_energy) atom_energy[u] = A.eps[r];
}

__global__ void __launch_bounds__(256) k_energy_total(EnergySum E) { energy_total(E.n, E.part, E.energy); }

#endif  // MLIP_MODEL_NODE_H
