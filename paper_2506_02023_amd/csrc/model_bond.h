// Kernels of the three-body (bond graph) variant.
// Part of model.hip (one translation unit): included inside namespace mlip, anonymous namespace.
#ifndef MLIP_MODEL_BOND_H
#define MLIP_MODEL_BOND_H

// ---------------------------------------------------------------- three-body (bond graph) kernels
//
// Benchmark configuration 4: bonds are the atom-graph edges within a smaller cutoff, two bonds interact when
// they share their centre atom (the paper's bond graph, Methods, "Distributing Bond Graphs").  All bonds of a
// centre are contiguous, so every kernel below works on one centre (or one bond) per wavefront with lane =
// feature and needs no atomics.  Notation: P_b = e0_b Wta, Q_b = e0_b Wtb, Wtc = rows 2F.. of Wt1,
//   h(b1, b2) = P_b1 + Q_b2 + T(c) Wtc,  S_b1 = sum_{b2 != b1} u_b2 SiLU(h),  m = S Wt2,  e1 = e0 + u SiLU(m).

//
// BT is the element type of the [bonds x F] arrays (P, Q, S, m, wb, e1bar, Sbar, Pbar, Qbar): float, or __bf16 in the
// bf16 precision mode, where these arrays are most of the bytes the bond kernels move.  Arithmetic is fp32 either way.

constexpr int kAngle = 8;

__device__ inline float silu_f(float x) { return x * __builtin_amdgcn_rcpf(1.0f + __expf(-x)); }
__device__ inline void silu_both(float x, float &s, float &ds)
{
    const float sg = __builtin_amdgcn_rcpf(1.0f + __expf(-x));
    s = x * sg;
    ds = fmaf(s, 1.0f - sg, sg);
}

// value of lane k (wave-uniform k) of a float register, as a wave-uniform value
__device__ inline float readlane_f32(float v, int k)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), k));
}

// T_n(c) = cos(n theta), dT_n/dc = n U_{n-1}(c), n = 0..7
__device__ inline void chebyshev(float c, float (&T)[kAngle], float (&dT)[kAngle])
{
    T[0] = 1.f; dT[0] = 0.f;
    T[1] = c;   dT[1] = 1.f;
    float Um = 1.f, Un = 2.f * c;   // U_0, U_1
#pragma unroll
    for (int n = 2; n < kAngle; ++n) {
        T[n] = 2.f * c * T[n - 1] - T[n - 2];
        dT[n] = (float)n * Un;
        const float Ux = 2.f * c * Un - Um;
        Um = Un;
        Un = Ux;
    }
}

// ---- angle terms of a centre's pairs of bonds on the matrix units
//
// Centres with at most kPairRegs bonds (12 on the benchmark's lattice) are processed by unordered pairs {a, o}, a < o, lane =
// feature, everything in registers: the bonds' rows and accumulators as arrays indexed by bond, the loops over a and o unrolled.
// T(c) Wtc (and dT/dc Wtc) of the pairs of two bonds a come from one tile of 32: pair (2 k, o) is row o, pair (2 k + 1, o) row
// 16 + o, the rows' cosines and Chebyshev values worked out with lane = pair.  With the pairs as the product's rows and
// the features as its columns a lane of the result holds one feature of half the pairs, and exchanging the halves
// of two result blocks leaves lane = feature with one register per pair: no LDS and no broadcast.
constexpr int kPairRegs = 16;

// T_n(c) = cos(n theta) or, DERIV, dT_n/dc = n U_{n-1}(c) as operands of the K = 8 product: lane half h takes n = 2 t + h,
// t = 0..3.   T_{n+2} = 2 T_2 T_n - T_{n-2}, the same for U
template <bool DERIV> __device__ inline Basis3 angle_operands(float c, int h)
{
    const float t2 = fmaf(2.0f * c, c, -1.0f), k2 = 2.0f * t2;
    float v[4];
    v[0] = DERIV ? (h ? 1.0f : 0.0f) : (h ? c : 1.0f);
    v[1] = DERIV ? (h ? k2 + 1.0f : 2.0f * c) : (h ? c * (k2 - 1.0f) : t2);
    v[2] = fmaf(k2, v[1], -v[0]);
    v[3] = fmaf(k2, v[2], -v[1]);
    if (DERIV)
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] *= (float)(2 * t) + (h ? 1.0f : 0.0f);
    return basis_operands(v);
}

template <int F> struct AngleWeights {   // Wtc packed as PACK_W1, per 32 features the three operands of gemm_k8_block
    bf16x8 hl[Dims<F>::NB], mm[Dims<F>::NB], hh[Dims<F>::NB];
    __device__ explicit AngleWeights(const float *__restrict__ pack, int lane)
    {
#pragma unroll
        for (int bo = 0; bo < Dims<F>::NB; ++bo) {
            const bf16x4 *A = reinterpret_cast<const bf16x4 *>(pack) + (bo * 3) * 64 + lane;
            const bf16x4 h = A[0], m = A[64], l = A[128];
            hl[bo] = __builtin_shufflevector(h, l, 0, 1, 2, 3, 4, 5, 6, 7);
            mm[bo] = __builtin_shufflevector(m, m, 0, 1, 2, 3, 4, 5, 6, 7);
            hh[bo] = __builtin_shufflevector(h, h, 0, 1, 2, 3, 4, 5, 6, 7);
        }
    }
    // one block of 32 features; PAIRS: the pairs are the result's rows and the features its columns (lanes), else the reverse
    template <bool PAIRS> __device__ f32x16 block(const Basis3 &v, int bo) const
    {
        f32x16 d;
#pragma unroll
        for (int r = 0; r < 16; ++r) d[r] = 0.f;
        d = PAIRS ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(v.lh, hl[bo], d, 0, 0, 0) : __builtin_amdgcn_mfma_f32_32x32x16_bf16(hl[bo], v.lh, d, 0, 0, 0);
        d = PAIRS ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(v.hm, mm[bo], d, 0, 0, 0) : __builtin_amdgcn_mfma_f32_32x32x16_bf16(mm[bo], v.hm, d, 0, 0, 0);
        return PAIRS ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(v.hm, hh[bo], d, 0, 0, 0) : __builtin_amdgcn_mfma_f32_32x32x16_bf16(hh[bo], v.hm, d, 0, 0, 0);
    }
    // out[p]: this lane's feature of row p's product (F = 32: both halves of the wavefront hold all features)
    __device__ void rows(const Basis3 &v, float (&out)[32]) const
    {
        constexpr int NB = Dims<F>::NB;
        f32x16 d[NB];
#pragma unroll
        for (int bo = 0; bo < NB; ++bo) d[bo] = block<true>(v, bo);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            // register r of half h holds row 8 (r / 4) + 4 h + r % 4; the upper half of block 0 and the lower half of the last
            // block change places
            const float lo = d[0][r], up = d[NB - 1][r];   // (a bit cast of a vector's element takes element 0)
            const unsigned x = __builtin_bit_cast(unsigned, lo), y = __builtin_bit_cast(unsigned, up);
            const auto sw = __builtin_amdgcn_permlane32_swap(x, y, false, false);
            out[8 * (r / 4) + (r & 3)] = __builtin_bit_cast(float, (unsigned)sw[0]);
            out[8 * (r / 4) + 4 + (r & 3)] = __builtin_bit_cast(float, (unsigned)sw[1]);
        }
    }
};

// cosines of tile k's pairs: lane (p, h) has pair (2 k + p / 16, p % 16); x, y, z: lane = bond (mod 16)
__device__ inline float pair_cosine(int k, int lane, float x, float y, float z)
{
    const int a = 2 * k + ((lane >> 4) & 1);
    return fmaf(__shfl(x, a, 64), x, fmaf(__shfl(y, a, 64), y, __shfl(z, a, 64) * z));
}

// S[b1][f] = sum_{b2 != b1, same centre} u[b2] SiLU(P[b1][f] + Q[b2][f] + sum_n T_n(c) Wtc[n][f])
// One wavefront per centre, lane = feature.  Bound by the vector unit: two SiLUs of two transcendentals each per pair and
// feature.  13.4 M pairs, fp32: 1566 us with vector angle terms, lane broadcasts and LDS accumulators, 687 us here; a branch
// per pair instead of one per four bonds took 1681 us (the chains of transcendentals had nothing to overlap with).
// Any number of bonds: ordered pairs, the angle basis of 64 bonds b2 at a time (lane = b2) handed to the feature lanes through
// wave-uniform registers.
template <int F, typename BT>
__device__ inline void triplet_fwd_any(int64_t b0, int64_t b1e, int lane, const float *__restrict__ rhat, const float *__restrict__ u,
                                       const BT *__restrict__ P, const BT *__restrict__ Q, const float *__restrict__ Wtc,
                                       BT *__restrict__ S)
{
    using IO = Elem<BT>;
    const int f = lane & (F - 1);
    float wc[kAngle];
#pragma unroll
    for (int n = 0; n < kAngle; ++n) wc[n] = Wtc[n * F + f];
    for (int64_t c0 = b0; c0 < b1e; c0 += 64) {   // bonds b2 in groups of 64 (one group unless the centre has more)
        const int nl = (int)min((int64_t)64, b1e - c0);
        const int64_t bl = min(c0 + lane, b1e - 1);
        const float xl = rhat[3 * bl], yl = rhat[3 * bl + 1], zl = rhat[3 * bl + 2], ul = u[bl];
        for (int64_t b1 = b0; b1 < b1e; ++b1) {
            const float p1 = IO::load(P + b1 * F + f);
            const float x1 = rhat[3 * b1], y1 = rhat[3 * b1 + 1], z1 = rhat[3 * b1 + 2];
            float T[kAngle], dT[kAngle];
            chebyshev(fmaf(x1, xl, fmaf(y1, yl, z1 * zl)), T, dT);   // lane = b2
            float acc = 0.f;
            for (int k = 0; k < nl; ++k) {
                if (c0 + k == b1) continue;
                float h = p1 + IO::load(Q + (c0 + k) * F + f);
#pragma unroll
                for (int n = 1; n < kAngle; ++n) h = fmaf(readlane_f32(T[n], k), wc[n], h);   // T_0 = 1
                acc = fmaf(readlane_f32(ul, k), silu_f(h + wc[0]), acc);
            }
            if (F == 64 || lane < F) {
                BT *sp = S + b1 * F + f;
                IO::store(sp, (c0 == b0) ? acc : IO::load(sp) + acc);
            }
        }
    }
}

// 17 to kPairBondsFwd bonds: unordered pairs as well, T(c) Wtc from wave-uniform registers, bond a's sum in a register and bond
// o's in a per-lane LDS row (accS, kPairBondsFwd rows of 64).
constexpr int kPairBondsFwd = 32;
template <int F, typename BT>
__device__ inline void triplet_fwd_lds(int nb, int64_t b0, int64_t b1e, int lane, float *accS, const float *__restrict__ rhat,
                                       const float *__restrict__ u, const BT *__restrict__ P, const BT *__restrict__ Q,
                                       const float *__restrict__ Wtc, BT *__restrict__ S)
{
    using IO = Elem<BT>;
    const int f = lane & (F - 1);
    float wc[kAngle];
#pragma unroll
    for (int n = 0; n < kAngle; ++n) wc[n] = Wtc[n * F + f];
    for (int b = 0; b < nb; ++b) accS[b * 64 + lane] = 0.f;
    const int64_t bl = min(b0 + lane, b1e - 1);
    const float xl = rhat[3 * bl], yl = rhat[3 * bl + 1], zl = rhat[3 * bl + 2], ul = u[bl];   // lane = bond
    for (int a = 0; a < nb; ++a) {
        const int64_t ba = b0 + a;
        const float pa = IO::load(P + ba * F + f), qa = IO::load(Q + ba * F + f);
        const float ua = readlane_f32(ul, a);
        float T[kAngle], dT[kAngle];
        chebyshev(fmaf(readlane_f32(xl, a), xl, fmaf(readlane_f32(yl, a), yl, readlane_f32(zl, a) * zl)), T, dT);   // lane = o
        float acc = 0.f;
        for (int o = a + 1; o < nb; ++o) {
            float tw = wc[0];   // T_0 = 1
#pragma unroll
            for (int n = 1; n < kAngle; ++n) tw = fmaf(readlane_f32(T[n], o), wc[n], tw);
            const float po = IO::load(P + (b0 + o) * F + f), qo = IO::load(Q + (b0 + o) * F + f);
            const float so = accS[o * 64 + lane];   // per-lane slot (read early, written at the end of the step;
                                                    // LDS float atomics measured an order of magnitude slower)
            acc = fmaf(readlane_f32(ul, o), silu_f(pa + qo + tw), acc);       // triplet (b1 = a, b2 = o)
            accS[o * 64 + lane] = fmaf(ua, silu_f(po + qa + tw), so);        // triplet (b1 = o, b2 = a)
        }
        accS[a * 64 + lane] += acc;
    }
    wave_lds_fence();
    if (F == 64 || lane < F)
        for (int b = 0; b < nb; ++b) IO::store(S + (b0 + b) * F + f, accS[b * 64 + lane]);
}

template <int F, typename BT>
__device__ inline void triplet_fwd_regs(int n, int64_t b0, int lane, const float *__restrict__ rhat, const float *__restrict__ u,
                                        const BT *__restrict__ P, const BT *__restrict__ Q, const float *__restrict__ WtcP,
                                        BT *__restrict__ S)
{
    using IO = Elem<BT>;
    constexpr int NR = kPairRegs;
    const int f = lane & (F - 1);
    const AngleWeights<F> W(WtcP, lane);
    const int64_t bl = b0 + min(lane & (NR - 1), n - 1);
    const float xl = rhat[3 * bl], yl = rhat[3 * bl + 1], zl = rhat[3 * bl + 2];   // lane = bond (mod 16)
    const float ul = (lane & (NR - 1)) < n ? u[bl] : 0.f;
    float Pr[NR], Qr[NR], Sr[NR];
#pragma unroll
    for (int o = 0; o < NR; ++o) {
        Pr[o] = Qr[o] = Sr[o] = 0.f;
        if (o < n) {
            Pr[o] = IO::load(P + (b0 + o) * F + f);
            Qr[o] = IO::load(Q + (b0 + o) * F + f);
        }
    }
#pragma unroll
    for (int k = 0; k < NR / 2; ++k) {
        if (2 * k + 1 >= n) break;
        float tw[32];
        W.rows(angle_operands<false>(pair_cosine(k, lane, xl, yl, zl), lane >> 5), tw);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int a = 2 * k + q;
            const float ua = readlane_f32(ul, a);
#pragma unroll
            for (int g = 0; g < NR; g += 4)   // bonds from n on have u = 0, their own sums are not stored
                if (g + 3 > a && g < n)
#pragma unroll
                    for (int o = g; o < g + 4; ++o)
                        if (o > a) {
                            const float t = tw[16 * q + o];
                            Sr[a] = fmaf(readlane_f32(ul, o), silu_f(Pr[a] + Qr[o] + t), Sr[a]);   // triplet (b1 = a, b2 = o)
                            Sr[o] = fmaf(ua, silu_f(Pr[o] + Qr[a] + t), Sr[o]);                    // triplet (b1 = o, b2 = a)
                        }
        }
    }
    if (F == 64 || lane < F)
#pragma unroll
        for (int o = 0; o < NR; ++o)
            if (o < n) IO::store(S + (b0 + o) * F + f, Sr[o]);
}

template <int F, typename BT>
__global__ void __launch_bounds__(256, 4)
k_triplet_fwd(int64_t N, const int64_t *__restrict__ bptr, const float *__restrict__ rhat, const float *__restrict__ u,
              const BT *__restrict__ P, const BT *__restrict__ Q, const float *__restrict__ Wtc, const float *__restrict__ WtcP,
              BT *__restrict__ S)
{
    __shared__ float acc_lds[4][kPairBondsFwd * 64];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t i = (int64_t)blockIdx.x * 4 + wave;
    if (i >= N) return;
    const int64_t b0 = bptr[i], b1e = bptr[i + 1];
    const int nb = __builtin_amdgcn_readfirstlane((int)(b1e - b0));
    if (nb <= 0) return;
    if (nb <= kPairRegs) {
        triplet_fwd_regs<F, BT>(nb, b0, lane, rhat, u, P, Q, WtcP, S);
        return;
    }
    if (nb <= kPairBondsFwd) triplet_fwd_lds<F, BT>(nb, b0, b1e, lane, acc_lds[wave], rhat, u, P, Q, Wtc, S);
    else triplet_fwd_any<F, BT>(b0, b1e, lane, rhat, u, P, Q, Wtc, S);
}

// Bond terms of a layer's rows, of up to kBatch partitions: out_i += sum over the bonds b = (i <- j) of wb[m_b] * from_j, forward m_b = b, from g
// and out a; reverse m_b the reverse bond (j <- i), whose filter multiplies g_i in row j, from abar and out gbar (no term if the sender is a
// ghost row: abar_j = 0, its owner adds that one).  One wavefront per centre, a row for F / 4 lanes of 16 bytes (8 in bf16), 16 bonds' rows in
// flight together whose places the lanes look up for themselves.  Bound by the bond rows (2.4 M bonds, 622 MB:
// 164 us per layer; 214 forward and 246 reverse with lane = feature, rows looked up one after another).
struct BondSumArgs {
    const int64_t *ptr;
    const int32_t *sender, *mirror;   // mirror == nullptr: forward
    const void *wb;
    const float *from;
    float *out;
};
struct BondSumBatch {
    int n;
    int64_t start[kBatch + 1];
    BondSumArgs s[kBatch];
};
template <int F, typename BT> __global__ void __launch_bounds__(256) k_bond_sum(BondSumBatch B)
{
    constexpr int kLanes = F / 4, kRows = 64 / kLanes, kTurns = 16 / kRows;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t gi = (int64_t)xcd_block() * 4 + wave;
    if (gi >= B.start[B.n]) return;
    const int part = batch_find(B.start, B.n, gi);
    const BondSumArgs &A = B.s[part];
    if (!A.ptr) return;   // (no bonds)
    const int64_t i = gi - B.start[part];
    const int sub = lane / kLanes, f = 4 * (lane % kLanes);
    const int64_t b0 = A.ptr[i], b1 = A.ptr[i + 1];
    if (b0 >= b1) return;
    float *out = A.out + i * F + f;
    const f32x4 before = *reinterpret_cast<const f32x4 *>(out);   // (requested with the indices)
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    for (int64_t bb = b0; bb < b1; bb += 16) {
        int64_t m[kTurns], j[kTurns];
#pragma unroll
        for (int t = 0; t < kTurns; ++t) {
            const int64_t b = bb + t * kRows + sub;
            m[t] = b < b1 ? (A.mirror ? (int64_t)A.mirror[b] : b) : -1;
            j[t] = A.sender[min(b, b1 - 1)];
        }
        f32x4 w[kTurns], x[kTurns];
#pragma unroll
        for (int t = 0; t < kTurns; ++t) {
            w[t] = x[t] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (m[t] >= 0) {
                w[t] = Elem<BT>::load4(static_cast<const BT *>(A.wb) + m[t] * F + f);
                x[t] = *reinterpret_cast<const f32x4 *>(A.from + j[t] * F + f);
            }
        }
#pragma unroll
        for (int t = 0; t < kTurns; ++t)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[c] = fmaf(w[t][c], x[t][c], acc[c]);
    }
#pragma unroll
    for (int off = kLanes; off < 64; off *= 2)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] += __shfl_xor(acc[c], off, 64);
    if (lane < kLanes) *reinterpret_cast<f32x4 *>(out) = before + acc;
}

// Reverse of k_triplet_fwd for one centre, any number of bonds, no LDS.  Pbar[b1] and rbar[b1] accumulate over the
// inner loop in registers; Qbar[b2], ubar[b2] and rbar[b2] are indexed by the inner bond, so they are accumulated
// in a second sweep with the roles of the loops exchanged (h is recomputed there): every triplet is evaluated twice.
template <int F, typename BT>
__device__ inline void
triplet_bwd_sweep(int64_t i, int lane, const int64_t *__restrict__ bptr, const float *__restrict__ rhat,
                  const float *__restrict__ u, const BT *__restrict__ P, const BT *__restrict__ Q,
                  const float *__restrict__ Wtc, const BT *__restrict__ Sbar, BT *__restrict__ Pbar,
                  BT *__restrict__ Qbar, float *__restrict__ ubar, float *__restrict__ rbar)
{
    using IO = Elem<BT>;
    const int f = lane & (F - 1);
    const bool on = (F == 64 || lane < F);
    float wc[kAngle];
#pragma unroll
    for (int n = 0; n < kAngle; ++n) wc[n] = Wtc[n * F + f];
    const int64_t b0 = bptr[i], be = bptr[i + 1];
    for (int64_t ba = b0; ba < be; ++ba) {
        const float xa = rhat[3 * ba], ya = rhat[3 * ba + 1], za = rhat[3 * ba + 2];
        const float pa = IO::load(P + ba * F + f), qa = IO::load(Q + ba * F + f), sa = IO::load(Sbar + ba * F + f), ua = u[ba];
        float pbar = 0.f, qbar = 0.f, ub = 0.f, rx = 0.f, ry = 0.f, rz = 0.f;
        for (int64_t bo = b0; bo < be; ++bo) {
            if (bo == ba) continue;
            const float xo = rhat[3 * bo], yo = rhat[3 * bo + 1], zo = rhat[3 * bo + 2];
            const float c = fmaf(xa, xo, fmaf(ya, yo, za * zo));
            float T[kAngle], dT[kAngle];
            chebyshev(c, T, dT);
            float tw = 0.f, dw = 0.f;   // T(c) Wtc and dT(c)/dc Wtc for this lane's feature
#pragma unroll
            for (int n = 0; n < kAngle; ++n) {
                tw = fmaf(T[n], wc[n], tw);
                dw = fmaf(dT[n], wc[n], dw);
            }
            // triplet (b1 = ba, b2 = bo): contributes to Pbar[ba] and, through c, to rbar[ba]
            float s1, ds1;
            silu_both(pa + IO::load(Q + bo * F + f) + tw, s1, ds1);
            const float h1 = sa * u[bo] * ds1;
            pbar += h1;
            // triplet (b1 = bo, b2 = ba): contributes to Qbar[ba], ubar[ba] and, through c, to rbar[ba]
            float s2, ds2;
            const float so = IO::load(Sbar + bo * F + f);
            silu_both(IO::load(P + bo * F + f) + qa + tw, s2, ds2);
            const float h2 = so * ua * ds2;
            qbar += h2;
            ub = fmaf(so, s2, ub);
            const float dc = on ? (h1 + h2) * dw : 0.f;   // this lane's share of dE/dc from both triplets
            rx = fmaf(dc, xo, rx);
            ry = fmaf(dc, yo, ry);
            rz = fmaf(dc, zo, rz);
        }
        if (!on) ub = 0.f;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            ub += __shfl_xor(ub, off, 64);
            rx += __shfl_xor(rx, off, 64);
            ry += __shfl_xor(ry, off, 64);
            rz += __shfl_xor(rz, off, 64);
        }
        if (on) {
            IO::store(Pbar + ba * F + f, pbar);
            IO::store(Qbar + ba * F + f, qbar);
        }
        if (lane == 0) {
            ubar[ba] += ub;
            rbar[3 * ba] = rx;
            rbar[3 * ba + 1] = ry;
            rbar[3 * ba + 2] = rz;
        }
    }
}


// Reverse of k_triplet_fwd, one centre per wavefront, lane = feature.  Centres with at most kPairRegs bonds by unordered pairs,
// every triplet evaluated once: what a pair contributes to its two bonds stays in registers, and dE/dc of the pair, a sum over
// the features, goes through an LDS tile that is summed with lane = pair; rbar is assembled from a small table at the end with
// lane = bond.  Other centres by triplet_bwd_sweep.  Bound by the vector unit as the forward kernel.  13.4 M pairs, fp32:
// 2672 us with vector angle terms and LDS accumulators, 1480 us here; three wavefronts per SIMD with 7 registers spilled against
// two without: the same there, 122 against 135 us in bf16 at 30,000 centres.
template <int F, typename BT>
__global__ void __launch_bounds__(256, 3)
k_triplet_bwd(int64_t N, const int64_t *__restrict__ bptr, const float *__restrict__ rhat, const float *__restrict__ u,
              const BT *__restrict__ P, const BT *__restrict__ Q, const float *__restrict__ Wtc, const float *__restrict__ WtcP,
              const BT *__restrict__ Sbar, BT *__restrict__ Pbar, BT *__restrict__ Qbar,
              float *__restrict__ ubar, float *__restrict__ rbar)
{
    using IO = Elem<BT>;
    constexpr int NR = kPairRegs, FS = Dims<64>::FS;
    __shared__ __align__(16) float tile_lds[4][32 * FS], dsym_lds[4][NR * NR];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t i = (int64_t)blockIdx.x * 4 + wave;
    if (i >= N) return;
    const int64_t b0 = bptr[i];
    const int n = __builtin_amdgcn_readfirstlane((int)(bptr[i + 1] - b0));
    if (n > NR) {
        triplet_bwd_sweep<F, BT>(i, lane, bptr, rhat, u, P, Q, Wtc, Sbar, Pbar, Qbar, ubar, rbar);
        return;
    }
    if (n <= 0) return;
    const int f = lane & (F - 1);
    const AngleWeights<F> W(WtcP, lane);
    const int64_t bl = b0 + min(lane & (NR - 1), n - 1);
    const float xl = rhat[3 * bl], yl = rhat[3 * bl + 1], zl = rhat[3 * bl + 2];   // lane = bond (mod 16)
    const float ul = (lane & (NR - 1)) < n ? u[bl] : 0.f;
    float *tile = tile_lds[wave], *dsym = dsym_lds[wave];
    float Pr[NR], Qr[NR], Sr[NR], aP[NR], aQ[NR], aU[NR];
#pragma unroll
    for (int o = 0; o < NR; ++o) {
        Pr[o] = Qr[o] = Sr[o] = aP[o] = aQ[o] = aU[o] = 0.f;
        if (o < n) {
            Pr[o] = IO::load(P + (b0 + o) * F + f);
            Qr[o] = IO::load(Q + (b0 + o) * F + f);
            Sr[o] = IO::load(Sbar + (b0 + o) * F + f);
        }
    }
#pragma unroll
    for (int k = 0; k < NR / 2; ++k) {
        if (2 * k + 1 >= n) break;
        const float c = pair_cosine(k, lane, xl, yl, zl);
        float tw[32];
        W.rows(angle_operands<false>(c, lane >> 5), tw);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int a = 2 * k + q;
            const float ua = readlane_f32(ul, a);
#pragma unroll
            for (int g = 0; g < NR; g += 4)   // bonds from n on have u = 0 and sbar = 0
                if (g + 3 > a && g < n)
#pragma unroll
                    for (int o = g; o < g + 4; ++o)
                        if (o > a) {
                            const float t = tw[16 * q + o], uo = readlane_f32(ul, o);
                            float s1, ds1, s2, ds2;
                            silu_both(Pr[a] + Qr[o] + t, s1, ds1);   // triplet (b1 = a, b2 = o)
                            silu_both(Pr[o] + Qr[a] + t, s2, ds2);   // triplet (b1 = o, b2 = a)
                            const float h1 = Sr[a] * uo * ds1, h2 = Sr[o] * ua * ds2;
                            aP[a] += h1;
                            aQ[o] += h1;
                            aP[o] += h2;
                            aQ[a] += h2;
                            aU[o] = fmaf(Sr[a], s1, aU[o]);
                            aU[a] = fmaf(Sr[o], s2, aU[a]);
                            tile[(16 * q + o) * FS + lane] = h1 + h2;
                        }
        }
        wave_lds_fence();
        {   // dE/dc = sum_f (dT/dc Wtc)_f (h1 + h2)_f, lane (p, h) half the features of pair p (rows without a pair: not used)
            const Basis3 dT = angle_operands<true>(c, lane >> 5);
            float s = 0.f;
#pragma unroll
            for (int bo = 0; bo < Dims<F>::NB; ++bo) {
                const f32x16 dw = W.template block<false>(dT, bo);
#pragma unroll
                for (int r = 0; r < 16; r += 4) {
                    const f32x4 hs = *reinterpret_cast<const f32x4 *>(tile + (lane & 31) * FS + 32 * bo + 2 * r + 4 * (lane >> 5));
#pragma unroll
                    for (int t = 0; t < 4; ++t) s = fmaf(dw[r + t], hs[t], s);
                }
            }
            s += __shfl_xor(s, 32, 64);
            const int a = 2 * k + ((lane >> 4) & 1), o = lane & 15;
            if (lane < 32 && o > a && o < n) dsym[a * NR + o] = s;
        }
        wave_lds_fence();
    }
    const bool on = (F == 64 || lane < F);
#pragma unroll
    for (int o = 0; o < NR; ++o) {
        tile[o * FS + lane] = aU[o];
        if (on && o < n) {
            IO::store(Pbar + (b0 + o) * F + f, aP[o]);
            IO::store(Qbar + (b0 + o) * F + f, aQ[o]);
        }
    }
    wave_lds_fence();
    {   // ubar: lane (bond, quarter of the features)
        const float *row = tile + (lane & 15) * FS + (F / 4) * (lane >> 4);
        float s = 0.f;
#pragma unroll
        for (int c = 0; c < F / 4; c += 4) {
            const f32x4 v = *reinterpret_cast<const f32x4 *>(row + c);
            s += (v[0] + v[1]) + (v[2] + v[3]);
        }
        s += __shfl_xor(s, 16, 64);
        s += __shfl_xor(s, 32, 64);
        if (lane < n) ubar[b0 + lane] += s;   // n <= 16
    }
    if (lane < n) {   // lane = bond: rbar_b = sum over the other bonds o of dE/dc{b, o} rhat_o
        float rx = 0.f, ry = 0.f, rz = 0.f;
        for (int o = 0; o < n; ++o) {
            if (o == lane) continue;
            const float dv = (o > lane) ? dsym[lane * NR + o] : dsym[o * NR + lane];
            rx = fmaf(dv, rhat[3 * (b0 + o)], rx);
            ry = fmaf(dv, rhat[3 * (b0 + o) + 1], ry);
            rz = fmaf(dv, rhat[3 * (b0 + o) + 2], rz);
        }
        rbar[3 * (b0 + lane)] = rx;
        rbar[3 * (b0 + lane) + 1] = ry;
        rbar[3 * (b0 + lane) + 2] = rz;
    }
}

// Forces of the bond part.  dE/dDelta_b = dbond rhat + (rbar - (rbar . rhat) rhat) / d for the bond vector
// Delta_b = r_j + S C - r_i; it pulls on j with + and on i with -.
__device__ inline void bond_gdelta(int64_t q, const float *__restrict__ dbond, const float *__restrict__ rbar,
                                   const float *__restrict__ rhat, const float *__restrict__ bd, float (&gd)[3])
{
    const float x = rhat[3 * q], y = rhat[3 * q + 1], z = rhat[3 * q + 2];
    const float ax = rbar[3 * q], ay = rbar[3 * q + 1], az = rbar[3 * q + 2];
    const float dot = fmaf(ax, x, fmaf(ay, y, az * z));
    const float inv = 1.0f / bd[q];
    gd[0] = fmaf(dbond[q], x, (ax - dot * x) * inv);
    gd[1] = fmaf(dbond[q], y, (ay - dot * y) * inv);
    gd[2] = fmaf(dbond[q], z, (az - dot * z) * inv);
}

// sum over the 16 lanes of a group
__device__ inline float sum16(float v)
{
#pragma unroll
    for (int off = 8; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// Gathered per centre, 16 lanes each (a thread per centre took its bonds one after another: 292 us at 2.4 M bonds, against
// 54): the bonds in which i is the sender are the reverse bonds of its own.   F_i = sum_b (gDelta_b - gDelta_mirror(b))
__global__ void __launch_bounds__(256)
k_bond_force(int64_t N, const int64_t *__restrict__ bptr, const int32_t *__restrict__ bmirror,
             const float *__restrict__ dbond, const float *__restrict__ rbar,
             const float *__restrict__ rhat, const float *__restrict__ bd, float *floc)
{
    const int64_t i = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
    if (i >= N) return;   // whole groups of 16 lanes leave together
    float fx = 0.f, fy = 0.f, fz = 0.f;
    const int64_t b1 = bptr[i + 1];
    for (int64_t b = bptr[i] + (threadIdx.x & 15); b < b1; b += 16) {
        const int64_t q = bmirror[b];   // -1: reverse bond held by the sender's partition (it reaches this atom as a ghost there)
        float own[3], rev[3] = {0.f, 0.f, 0.f};
        bond_gdelta(b, dbond, rbar, rhat, bd, own);
        if (q >= 0) bond_gdelta(q, dbond, rbar, rhat, bd, rev);
        fx += own[0] - rev[0];
        fy += own[1] - rev[1];
        fz += own[2] - rev[2];
    }
    fx = sum16(fx);
    fy = sum16(fy);
    fz = sum16(fz);
    if ((threadIdx.x & 15) == 0) {
        floc[3 * i] = fx;   // (the radial part's rows add to it)
        floc[3 * i + 1] = fy;
        floc[3 * i + 2] = fz;
    }
}

// Ghost rows: a ghost atom i is the sender of bonds (j <- i) held by this partition; each pulls on it with +dE/dDelta.
// Gathered over the ghost's sub-row through the reverse edges, 16 lanes each.
__global__ void __launch_bounds__(256)
k_bond_force_ghost(int64_t n_ghost, int64_t n_owned, const int64_t *__restrict__ row_ptr,
                   const int32_t *__restrict__ mirror, const int32_t *__restrict__ bond_of_edge,
                   const float *__restrict__ dbond, const float *__restrict__ rbar,
                   const float *__restrict__ rhat, const float *__restrict__ bd, float *floc)
{
    const int64_t k = (int64_t)blockIdx.x * 16 + (threadIdx.x >> 4);
    if (k >= n_ghost) return;
    const int64_t r = n_owned + k, e1 = row_ptr[r + 1];
    float fx = 0.f, fy = 0.f, fz = 0.f;
    for (int64_t e = row_ptr[r] + (threadIdx.x & 15); e < e1; e += 16) {
        const int64_t q = bond_of_edge[mirror[e]];
        if (q < 0) continue;
        float gd[3];
        bond_gdelta(q, dbond, rbar, rhat, bd, gd);
        fx -= gd[0];
        fy -= gd[1];
        fz -= gd[2];
    }
    fx = sum16(fx);
    fy = sum16(fy);
    fz = sum16(fz);
    if ((threadIdx.x & 15) == 0) {
        floc[3 * r] = fx;   // (the radial part's rows add to it)
        floc[3 * r + 1] = fy;
        floc[3 * r + 2] = fz;
    }
}

// ---- F x F products over the bonds, fused with what surrounds them
//
// As in the node kernel, a wavefront takes 32 bonds whose rows are loaded in the accumulator layout, so the products chain in
// registers and only the packed operands sit in LDS; each stage reads or writes every [bonds x F] array it touches once.
//   HEAD       e0 = bbond(d) We0 (registers only, never stored: TAIL recomputes it);  P = e0 Wta;  Q = e0 Wtb
//   TAIL       m = S Wt2;  e1 = e0 + u SiLU(m) (registers only);  wb_l = e1 Wb_l for every layer l
//   EBAR       e1bar = sum over the layers l of (abar_l,recv * g_l,send) Wb_l^T, from the kept per-layer abar and g rows;
//              ubar = sum_f e1bar SiLU(m);  mbar = e1bar u SiLU'(m) (registers only);  Sbar = mbar Wt2^T
//   E0BAR      e0bar = e1bar + Pbar Wta^T + Qbar Wtb^T (registers only);
//              dbond = sum_f e0bar (We0^T dbbond/dd) + ubar du/dd
// Bound by the arrays' bytes.  At 2.4 M bonds, 622 MB per fp32 array, in us with fp32 MFMA and the rows staged through LDS ->
// here: HEAD 492 -> 356, TAIL 951 -> 816, EBAR 1354 -> 857, E0BAR 463 -> 360.
enum { BOND_HEAD = 0, BOND_TAIL = 1, BOND_EBAR = 2, BOND_E0BAR = 3 };

struct BondArgs {                      // one partition
    int64_t n;                         // bonds
    const float *d, *u, *du;           // [n] length, envelope at the bond cutoff, its derivative
    const int32_t *edge, *sender;      // [n] edge index, sender row of a bond
    const int32_t *recv;               // receiver row of an edge
    const float *We0p;                 // We0 packed for the K = 8 product (PACK_W1)
    BasisParams bp;                    // radial basis at the bond cutoff
    const float *W[4];                 // packed F x F operands of the stage (TAIL: Wt2, then the first layers' Wb;
                                       // EBAR: Wt2^T, then the first layers' Wb^T)
    const float *Wx;                   // TAIL, EBAR: the packs of the layers beyond the third (read from global memory)
    int n_layers;                      // TAIL, EBAR
    size_t wb_stride;                  // TAIL: elements between two layers' wb
    // [bonds x F] arrays, elements of type BT (fp32, or bf16 in the bf16 mode)
    void *P, *Q;                       // HEAD out
    const void *S;                     // TAIL in
    void *m, *wb;                      // TAIL out; EBAR reads m
    const float *abar, *g;             // EBAR in: kept per-layer node rows, layer l at abar + l abar_stride, g + l g_stride
    size_t abar_stride, g_stride;
    void *e1bar;                       // EBAR out; E0BAR in (BT)
    float *ubar;                       // EBAR out; E0BAR in
    void *Sbar;                        // EBAR out (BT)
    const void *Pbar, *Qbar;           // E0BAR in (BT)
    float *dbond;                      // E0BAR out
};

template <int STAGE> struct BondStage {
    static constexpr bool PER_LAYER = (STAGE == BOND_TAIL || STAGE == BOND_EBAR);   // one operand pack per layer
    static constexpr int NPACK = PER_LAYER ? 4 : 2;
    static constexpr int NW = 8;                          // wavefronts per block
    static constexpr int STAGE_FS = 36;                   // EBAR: row stride of a wavefront's 32 x 32 staging tile
    static constexpr int TILE = STAGE == BOND_EBAR ? 32 * STAGE_FS : 0;
    static constexpr int BLOCKS = PER_LAYER ? 256 : 512;  // blocks in flight
};

// PREC: the F x F products follow the precision mode of the filter MLP's (fp32 as three-part bf16; bf16 operands; split-fp16
// triples; packs prepared accordingly, activations converted in registers, fp32 accumulation); the K = 8 products are fp32 products
// (three-part bf16) in every mode.
// The [bonds x F] arrays are bf16 in the bf16 mode and fp32 otherwise.
template <int PREC> struct BondElem { typedef float type; };
template <> struct BondElem<kPrecBf16> { typedef __bf16 type; };

template <int F, int STAGE, int PREC>
__global__ void __launch_bounds__(BondStage<STAGE>::NW * 64) k_bond_mlp(BondArgs A)
{
    using BT = typename BondElem<PREC>::type;
    using IO = Elem<BT>;
    constexpr int NB = Dims<F>::NB, NW = BondStage<STAGE>::NW, NPACK = BondStage<STAGE>::NPACK, PACK = pack_floats<F>(PREC);
    extern __shared__ float packs[];
    const int n_lds_layers = BondStage<STAGE>::PER_LAYER ? min(A.n_layers, 3) : 0;
    const int n_packs = BondStage<STAGE>::PER_LAYER ? 1 + n_lds_layers : NPACK;
    LdsFill<PACK / 4, NW * 64> fill[NPACK];
#pragma unroll
    for (int q = 0; q < NPACK; ++q)
        if (q < n_packs) fill[q].load(A.W[q]);
#pragma unroll
    for (int q = 0; q < NPACK; ++q)
        if (q < n_packs) fill[q].store(packs + q * PACK);
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int c32 = lane & 31, h4 = 4 * (lane >> 5);
    const int64_t n_tiles = (A.n + 31) / 32;
    const int64_t stride = (int64_t)gridDim.x * NW;

    // rows in accumulator layout: lane (c32, h) holds features 32 b + 8 a + 4 h + (0..3) of bond c32, as loaded until used
    typedef typename IO::raw4 raw4;
    auto load_rows = [&](const void *Yv, int64_t row, bool ok, raw4 (&v)[NB][4]) {
        const BT *Y = static_cast<const BT *>(Yv);
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                v[b][a] = raw4{};   // all-zero bits are 0.0 in either type
                if (ok) v[b][a] = IO::load4_raw(Y + row * F + 32 * b + 8 * a + h4);
            }
    };
    auto widen_rows = [&](const raw4 (&v)[NB][4], f32x16 (&x)[NB]) {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const f32x4 w = IO::widen4(v[b][a]);
#pragma unroll
                for (int c = 0; c < 4; ++c) x[b][4 * a + c] = w[c];
            }
    };
    auto store_rows = [&](void *Yv, int64_t row, bool ok, const f32x16 (&acc)[NB]) {
        BT *Y = static_cast<BT *>(Yv);
        if (ok)
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    const f32x4 v = {acc[b][4 * a], acc[b][4 * a + 1], acc[b][4 * a + 2], acc[b][4 * a + 3]};
                    IO::store4(Y + row * F + 32 * b + 8 * a + h4, v);
                }
    };
    // out (+)= M in
    auto mul = [&](auto accumulate, const float *pack, const f32x16 (&in)[NB], f32x16 (&out)[NB]) {
        constexpr bool ACC = decltype(accumulate)::value;
        if (PREC == kPrecBf16) gemm_rl_bf16<F, ACC>(reinterpret_cast<const __bf16 *>(pack), in, out, lane);
        else if (PREC == kPrecF16x3) gemm_rl_f16x3<F, ACC>(reinterpret_cast<const _Float16 *>(pack), in, out, lane);
        else gemm_rl_bf16x3<F, ACC>(reinterpret_cast<const __bf16 *>(pack), in, out, lane);
    };
    using Fresh = std::false_type;
    using Add = std::true_type;

    raw4 pre[NB][4], pre2[NB][4];
    int64_t ti = (int64_t)wave * gridDim.x + blockIdx.x;   // few tiles: one per block
    // EBAR gathers its rows 8 lanes to 128 consecutive bytes of a row and turns them into the accumulator layout through a small
    // LDS tile (gathered in that layout directly, 16 bytes a lane, every line was fetched several times: 1586 us against 857 us)
    f32x4 fa[NB][4], fg[NB][4];
    int32_t gi[4], gj[4];   // receiver and sender rows of tile rows 8 q + lane / 8 (-1: past the end)
    auto load_factors = [&](int l) {   // dE/dwb_l of a bond = abar_l[receiver] * g_l[sender]
        const float *al = A.abar + (size_t)l * A.abar_stride, *gl = A.g + (size_t)l * A.g_stride;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                fa[b][q] = fg[b][q] = f32x4{0.f, 0.f, 0.f, 0.f};
                if (gi[q] >= 0) {
                    fa[b][q] = *reinterpret_cast<const f32x4 *>(al + (int64_t)gi[q] * F + 32 * b + 4 * (lane & 7));
                    fg[b][q] = *reinterpret_cast<const f32x4 *>(gl + (int64_t)gj[q] * F + 32 * b + 4 * (lane & 7));
                }
            }
    };
    auto turn_factors = [&](f32x16 (&x)[NB]) {
        constexpr int FS = BondStage<STAGE>::STAGE_FS;
        float *tile = packs + NPACK * PACK + wave * BondStage<STAGE>::TILE;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<f32x4 *>(tile + (8 * q + (lane >> 3)) * FS + 4 * (lane & 7)) = fa[b][q] * fg[b][q];
            wave_lds_fence();
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const f32x4 v = *reinterpret_cast<const f32x4 *>(tile + c32 * FS + 8 * a + h4);
#pragma unroll
                for (int c = 0; c < 4; ++c) x[b][4 * a + c] = v[c];
            }
            wave_lds_fence();
        }
    };
    auto fetch = [&](int64_t t) {   // what a tile needs first
        const int64_t row = t * 32 + c32;
        const bool ok = row < A.n;
        if (STAGE == BOND_TAIL) load_rows(A.S, row, ok, pre);
        if (STAGE == BOND_E0BAR) load_rows(A.Pbar, row, ok, pre);
        if (STAGE == BOND_EBAR) {
            const int32_t ri = ok ? A.recv[A.edge[row]] : -1, rj = ok ? A.sender[row] : -1;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                gi[q] = __shfl(ri, 8 * q + (lane >> 3), 64);
                gj[q] = __shfl(rj, 8 * q + (lane >> 3), 64);
            }
            if (A.n_layers > 0) load_factors(0);
        }
    };
    if (ti < n_tiles) fetch(ti);
    for (; ti < n_tiles; ti += stride) {
        const int64_t row = ti * 32 + c32;
        const bool ok = row < A.n;
        const bool more = ti + stride < n_tiles;
        f32x16 acc[NB];

        if (STAGE == BOND_HEAD) {
            float bb[4], db[4];
            radial_basis<false>(ok ? A.d[row] : A.bp.rc, A.bp, lane >> 5, bb, db);   // 0 at the cutoff
            f32x16 e0[NB];
            gemm_k8<F>(A.We0p, bb, e0, lane);
            mul(Fresh{}, packs, e0, acc);
            store_rows(A.P, row, ok, acc);
            mul(Fresh{}, packs + PACK, e0, acc);
            store_rows(A.Q, row, ok, acc);
        } else if (STAGE == BOND_TAIL) {
            f32x16 e1[NB];
            widen_rows(pre, e1);
            const float uc = ok ? A.u[row] : 0.f;
            const float dc = ok ? A.d[row] : A.bp.rc;
            if (more) fetch(ti + stride);
            mul(Fresh{}, packs, e1, acc);
            store_rows(A.m, row, ok, acc);
            {
                float bb[4], db[4];
                radial_basis<false>(dc, A.bp, lane >> 5, bb, db);
                gemm_k8<F>(A.We0p, bb, e1, lane);   // e0, as in HEAD
            }
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) e1[b][r] = fmaf(uc, silu_f(acc[b][r]), e1[b][r]);
            for (int l = 0; l < A.n_layers; ++l) {
                mul(Fresh{}, l < 3 ? packs + (1 + l) * PACK : A.Wx + (size_t)(l - 3) * Dims<F>::PACK3, e1, acc);
                store_rows(static_cast<BT *>(A.wb) + (size_t)l * A.wb_stride, row, ok, acc);
            }
        } else if (STAGE == BOND_EBAR) {
            load_rows(A.m, row, ok, pre);   // needed after the products
            const float uc = ok ? A.u[row] : 0.f;
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[b][r] = 0.f;
            f32x16 x[NB];
            for (int l = 0; l < A.n_layers; ++l) {
                turn_factors(x);
                if (l + 1 < A.n_layers) load_factors(l + 1);   // in flight during this layer's product
                else if (more) fetch(ti + stride);
                mul(Add{}, l < 3 ? packs + (1 + l) * PACK : A.Wx + (size_t)(l - 3) * Dims<F>::PACK3, x, acc);
            }
            store_rows(A.e1bar, row, ok, acc);
            float part = 0.f;
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    float sv, ds;
                    silu_both(IO::widen4(pre[b][r / 4])[r % 4], sv, ds);
                    part = fmaf(acc[b][r], sv, part);
                    x[b][r] = acc[b][r] * uc * ds;   // mbar
                }
            part += __shfl_xor(part, 32, 64);
            if (ok && h4 == 0) A.ubar[row] = part;
            mul(Fresh{}, packs, x, acc);
            store_rows(A.Sbar, row, ok, acc);
        } else {   // BOND_E0BAR
            f32x16 x[NB];
            widen_rows(pre, x);
            load_rows(A.Qbar, row, ok, pre);   // in flight during the first product
            load_rows(A.e1bar, row, ok, pre2);
            mul(Fresh{}, packs, x, acc);
            widen_rows(pre, x);
            if (more) fetch(ti + stride);
            mul(Add{}, packs + PACK, x, acc);
            float bb[4], db[4];
            radial_basis<true>(ok ? A.d[row] : A.bp.rc, A.bp, lane >> 5, bb, db);
            gemm_k8<F>(A.We0p, db, x, lane);   // We0^T dbbond/dd
            float part = 0.f;
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) part = fmaf(IO::widen4(pre2[b][r / 4])[r % 4] + acc[b][r], x[b][r], part);
            part += __shfl_xor(part, 32, 64);
            if (ok && h4 == 0) A.dbond[row] = fmaf(A.ubar[row], A.du[row], part);
        }
    }
}

#endif  // MLIP_MODEL_BOND_H
