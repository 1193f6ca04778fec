// Types, the radial basis, packed weight operands and the MFMA tile products shared by the model kernels.
// Part of model.hip (one translation unit): included inside namespace mlip, anonymous namespace.
#ifndef MLIP_MODEL_TILES_H
#define MLIP_MODEL_TILES_H

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));

constexpr int kBufferFlags = 0x00020000;  // raw 32-bit buffer descriptor word 3 on gfx9-family targets
constexpr float kPi = 3.14159265358979323846f;

__device__ inline void wave_lds_fence()
{
    // LDS operations of one wavefront execute in program order; this only stops the
    // compiler from moving them across the point where lanes exchange roles.
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Element access for arrays that are kept as fp32 or, in the bf16 precision mode, as bf16: rounded to nearest even
// on the way out, exact on the way in.  load4 / store4 move four consecutive elements; load4_raw returns them
// as loaded and widen4 converts later, so that a prefetch does not have to wait for its data to convert it.
template <typename T> struct Elem;
template <> struct Elem<float> {
    static __device__ inline float load(const float *p) { return *p; }
    static __device__ inline void store(float *p, float v) { *p = v; }
    typedef f32x4 raw4;
    static __device__ inline raw4 load4_raw(const float *p) { return *reinterpret_cast<const f32x4 *>(p); }
    static __device__ inline f32x4 widen4(raw4 w) { return w; }
    static __device__ inline f32x4 load4(const float *p) { return *reinterpret_cast<const f32x4 *>(p); }
    static __device__ inline void store4(float *p, f32x4 v) { *reinterpret_cast<f32x4 *>(p) = v; }
};
template <> struct Elem<__bf16> {
    static __device__ inline float load(const __bf16 *p)
    {
        return __builtin_bit_cast(float, (unsigned)*reinterpret_cast<const unsigned short *>(p) << 16);
    }
    static __device__ inline void store(__bf16 *p, float v) { *p = (__bf16)v; }
    typedef uint2 raw4;
    static __device__ inline raw4 load4_raw(const __bf16 *p) { return *reinterpret_cast<const uint2 *>(p); }
    static __device__ inline f32x4 widen4(raw4 w)
    {
        return f32x4{__builtin_bit_cast(float, w.x << 16), __builtin_bit_cast(float, w.x & 0xffff0000u),
                     __builtin_bit_cast(float, w.y << 16), __builtin_bit_cast(float, w.y & 0xffff0000u)};
    }
    static __device__ inline f32x4 load4(const __bf16 *p) { return widen4(load4_raw(p)); }
    static __device__ inline void store4(__bf16 *p, f32x4 v)
    {
        const bf16x2 lo = __builtin_convertvector(f32x2{v[0], v[1]}, bf16x2);
        const bf16x2 hi = __builtin_convertvector(f32x2{v[2], v[3]}, bf16x2);
        uint2 w;
        w.x = __builtin_bit_cast(unsigned, lo);
        w.y = __builtin_bit_cast(unsigned, hi);
        *reinterpret_cast<uint2 *>(p) = w;
    }
};

__device__ inline float sigmoidf_fast(float x) { return __builtin_amdgcn_rcpf(1.0f + __expf(-x)); }

// The edge kernels evaluate SiLU on pre-scaled pre-activations t' = c t with c = -log2(e):
// sigmoid(t) = 1 / (1 + 2^t'), so the scaling multiply disappears (c is folded into the packed W1,
// 1/c into the packed W2 that consumes s' = c SiLU(t)).
constexpr float kSiluScale = -1.4426950408889634f;
constexpr float kSiluScaleInv = -0.6931471805599453f;
__device__ inline float sigmoid_scaled(float tp) { return __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(tp)); }

// A block of THREADS threads brings N4 times 16 bytes into LDS: every piece is requested before the first is stored.  (A plain loop
// waits for each piece in turn, 0.6 us a round.)
template <int N4, int THREADS> struct LdsFill {
    static constexpr int kEach = (N4 + THREADS - 1) / THREADS;
    f32x4 v[kEach];
    __device__ inline void load(const void *src)
    {
#pragma unroll
        for (int i = 0; i < kEach; ++i)
            if ((i + 1) * THREADS <= N4 || i * THREADS + (int)threadIdx.x < N4) v[i] = reinterpret_cast<const f32x4 *>(src)[i * THREADS + threadIdx.x];
    }
    __device__ inline void store(void *lds) const
    {
#pragma unroll
        for (int i = 0; i < kEach; ++i)
            if ((i + 1) * THREADS <= N4 || i * THREADS + (int)threadIdx.x < N4) reinterpret_cast<f32x4 *>(lds)[i * THREADS + threadIdx.x] = v[i];
    }
};

struct BasisParams {
    float rc, inv_rc;
    float pc0;   // p (p + 1) (p + 2) / 2, the factor of the envelope's derivative
    int p;
};

// The basis has K = 8 functions b_n = sin((n+1) pi x) / d * u(x), n = 0..7.  The two lanes (c, h), h = 0, 1, that hold an item in
// the MFMA layouts take four each: b[t] = b_n with n = 2 t + h and, if DERIV, db[t] = d b_n / d d.
template <bool DERIV>
__device__ inline void radial_basis(float d, const BasisParams &bp, int h, float (&b)[4], float (&db)[4])
{
    float x = fminf(d * bp.inv_rc, 1.0f);
    // sin(pi x), cos(pi x) on [0,1]: with z = pi (x - 1/2) in [-pi/2, pi/2], sin(pi x) = cos z and
    // cos(pi x) = -sin z; Taylor polynomials to z^12 / z^13 (truncation below 1e-8)
    const float z = kPi * (x - 0.5f), z2 = z * z;
    float s1 = 1.0f + z2 * (-0.5f + z2 * (4.16666667e-2f + z2 * (-1.38888889e-3f + z2 * (2.48015873e-5f +
               z2 * (-2.75573192e-7f + z2 * 2.08767570e-9f)))));
    float c1v = -z * (1.0f + z2 * (-1.66666667e-1f + z2 * (8.33333333e-3f + z2 * (-1.98412698e-4f +
                z2 * (2.75573192e-6f + z2 * (-2.50521084e-8f + z2 * 1.60590438e-10f))))));
    // envelope in factored form, free of cancellation near the cutoff where it goes to zero with its first two
    // derivatives:  u(x) = (1 - x)^3 sum_{k < p} C(k + 2, 2) x^k  (the same polynomial as 1 - (p+1)(p+2)/2 x^p
    // + p(p+2) x^(p+1) - p(p+1)/2 x^(p+2)),  u'(x) = -p(p+1)(p+2)/2 x^(p-1) (1 - x)^2
    const float w1 = 1.0f - x;
    float xpm1 = 1.0f;
    float q = (float)(bp.p * (bp.p + 1) / 2);
    for (int k = bp.p - 2; k >= 0; --k) {
        q = fmaf(q, x, (float)((k + 1) * (k + 2) / 2));
        xpm1 *= x;
    }
    const float w2 = w1 * w1;
    const float u = w2 * w1 * q;
    const float inv_d = __builtin_amdgcn_rcpf(d);
    float du_term = 0.f;  // u'/rc - u/d
    if (DERIV) {
        const float du = -bp.pc0 * xpm1 * w2;
        du_term = du * bp.inv_rc - u * inv_d;
    }
    const float u_rc = u * bp.inv_rc;
    // sin and cos of (n+1) pi x: from pi x or 2 pi x on in steps of 2 pi x.  The cosine of 2 pi x from the smaller of the two
    // squares: rms error of the eight sines 6.8e-8 (8.0e-8 in steps of pi x, 10.6e-8 with 1 - 2 s^2 alone)
    const float s2 = 2.0f * s1 * c1v, c2 = fabsf(s1) < fabsf(c1v) ? fmaf(-2.0f * s1, s1, 1.0f) : fmaf(2.0f * c1v, c1v, -1.0f);
    float sn = h ? s2 : s1, cn = h ? c2 : c1v;
    const float pi_n = h ? 2.0f * kPi : kPi, u_d = u * inv_d;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        b[t] = sn * u_d;
        if (DERIV) db[t] = fmaf((float)(2 * t) * kPi + pi_n, cn * u_rc, sn * du_term) * inv_d;
        const float sx = sn * c2 + cn * s2;
        cn = cn * c2 - sn * s2;
        sn = sx;
    }
}

// ---------------------------------------------------------------- packed weights
//
// F x F operands are packed as the A operands of v_mfma_f32_32x32x16_{bf16,f16}: matrix M[o][k] = W[k][o] (trans, y = x W) or
// W[o][k] (y = x W^T), index
//   (((bo * NB + bi) * 2 + q) * 64 + lane) * 8 + t  ->  M[32 bo + lane % 32][32 bi + 8 (r / 4) + 4 (lane / 32) + r % 4],
// r = 8 q + t: element t of lane-half h of MFMA (bi, q) pairs with accumulator register r of a chained product
// (or with the same feature of an item-major LDS row).
// PACK_W1: K = 8 rows as three-part bf16, index ((bo * 3 + part) * 64 + lane) * 4 + t  ->  part of W1[2 t + lane / 32][32 bo + lane % 32].
//
// PACK_FF_BF16X3: every fp32 value as three bf16 parts (split_bf16x3), one pack of each after the other; the fp32 mode and
// the node kernels.  PACK_FF_BF16: rounded to bf16; the bf16 mode.  PACK_FF_BF16X3_ALT: three parts, the weights of odd output
// features negated, so that their sums come out negated: aligning the products of one instruction, the matrix unit cuts bits
// off towards minus infinity, which shifts every sum of unit size by -7.4e-9 on average (fp32 MFMA: 1e-10).  The readout's
// weights wr2 may all have one sign, and the shift then adds up in the total energy; with every other feature negated it
// cancels (mean error of the energy of 3,880 atoms over 60 models, fp32 MFMA / all features alike / here: L = 3 1.36e-7 /
// 1.48e-7 / 1.33e-7, L = 1 4.0e-8 / 6.0e-8 / 4.2e-8, L = 0 1.9e-8 / 3.3e-8 / 1.5e-8).  Elsewhere it meets weights of both signs.
//
// Split-fp16 form of the same operand: every fp32 value v is kept as hi + lo, hi = fp16(v), lo = fp16(v - hi)
// (22 significant bits together); a product of two such values is taken as hi hi + hi lo + lo hi with fp32
// accumulation.  What is dropped (lo lo, and the rounding of the two lo parts) is about 3 * 2^-22 of the term,
// the size of the rounding an fp32 accumulation of 64 terms makes anyway, at 3/16 of the fp32 MFMA's matrix time.
// hi parts first (F * F halves), then lo parts.
//
// Operand packs a call needs are made by one launch: one job per pack (blockIdx.y), one thread per element.  Every
// pack in a launch of its own took 2 us of device time and a launch each, 20 to 26 per model.
enum { PACK_W1 = 0, PACK_FF_BF16 = 1, PACK_FF_F16X2 = 2, PACK_FF_BF16X3 = 3, PACK_FF_BF16X3_ALT = 4 };
struct PackJob {
    const float *W;
    float *out;
    float scale;
    int16_t kind, trans;
};
constexpr int kPackJobs = 66;   // 8 layers x 8 packs and the readout's two; the bond part has 6 + 2 x 8 + 2
struct PackBatch {
    int n, F;
    int32_t *clear;   // words to clear
    int n_clear;
    PackJob job[kPackJobs];
    void add(const float *W, float *out, int kind, int trans, float scale) { job[n++] = PackJob{W, out, scale, (int16_t)kind, (int16_t)trans}; }
};

__global__ void k_pack(PackBatch B)
{
    const PackJob &J = B.job[blockIdx.y];
    if (blockIdx.x == 0 && blockIdx.y == 0)
        for (int i = threadIdx.x; i < B.n_clear; i += blockDim.x) B.clear[i] = 0;
    const int F = B.F, NB = F / 32;
    const float *__restrict__ W = J.W;
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    auto part3 = [](float v, int part) {   // split_bf16x3, one part
        const __bf16 hi = (__bf16)v;
        const float r = v - (float)hi;
        const __bf16 mid = (__bf16)r;
        return part == 0 ? hi : part == 1 ? mid : (__bf16)(r - (float)mid);
    };
    if (J.kind == PACK_W1) {
        if (idx >= NB * 3 * 64 * 4) return;
        const int t = idx & 3, lane = (idx >> 2) & 63, part = (idx >> 8) % 3, bo = (idx >> 8) / 3;
        reinterpret_cast<__bf16 *>(J.out)[idx] = part3(J.scale * W[(2 * t + (lane >> 5)) * F + 32 * bo + (lane & 31)], part);
        return;
    }
    if (idx >= F * F) return;
    const int bb = idx >> 10, bi = bb % NB, bo = bb / NB;
    const int t = idx & 7, lane = (idx >> 3) & 63, q = (idx >> 9) & 1, r = 8 * q + t;
    const int o = 32 * bo + (lane & 31);
    const int k = 32 * bi + 8 * (r / 4) + 4 * (lane >> 5) + (r & 3);
    const float scale = J.kind == PACK_FF_BF16X3_ALT && (o & 1) ? -J.scale : J.scale;
    const float v = scale * (J.trans ? W[k * F + o] : W[o * F + k]);
    if (J.kind == PACK_FF_BF16) {
        reinterpret_cast<__bf16 *>(J.out)[idx] = (__bf16)v;
    } else if (J.kind == PACK_FF_BF16X3 || J.kind == PACK_FF_BF16X3_ALT) {
        for (int q = 0; q < 3; ++q) reinterpret_cast<__bf16 *>(J.out)[q * F * F + idx] = part3(v, q);
    } else {
        const _Float16 h = (_Float16)v;
        reinterpret_cast<_Float16 *>(J.out)[idx] = h;
        reinterpret_cast<_Float16 *>(J.out)[F * F + idx] = (_Float16)(v - (float)h);
    }
}

__device__ inline void split_f16(const float (&v)[8], f16x8 &hi, f16x8 &lo)
{
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
        const f32x2 p = {v[i], v[i + 1]};
        const f16x2 h = __builtin_convertvector(p, f16x2);
        const f16x2 l = __builtin_convertvector(p - __builtin_convertvector(h, f32x2), f16x2);
        hi[i] = h[0];
        hi[i + 1] = h[1];
        lo[i] = l[0];
        lo[i + 1] = l[1];
    }
}

__device__ inline bf16x8 to_bf16x8(const float (&v)[8])
{
    bf16x8 o;
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
        const f32x2 p = {v[i], v[i + 1]};
        const bf16x2 h = __builtin_convertvector(p, bf16x2);   // round to nearest even, two per instruction
        o[i] = h[0];
        o[i + 1] = h[1];
    }
    return o;
}

// v = h + m + l with three bf16 parts, exactly unless l underflows: 8 significant bits each, rounded to nearest, what
// is left after each part is exact in fp32.  An infinity (and what rounds to one: beyond 3.39e38) becomes NaN.
__device__ inline void split_bf16x3(const float (&v)[8], bf16x8 &h, bf16x8 &m, bf16x8 &l)
{
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
        const f32x2 p = {v[i], v[i + 1]};
        const bf16x2 ph = __builtin_convertvector(p, bf16x2);
        const f32x2 r = p - __builtin_convertvector(ph, f32x2);
        const bf16x2 pm = __builtin_convertvector(r, bf16x2);
        const f32x2 r2 = r - __builtin_convertvector(pm, f32x2);
        const bf16x2 pl = __builtin_convertvector(r2, bf16x2);
        h[i] = ph[0]; h[i + 1] = ph[1];
        m[i] = pm[0]; m[i + 1] = pm[1];
        l[i] = pl[0]; l[i + 1] = pl[1];
    }
}

template <int F> struct Dims {
    static constexpr int NB = F / 32;
    static constexpr int FS = F + 4;      // LDS row stride of an item-major tile
    static constexpr int TILE = 32 * FS;  // floats per 32-item tile
    static constexpr int PACK1 = NB * 3 * 64 * 2;   // floats of a K = 8 pack
    static constexpr int PACK3 = F * F * 3 / 2;   // floats of a three-part bf16 pack
};

// out[bo] = sum_k M[.][k] in[k][.], `in` held in accumulator layout (chained product), in bf16: weights as a bf16 pack in
// LDS, the chained operand rounded to bf16, fp32 accumulation
template <int F, bool ACCUMULATE = false>
__device__ inline void gemm_rl_bf16(const __bf16 *__restrict__ Ap, const f32x16 (&in)[Dims<F>::NB],
                                    f32x16 (&out)[Dims<F>::NB], int lane)
{
    constexpr int NB = Dims<F>::NB;
    const bf16x8 *A = reinterpret_cast<const bf16x8 *>(Ap) + lane;
    if (!ACCUMULATE)
#pragma unroll
        for (int bo = 0; bo < NB; ++bo)
#pragma unroll
            for (int r = 0; r < 16; ++r) out[bo][r] = 0.f;
#pragma unroll
    for (int bi = 0; bi < NB; ++bi)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            float v[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) v[t] = in[bi][8 * q + t];
            const bf16x8 b = to_bf16x8(v);
#pragma unroll
            for (int bo = 0; bo < NB; ++bo)
                out[bo] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[((bo * NB + bi) * 2 + q) * 64], b, out[bo], 0, 0, 0);
        }
}

// the same with the B operand taken from an item-major LDS row of this lane's item (fp32, rounded here)
template <int F, bool ACCUMULATE = false>
__device__ inline void gemm_row_bf16(const __bf16 *__restrict__ Ap, const float *row, f32x16 (&out)[Dims<F>::NB], int lane)
{
    constexpr int NB = Dims<F>::NB;
    const int h = lane >> 5;
    const bf16x8 *A = reinterpret_cast<const bf16x8 *>(Ap) + lane;
    if (!ACCUMULATE)
#pragma unroll
        for (int bo = 0; bo < NB; ++bo)
#pragma unroll
            for (int r = 0; r < 16; ++r) out[bo][r] = 0.f;
#pragma unroll
    for (int bi = 0; bi < NB; ++bi)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const f32x4 lo4 = *reinterpret_cast<const f32x4 *>(row + 32 * bi + 16 * q + 4 * h);
            const f32x4 hi4 = *reinterpret_cast<const f32x4 *>(row + 32 * bi + 16 * q + 8 + 4 * h);
            const float v[8] = {lo4[0], lo4[1], lo4[2], lo4[3], hi4[0], hi4[1], hi4[2], hi4[3]};
            const bf16x8 b = to_bf16x8(v);
#pragma unroll
            for (int bo = 0; bo < NB; ++bo)
                out[bo] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A[((bo * NB + bi) * 2 + q) * 64], b, out[bo], 0, 0, 0);
        }
}

// gemm_rl and gemm_row in split fp16 (three MFMAs of depth 16 per 16 k-values)
template <int F, bool ACCUMULATE = false>
__device__ inline void gemm_rl_f16x3(const _Float16 *__restrict__ Ap, const f32x16 (&in)[Dims<F>::NB],
                                     f32x16 (&out)[Dims<F>::NB], int lane)
{
    constexpr int NB = Dims<F>::NB;
    const f16x8 *Ah = reinterpret_cast<const f16x8 *>(Ap) + lane;
    const f16x8 *Al = reinterpret_cast<const f16x8 *>(Ap + F * F) + lane;
    if (!ACCUMULATE)
#pragma unroll
        for (int bo = 0; bo < NB; ++bo)
#pragma unroll
            for (int r = 0; r < 16; ++r) out[bo][r] = 0.f;
#pragma unroll
    for (int bi = 0; bi < NB; ++bi)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            float v[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) v[t] = in[bi][8 * q + t];
            f16x8 bh, bl;
            split_f16(v, bh, bl);
#pragma unroll
            for (int bo = 0; bo < NB; ++bo) {
                const f16x8 ah = Ah[((bo * NB + bi) * 2 + q) * 64], al = Al[((bo * NB + bi) * 2 + q) * 64];
                out[bo] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, bh, out[bo], 0, 0, 0);   // small terms first
                out[bo] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bl, out[bo], 0, 0, 0);
                out[bo] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bh, out[bo], 0, 0, 0);
            }
        }
}

template <int F, bool ACCUMULATE = false>
__device__ inline void gemm_row_f16x3(const _Float16 *__restrict__ Ap, const float *row, f32x16 (&out)[Dims<F>::NB], int lane)
{
    constexpr int NB = Dims<F>::NB;
    const int h = lane >> 5;
    const f16x8 *Ah = reinterpret_cast<const f16x8 *>(Ap) + lane;
    const f16x8 *Al = reinterpret_cast<const f16x8 *>(Ap + F * F) + lane;
    if (!ACCUMULATE)
#pragma unroll
        for (int bo = 0; bo < NB; ++bo)
#pragma unroll
            for (int r = 0; r < 16; ++r) out[bo][r] = 0.f;
#pragma unroll
    for (int bi = 0; bi < NB; ++bi)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const f32x4 lo4 = *reinterpret_cast<const f32x4 *>(row + 32 * bi + 16 * q + 4 * h);
            const f32x4 hi4 = *reinterpret_cast<const f32x4 *>(row + 32 * bi + 16 * q + 8 + 4 * h);
            const float v[8] = {lo4[0], lo4[1], lo4[2], lo4[3], hi4[0], hi4[1], hi4[2], hi4[3]};
            f16x8 bh, bl;
            split_f16(v, bh, bl);
#pragma unroll
            for (int bo = 0; bo < NB; ++bo) {
                const f16x8 ah = Ah[((bo * NB + bi) * 2 + q) * 64], al = Al[((bo * NB + bi) * 2 + q) * 64];
                out[bo] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, bh, out[bo], 0, 0, 0);
                out[bo] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bl, out[bo], 0, 0, 0);
                out[bo] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bh, out[bo], 0, 0, 0);
            }
        }
}

// fp32 products as three-part bf16 operands: x y = (h + m + l)(h' + m' + l'), of which the six largest terms (down to
// 2^-18 of the product) are taken, smallest first (l m', m l' and l l' are together below 2^-25 of it, half an fp32 rounding).  24 MFMAs of a
// chain round at full size for 64 terms, where the fp32 instruction makes 32.  The A operands of the next step are
// requested before the MFMAs of this one.
template <int F, bool ACCUMULATE, class Values>
__device__ inline void gemm_bf16x3(const __bf16 *__restrict__ Ap, Values values, f32x16 (&out)[Dims<F>::NB], int lane)
{
    constexpr int NB = Dims<F>::NB, STEPS = NB * 2 * NB;
    const bf16x8 *A = reinterpret_cast<const bf16x8 *>(Ap) + lane;
    if (!ACCUMULATE)
#pragma unroll
        for (int bo = 0; bo < NB; ++bo)
#pragma unroll
            for (int r = 0; r < 16; ++r) out[bo][r] = 0.f;
    auto at = [](int st) { return ((st % NB) * NB * 2 + st / NB) * 64; };   // step st: k block st / NB, output block st % NB
    bf16x8 a[3], bh, bm, bl;
#pragma unroll
    for (int q = 0; q < 3; ++q) a[q] = A[at(0) + q * (F * F / 8)];
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
        const int bo = st % NB;
        bf16x8 an[3] = {a[0], a[1], a[2]};
        if (st + 1 < STEPS)
#pragma unroll
            for (int q = 0; q < 3; ++q) an[q] = A[at(st + 1) + q * (F * F / 8)];
        if (bo == 0) {
            float v[8];
            values(st / NB, v);
            split_bf16x3(v, bh, bm, bl);
        }
        out[bo] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[2], bh, out[bo], 0, 0, 0);
        out[bo] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], bl, out[bo], 0, 0, 0);
        out[bo] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], bm, out[bo], 0, 0, 0);
        out[bo] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1], bh, out[bo], 0, 0, 0);
        out[bo] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], bm, out[bo], 0, 0, 0);
        out[bo] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0], bh, out[bo], 0, 0, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 6, 0);
#pragma unroll
        for (int q = 0; q < 3; ++q) a[q] = an[q];
    }
}

// the B operand in accumulator layout (chained product) ...
template <int F, bool ACCUMULATE = false>
__device__ inline void gemm_rl_bf16x3(const __bf16 *__restrict__ Ap, const f32x16 (&in)[Dims<F>::NB],
                                      f32x16 (&out)[Dims<F>::NB], int lane)
{
    gemm_bf16x3<F, ACCUMULATE>(Ap, [&](int s, float (&v)[8]) {
#pragma unroll
        for (int t = 0; t < 8; ++t) v[t] = in[s / 2][8 * (s % 2) + t];
    }, out, lane);
}

// ... or from an item-major LDS row of this lane's item
template <int F, bool ACCUMULATE = false>
__device__ inline void gemm_row_bf16x3(const __bf16 *__restrict__ Ap, const float *row, f32x16 (&out)[Dims<F>::NB], int lane)
{
    const int h = lane >> 5;
    gemm_bf16x3<F, ACCUMULATE>(Ap, [&](int s, float (&v)[8]) {
        const f32x4 lo4 = *reinterpret_cast<const f32x4 *>(row + 16 * s + 4 * h);
        const f32x4 hi4 = *reinterpret_cast<const f32x4 *>(row + 16 * s + 8 + 4 * h);
#pragma unroll
        for (int t = 0; t < 4; ++t) { v[t] = lo4[t]; v[4 + t] = hi4[t]; }
    }, out, lane);
}

// K = 8 product with the basis, out[bo] (one block of 32 features) = sum_n W1[n][.] v[n]: operands in three bf16 parts as in
// gemm_bf16x3.  A lane's four values fill half of its eight places along k of an MFMA, so three MFMAs hold the six terms:
// (l + h)(h' + l') as l h' + h l', (h + m) m', (h + m) h'.
// The work of 8 fp32 MFMAs of half the rate, and each lane evaluates the four basis functions it feeds in, not all eight:
// 3.31 -> 3.18 ms for the forward, 2.90 -> 2.87 ms for the reverse launch at a million atoms (44 M edges); forces against 64 bits
// 8.0e-7 (8.1e-7 before; rms relative, geometric mean of 41 systems).
struct Basis3 { bf16x8 hm, lh; };   // an item's values as the MFMAs' B operands
__device__ inline Basis3 basis_operands(const float (&v)[4])
{
    Basis3 o;
#pragma unroll
    for (int i = 0; i < 4; i += 2) {
        const f32x2 p = {v[i], v[i + 1]};
        const bf16x2 ph = __builtin_convertvector(p, bf16x2);
        const f32x2 r = p - __builtin_convertvector(ph, f32x2);
        const bf16x2 pm = __builtin_convertvector(r, bf16x2);
        const bf16x2 pl = __builtin_convertvector(r - __builtin_convertvector(pm, f32x2), bf16x2);
        o.hm[i] = ph[0]; o.hm[i + 1] = ph[1];
        o.hm[4 + i] = pm[0]; o.hm[5 + i] = pm[1];
        o.lh[i] = pl[0]; o.lh[i + 1] = pl[1];
        o.lh[4 + i] = ph[0]; o.lh[5 + i] = ph[1];
    }
    return o;
}

template <int F> __device__ inline void gemm_k8_block(const float *__restrict__ A1, const Basis3 &v, int bo, f32x16 &out, int lane)
{
    const bf16x4 *A = reinterpret_cast<const bf16x4 *>(A1) + (bo * 3) * 64 + lane;
    const bf16x4 h = A[0], m = A[64], l = A[128];
#pragma unroll
    for (int r = 0; r < 16; ++r) out[r] = 0.f;
    out = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_shufflevector(h, l, 0, 1, 2, 3, 4, 5, 6, 7), v.lh, out, 0, 0, 0);
    out = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_shufflevector(m, m, 0, 1, 2, 3, 4, 5, 6, 7), v.hm, out, 0, 0, 0);
    out = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_shufflevector(h, h, 0, 1, 2, 3, 4, 5, 6, 7), v.hm, out, 0, 0, 0);
}
template <int F> __device__ inline void gemm_k8(const float *__restrict__ A1, const float (&v)[4], f32x16 (&out)[Dims<F>::NB], int lane)
{
    const Basis3 o = basis_operands(v);
#pragma unroll
    for (int bo = 0; bo < Dims<F>::NB; ++bo) gemm_k8_block<F>(A1, o, bo, out[bo], lane);
}

// accumulator layout -> item-major LDS tile
template <int F>
__device__ inline void regs_to_tile(const f32x16 (&v)[Dims<F>::NB], float *tile, int lane)
{
    constexpr int NB = Dims<F>::NB;
    constexpr int FS = Dims<F>::FS;
    const int c32 = lane & 31, h = lane >> 5;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            f32x4 x = {v[b][4 * a], v[b][4 * a + 1], v[b][4 * a + 2], v[b][4 * a + 3]};
            *reinterpret_cast<f32x4 *>(tile + c32 * FS + 32 * b + 8 * a + 4 * h) = x;
        }
}

#endif  // MLIP_MODEL_TILES_H
