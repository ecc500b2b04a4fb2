// Learned shape-function surrogate (an addition to the paper's method).
//
// A 6 -> 128 -> 128 -> 27 GELU network maps the features of one (marker,
// component) support -- the in-cell offsets xi_d = (X - X_0)/H_d and the
// spacing ratios rho_d = (X_{+1} - X_0)/(X_0 - X_{-1}), which fix the exact
// MLS shape function of eq. 3-6 -- to its 27 shape-function values.
//
// Arithmetic: every matrix product runs on the matrix cores as "split BF16":
// an FP32 operand v is held as hi = bf16(v) and lo = bf16(v - hi), and
// hi*hi + hi*lo + lo*hi is accumulated in FP32 (the dropped lo*lo term and
// the rounding of lo leave a relative error near 2^-17 per product).
//
// Training: a step is three launches.  k_mlp_pass takes 16 samples per
// workgroup through the forward pass, the loss and the backward pass with all
// activations in registers, and leaves the layers' inputs and output gradients
// in memory; k_mlp_wgrad forms the weight gradients from them in chunks of the
// batch; k_mlp_update sums the chunks in order, applies Adam and refreshes the
// packed operands.  Every reduction has a fixed order, so a training run is
// reproducible.
//
// Inference (mls_build with MLS_LEARNED): one wavefront per (64-marker block,
// component) computes the features, evaluates the network for 32 markers at a
// time with the three layers chained through registers, and checks the
// result against the consistency conditions of MLS with a linear basis:
//   r0 = |sum_k phi_k - 1|,  r1 = max_d |sum_k phi_k s_dk|
// (partition of unity, reproduction of linear fields; s_dk the offset of node
// k from the marker along d in units of H_d).  A marker whose residual is not
// below the tolerance is rebuilt with exact MLS on the same wavefront.
#include <cmath>
#include <cstring>

#include "mls_exact.h"

namespace mls {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kBlock = 256;
constexpr int kLearnBlock = 512;        // 8 wavefronts share one copy of the network in LDS

// ---- activation ------------------------------------------------------------
// The standard normal tail Q(x) = 1 - Phi(x) = erfc(x / sqrt 2) / 2 for x >= 0
// from the rational approximation of Abramowitz & Stegun, Handbook of
// Mathematical Functions, formula 7.1.26 (|error of erf| <= 1.5e-7):
//   erfc(y) ~ t (a1 + t (a2 + t (a3 + t (a4 + t a5)))) exp(-y^2),  t = 1 / (1 + p y).
// ez receives exp(-x^2 / 2).
__device__ __forceinline__ float normal_tail(float x, float &ez)
{
    const float yv = x * 0.70710678118654752f;
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, yv, 1.0f));
    const float poly =
        t * fmaf(t, fmaf(t, fmaf(t, fmaf(t, 1.061405429f, -1.453152027f), 1.421413741f), -0.284496736f), 0.254829592f);
    ez = __builtin_amdgcn_exp2f(x * x * -0.72134752044448170f);   // exp(-x^2/2) = 2^(-x^2 log2(e) / 2)
    return 0.5f * poly * ez;
}

// gelu(z) = z Phi(z)
__device__ __forceinline__ float gelu(float z)
{
    float ez;
    const float q = normal_tail(fabsf(z), ez);
    return z * (z >= 0.0f ? 1.0f - q : q);
}

// The same with its derivative gelu'(z) = Phi(z) + z phi(z), phi(z) =
// exp(-z^2/2) / sqrt(2 pi).
__device__ __forceinline__ float gelu(float z, float &dz)
{
    float ez;
    const float q = normal_tail(fabsf(z), ez);
    const float cdf = z >= 0.0f ? 1.0f - q : q;
    dz = cdf + z * ez * 0.39894228040143268f;
    return z * cdf;
}

__device__ __forceinline__ void split_bf16(float v, __bf16 &hi, __bf16 &lo)
{
    hi = (__bf16)v;
    lo = (__bf16)(v - (float)hi);
}

// The same of two values, with v - hi as a two-term dot product whose other
// factor picks one half of the packed hi, in place of an unpacking shift and a
// subtraction.  The difference is exact in FP32 either way.  An infinity or NaN
// spreads to its neighbour's lo; both belong to one row of a product, which it
// makes non-finite anyway.  (The factors are hidden from the compiler: as
// constants it encoded {-1, 0} as -1 in both halves.)
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void split_bf16_pair(float v0, float v1, bf16x2 &hi, bf16x2 &lo)
{
    uint32_t first = 0x0000bf80u, second = 0xbf800000u;   // -1 in one half
    asm("" : "+s"(first));
    asm("" : "+s"(second));
    hi = bf16x2{(__bf16)v0, (__bf16)v1};
    lo = bf16x2{(__bf16)__builtin_amdgcn_fdot2_f32_bf16(hi, __builtin_bit_cast(bf16x2, first), v0, false),
                (__bf16)__builtin_amdgcn_fdot2_f32_bf16(hi, __builtin_bit_cast(bf16x2, second), v1, false)};
}

__device__ __forceinline__ f32x16 mfma3(bf16x8 ah, bf16x8 al, bf16x8 bh, bf16x8 bl, f32x16 c)
{
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bh, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah, bl, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bh, c, 0, 0, 0);
    return c;
}

// ---- training -----------------------------------------------------------------

// Row of batch entry b: idx[b] if idx is given, else b.  An index outside
// [0, rows) raises MLS_E_ARG on the device and reads row 0 instead.
__device__ __forceinline__ int64_t batch_row(const int64_t *idx, int64_t b, int64_t rows, ErrWord *err)
{
    if (!idx) return b;
    const int64_t r = idx[b];
    if (r < 0 || r >= rows) {
        raise_error(err, b, MLS_E_ARG);
        return 0;
    }
    return r;
}

// Offsets of the three support nodes from the marker along each axis in
// units of H, from the features: nodes at -2/(1+rho), 0, 2 rho/(1+rho)
// relative to the home node, the marker at xi.
__device__ __forceinline__ void node_offsets(const float *f, float s[3][3])
{
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const float xi = f[d], rho = f[3 + d];
        const float inv = 1.0f / (1.0f + rho);
        s[d][0] = -2.0f * inv - xi;
        s[d][1] = -xi;
        s[d][2] = 2.0f * rho * inv - xi;
    }
}

// Operands of the training kernels: every weight matrix as the A operands of
// v_mfma_f32_16x16x32_bf16 (lane l: output row l % 16, eight inputs), split
// into a high and a low BF16 part.  Slot s holds
//   0 + T        W1^T, rows 16 T .. (hidden units), inputs the 6 features
//   8 + 4 T + kb W2^T, rows 16 T .., inputs of k block kb
//   40 + 4 T + kb W3^T, rows 16 T .. (27 outputs)
//   48 + T       W3, rows 16 T .. (hidden units), inputs the 27 outputs
//   56 + 4 T + kb W2, rows 16 T .. (first-layer units), inputs of block kb
// A result tile leaves rows 4 (l / 16) + j of column l % 16 in registers j < 4,
// so two tiles in a row are the B operand of the next product if its k slot
// (l / 16, i) stands for input 32 kb + 16 (i / 4) + 4 (l / 16) + i % 4: the
// products chain through registers without a shuffle.
typedef float f32x4v __attribute__((ext_vector_type(4)));
constexpr int kTrainSlots = 88;
constexpr size_t kTrainImageBytes = (size_t)kTrainSlots * 2 * 64 * 16;

// Writes parameter p (value v) into its one or two places of the image.
__device__ __forceinline__ void pack_train(__bf16 *img, int p, float v)
{
    __bf16 hi, lo;
    split_bf16(v, hi, lo);
    auto put = [&](int slot, int lane, int e) {
        img[(((slot * 2) * 64) + lane) * 8 + e] = hi;
        img[(((slot * 2 + 1) * 64) + lane) * 8 + e] = lo;
    };
    // k slot of input q within its block of 32
    auto grp = [](int q) { return (q >> 2) & 3; };
    auto elt = [](int q) { return ((q >> 4) & 1) * 4 + (q & 3); };
    if (p < kOffB1) {
        const int i = p / kMlpHidden, o = p % kMlpHidden;
        put(o >> 4, o & 15, i);
    } else if (p >= kOffW2 && p < kOffB2) {
        const int i = (p - kOffW2) / kMlpHidden, o = (p - kOffW2) % kMlpHidden;
        put(8 + 4 * (o >> 4) + (i >> 5), 16 * grp(i) + (o & 15), elt(i));
        put(56 + 4 * (i >> 4) + (o >> 5), 16 * grp(o) + (i & 15), elt(o));
    } else if (p >= kOffW3 && p < kOffB3) {
        const int i = (p - kOffW3) / kMlpOut, o = (p - kOffW3) % kMlpOut;
        put(40 + 4 * (o >> 4) + (i >> 5), 16 * grp(i) + (o & 15), elt(i));
        put(48 + (i >> 4), 16 * grp(o) + (i & 15), elt(o));
    }
}

__global__ void __launch_bounds__(kBlock) k_pack_train(const float *__restrict__ P, __bf16 *__restrict__ img)
{
    const int p = blockIdx.x * kBlock + threadIdx.x;
    if (p < kMlpParams) pack_train(img, p, P[p]);
}

// One operand slot (high and low part) of a lane, and the split product with it.
struct Slot {
    bf16x8 hi, lo;
};
__device__ __forceinline__ Slot slot_at(const uint4 *img, int slot, int lane)
{
    return {__builtin_bit_cast(bf16x8, img[(slot * 2) * 64 + lane]),
            __builtin_bit_cast(bf16x8, img[(slot * 2 + 1) * 64 + lane])};
}
__device__ __forceinline__ f32x4v mfma3_16(const Slot &a, const Slot &b, f32x4v c)
{
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.hi, b.hi, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.hi, b.lo, c, 0, 0, 0);
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.lo, b.hi, c, 0, 0, 0);
    return c;
}

// What a training pass leaves for the weight gradients: per layer the inputs
// (u, h1, h2) and the gradients of the pre-activations (d1, d2, dy), 16 samples
// after 16, the 16 values of a unit together, so that the operand of 32 units
// by 16 samples is one run of 2 KB (with a unit's whole batch in one run a load
// touches 32 lines).  Mp samples, a multiple of 32, zeros past the batch.
struct TrainBufs {
    float *u, *h1, *h2, *d1, *d2, *dy;   // kTrainIn, 4 x 128 and kTrainOut units
    float *part;                         // [chunks][kPartStride] weight-gradient sums
    float *loss;                         // [Mp / 16], one per 16 samples
    int64_t Mp;
    int chunks, chunk;                   // chunk: samples per chunk, a multiple of 32
};
constexpr int kTrainIn = 8, kTrainOut = 32;   // units stored for the features and the outputs
constexpr int kPartStride = (kMlpParams + 63) / 64 * 64;

// Forward pass of 16 samples per workgroup, and with TRAIN the loss
//   L = mean_{b,k} (y - t)^2 + mu mean_b [(sum_k y - 1)^2 + sum_d (sum_k y s_dk)^2]
// (one partial sum per workgroup) and the backward pass.  What bounds it is
// latency: a batch of 8192 is 512 groups of samples, and each is a chain of
// five matrix products.  So the 128 units of a layer are shared out over four
// wavefronts, 32 each (lane l: sample l % 16, eight units), which is one k
// block of the next product: its split operand goes to the others through
// LDS, one barrier a layer.  The weights a wavefront needs next are requested
// a layer ahead.  8192 samples: 16 us; with all units in one wavefront 33 us,
// and as one product kernel per layer with activations through memory 290 us.
constexpr int kPassWaves = 4;
template <bool TRAIN>
__global__ void __launch_bounds__(64 * kPassWaves)
k_mlp_pass(int64_t M, const float *__restrict__ feat, int64_t rows, const int64_t *__restrict__ idx,
           const float *__restrict__ norm, const float *__restrict__ P, const uint4 *__restrict__ img,
           const float *__restrict__ target, float mu, float *__restrict__ Y, const TrainBufs tb, ErrWord *err)
{
    __shared__ bf16x8 ops[TRAIN ? 3 : 2][4][2][64];   // h1, h2 and d2 as operands
    const int lane = threadIdx.x & 63, s = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t b = (int64_t)blockIdx.x * 16 + s;
    const bool in = b < M;
    // place of this lane's sample and unit i in a buffer of `units` units
    auto at = [&](int units, int i) { return ((int64_t)blockIdx.x * units + i) * 16 + s; };
    Slot w1[2], w2[2][4];
#pragma unroll
    for (int t = 0; t < 2; ++t) w1[t] = slot_at(img, 2 * w + t, lane);
    int64_t row = 0;
    if (in) row = w == 0 && g == 0 ? batch_row(idx, b, rows, err) : (idx ? idx[b] : b);
    if (row < 0 || row >= rows) row = 0;   // reported by batch_row
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) w2[t][kb] = slot_at(img, 8 + 4 * (2 * w + t) + kb, lane);
    float f[6];
    Slot u;
#pragma unroll
    for (int q = 0; q < 6; ++q) f[q] = feat[row * 6 + q];
    float tg[8];   // this lane's targets (outputs 16 (q / 4) + 4 g + q % 4)
    if constexpr (TRAIN) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int k = 16 * (q >> 2) + 4 * g + (q & 3);
            tg[q] = target[row * kMlpOut + (k < kMlpOut ? k : 0)];
        }
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        float v = 0.0f;
        if (i < kMlpIn) v = in ? (f[i] - norm[i]) * norm[6 + i] : 0.0f;
        if (TRAIN && i < kMlpIn && w == 0 && g == 0) tb.u[at(kTrainIn, i)] = v;
        __bf16 p, r;
        split_bf16(g == 0 ? v : 0.0f, p, r);
        u.hi[i] = p; u.lo[i] = r;
    }
    float g1[TRAIN ? 8 : 1], g2[TRAIN ? 8 : 1];
    // activations of this wavefront's 32 units: k block w of the next operand,
    // and in training the derivatives and stored values
    auto activate = [&](const f32x4v (&z)[2], float *gr, float *h, int to) {
        Slot o;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            float a;
            if constexpr (TRAIN) {
                a = gelu(z[q >> 2][q & 3], gr[q]);
                h[at(kMlpHidden, 32 * w + 16 * (q >> 2) + 4 * g + (q & 3))] = a;
            } else {
                a = gelu(z[q >> 2][q & 3]);
            }
            __bf16 p, r;
            split_bf16(a, p, r);
            o.hi[q] = p; o.lo[q] = r;
        }
        ops[to][w][0][lane] = o.hi;
        ops[to][w][1][lane] = o.lo;
    };
    f32x4v z[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
        z[t] = mfma3_16(w1[t], u, *reinterpret_cast<const f32x4v *>(P + kOffB1 + 32 * w + 16 * t + 4 * g));
    activate(z, g1, tb.h1, 0);
    Slot w3[TRAIN ? 2 : 1][4];   // forward only: wavefronts 0 and 1 take an output tile each
#pragma unroll
    for (int t = 0; t < (TRAIN ? 2 : 1); ++t)
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) w3[t][kb] = slot_at(img, 40 + 4 * (TRAIN ? t : (w & 1)) + kb, lane);
#pragma unroll
    for (int t = 0; t < 2; ++t) z[t] = *reinterpret_cast<const f32x4v *>(P + kOffB2 + 32 * w + 16 * t + 4 * g);
    __syncthreads();
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
        const Slot o = {ops[0][kb][0][lane], ops[0][kb][1][lane]};
#pragma unroll
        for (int t = 0; t < 2; ++t) z[t] = mfma3_16(w2[t][kb], o, z[t]);
    }
    activate(z, g2, tb.h2, 1);
    if constexpr (!TRAIN) {
        __syncthreads();
        if (w >= 2) return;
        f32x4v y;
#pragma unroll
        for (int j = 0; j < 4; ++j) y[j] = 16 * w + 4 * g + j < kMlpOut ? P[kOffB3 + 16 * w + 4 * g + j] : 0.0f;
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) y = mfma3_16(w3[0][kb], Slot{ops[1][kb][0][lane], ops[1][kb][1][lane]}, y);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = 16 * w + 4 * g + j;
            if (in && k < kMlpOut) Y[b * kMlpOut + k] = y[j];
        }
        return;
    } else {
        Slot v3[2], v2[2][4];   // W3 and W2 for the way back
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            v3[t] = slot_at(img, 48 + 2 * w + t, lane);
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) v2[t][kb] = slot_at(img, 56 + 4 * (2 * w + t) + kb, lane);
        }
        f32x4v y[2];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int k = 16 * (q >> 2) + 4 * g + (q & 3);
            y[q >> 2][q & 3] = k < kMlpOut ? P[kOffB3 + k] : 0.0f;
        }
        __syncthreads();
        // every wavefront forms all outputs (24 products more, no exchange)
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
            const Slot o = {ops[1][kb][0][lane], ops[1][kb][1][lane]};
#pragma unroll
            for (int t = 0; t < 2; ++t) y[t] = mfma3_16(w3[t][kb], o, y[t]);
        }
        // loss and dL/dy; a sample's outputs are spread over lanes s, s + 16, ...
        float sn[3][3];
        node_offsets(f, sn);
        float e[8], sx[8], sy[8], sz[8];
        float se = 0.0f, r0 = 0.0f, r1 = 0.0f, r2 = 0.0f, r3 = 0.0f;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int k = 16 * (q >> 2) + 4 * g + (q & 3);
            const bool out = k < kMlpOut;
            const float yv = out ? y[q >> 2][q & 3] : 0.0f;
            e[q] = out ? yv - tg[q] : 0.0f;
            const int ax = k % 3, ay = (k / 3) % 3, az = k / 9;
            sx[q] = ax == 0 ? sn[0][0] : (ax == 1 ? sn[0][1] : sn[0][2]);
            sy[q] = ay == 0 ? sn[1][0] : (ay == 1 ? sn[1][1] : sn[1][2]);
            sz[q] = az == 0 ? sn[2][0] : (az == 1 ? sn[2][1] : sn[2][2]);
            se += e[q] * e[q];
            r0 += yv; r1 += yv * sx[q]; r2 += yv * sy[q]; r3 += yv * sz[q];
        }
#pragma unroll
        for (int o = 16; o < 64; o <<= 1) {
            se += __shfl_xor(se, o);
            r0 += __shfl_xor(r0, o); r1 += __shfl_xor(r1, o); r2 += __shfl_xor(r2, o); r3 += __shfl_xor(r3, o);
        }
        r0 -= 1.0f;
        const float inv_m = 1.0f / (float)M;
        float l = in && g == 0 ? se * inv_m * (1.0f / kNe) + mu * inv_m * (r0 * r0 + r1 * r1 + r2 * r2 + r3 * r3) : 0.0f;
#pragma unroll
        for (int o = 1; o < 16; o <<= 1) l += __shfl_xor(l, o);
        if (w == 0 && lane == 0) tb.loss[blockIdx.x] = l;
        const float ce = 2.0f * inv_m * (1.0f / kNe), cr = 2.0f * mu * inv_m;
        Slot dy;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int k = 16 * (q >> 2) + 4 * g + (q & 3);
            const float d = in && k < kMlpOut ? ce * e[q] + cr * (r0 + r1 * sx[q] + r2 * sy[q] + r3 * sz[q]) : 0.0f;
            if (w == 0) tb.dy[at(kTrainOut, k)] = d;
            __bf16 p, r;
            split_bf16(d, p, r);
            dy.hi[q] = p; dy.lo[q] = r;
        }
        // back through the layers: d2 = (W3 dy) gelu'(z2), d1 = (W2 d2) gelu'(z1)
        Slot o;
#pragma unroll
        for (int t = 0; t < 2; ++t) z[t] = mfma3_16(v3[t], dy, f32x4v{0.f, 0.f, 0.f, 0.f});
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const float v = z[q >> 2][q & 3] * g2[q];
            tb.d2[at(kMlpHidden, 32 * w + 16 * (q >> 2) + 4 * g + (q & 3))] = v;
            __bf16 p, r;
            split_bf16(v, p, r);
            o.hi[q] = p; o.lo[q] = r;
        }
        ops[2][w][0][lane] = o.hi;
        ops[2][w][1][lane] = o.lo;
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 2; ++t) z[t] = f32x4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
            const Slot d = {ops[2][kb][0][lane], ops[2][kb][1][lane]};
#pragma unroll
            for (int t = 0; t < 2; ++t) z[t] = mfma3_16(v2[t][kb], d, z[t]);
        }
#pragma unroll
        for (int q = 0; q < 8; ++q)
            tb.d1[at(kMlpHidden, 32 * w + 16 * (q >> 2) + 4 * g + (q & 3))] = z[q >> 2][q & 3] * g1[q];
    }
}

// Weight gradients of one chunk of samples: [dW; db](i, o) = sum_s X(i, s)
// D(o, s) for RT x CT tiles of 32 x 32, with the bias gradient (the sum of D)
// by the wavefront that holds the first rows.  Operands are split as they are
// loaded; v_mfma_f32_32x32x16_bf16: lane l holds row / column l % 32 and
// samples 8 (l / 32) + i; result register j is row 8 (j / 4) + 4 (l / 32) +
// j % 4, column l % 32.
template <int RT, int CT>
__device__ __forceinline__ void wgrad_tiles(const float *__restrict__ X, int x_units, int x_rows,
                                            const float *__restrict__ D, int d_units, int64_t beg, int64_t end,
                                            float *__restrict__ W, int n_out, int stride, float *__restrict__ bias)
{
    const int lane = threadIdx.x & 63, r = lane & 31, h = lane >> 5;
    f32x16 acc[RT][CT] = {};
    float bsum[CT] = {};
    auto load8 = [&](const float *p, bool on, float (&v)[8]) {
        const float4 a = on ? *reinterpret_cast<const float4 *>(p) : make_float4(0.f, 0.f, 0.f, 0.f);
        const float4 c = on ? *reinterpret_cast<const float4 *>(p + 4) : make_float4(0.f, 0.f, 0.f, 0.f);
        v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = c.x; v[5] = c.y; v[6] = c.z; v[7] = c.w;
    };
    auto split8 = [](const float (&v)[8], bf16x8 &hi, bf16x8 &lo) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            __bf16 p, q;
            split_bf16(v[i], p, q);
            hi[i] = p; lo[i] = q;
        }
    };
    // the loads of kAhead products are in flight together
    constexpr int kAhead = 4;
    for (int64_t s0 = beg; s0 < end; s0 += 16 * kAhead) {
        float xv[kAhead][RT][8], dv[kAhead][CT][8];
#pragma unroll
        for (int n = 0; n < kAhead; ++n) {
            const int64_t blk = (s0 >> 4) + n;
            const bool on = s0 + 16 * n < end;
#pragma unroll
            for (int q = 0; q < RT; ++q) load8(X + ((blk * x_units + 32 * q + r) << 4) + 8 * h, on && 32 * q + r < x_rows, xv[n][q]);
#pragma unroll
            for (int q = 0; q < CT; ++q) load8(D + ((blk * d_units + 32 * q + r) << 4) + 8 * h, on, dv[n][q]);
        }
#pragma unroll
        for (int n = 0; n < kAhead; ++n) {
            bf16x8 dh[CT], dl[CT];
#pragma unroll
            for (int q = 0; q < CT; ++q) {
                const float(&d)[8] = dv[n][q];
                split8(d, dh[q], dl[q]);
                bsum[q] += ((d[0] + d[1]) + (d[2] + d[3])) + ((d[4] + d[5]) + (d[6] + d[7]));
            }
#pragma unroll
            for (int q = 0; q < RT; ++q) {
                bf16x8 xh, xl;
                split8(xv[n][q], xh, xl);
#pragma unroll
                for (int t = 0; t < CT; ++t) acc[q][t] = mfma3(xh, xl, dh[t], dl[t], acc[q][t]);
            }
        }
    }
#pragma unroll
    for (int q = 0; q < RT; ++q)
#pragma unroll
        for (int t = 0; t < CT; ++t)
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int i = 32 * q + 8 * (j / 4) + 4 * h + (j % 4), o = 32 * t + r;
                if (i < x_rows && o < n_out) W[(int64_t)i * stride + o] = acc[q][t][j];
            }
    if (bias) {
#pragma unroll
        for (int t = 0; t < CT; ++t) {
            const float v = bsum[t] + __shfl_xor(bsum[t], 32);
            if (h == 0 && 32 * t + r < n_out) bias[32 * t + r] = v;
        }
    }
}

// One wavefront per (job, chunk), two tiles each so that four rounds of loads
// fit the registers at once: jobs 0..7 the row tiles and column halves of dW2,
// 8 and 9 the row halves of dW3, 10 and 11 the column halves of dW1.  At most
// 64 chunks of at least 128 samples: 768 wavefronts for a batch of 8192
// (8 us).
constexpr int kWgradJobs = 12;
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(1, 2))) k_mlp_wgrad(const TrainBufs tb)
{
    // the jobs of a chunk run on one XCD (workgroup b runs on XCD b % 8), whose
    // L2 then reads the chunk from memory once instead of all eight (9.4 -> 7.9
    // us for a batch of 8192)
    const int job = (blockIdx.x >> 3) % kWgradJobs, ch = (blockIdx.x >> 3) / kWgradJobs * 8 + (blockIdx.x & 7);
    if (ch >= tb.chunks) return;
    const int64_t beg = (int64_t)ch * tb.chunk, end = min(beg + tb.chunk, tb.Mp);
    float *P = tb.part + (int64_t)ch * kPartStride;
    if (job < 8) {
        const int i0 = (job & 3) * 32, o0 = (job >> 2) * 64;
        wgrad_tiles<1, 2>(tb.h1 + i0 * 16, kMlpHidden, 32, tb.d2 + o0 * 16, kMlpHidden, beg, end,
                          P + kOffW2 + i0 * kMlpHidden + o0, 64, kMlpHidden, i0 == 0 ? P + kOffB2 + o0 : nullptr);
    } else if (job < 10) {
        const int i0 = (job - 8) * 64;
        wgrad_tiles<2, 1>(tb.h2 + i0 * 16, kMlpHidden, 64, tb.dy, kTrainOut, beg, end, P + kOffW3 + i0 * kMlpOut,
                          kMlpOut, kMlpOut, i0 == 0 ? P + kOffB3 : nullptr);
    } else {
        const int o0 = (job - 10) * 64;
        wgrad_tiles<1, 2>(tb.u, kTrainIn, kMlpIn, tb.d1 + o0 * 16, kMlpHidden, beg, end, P + kOffW1 + o0, 64,
                          kMlpHidden, P + kOffB1 + o0);
    }
}

// Adam (Kingma & Ba, 2015): learning rate, betas, bias corrections 1 - beta^t.
struct AdamArgs {
    float *p, *m1, *m2;
    __bf16 *img;
    float lr, b1, b2, eps, c1, c2;
};

// Sums the chunks of every parameter's gradient: four threads a quarter of the
// chunks each, in order, then the quarters in order (one thread per parameter
// waits for 64 loads in a row, 8 us instead of 5).  ADAM: updates the parameter
// and its places in the packed operands; else stores the gradient.  The last
// workgroup sums the loss (each thread a strided share in order, then a fixed
// tree).
constexpr int kUpdateBlock = 256;
template <bool ADAM>
__global__ void __launch_bounds__(kUpdateBlock)
k_mlp_update(const TrainBufs tb, float *__restrict__ grad, const AdamArgs ad, float *__restrict__ loss)
{
    __shared__ float sh[kUpdateBlock];
    if (blockIdx.x == gridDim.x - 1) {
        float a = 0.0f;
        for (int64_t i = threadIdx.x; i < tb.Mp / 16; i += kUpdateBlock) a += tb.loss[i];
        sh[threadIdx.x] = a;
        for (int o = kUpdateBlock / 2; o > 0; o >>= 1) {
            __syncthreads();
            if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        }
        if (threadIdx.x == 0) *loss = sh[0];
        return;
    }
    const int p = blockIdx.x * 64 + (threadIdx.x & 63), quarter = threadIdx.x >> 6;
    const int per = (tb.chunks + 3) / 4;
    const int c0 = quarter * per, c1 = min(c0 + per, tb.chunks);
    float sum = 0.0f;   // (rows of kPartStride floats, a multiple of 64: p is in bounds)
#pragma unroll 16
    for (int c = c0; c < c1; ++c) sum += tb.part[(int64_t)c * kPartStride + p];
    sh[threadIdx.x] = sum;
    __syncthreads();
    if (quarter > 0 || p >= kMlpParams) return;
    const float gi = ((sh[p & 63] + sh[64 + (p & 63)]) + sh[128 + (p & 63)]) + sh[192 + (p & 63)];
    if constexpr (!ADAM) {
        grad[p] = gi;
    } else {
        const float a = ad.b1 * ad.m1[p] + (1.0f - ad.b1) * gi;
        const float q = ad.b2 * ad.m2[p] + (1.0f - ad.b2) * gi * gi;
        ad.m1[p] = a;
        ad.m2[p] = q;
        const float v = ad.p[p] - ad.lr * (a / ad.c1) / (sqrtf(q / ad.c2) + ad.eps);
        ad.p[p] = v;
        pack_train(ad.img, p, v);
    }
}

// Features of every (component, marker): feat[(c n + l) 6 + q] = xi_x, xi_y,
// xi_z, rho_x, rho_y, rho_z of component c's support; NaN (and a device
// error) if the support leaves the grid.
__global__ void __launch_bounds__(kBlock)
k_features(const Grid *__restrict__ gp, int64_t n, const float *__restrict__ x, const float *__restrict__ y,
           const float *__restrict__ z, float *__restrict__ feat, ErrWord *err)
{
    const Grid &g = *gp;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < 3 * n; i += (int64_t)gridDim.x * blockDim.x) {
        const int c = (int)(i / n);
        const int64_t l = i - (int64_t)c * n;
        const double px = (double)x[l], py = (double)y[l], pz = (double)z[l];
        AxisGeo G[3];
        bool ok = axis_geo(g.ax[0], c == 0, px, G[0]);
        ok = ok && axis_geo(g.ax[1], c == 1, py, G[1]);
        ok = ok && axis_geo(g.ax[2], c == 2, pz, G[2]);
        float *f = feat + i * 6;
        if (!ok) {
            raise_error(err, l, isfinite(px) && isfinite(py) && isfinite(pz) ? MLS_E_SUPPORT : MLS_E_NONFINITE);
            for (int q = 0; q < 6; ++q) f[q] = __builtin_nanf("");
            continue;
        }
        f[0] = G[0].xi; f[1] = G[1].xi; f[2] = G[2].xi;
        f[3] = G[0].rho; f[4] = G[1].rho; f[5] = G[2].rho;
    }
}

// ---- inference image ---------------------------------------------------------
// Slot s of the image is (layer, output tile T, k block kb): layer 1 slots
// 0..3 (T), layer 2 slots 4 + 8 T + kb, layer 3 slots 36 + kb.  For lane l the
// A operand holds output row o = 32 T + l % 32 and, in its eight k slots, the
// inputs
//   layer 1:     8 (l / 32) + i                        (features, 6 used)
//   layers 2, 3: 32 (kb / 2) + 16 (kb % 2) + 8 (i / 4) + 4 (l / 32) + i % 4,
// the order in which the previous layer's result registers hold the hidden
// units (register j of tile T is unit 32 T + 8 (j / 4) + 4 (l / 32) + j % 4),
// so those registers serve directly as the next B operand.
__device__ __forceinline__ int layer_input(int layer, int kb, int h, int i)
{
    if (layer == 1) return 8 * h + i;
    return 32 * (kb / 2) + 16 * (kb % 2) + 8 * (i / 4) + 4 * h + (i % 4);
}

__global__ void k_pack(const float *__restrict__ P, const float *__restrict__ norm, uint4 *__restrict__ ops,
                       float *__restrict__ tail)
{
    const int tid = blockIdx.x * blockDim.x + threadIdx.x;
    if (tid < kMlpImageOps) {
        const int lane = tid & 63, part = (tid >> 6) & 1, slot = tid >> 7;
        int layer, T, kb;
        if (slot < 4) { layer = 1; T = slot; kb = 0; }
        else if (slot < 36) { layer = 2; T = (slot - 4) / 8; kb = (slot - 4) % 8; }
        else { layer = 3; T = 0; kb = slot - 36; }
        const int o = 32 * T + (lane & 31), h = lane >> 5;
        uint32_t v16[8];
        for (int i = 0; i < 8; ++i) {
            const int in = layer_input(layer, kb, h, i);
            float v = 0.0f;
            if (layer == 1) v = in < kMlpIn ? P[kOffW1 + in * kMlpHidden + o] : 0.0f;
            else if (layer == 2) v = P[kOffW2 + in * kMlpHidden + o];
            else v = o < kMlpOut ? P[kOffW3 + in * kMlpOut + o] : 0.0f;
            __bf16 hi, lo;
            split_bf16(v, hi, lo);
            const __bf16 sel = part ? lo : hi;
            v16[i] = (uint32_t)__builtin_bit_cast(uint16_t, sel);
        }
        ops[tid] = make_uint4(v16[0] | v16[1] << 16, v16[2] | v16[3] << 16, v16[4] | v16[5] << 16,
                              v16[6] | v16[7] << 16);
    }
    if (tid < kMlpImageFloats) {
        float v;
        if (tid < kMlpHidden) v = P[kOffB1 + tid];
        else if (tid < 2 * kMlpHidden) v = P[kOffB2 + tid - kMlpHidden];
        else if (tid < 2 * kMlpHidden + 32)
            v = (tid - 2 * kMlpHidden) < kMlpOut ? P[kOffB3 + tid - 2 * kMlpHidden] : 0.0f;
        else v = norm[tid - 2 * kMlpHidden - 32];
        tail[tid] = v;
    }
}

// ---- fused learned build -----------------------------------------------------

__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

__device__ __forceinline__ bf16x8 op_at(const uint4 *img, int slot, int part, int lane)
{
    return __builtin_bit_cast(bf16x8, img[(slot * 2 + part) * 64 + lane]);
}

// Accumulator initialised with the bias of output tile T in result layout.
__device__ __forceinline__ f32x16 bias_tile(const float *b, int T, int h)
{
    f32x16 acc;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float4 v = *reinterpret_cast<const float4 *>(b + 32 * T + 8 * q + 4 * h);
        acc[4 * q + 0] = v.x; acc[4 * q + 1] = v.y; acc[4 * q + 2] = v.z; acc[4 * q + 3] = v.w;
    }
    return acc;
}

// gelu(z) = max(z, 0) - |z| Q(|z|) from the cubic table of the network image
// (inference only; training keeps the closed form above).  Beyond |z| = 6 the
// last interval's end value, 6 Q(6) < 6e-9, stands in for |z| Q(|z|).
// gelu_rows reads the table rows of result registers 8 q .. 8 q + 7;
// gelu_operand makes their GELU the split B operand of the next layer.
struct GeluRows {
    float4 c[8];
    float s[8];
};
__device__ __forceinline__ GeluRows gelu_rows(const f32x16 &acc, int q, const float4 *tab)
{
    GeluRows r;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float t = fminf(fabsf(acc[8 * q + i]) * (float)kGeluPerUnit, 95.99999f);
        r.c[i] = tab[(int)t];
        r.s[i] = __builtin_amdgcn_fractf(t);
    }
    return r;
}

__device__ __forceinline__ void gelu_operand(const f32x16 &acc, int q, const GeluRows &r, bf16x8 &hi, bf16x8 &lo)
{
    // max(z, 0) is taken as z - min(z, 0), which passes a NaN argument on to
    // the result, and min(z, 0) as the median of z, 0 and -infinity (the lower
    // of the others for a NaN; hidden from the compiler, which would make it a
    // minimum and quiet its argument with a further operation)
    float low = -__builtin_inff();
    asm("" : "+s"(low));
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float z = acc[8 * q + i], t = r.s[i];
        const float p = fmaf(fmaf(fmaf(r.c[i].w, t, r.c[i].z), t, r.c[i].y), t, r.c[i].x);
        v[i] = (z - __builtin_amdgcn_fmed3f(z, 0.0f, low)) - p;
    }
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
        bf16x2 p, l;
        split_bf16_pair(v[i], v[i + 1], p, l);
        hi[i] = p.x; hi[i + 1] = p.y;
        lo[i] = l.x; lo[i + 1] = l.y;
    }
}

// Network output for the 32 markers whose features lane l % 32 holds (ft);
// returns the 32 x 32 result tile (rows 0..26 are the outputs).
__device__ __forceinline__ f32x16 evaluate(const uint4 *img, const float *b1, const float *b2, const float *b3,
                                           const float *norm, const float4 *tab, const float ft[6], int lane)
{
    const int h = lane >> 5;
    bf16x8 uh, ul;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        float v = 0.0f;
        if (i < kMlpIn) v = (ft[i] - norm[i]) * norm[6 + i];
        v = h ? 0.0f : v;
        __bf16 p, r;
        split_bf16(v, p, r);
        uh[i] = p; ul[i] = r;
    }
    // Layer 2 is accumulated k block by k block: each 32-unit tile of layer 1
    // is computed, activated and consumed by the four layer-2 output tiles
    // at once, so only its own registers are live instead of all of layer 1.
    // The matrix products of a step are issued between the vector operations
    // that activate the next step's operand: a product occupies the matrix
    // core for as long as eight of them take to issue, a wavefront issues in
    // order, and with two wavefronts per SIMD (the network image and the staged
    // rows fill the LDS) nothing else fills the gaps.  Each accumulator sums
    // its k blocks in order.  Learned step of 2.56e6 markers in the channel:
    // 2460 us as the compiler ordered it (two table reads, then a wait, 64
    // times), 2430 with a step's table rows and operands requested together,
    // 2365 interleaved.
    f32x16 acc[4];
#pragma unroll
    for (int T = 0; T < 4; ++T) acc[T] = bias_tile(b2, T, h);
    f32x16 a = bias_tile(b1, 0, h);
    a = mfma3(op_at(img, 0, 0, lane), op_at(img, 0, 1, lane), uh, ul, a);
    bf16x8 bh, bl;
    gelu_operand(a, 0, gelu_rows(a, 0, tab), bh, bl);
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        // operand of the next step: the other half of this tile, or the first
        // half of the next
        f32x16 an = a;
        if ((s & 1) && s < 7) {
            const int T1 = (s + 1) / 2;
            an = bias_tile(b1, T1, h);
            an = mfma3(op_at(img, T1, 0, lane), op_at(img, T1, 1, lane), uh, ul, an);
        }
        bf16x8 wh[4], wl[4], nh, nl;
#pragma unroll
        for (int T = 0; T < 4; ++T) {
            wh[T] = op_at(img, 4 + 8 * T + s, 0, lane);
            wl[T] = op_at(img, 4 + 8 * T + s, 1, lane);
        }
        GeluRows rows;
        if (s < 7) rows = gelu_rows(an, (s + 1) & 1, tab);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int T = 0; T < 4; ++T) acc[T] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wh[T], bh, acc[T], 0, 0, 0);
#pragma unroll
        for (int T = 0; T < 4; ++T) acc[T] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wh[T], bl, acc[T], 0, 0, 0);
#pragma unroll
        for (int T = 0; T < 4; ++T) acc[T] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wl[T], bh, acc[T], 0, 0, 0);
        if (s < 7) {
            gelu_operand(an, (s + 1) & 1, rows, nh, nl);
#pragma unroll
            for (int k = 0; k < 12; ++k) {
                __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x2, 7, 0);
            }
            bh = nh; bl = nl;
            a = an;
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    f32x16 y3 = bias_tile(b3, 0, h);
    gelu_operand(acc[0], 0, gelu_rows(acc[0], 0, tab), bh, bl);
#pragma unroll
    for (int s = 0; s < 8; ++s) {
        const bf16x8 wh = op_at(img, 36 + s, 0, lane), wl = op_at(img, 36 + s, 1, lane);
        GeluRows rows;
        bf16x8 nh, nl;
        if (s < 7) rows = gelu_rows(acc[(s + 1) / 2], (s + 1) & 1, tab);
        __builtin_amdgcn_sched_barrier(0);
        y3 = mfma3(wh, wl, bh, bl, y3);
        if (s < 7) {
            gelu_operand(acc[(s + 1) / 2], (s + 1) & 1, rows, nh, nl);
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x2, 24, 0);
            }
            bh = nh; bl = nl;
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    return y3;
}

// Rows of one wavefront staged in LDS for the fused interpolation (after the
// network image): 27 values of 64 rows, node-major like the stored rows.
constexpr size_t kLearnStageBytes = (size_t)(kLearnBlock / 64) * kNe * 64 * sizeof(float);

__global__ void __launch_bounds__(kLearnBlock)
k_build_learned(const Grid *__restrict__ gp, const Weight W, float tau, float tol, int64_t n,
                const float *__restrict__ x, const float *__restrict__ y, const float *__restrict__ z,
                const uint4 *__restrict__ image, uint32_t *__restrict__ home, float *__restrict__ phi,
                uint8_t *__restrict__ route, ErrWord *err, DevStats *st, const uint32_t *__restrict__ order,
                const LearnedInterp li)
{
    extern __shared__ uint4 lds[];
    // the GELU table in a static LDS array (placed first, so its rows are
    // addressed with small immediate offsets)
    __shared__ float4 tab[kGeluIntervals];
    constexpr int kWords = (int)(kMlpImageBytes / 16);
    for (int i = threadIdx.x; i < kWords; i += kLearnBlock) lds[i] = image[i];
    if (threadIdx.x < kGeluIntervals)
        tab[threadIdx.x] = reinterpret_cast<const float4 *>(reinterpret_cast<const char *>(image) +
                                                            kMlpImageTableOffset)[threadIdx.x];
    __syncthreads();
    const float *b1 = reinterpret_cast<const float *>(lds + kMlpImageOps);
    const float *b2 = b1 + kMlpHidden, *b3 = b2 + kMlpHidden, *norm = b3 + 32;

    const Grid &g = *gp;
    const int lane = threadIdx.x & 63, h = lane >> 5, r = lane & 31;
    float *const stage = reinterpret_cast<float *>(reinterpret_cast<char *>(lds) + kMlpImageBytes) +
                         wave_id() * (kNe * 64);
    const int64_t items = ((n + 63) >> 6) * 3;
    const int64_t wstride = (int64_t)gridDim.x * (kLearnBlock / 64);
    unsigned long long routed = 0, n_fb = 0, n_ok = 0;
    float kmax = 0.0f;
    for (int64_t it = (int64_t)blockIdx.x * (kLearnBlock / 64) + wave_id(); it < items; it += wstride) {
        const int64_t blk = it / 3;
        const int c = (int)(it - blk * 3);
        const int64_t l = (blk << 6) + lane;
        // the marker of row l (rows in tile order in the time step)
        const int64_t mk = l < n ? (order ? (int64_t)order[l] : l) : 0;
        float *out = phi + (((blk * 3 + c) * kNe) << 6);          // + k * 64 + marker in block
        uint32_t *hout = home + ((blk * 3 + c) << 6) + lane;
        uint8_t *rout = route ? route + ((blk * 3 + c) << 6) : nullptr;
        float f[6] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        bool ok = false;
        uint32_t hv = 0xffffffffu;
        if (l < n) {
            const double px = (double)x[mk], py = (double)y[mk], pz = (double)z[mk];
            AxisGeo G[3];
            ok = axis_geo(g.ax[0], c == 0, px, G[0]);
            ok = ok && axis_geo(g.ax[1], c == 1, py, G[1]);
            ok = ok && axis_geo(g.ax[2], c == 2, pz, G[2]);
            if (!ok) {
                mark_failed(err, mk, px, py, pz, hout, out + lane, rout ? rout + lane : nullptr);
            } else {
                hv = pack_home(G[0].ih, G[1].ih, G[2].ih);
                *hout = hv;
                f[0] = G[0].xi; f[1] = G[1].xi; f[2] = G[2].xi;
                f[3] = G[0].rho; f[4] = G[1].rho; f[5] = G[2].rho;
            }
        }
        const unsigned long long good = __ballot(ok);
        unsigned long long accept = 0;
#pragma unroll 1
        for (int t = 0; t < 2; ++t) {
            const uint32_t gt = (uint32_t)(good >> (32 * t));
            if (gt == 0) continue;
            const int src = 32 * t + r;
            float ft[6];
#pragma unroll
            for (int q = 0; q < 6; ++q) ft[q] = __shfl(f[q], src);
            const f32x16 yv = evaluate(lds, b1, b2, b3, norm, tab, ft, lane);
            // consistency residuals; a marker's outputs are split between lanes r and r + 32
            float s[3][3];
            node_offsets(ft, s);
            float sy = 0.0f, r1x = 0.0f, r1y = 0.0f, r1z = 0.0f;
            // the offsets of a row are picked by a bit mask on h, so that the
            // array stays in registers (a select of two elements would become
            // a select of two addresses and put the array in scratch)
            const uint32_t hm = h ? 0xffffffffu : 0u;
            auto pick = [hm](float a0, float a1) {
                return __builtin_bit_cast(float, (__builtin_bit_cast(uint32_t, a1) & hm) |
                                                     (__builtin_bit_cast(uint32_t, a0) & ~hm));
            };
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const int k0 = 8 * (j / 4) + (j % 4), k1 = k0 + 4;   // output row for h = 0, 1
                const int kk1 = k1 < kNe ? k1 : 0;
                const bool valid = h ? (k1 < kNe) : true;
                const float sx = pick(s[0][k0 % 3], s[0][kk1 % 3]);
                const float sv = pick(s[1][(k0 / 3) % 3], s[1][(kk1 / 3) % 3]);
                const float sz = pick(s[2][k0 / 9], s[2][kk1 / 9]);
                const float yj = valid ? yv[j] : 0.0f;
                sy += yj;
                r1x += yj * sx;
                r1y += yj * sv;
                r1z += yj * sz;
            }
            sy += __shfl_xor(sy, 32);
            r1x += __shfl_xor(r1x, 32);
            r1y += __shfl_xor(r1y, 32);
            r1z += __shfl_xor(r1z, 32);
            const float res = fmaxf(fmaxf(fabsf(sy - 1.0f), fabsf(r1x)), fmaxf(fabsf(r1y), fabsf(r1z)));
            const bool pass = ((gt >> r) & 1u) && res < tol;   // NaN fails
            if (pass) {
#pragma unroll
                for (int j = 0; j < 16; ++j) {
                    const int k = 8 * (j / 4) + 4 * h + (j % 4);
                    if (k < kNe) {
                        out[k * kLanes + 32 * t + r] = yv[j];
                        if (li.U) stage[k * 64 + 32 * t + r] = yv[j];
                    }
                }
                if (rout && h == 0) rout[32 * t + r] = 2;
            }
            const unsigned long long pb = __ballot(pass);
            accept |= (pb & 0xffffffffull) << (32 * t);
        }
        const unsigned long long rej = good & ~accept;
        n_ok += (unsigned long long)__popcll(accept);
        n_fb += (unsigned long long)__popcll(rej);
        if ((rej >> lane) & 1ull) {
            const double px = (double)x[mk], py = (double)y[mk], pz = (double)z[mk];
            AxisGeo G[3];
            axis_geo(g.ax[0], c == 0, px, G[0]);
            axis_geo(g.ax[1], c == 1, py, G[1]);
            axis_geo(g.ax[2], c == 2, pz, G[2]);
            float ph[kNe];
            exact_from_geo(g, W, tau, c, mk, px, py, pz, G, out + lane, rout ? rout + lane : nullptr, 4, err, routed,
                           kmax, ph);
            if (li.U) {
#pragma unroll
                for (int k = 0; k < kNe; ++k) stage[k * 64 + lane] = ph[k];
            }
        }
        if (li.U) {
            // Interpolation (eq. 6), direct forcing and c_l F_l (eq. 8) of the
            // rows just built, from the wavefront's LDS copy of them: the same
            // arithmetic as interpolating the stored rows, without reading
            // them back from memory.  U and F go out by marker, c_l F_l by row,
            // and the largest |c_l F_l| per spreading tile into tmax.
            __builtin_amdgcn_s_waitcnt(0xc07f);   // lgkmcnt(0): this wavefront's LDS writes are done
            __builtin_amdgcn_wave_barrier();
            asm volatile("" ::: "memory");
            const bool in = l < n;
            float acc = __builtin_nanf(""), fo = __builtin_nanf(""), cfv = 0.0f;
            if (ok) {
                int i, j, k;
                unpack_home(hv, i, j, k);
                const float *q = c == 0 ? li.u : (c == 1 ? li.v : li.w);
                uint32_t oy[3], oz[3];
                support_rows(j, k, g.dims[c][0], g.dims[c][1], g.dims[c][2], oy, oz);
                float qv[kNe];
                load_rows(q, i, g.dims[c][0], oy, oz, qv);
                float ph[kNe];
#pragma unroll
                for (int kk = 0; kk < kNe; ++kk) ph[kk] = stage[kk * 64 + lane];
                wrap_rows(q, i, j, k, g.dims[c][0], g.dims[c][1], g.dims[c][2], qv);
                acc = 0.0f;
#pragma unroll
                for (int kk = 0; kk < kNe; ++kk) acc += ph[kk] * qv[kk];
                const float vbv = li.vb ? li.vb[c * n + mk] : 0.0f;
                fo = (vbv - acc) * li.inv_dt;
                cfv = eq8_coef_built(g, c, i, j, k, ph, li.area[mk] * fo);
                if (!(fabsf(cfv) <= 3.0e38f)) raise_error(err, mk, MLS_E_RANGE);
            }
            if (in) {
                li.U[c * n + mk] = acc;
                li.F[c * n + mk] = fo;
                li.cf[c * li.cf_stride + l] = ok ? cfv : 0.0f;
            }
            const uint32_t tl = in ? li.tile_of_marker[mk] : (uint32_t)g.ntiles;
            wave_key_max(li.tmax + c * li.tstride, ok && tl < (uint32_t)g.ntiles ? (int64_t)tl : -1,
                         finite_abs(cfv));
            // the next item's stage writes come after every lane's reads
            __builtin_amdgcn_s_waitcnt(0xc07f);
            __builtin_amdgcn_wave_barrier();
            asm volatile("" ::: "memory");
        }
    }
    wave_stats(st, routed, kmax);
    if (lane == 0) {
        DevStats &d = stat_slot(st);
        if (n_fb) atomicAdd(&d.fallbacks, n_fb);
        if (n_ok) atomicAdd(&d.learned, n_ok);
    }
}

int grid_for(int64_t work, int cu)
{
    int64_t b = (work + kBlock - 1) / kBlock;
    const int64_t cap = (int64_t)cu * 32;
    if (b > cap) b = cap;
    return (int)(b < 1 ? 1 : b);
}

}  // namespace

// ---- host side ---------------------------------------------------------------

// The inference GELU table: f(a) = a Q(a), Q(a) = erfc(a / sqrt 2) / 2, on
// intervals of width 1/16 as cubic Hermite pieces in s = 16 a - i (value and
// derivative f'(a) = Q(a) - a phi(a) matched at both ends), in FP64.
static void gelu_table(float *t)
{
    auto f = [](double a) { return 0.5 * a * std::erfc(a * 0.70710678118654752440); };
    auto df = [](double a) {
        return 0.5 * std::erfc(a * 0.70710678118654752440) - a * std::exp(-0.5 * a * a) * 0.39894228040143267794;
    };
    const double h = 1.0 / kGeluPerUnit;
    for (int i = 0; i < kGeluIntervals; ++i) {
        const double a0 = i * h, a1 = (i + 1) * h;
        const double f0 = f(a0), f1 = f(a1), d0 = df(a0) * h, d1 = df(a1) * h;
        t[4 * i + 0] = (float)f0;
        t[4 * i + 1] = (float)d0;
        t[4 * i + 2] = (float)(3.0 * (f1 - f0) - 2.0 * d0 - d1);
        t[4 * i + 3] = (float)(2.0 * (f0 - f1) + d0 + d1);
    }
}

hipError_t mlp_alloc(Ctx &c)
{
    Mlp &net = c.mlp;
    if (net.params) return hipSuccess;
    const size_t floats = 3 * (size_t)kMlpParams + 12 + 4;
    const size_t head = (floats * sizeof(float) + 255) & ~(size_t)255;
    char *block = nullptr;
    const size_t image = (kMlpImageBytes + 255) & ~(size_t)255;
    hipError_t e = hipMalloc((void **)&block, head + image + kTrainImageBytes);
    if (e != hipSuccess) return e;
    float *fp = reinterpret_cast<float *>(block);
    net.params = fp;
    net.m1 = fp + kMlpParams;
    net.m2 = fp + 2 * kMlpParams;
    net.norm = fp + 3 * kMlpParams;
    net.loss = net.norm + 12;
    net.image = block + head;
    net.train_image = block + head + image;
    e = hipMemset(net.train_image, 0, kTrainImageBytes);   // slots of no parameter stay zero
    if (e != hipSuccess) {
        hipFree(block);
        net.params = nullptr;
        return e;
    }
    float tab[4 * kGeluIntervals];
    gelu_table(tab);
    e = hipMemcpy(static_cast<char *>(net.image) + kMlpImageTableOffset, tab, sizeof(tab), hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        hipFree(block);
        net.params = nullptr;
        return e;
    }
    return hipFuncSetAttribute((const void *)k_build_learned, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)(kMlpImageBytes + kLearnStageBytes));
}

void mlp_free(Ctx &c)
{
    Mlp &net = c.mlp;
    if (net.params) hipFree(net.params);
    if (net.scratch) hipFree(net.scratch);
    net = Mlp{};
}

hipError_t mlp_pack(Ctx &c, hipStream_t s)
{
    Mlp &net = c.mlp;
    uint4 *ops = static_cast<uint4 *>(net.image);
    float *tail = reinterpret_cast<float *>(ops + kMlpImageOps);
    hipLaunchKernelGGL(k_pack, dim3((kMlpImageOps + kBlock - 1) / kBlock), dim3(kBlock), 0, s, net.params, net.norm,
                       ops, tail);
    net.image_version = net.version;
    return hipGetLastError();
}

LearnedInterp learned_interp(const Ctx &c, const float *u, const float *v, const float *w, const float *vb,
                             const float *area, float dt, float *U, float *F)
{
    LearnedInterp li;
    li.u = u; li.v = v; li.w = w; li.vb = vb; li.area = area;
    li.inv_dt = 1.0f / dt;
    li.U = U; li.F = F;
    li.cf = c.cf_rows; li.cf_stride = c.cf_stride;
    li.tile_of_marker = c.marker_tile;
    li.tmax = c.tile_fmax; li.tstride = c.g.ntiles + 1;
    return li;
}

hipError_t launch_build_learned(Ctx &c, int64_t n, const float *x, const float *y, const float *z, uint32_t *home,
                                float *phi, uint8_t *route, hipStream_t s, const uint32_t *order,
                                const LearnedInterp *interp)
{
    if (n == 0) return hipSuccess;
    Mlp &net = c.mlp;
    if (net.image_version != net.version) {
        hipError_t e = mlp_pack(c, s);
        if (e != hipSuccess) return e;
    }
    const float tau = (float)(c.opts.kappa_tau > 3.0e38 ? 3.0e38 : c.opts.kappa_tau);
    const float tol = (float)(c.opts.fallback_tol > 3.0e38 ? 3.0e38 : c.opts.fallback_tol);
    const int64_t waves = ((n + 63) / 64) * 3;
    int64_t blocks = (waves + kLearnBlock / 64 - 1) / (kLearnBlock / 64);
    if (blocks > c.cu_count) blocks = c.cu_count;
    const LearnedInterp li = interp ? *interp : LearnedInterp{};
    hipLaunchKernelGGL(k_build_learned, dim3((unsigned)blocks), dim3(kLearnBlock),
                       kMlpImageBytes + (li.U ? kLearnStageBytes : 0), s, c.d_grid, c.w, tau, tol, n, x, y, z,
                       static_cast<const uint4 *>(net.image), home, phi, route, c.err, c.stats, order, li);
    return hipGetLastError();
}

hipError_t launch_features(const Ctx &c, int64_t n, const float *x, const float *y, const float *z, float *feat,
                           hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_features, dim3(grid_for(3 * n, c.cu_count)), dim3(kBlock), 0, s, c.d_grid, n, x, y, z,
                       feat, c.err);
    return hipGetLastError();
}

// Samples of a batch as the training buffers hold them, and its chunks.
static int64_t train_pad(int64_t M) { return (M + 31) / 32 * 32; }
static int train_chunk(int64_t Mp)
{
    const int64_t c = std::max<int64_t>(128, (Mp + 63) / 64);
    return (int)((c + 31) / 32 * 32);
}

static size_t train_floats(int64_t M)
{
    const int64_t Mp = train_pad(M);
    const int64_t chunks = (Mp + train_chunk(Mp) - 1) / train_chunk(Mp);
    return (size_t)(Mp * (kTrainIn + 4 * kMlpHidden + kTrainOut) + chunks * kPartStride + Mp / 16 + 64);
}

static TrainBufs train_bufs(const Ctx &c, int64_t M)
{
    TrainBufs t;
    t.Mp = train_pad(M);
    t.chunk = train_chunk(t.Mp);
    t.chunks = (int)((t.Mp + t.chunk - 1) / t.chunk);
    t.u = c.mlp.scratch;
    t.h1 = t.u + kTrainIn * t.Mp;
    t.h2 = t.h1 + kMlpHidden * t.Mp;
    t.d1 = t.h2 + kMlpHidden * t.Mp;
    t.d2 = t.d1 + kMlpHidden * t.Mp;
    t.dy = t.d2 + kMlpHidden * t.Mp;
    t.part = t.dy + kTrainOut * t.Mp;
    t.loss = t.part + (int64_t)t.chunks * kPartStride;
    return t;
}

hipError_t mlp_reserve(Ctx &c, int64_t M)
{
    Mlp &net = c.mlp;
    if (M <= net.cap_batch) return hipSuccess;
    hipError_t e = hipDeviceSynchronize();
    if (e != hipSuccess) return e;
    ++c.scratch_gen;
    if (net.scratch) hipFree(net.scratch);
    net.scratch = nullptr;
    net.cap_batch = 0;
    // enough for any smaller batch too: its samples take less, its chunks at most 64
    const size_t floats = train_floats(M) + (size_t)64 * kPartStride;
    e = hipMalloc((void **)&net.scratch, floats * sizeof(float));
    if (e != hipSuccess) return e;
    net.cap_batch = M;
    return hipSuccess;
}

// Packs the parameters into the training kernels' operands (the image follows
// the parameters at all times: the update refreshes it as it goes, a load packs
// it anew, so every pass, captured or not, reads the current weights).
hipError_t mlp_pack_train(Ctx &c, hipStream_t s)
{
    Mlp &net = c.mlp;
    hipLaunchKernelGGL(k_pack_train, dim3((kMlpParams + kBlock - 1) / kBlock), dim3(kBlock), 0, s, net.params,
                       static_cast<__bf16 *>(net.train_image));
    return hipGetLastError();
}

hipError_t mlp_forward_batch(Ctx &c, int64_t M, const float *feat, int64_t rows, const int64_t *idx, float *Yout,
                             hipStream_t s)
{
    if (M == 0) return hipSuccess;
    Mlp &net = c.mlp;
    hipLaunchKernelGGL(k_mlp_pass<false>, dim3((unsigned)((M + 15) / 16)), dim3(64 * kPassWaves), 0, s, M, feat,
                       rows, idx, net.norm, net.params, static_cast<const uint4 *>(net.train_image), nullptr, 0.0f, Yout,
                       TrainBufs{}, c.err);
    return hipGetLastError();
}

// Forward, backward and the chunks of the weight gradients of a batch.
static TrainBufs launch_train_pass(Ctx &c, int64_t M, const float *feat, const float *target, int64_t rows,
                                   const int64_t *idx, float mu, hipStream_t s)
{
    Mlp &net = c.mlp;
    const TrainBufs tb = train_bufs(c, M);
    hipLaunchKernelGGL(k_mlp_pass<true>, dim3((unsigned)(tb.Mp / 16)), dim3(64 * kPassWaves), 0, s, M, feat, rows,
                       idx, net.norm, net.params, static_cast<const uint4 *>(net.train_image), target, mu, nullptr, tb, c.err);
    hipLaunchKernelGGL(k_mlp_wgrad, dim3((unsigned)(kWgradJobs * round_up8(tb.chunks))), dim3(64), 0, s, tb);
    return tb;
}

constexpr unsigned kUpdateBlocks = (kMlpParams + 63) / 64 + 1;   // and one for the loss

hipError_t mlp_grad_batch(Ctx &c, int64_t M, const float *feat, const float *target, int64_t rows,
                          const int64_t *idx, float mu, float *grad, float *loss, hipStream_t s)
{
    if (M == 0) return hipSuccess;
    const TrainBufs tb = launch_train_pass(c, M, feat, target, rows, idx, mu, s);
    hipLaunchKernelGGL(k_mlp_update<false>, dim3(kUpdateBlocks), dim3(kUpdateBlock), 0, s, tb, grad, AdamArgs{}, loss);
    return hipGetLastError();
}

hipError_t mlp_train_batch(Ctx &c, int64_t M, const float *feat, const float *target, int64_t rows,
                           const int64_t *idx, float mu, float lr, float *loss, hipStream_t s)
{
    if (M == 0) return hipSuccess;
    Mlp &net = c.mlp;
    const TrainBufs tb = launch_train_pass(c, M, feat, target, rows, idx, mu, s);
    net.adam_step += 1;
    const double b1 = 0.9, b2 = 0.999;
    AdamArgs ad;
    ad.p = net.params; ad.m1 = net.m1; ad.m2 = net.m2;
    ad.img = static_cast<__bf16 *>(net.train_image);
    ad.lr = lr; ad.b1 = (float)b1; ad.b2 = (float)b2; ad.eps = 1e-8f;
    ad.c1 = (float)(1.0 - std::pow(b1, (double)net.adam_step));
    ad.c2 = (float)(1.0 - std::pow(b2, (double)net.adam_step));
    hipLaunchKernelGGL(k_mlp_update<true>, dim3(kUpdateBlocks), dim3(kUpdateBlock), 0, s, tb, nullptr, ad, loss);
    net.version += 1;
    return hipGetLastError();
}

}  // namespace mls
