// Derivative shape functions: the gradient, with respect to the marker
// position, of the exact MLS approximation of eq. 6 (the weights, and so A
// and B, move with the marker), and the cell-centred staggering of the
// pressure.  These give velocity gradients and pressure at the markers, the
// further MLS operations that moving and deforming bodies need.
//
// In the marker-centred basis p = [1, s] (s = (node - x)/H) with
// gamma = A^-1 e0, beta_d = A^-1 e_{1+d} and eta_d = A^-1 dA_d gamma,
//   phi_k = W_k (gamma . p_k),
//   d phi_k / d xi_d = dW_dk (gamma . p_k) + W_k ((beta_d - eta_d) . p_k),
// where dW_dk = -w'(s_dk) prod_{e != d} w(s_ek) and dA_d = sum_k dW_dk
// p_k p_k^T, assembled from separable moments like A itself (the moments of
// axis d taken with w' in place of w).  The physical derivative divides by
// H_d.  The solve runs in FP32 with the condition bound of the exact build;
// a (marker, staggering) above the routing threshold, or whose interpolated
// result is not finite, is queued and redone in FP64 from the position by a
// second kernel, which keeps the registers of the double-precision state off the
// FP32 kernel.
#include "mls_device.h"

namespace mls {

namespace {

constexpr int kGradBlock = 256;

__device__ __forceinline__ int comp_dim(const Grid &g, int c, int d)
{
    return c < 3 ? g.dims[c][d] : g.ax[d].n;
}

template <typename T>
__device__ __forceinline__ void sym_mul(const T A[10], const T v[4], T out[4])
{
    out[0] = A[0] * v[0] + A[1] * v[1] + A[2] * v[2] + A[3] * v[3];
    out[1] = A[1] * v[0] + A[4] * v[1] + A[5] * v[2] + A[6] * v[3];
    out[2] = A[2] * v[0] + A[5] * v[1] + A[7] * v[2] + A[8] * v[3];
    out[3] = A[3] * v[0] + A[6] * v[1] + A[8] * v[2] + A[9] * v[3];
}

// Coefficients of one (marker, staggering): weights w, derivatives wd,
// gamma and cd[d] = beta_d - eta_d.  FP32: returns false (caller goes to
// FP64) if A is not numerically positive definite or the condition bound
// exceeds tau.  FP64: returns false if A is singular.
template <typename T>
struct GradCoef {
    T s[3][3], w[3][3], wd[3][3], gam[4], cd[3][4], rH[3];
};

template <typename T>
__device__ __forceinline__ bool grad_coef(const Weight &Wt, T tau, GradCoef<T> &q, float &kmax)
{
    Moments<T> m[3], md[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        T m0 = 0, m1 = 0, m2 = 0, d0 = 0, d1 = 0, d2 = 0;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            T v, dv;
            weight1_ds(Wt, q.s[d][a], v, dv);
            q.w[d][a] = v;
            q.wd[d][a] = dv;
            const T sa = q.s[d][a];
            m0 += v; m1 += v * sa; m2 += v * sa * sa;
            d0 += dv; d1 += dv * sa; d2 += dv * sa * sa;
        }
        m[d] = {m0, m1, m2};
        md[d] = {-d0, -d1, -d2};   // dW_dk carries -w'
    }
    T A[10], L[10];
    assemble(m[0], m[1], m[2], A);
    if (!cholesky4(A, L)) return false;
    if (sizeof(T) == 4) {
        const T kap = cond_bound_and_gamma(A, L, q.gam);
        kmax = fmaxf(kmax, isfinite((float)kap) ? (float)kap : 3.0e38f);
        if (!(kap <= tau)) return false;
    } else {
        const T e0[4] = {1, 0, 0, 0};
        chol_solve(L, e0, q.gam);
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        T e[4] = {0, 0, 0, 0};
        e[1 + d] = 1;
        T beta[4], dA[10], v[4], eta[4];
        chol_solve(L, e, beta);
        assemble(d == 0 ? md[0] : m[0], d == 1 ? md[1] : m[1], d == 2 ? md[2] : m[2], dA);
        sym_mul(dA, q.gam, v);
        chol_solve(L, v, eta);
#pragma unroll
        for (int i = 0; i < 4; ++i) q.cd[d][i] = beta[i] - eta[i];
    }
    return true;
}

// phi_k (returned) and its physical derivatives at the node with offsets s,
// weights w and weight derivatives wd along the axes.
template <typename T>
__device__ __forceinline__ T node_phi(const GradCoef<T> &q, T sx, T sy, T sz, T wx, T wy, T wz, T dx, T dy, T dz,
                                      T dph[3])
{
    const T W = wx * wy * wz;
    const T gp = q.gam[0] + q.gam[1] * sx + q.gam[2] * sy + q.gam[3] * sz;
    const T dW[3] = {-dx * wy * wz, -wx * dy * wz, -wx * wy * dz};
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const T cp = q.cd[d][0] + q.cd[d][1] * sx + q.cd[d][2] * sy + q.cd[d][3] * sz;
        dph[d] = (dW[d] * gp + W * cp) * q.rH[d];
    }
    return W * gp;
}

// Visits the 27 support nodes (x fastest) with phi_k and the physical
// derivatives; the loops unroll fully so every index is a constant.  With
// RECOMPUTE the 1-D weights are evaluated again from the offsets instead of
// read from q (fewer live registers for the FP64 route).
template <bool RECOMPUTE, typename T, typename F>
__device__ __forceinline__ void for_each_node(const GradCoef<T> &q, const Weight &Wt, F &&f)
{
#pragma unroll
    for (int c = 0; c < 3; ++c) {
#pragma unroll
        for (int b = 0; b < 3; ++b) {
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const T sx = q.s[0][a], sy = q.s[1][b], sz = q.s[2][c];
                T wx, wy, wz, dx, dy, dz, dph[3];
                if (RECOMPUTE) {
                    weight1_ds(Wt, sx, wx, dx);
                    weight1_ds(Wt, sy, wy, dy);
                    weight1_ds(Wt, sz, wz, dz);
                } else {
                    wx = q.w[0][a]; wy = q.w[1][b]; wz = q.w[2][c];
                    dx = q.wd[0][a]; dy = q.wd[1][b]; dz = q.wd[2][c];
                }
                const T ph = node_phi(q, sx, sy, sz, wx, wy, wz, dx, dy, dz, dph);
                f(a, b, c, ph, dph);
            }
        }
    }
}

// The same nodes in the same order with a loop over the z layers, f(a, b, z[c],
// ...): nine nodes of FP64 state are live at a time.  With all 27 unrolled the
// kernel below kept 276 to 524 bytes a lane in scratch.
template <typename F>
__device__ __forceinline__ void for_each_node_layer(const GradCoef<double> &q, const int64_t z[3], F &&f)
{
#pragma unroll 1
    for (int c = 0; c < 3; ++c) {
        auto at = [c](const auto v[3]) { return c == 0 ? v[0] : (c == 1 ? v[1] : v[2]); };
        const double sz = at(q.s[2]), wz = at(q.w[2]), dz = at(q.wd[2]);
        const int64_t zc = at(z);
#pragma unroll
        for (int b = 0; b < 3; ++b) {
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                double dph[3];
                const double ph = node_phi(q, q.s[0][a], q.s[1][b], sz, q.w[0][a], q.w[1][b], wz, q.wd[0][a],
                                           q.wd[1][b], dz, dph);
                f(a, b, zc, ph, dph);
            }
        }
    }
}

// Geometry of one (marker, staggering c): FP32 offsets and 1/H; false if a
// support leaves a wall axis.  ih receives the wrapped home per axis.
__device__ __forceinline__ bool grad_geo(const Grid &g, int c, const double p[3], GradCoef<float> &q, int ih[3])
{
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        AxisGeo G;
        double rH;
        if (!axis_geo(g.ax[d], d == c, p[d], G, rH)) return false;
        q.s[d][0] = G.s[0]; q.s[d][1] = G.s[1]; q.s[d][2] = G.s[2];
        q.rH[d] = (float)rH;
        ih[d] = G.ih;
    }
    return true;
}

__device__ __forceinline__ void grad_geo_d(const Grid &g, int c, const double p[3], GradCoef<double> &q)
{
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        double H;
        axis_offsets_d(g.ax[d], d == c, p[d], q.s[d], H);
        q.rH[d] = 1.0 / H;
    }
}

// FP64 route of one (marker, staggering).  Shape functions: phi/dphi at the
// marker's first entries, kLanes apart.
__device__ __forceinline__ bool build_grad_fp64(const Grid &g, const Weight &Wt, int c, double px, double py, double pz,
                                             float *ph, float *dp)
{
    const double p[3] = {px, py, pz};
    GradCoef<double> qd;
    grad_geo_d(g, c, p, qd);
    float kmax = 0.f;
    const bool ok = grad_coef(Wt, 0.0, qd, kmax);
    const float nan = __builtin_nanf("");
    for_each_node<true>(qd, Wt, [&](int a, int b, int cz, double v, const double dv[3]) {
        const int k = a + 3 * b + 9 * cz;
        ph[k * kLanes] = ok ? (float)v : nan;
        dp[k * kLanes] = ok ? (float)dv[0] : nan;
        dp[(kNe + k) * kLanes] = ok ? (float)dv[1] : nan;
        dp[(2 * kNe + k) * kLanes] = ok ? (float)dv[2] : nan;
    });
    return ok;
}

// Value and gradient: out[0] = sum phi q, out[1 + d] = sum dphi_d (q - q0).
// q0 = 0 for a pair above the routing threshold.  For one that FP32 solved to a
// result that is not finite, q0 is the home value, the terms of the FP32 sums:
// an infinite or NaN field value passes through them as it does there, and
// sums that only FP32 cannot hold come out finite.
__device__ __forceinline__ bool interp_grad_fp64(const Grid &g, const Weight &Wt, int c, double px, double py,
                                              double pz, const float *fq, const int64_t ox[3], const int64_t oy[3],
                                              const int64_t oz[3], double q0, float out[4])
{
    const double p[3] = {px, py, pz};
    GradCoef<double> qd;
    grad_geo_d(g, c, p, qd);
    float kmax = 0.f;
    const bool ok = grad_coef(Wt, 0.0, qd, kmax);
    double ad = 0.0, gd[3] = {0.0, 0.0, 0.0};
    for_each_node_layer(qd, oz, [&](int a, int b, int64_t z0, double ph, const double dv[3]) {
        const double fv = (double)fq[z0 + oy[b] + ox[a]], df = fv - q0;
        ad += ph * fv;
        gd[0] += dv[0] * df; gd[1] += dv[1] * df; gd[2] += dv[2] * df;
    });
    const float nan = __builtin_nanf("");
    out[0] = ok ? (float)ad : nan;
    for (int d = 0; d < 3; ++d) out[1 + d] = ok ? (float)gd[d] : nan;
    return ok;
}

__device__ __forceinline__ void count_fp64(DevStats *stats, unsigned long long routed)
{
    if (routed) atomicAdd(&stat_slot(stats).fp64_solves, routed);
}

// Queue of the (marker, staggering) pairs that a second kernel redoes: q[0]
// entries, q[1] the workgroups done with them, q[2 + i] = 4 l + c, with
// kDirect set for a pair that FP32 solved to a result that is not finite.  The
// second kernel leaves both counts at zero for the next call; if a launch of
// the two fails, the next call clears them first (reserve_queue).
constexpr int kQueueHead = 2;
constexpr uint32_t kDirect = 0x80000000u;   // 4 l + c stays below it (at most 0x1fffffff markers)

// Appends e (of marker l) of every lane with on set, one reservation per
// wavefront; every active lane calls it.  cap entries fit: what calls that
// overlap on one context would append beyond them is left out and reported.
__device__ __forceinline__ void enqueue(uint32_t *queue, uint32_t cap, bool on, uint32_t e, int64_t l, ErrWord *err)
{
    const unsigned long long mask = __ballot(on);
    if (!mask) return;
    const int lane = threadIdx.x & 63, lead = __ffsll((long long)mask) - 1;
    uint32_t slot = 0;
    if (lane == lead) slot = atomicAdd(&queue[0], (uint32_t)__popcll(mask));
    slot = __shfl(slot, lead) + (uint32_t)__popcll(mask & ((1ull << lane) - 1ull));
    if (on) {
        if (slot < cap) queue[kQueueHead + slot] = e;
        else raise_error(err, l, MLS_E_HIP);
    }
}

__global__ void k_queue_clear(uint32_t *queue)
{
    if (threadIdx.x < kQueueHead) queue[threadIdx.x] = 0u;
}

// Called by every thread of the second kernel once it is done with the cnt
// entries: the last workgroup clears the counts.
__device__ __forceinline__ void queue_done(uint32_t *queue, uint32_t cnt)
{
    if (cnt == 0) return;
    __syncthreads();
    if (threadIdx.x == 0 && atomicAdd(&queue[1], 1u) == gridDim.x - 1) queue[0] = queue[1] = 0u;
}

// Shape functions and derivatives of one staggering, blocked by 64 markers:
// home[l], phi[(b*27 + k)*64 + r], dphi[((b*3 + d)*27 + k)*64 + r].
__global__ void __launch_bounds__(kGradBlock)
k_build_grad(const Grid *__restrict__ gp, Weight Wt, float tau, int c, int64_t n, const float *__restrict__ x,
             const float *__restrict__ y, const float *__restrict__ z, uint32_t *__restrict__ home,
             float *__restrict__ phi, float *__restrict__ dphi, uint32_t *queue, uint32_t qcap, ErrWord *err,
             DevStats *stats)
{
    const Grid &g = *gp;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    unsigned long long routed = 0;
    float kmax = 0.f;
    const int64_t npad = (n + kLanes - 1) / kLanes * kLanes;
    for (int64_t l = xcd_block() * blockDim.x + threadIdx.x; l < npad; l += stride) {
        const int64_t b = l / kLanes, r = l % kLanes;
        float *ph = phi + b * kNe * kLanes + r;
        float *dp = dphi + b * 3 * kNe * kLanes + r;
        if (l >= n) {   // padding lanes of the last block
            home[l] = 0xffffffffu;
            for (int k = 0; k < kNe; ++k) ph[k * kLanes] = 0.f;
            for (int k = 0; k < 3 * kNe; ++k) dp[k * kLanes] = 0.f;
            continue;
        }
        const double p[3] = {(double)x[l], (double)y[l], (double)z[l]};
        GradCoef<float> q;
        int ih[3];
        if (!grad_geo(g, c, p, q, ih)) {
            raise_error(err, l, isfinite(p[0]) && isfinite(p[1]) && isfinite(p[2]) ? MLS_E_SUPPORT
                                                                                      : MLS_E_NONFINITE);
            home[l] = 0xffffffffu;
            for (int k = 0; k < kNe; ++k) ph[k * kLanes] = __builtin_nanf("");
            for (int k = 0; k < 3 * kNe; ++k) dp[k * kLanes] = __builtin_nanf("");
            continue;
        }
        st_stream(&home[l], (uint32_t)ih[0] | ((uint32_t)ih[1] << 11) | ((uint32_t)ih[2] << 22));
        if (grad_coef(Wt, tau, q, kmax)) {
            for_each_node<false>(q, Wt, [&](int a, int b, int cz, float v, const float dv[3]) {
                const int k = a + 3 * b + 9 * cz;
                st_stream(&ph[k * kLanes], v);
                st_stream(&dp[k * kLanes], dv[0]);
                st_stream(&dp[(kNe + k) * kLanes], dv[1]);
                st_stream(&dp[(2 * kNe + k) * kLanes], dv[2]);
            });
        } else {
            ++routed;
            enqueue(queue, qcap, true, (uint32_t)(4 * l + c), l, err);
        }
    }
    count_fp64(stats, routed);
}

// Value (out[0]) and gradient (out[1 + d]) of a field over one support in
// FP32, without forming the shape functions.  With df_k = q_k - q_home and the
// vectors T = sum_k W_k p_k df_k and T_d = sum_k dW_dk p_k df_k, the solution
// z of A z = T gives them all:
//   value = q_home + sum_k phi_k df_k = q_home + z_0   (sum_k phi_k = 1),
//   d/dxi_d = gamma . T_d + (beta_d - eta_d) . T = gamma . T_d + z_{1+d} - z . (dA_d gamma),
// one solve instead of the seven of grad_coef.  (The sums over df instead of q
// use sum_k dphi_dk = 0 and are O(h |grad q|) instead of O(|q|), which spares
// FP32 the cancellation of an O(|q|/h) sum down to O(|grad q|).)  The weights
// are products of three axes, so the 16 sums are contracted axis by axis: 237
// multiply-adds for the 27 nodes, where visiting each node takes about 950
// operations.  Returns false if the pair goes to FP64.
// wrap() puts the values of wrapping stencils in place, once they are needed.
template <typename F>
__device__ __forceinline__ bool value_and_grad(const Weight &Wt, float tau, const float s[3][3], const float rH[3],
                                               const float (&qv)[kNe], F &&wrap, float out[4], float &kmax)
{
    // per axis and node: w, w s, -w', -w' s (the factors of W_k p_k and dW_dk p_k)
    float w0[3][3], w1[3][3], d0[3][3], d1[3][3];
    Moments<float> m[3], md[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        float a0 = 0.f, a1 = 0.f, a2 = 0.f, b0 = 0.f, b1 = 0.f, b2 = 0.f;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            float v, dv;
            weight1_ds(Wt, s[d][a], v, dv);
            w0[d][a] = v;
            w1[d][a] = v * s[d][a];
            d0[d][a] = -dv;
            d1[d][a] = -dv * s[d][a];
            a0 += w0[d][a]; a1 += w1[d][a]; a2 += w1[d][a] * s[d][a];
            b0 += d0[d][a]; b1 += d1[d][a]; b2 += d1[d][a] * s[d][a];
        }
        m[d] = {a0, a1, a2};
        md[d] = {b0, b1, b2};
    }
    float A[10], L[10], gam[4];
    assemble(m[0], m[1], m[2], A);
    bool ok = cholesky4(A, L);
    if (ok) {
        const float kap = cond_bound_and_gamma(A, L, gam);
        kmax = fmaxf(kmax, isfinite(kap) ? kap : 3.0e38f);
        ok = kap <= tau;
    }
    wrap();   // (votes over the wavefront: every lane comes here)
    if (!ok) return false;
    // x, then y, then z: names give the factor kind per axis (0: w, 1: w s, 2: -w', 3: -w' s)
    const float fh = qv[13];
    float T[4] = {0.f, 0.f, 0.f, 0.f}, Tx[4] = {0.f, 0.f, 0.f, 0.f}, Ty[4] = {0.f, 0.f, 0.f, 0.f},
          Tz[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        float p00 = 0.f, p10 = 0.f, p01 = 0.f, p20 = 0.f, p30 = 0.f, p21 = 0.f, p02 = 0.f, p12 = 0.f, p03 = 0.f;
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            float r0 = 0.f, r1 = 0.f, r2 = 0.f, r3 = 0.f;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const float df = qv[a + 3 * b + 9 * c] - fh;
                r0 += w0[0][a] * df; r1 += w1[0][a] * df; r2 += d0[0][a] * df; r3 += d1[0][a] * df;
            }
            p00 += r0 * w0[1][b]; p10 += r1 * w0[1][b]; p01 += r0 * w1[1][b];
            p20 += r2 * w0[1][b]; p30 += r3 * w0[1][b]; p21 += r2 * w1[1][b];
            p02 += r0 * d0[1][b]; p12 += r1 * d0[1][b]; p03 += r0 * d1[1][b];
        }
        T[0] += p00 * w0[2][c]; T[1] += p10 * w0[2][c]; T[2] += p01 * w0[2][c]; T[3] += p00 * w1[2][c];
        Tx[0] += p20 * w0[2][c]; Tx[1] += p30 * w0[2][c]; Tx[2] += p21 * w0[2][c]; Tx[3] += p20 * w1[2][c];
        Ty[0] += p02 * w0[2][c]; Ty[1] += p12 * w0[2][c]; Ty[2] += p03 * w0[2][c]; Ty[3] += p02 * w1[2][c];
        Tz[0] += p00 * d0[2][c]; Tz[1] += p10 * d0[2][c]; Tz[2] += p01 * d0[2][c]; Tz[3] += p00 * d1[2][c];
    }
    float z[4];
    chol_solve(L, T, z);
    out[0] = fh + z[0];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        float dA[10], v[4];
        assemble(d == 0 ? md[0] : m[0], d == 1 ? md[1] : m[1], d == 2 ? md[2] : m[2], dA);
        sym_mul(dA, gam, v);
        const float *t = d == 0 ? Tx : (d == 1 ? Ty : Tz);
        const float g = gam[0] * t[0] + gam[1] * t[1] + gam[2] * t[2] + gam[3] * t[3];
        out[1 + d] = rH[d] * (g + (z[1 + d] - (z[0] * v[0] + z[1] * v[1] + z[2] * v[2] + z[3] * v[3])));
    }
    return true;
}

// Value and gradient of the MLS approximation of the fields at the markers:
// for c in 0..NC-1 (u, v, w, then the cell-centred p when given),
// val[c][l] = sum_k phi_k q_c[node_k], grad[3c + d][l] = sum_k dphi_dk q_c.
// One wavefront per (64 markers, staggering), the staggerings of 64 markers
// side by side on one XCD, so that few markers too reach all compute units.
// Bound by the vector ALU.  2.56 M markers of a stretched channel with pressure
// 0.36 ms, 20,480 markers without 9 us; with the node-by-node sums and all
// staggerings in one wavefront 0.73 ms and 19 us.  A pair whose result is not
// finite is queued for the FP64 sums, which pass an infinite field value on as
// they meet it, unless a NaN in its support makes it NaN whatever the sums (with
// all fields NaN 0.63 ms instead of 4.2).
template <int NC>
__global__ void __launch_bounds__(kGradBlock)
k_interp_grad(const Grid *__restrict__ gp, Weight Wt, float tau, int64_t n, const float *__restrict__ x,
              const float *__restrict__ y, const float *__restrict__ z, const float *__restrict__ u,
              const float *__restrict__ v, const float *__restrict__ w, const float *__restrict__ pf,
              float *__restrict__ val, float *__restrict__ grad, float *__restrict__ pval,
              float *__restrict__ pgrad, uint32_t *queue, uint32_t qcap, ErrWord *err, DevStats *stats)
{
    const Grid &g = *gp;
    const int gw = (int)xcd_block() * (kGradBlock / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = gw % NC;
    const int64_t stride = (int64_t)(gridDim.x * (kGradBlock / 64) / NC) * 64;
    const float *fq = c == 0 ? u : (c == 1 ? v : (c == 2 ? w : pf));
    float *vo = c < 3 ? (val ? val + (int64_t)c * n : nullptr) : pval;
    float *go = c < 3 ? grad + (int64_t)3 * c * n : pgrad;
    const int nx = comp_dim(g, c, 0), ny = comp_dim(g, c, 1), nz = comp_dim(g, c, 2);
    unsigned long long routed = 0;
    float kmax = 0.f;
    for (int64_t l = (int64_t)(gw / NC) * 64 + (threadIdx.x & 63); l < n; l += stride) {
        const double p[3] = {(double)x[l], (double)y[l], (double)z[l]};
        float s[3][3], rH[3];
        int ih[3] = {1, 0, 0};
        bool ok = true;
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            AxisGeo G;
            double r;
            ok = ok && axis_geo(g.ax[d], d == c, p[d], G, r);
            if (ok) {
                s[d][0] = G.s[0]; s[d][1] = G.s[1]; s[d][2] = G.s[2];
                rH[d] = (float)r;
                ih[d] = G.ih;
            }
        }
        if (!ok) {
            raise_error(err, l, isfinite(p[0]) && isfinite(p[1]) && isfinite(p[2]) ? MLS_E_SUPPORT
                                                                                      : MLS_E_NONFINITE);
            const float nan = __builtin_nanf("");
            if (vo) vo[l] = nan;
            if (go) { go[l] = nan; go[n + l] = nan; go[2 * n + l] = nan; }
            continue;
        }
        uint32_t oy[3], oz[3];
        support_rows(ih[1], ih[2], nx, ny, nz, oy, oz);
        // the 27 field values are requested before the solve, which hides
        // their latency
        float qv[kNe];
        load_rows(fq, ih[0], nx, oy, oz, qv);
        float o[4] = {0.f, 0.f, 0.f, 0.f};
        const bool fp32 = value_and_grad(
            Wt, tau, s, rH, qv, [&]() { wrap_rows(fq, ih[0], ih[1], ih[2], nx, ny, nz, qv); }, o, kmax);
        if (!fp32) ++routed;
        const bool finite = fabsf(o[0]) <= 3.0e38f && fabsf(o[1]) <= 3.0e38f && fabsf(o[2]) <= 3.0e38f &&
                            fabsf(o[3]) <= 3.0e38f;
        bool redo = !fp32 || !finite;
        if (__any(redo)) {
            // A NaN in the support makes every sum NaN: nothing to redo (fields
            // may be NaN wherever the solver has no values, near every marker of
            // a body).  The values are loaded again, a row at a time, so that
            // this costs the kernel no registers.  (On a wall axis a home is
            // never an end node, so no neighbour wraps.)
            bool some_nan = false;
            if (fp32 && !finite) {
#pragma unroll 1
                for (int r = 0; r < 9; ++r) {
                    const int y1 = nb_index(ih[1], r % 3 - 1, ny, 1), z1 = nb_index(ih[2], r / 3 - 1, nz, 1);
                    const float *row = fq + ((int64_t)z1 * ny + y1) * nx;
#pragma unroll
                    for (int a = -1; a < 2; ++a) {
                        const float q = row[nb_index(ih[0], a, nx, 1)];
                        some_nan = some_nan || q != q;
                    }
                }
            }
            if (some_nan) {
                redo = false;
                o[0] = o[1] = o[2] = o[3] = __builtin_nanf("");
            }
            // the second kernel writes what is queued
            enqueue(queue, qcap, redo, (uint32_t)(4 * l + c) | (fp32 ? kDirect : 0u), l, err);
        }
        if (vo) vo[l] = o[0];
        if (go) { go[l] = o[1]; go[n + l] = o[2]; go[2 * n + l] = o[3]; }
    }
    count_fp64(stats, routed);
}

// FP64 redo of the queued (marker, staggering) pairs.
__global__ void __launch_bounds__(kGradBlock)
k_build_grad_fp64(const Grid *__restrict__ gp, Weight Wt, int64_t n, const float *__restrict__ x,
                  const float *__restrict__ y, const float *__restrict__ z, float *__restrict__ phi,
                  float *__restrict__ dphi, uint32_t *queue, uint32_t qcap, ErrWord *err)
{
    const Grid &g = *gp;
    const uint32_t cnt = min(queue[0], qcap);
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < cnt; i += gridDim.x * blockDim.x) {
        const uint32_t e = queue[kQueueHead + i];
        const int64_t l = e >> 2;
        const int c = (int)(e & 3u);
        if (l >= n) continue;
        const int64_t b = l / kLanes, r = l % kLanes;
        if (!build_grad_fp64(g, Wt, c, (double)x[l], (double)y[l], (double)z[l], phi + b * kNe * kLanes + r,
                             dphi + b * 3 * kNe * kLanes + r))
            raise_error(err, l, MLS_E_SINGULAR);
    }
    queue_done(queue, cnt);
}

__global__ void __launch_bounds__(kGradBlock)
k_interp_grad_fp64(const Grid *__restrict__ gp, Weight Wt, int64_t n, const float *__restrict__ x,
                   const float *__restrict__ y, const float *__restrict__ z, const float *__restrict__ u,
                   const float *__restrict__ v, const float *__restrict__ w, const float *__restrict__ pf,
                   float *__restrict__ val, float *__restrict__ grad, float *__restrict__ pval,
                   float *__restrict__ pgrad, uint32_t *queue, uint32_t qcap, ErrWord *err)
{
    const Grid &g = *gp;
    const uint32_t cnt = min(queue[0], qcap);
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < cnt; i += gridDim.x * blockDim.x) {
        const uint32_t e = queue[kQueueHead + i];
        const int64_t l = (e & ~kDirect) >> 2;
        const int c = (int)(e & 3u);
        if (l >= n || (c == 3 && !pf)) continue;
        const double p[3] = {(double)x[l], (double)y[l], (double)z[l]};
        int ih[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            AxisGeo G;
            axis_geo(g.ax[d], d == c, p[d], G);   // located by the FP32 pass
            ih[d] = G.ih;
        }
        const int nx = comp_dim(g, c, 0), ny = comp_dim(g, c, 1), nz = comp_dim(g, c, 2);
        int64_t ox[3], oy[3], oz[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            ox[a] = nb_index(ih[0], a - 1, nx, g.ax[0].periodic);
            oy[a] = (int64_t)nb_index(ih[1], a - 1, ny, g.ax[1].periodic) * nx;
            oz[a] = (int64_t)nb_index(ih[2], a - 1, nz, g.ax[2].periodic) * nx * ny;
        }
        const float *fq = c == 0 ? u : (c == 1 ? v : (c == 2 ? w : pf));
        float o4[4];
        const double q0 = e & kDirect ? (double)fq[oz[1] + oy[1] + ox[1]] : 0.0;
        if (!interp_grad_fp64(g, Wt, c, p[0], p[1], p[2], fq, ox, oy, oz, q0, o4)) raise_error(err, l, MLS_E_SINGULAR);
        float *vo = c < 3 ? val : pval;
        float *go = c < 3 ? grad + (int64_t)3 * c * n : pgrad;
        if (vo) vo[c < 3 ? (int64_t)c * n + l : l] = o4[0];
        if (go) { go[l] = o4[1]; go[n + l] = o4[2]; go[2 * n + l] = o4[3]; }
    }
    queue_done(queue, cnt);
}

unsigned grad_blocks(const Ctx &c, int64_t work)
{
    int64_t b = (work + kGradBlock - 1) / kGradBlock;
    b = std::min(b, (int64_t)c.cu_count * 16);
    return (unsigned)round_up8(std::max<int64_t>(b, 1));
}

}  // namespace

// The queue holds up to 4 n entries (one per marker and staggering).  Its
// counts are cleared before the first use, on growth and after a failed launch;
// the stream is waited for then, so that they are clear for a call on any
// stream (and a capture, whose replays would clear them instead, is refused).
static hipError_t reserve_queue(Ctx &c, int64_t n, hipStream_t s)
{
    const int64_t need = kQueueHead + 4 * n;
    if (need <= c.grad_queue_cap && c.grad_queue_clear) return hipSuccess;
    hipError_t e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    c.grad_queue_clear = false;
    if (need > c.grad_queue_cap) {
        hipFree(c.grad_queue);
        c.grad_queue = nullptr;
        c.grad_queue_cap = 0;
        e = hipMalloc((void **)&c.grad_queue, (size_t)need * sizeof(uint32_t));
        if (e != hipSuccess) return e;
        c.grad_queue_cap = need;
    }
    hipLaunchKernelGGL(k_queue_clear, dim3(1), dim3(64), 0, s, c.grad_queue);
    e = hipGetLastError();
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    c.grad_queue_clear = e == hipSuccess;
    return e;
}

// The status of a call's launches.
static hipError_t queue_status(Ctx &c)
{
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) c.grad_queue_clear = false;
    return e;
}

hipError_t launch_build_grad(Ctx &c, int64_t n, const float *x, const float *y, const float *z, int stagger,
                             uint32_t *home, float *phi, float *dphi, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipError_t e = reserve_queue(c, n, s);
    if (e != hipSuccess) return e;
    const uint32_t qcap = (uint32_t)(c.grad_queue_cap - kQueueHead);
    const int64_t npad = (n + kLanes - 1) / kLanes * kLanes;
    hipLaunchKernelGGL(k_build_grad, dim3(grad_blocks(c, npad)), dim3(kGradBlock), 0, s, c.d_grid, c.w,
                       (float)c.opts.kappa_tau, stagger, n, x, y, z, home, phi, dphi, c.grad_queue, qcap, c.err,
                       c.stats);
    hipLaunchKernelGGL(k_build_grad_fp64, dim3(round_up8(c.cu_count)), dim3(kGradBlock), 0, s, c.d_grid, c.w, n, x, y,
                       z, phi, dphi, c.grad_queue, qcap, c.err);
    return queue_status(c);
}

hipError_t launch_interp_grad(Ctx &c, int64_t n, const float *x, const float *y, const float *z, const float *u,
                              const float *v, const float *w, const float *p, float *U, float *G, float *P, float *GP,
                              hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipError_t e = reserve_queue(c, n, s);
    if (e != hipSuccess) return e;
    const uint32_t qcap = (uint32_t)(c.grad_queue_cap - kQueueHead);
    // three or four wavefronts per 64 markers, a multiple of 24 workgroups (8 XCDs)
    const int nc = p ? 4 : 3;
    int64_t blocks = ((n + 63) / 64 * nc + kGradBlock / 64 - 1) / (kGradBlock / 64);
    blocks = std::min(blocks, (int64_t)c.cu_count * 32);
    const dim3 grid((unsigned)((blocks + kBuildGridMultiple - 1) / kBuildGridMultiple * kBuildGridMultiple));
    if (p)
        hipLaunchKernelGGL(k_interp_grad<4>, grid, dim3(kGradBlock), 0, s, c.d_grid, c.w, (float)c.opts.kappa_tau, n, x,
                           y, z, u, v, w, p, U, G, P, GP, c.grad_queue, qcap, c.err, c.stats);
    else
        hipLaunchKernelGGL(k_interp_grad<3>, grid, dim3(kGradBlock), 0, s, c.d_grid, c.w, (float)c.opts.kappa_tau, n, x,
                           y, z, u, v, w, p, U, G, P, GP, c.grad_queue, qcap, c.err, c.stats);
    hipLaunchKernelGGL(k_interp_grad_fp64, dim3(round_up8(c.cu_count)), dim3(kGradBlock), 0, s, c.d_grid, c.w, n, x,
                       y, z, u, v, w, p, U, G, P, GP, c.grad_queue, qcap, c.err);
    return queue_status(c);
}

}  // namespace mls
