// Gaussian-mixture log-likelihood and its full reverse-mode gradient (the
// workload of Sec. 7.6; accumulators turned into reductions and contractions
// as in Sec. 6.1).
//
// Objective (precision-Cholesky parametrisation; the paper leaves the
// definition to its benchmark suite, this is the textbook mixture):
//   Q_k = diag(exp q_k) + L_k (L_k strictly lower, row-major packed in l_k),
//   z_ik = Q_k (x_i - mu_k) = Q_k x_i - c_k with c_k = Q_k mu_k,
//   s_ik = alpha_k + sum_d q_kd - |z_ik|^2 / 2,
//   loglik = sum_i LSE_k s_ik - N LSE(alpha) - N D/2 log(2 pi).
//
// Forward sweep: per 32-point tile a wave forms Z^T = Q_k X^T on MFMA (only the
// lower-triangular 32x32 blocks of Q_k), squares and sums z in FP64, and keeps an
// online FP64 log-sum-exp over k.  LSE_i is the per-point checkpoint of the
// reverse sweep.  Two forms of both sweeps: FP32 MFMA 32x32x2 (gmm_fwd_kernel,
// gmm_bwd_kernel), and for long inputs (gmm_split) every FP32 value as three bf16
// ones on bf16 MFMA (gmm_fwd_split_kernel, gmm_bwd_split_kernel).
//
// Return sweep: with w_ik = ell_bar * exp(s_ik - LSE_i) (s_ik recomputed,
// Sec. 4.1), the parameter adjoints are
//   G_k = sum_i w_ik z_ik y_ik^T = Q_k S_k with S_k = sum_i w_ik y_ik y_ik^T
//         (y = x - mu_k; S_k is an MFMA contraction over points of the
//         weighted and plain Y tiles, the product with Q_k is FP64),
//   v_k = sum_i w_ik z_ik = Q_k sum_i w_ik y_ik, W_k = sum_i w_ik,
//   alpha_bar_k = W_k - N ell_bar softmax(alpha)_k,
//   mu_bar_k = Q_k^T v_k,
//   q_bar_kd = W_k - exp(q_kd) G_k[d][d],
//   l_bar_k[r,c] = -G_k[r][c]  (r > c).
// Per component and point chunk FP32 partials of S_k and u_k = sum_i w_ik y_ik are
// written, which are summed in FP64 in a fixed order; a per-component kernel then
// forms G_k and v_k and applies the parameter maps.  The FP32 form accumulates in
// the MFMA registers over at most 4,096 points per wave; the bf16 form sums each
// tile of 32 or 64 points from zero and adds the tiles' sums over at most 32,768
// points.
#include <math.h>

#include <algorithm>

#include "common.h"
#include "prims.h"

namespace pvjp {

typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ f32x16 mfma32(float a, float b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// Result layout of a 32x32 MFMA: lane l, item t holds row drow(t, l) and
// column l % 32.
__device__ __forceinline__ int drow(int t, int lane) { return 8 * (t >> 2) + 4 * (lane >> 5) + (t & 3); }

// Operand layout of a 32x32x2 MFMA step: lane l supplies A[l % 32][l / 32] and
// B[l / 32][l % 32]; the contraction index of step s, half h, is c = 2s + h.
template <int D>
struct Gm {
    static constexpr int RT = D / 32;                    // 32-row tiles of Q_k
    static constexpr int S = D / 2;                      // steps over a full row
    static constexpr int NF = 16 * RT * (RT + 1) / 2;    // A fragments in the lower triangle
    static constexpr int NGT = RT * (RT + 1) / 2;        // lower-triangular 32x32 blocks of G_k
};

// Fragment index of row tile rt, step s (rt's row needs steps s < 16 (rt+1)).
__host__ __device__ constexpr int fidx(int rt, int s) { return 8 * rt * (rt + 1) + s; }

// X tile of 32 points in LDS, row-major [p][c] with an XOR swizzle that keeps
// both the point-major and the column-major fragment reads conflict-free.
template <int D>
__device__ __forceinline__ int xs_at(int p, int c) {
    return p * D + (c ^ (D == 64 ? 2 * p : 2 * (p >> 1)));
}

constexpr double kLog2Pi = 1.8378770664093454835606594728112;

// -------------------------------------------------------------------- prep
template <int D>
__global__ __launch_bounds__(256) void gmm_prep_kernel(const float* __restrict__ alpha, const float* __restrict__ mu,
                                                       const float* __restrict__ q, const float* __restrict__ l,
                                                       int K, float* __restrict__ Qf, float* __restrict__ cvec,
                                                       double* __restrict__ bias, double* __restrict__ lse_alpha) {
    using C = Gm<D>;
    const int k = blockIdx.x;
    const int64_t tri = (int64_t)D * (D - 1) / 2;
    __shared__ float Q[D][D + 1];
    for (int e = threadIdx.x; e < D * D; e += blockDim.x) {
        const int r = e / D, c = e % D;
        float v = 0.f;
        if (r == c)
            v = (float)exp((double)q[(int64_t)k * D + r]);
        else if (r > c)
            v = l[(int64_t)k * tri + r * (r - 1) / 2 + c];
        Q[r][c] = v;
    }
    __syncthreads();
    for (int r = threadIdx.x; r < D; r += blockDim.x) {
        double acc = 0.0;
        for (int c = 0; c <= r; ++c) acc += (double)Q[r][c] * (double)mu[(int64_t)k * D + c];
        cvec[(int64_t)k * D + r] = (float)acc;
    }
    for (int e = threadIdx.x; e < C::NF * 64; e += blockDim.x) {
        const int f = e / 64, lane = e % 64;
        const int rt = (f < 16) ? 0 : 1;
        const int s = f - fidx(rt, 0);
        Qf[((int64_t)k * C::NF + f) * 64 + lane] = Q[32 * rt + (lane & 31)][2 * s + (lane >> 5)];
    }
    // One wave each for the bias and (block 0) LSE(alpha): with one thread the
    // K exponentials in a row took most of the kernel (37 -> 14 us at K = 200).
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (w == 0) {
        double b = lane < D ? (double)q[(int64_t)k * D + lane] : 0.0;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) b += __shfl_xor(b, d, kWave);
        if (lane == 0) bias[k] = (double)alpha[k] + b;
    }
    if (w == 1 && k == 0) {
        double mx = -INFINITY;
        for (int j = lane; j < K; j += 64) mx = fmax(mx, (double)alpha[j]);
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) mx = fmax(mx, __shfl_xor(mx, d, kWave));
        double s = 0.0;
        for (int j = lane; j < K; j += 64) s += exp((double)alpha[j] - mx);
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d, kWave);
        if (lane == 0) *lse_alpha = mx + log(s);
    }
}

// The wave's share of a 32-point X tile in registers (loaded ahead of use)
// and its store into the LDS tile.
template <int D>
struct XRegs {
    float4 v[(32 * D) / 256];
};

template <int D>
__device__ __forceinline__ void load_x(const float* __restrict__ X, int64_t N, int64_t p0, XRegs<D>& r) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int q = 0; q < (32 * D) / 256; ++q) {
        const int e = 4 * (lane + 64 * q);  // 4 consecutive floats of one point
        const int64_t p = p0 + e / D;
        r.v[q] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (p < N) r.v[q] = *reinterpret_cast<const float4*>(X + p * D + e % D);
    }
}

template <int D>
__device__ __forceinline__ void store_x(const XRegs<D>& r, float* xs) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int q = 0; q < (32 * D) / 256; ++q) {
        const int e = 4 * (lane + 64 * q);
        const int pt = e / D, c = e % D;
        xs[xs_at<D>(pt, c)] = r.v[q].x;
        xs[xs_at<D>(pt, c + 1)] = r.v[q].y;
        xs[xs_at<D>(pt, c + 2)] = r.v[q].z;
        xs[xs_at<D>(pt, c + 3)] = r.v[q].w;
    }
}

template <int D>
__device__ __forceinline__ void stage_x(const float* __restrict__ X, int64_t N, int64_t p0, float* xs) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int q = 0; q < (32 * D) / 256; ++q) {
        const int e = 4 * (lane + 64 * q);  // 4 consecutive floats of one point
        const int pt = e / D, c = e % D;
        const int64_t p = p0 + pt;
        float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
        if (p < N) v = *reinterpret_cast<const float4*>(X + p * D + c);
        xs[xs_at<D>(pt, c)] = v.x;
        xs[xs_at<D>(pt, c + 1)] = v.y;
        xs[xs_at<D>(pt, c + 2)] = v.z;
        xs[xs_at<D>(pt, c + 3)] = v.w;
    }
}

// z = Q_k x - c_k for the wave's 32 points (column j = lane % 32) as MFMA
// accumulators, with Q_k's fragments (qs[f * 64 + lane]), c_k (cs[r]) and
// the X tile (xs, the wave's 32 points) read from LDS; the row tiles' MFMA
// chains are interleaved.  Each accumulator sees the operands in step order
// s = 0, 1, ..., the same as the forward sweep's chains, so z and |z|^2 are
// bit-identical to the forward's.  Returns sum_r z_r^2 in FP64 for the
// lane's point.
template <int D>
__device__ __forceinline__ double tile_znorm_lds(const float* qs, const float* cs, const float* xs,
                                                 f32x16 (&acc)[Gm<D>::RT]) {
    using C = Gm<D>;
    const int lane = threadIdx.x & 63;
    const int j = lane & 31, h = lane >> 5;
#pragma unroll
    for (int rt = 0; rt < C::RT; ++rt)
#pragma unroll
        for (int t = 0; t < 16; ++t) acc[rt][t] = 0.f;
#pragma unroll 8
    for (int s = 0; s < C::S; ++s) {
        const float bx = xs[xs_at<D>(j, 2 * s + h)];
#pragma unroll
        for (int rt = 0; rt < C::RT; ++rt)
            if (s < 16 * (rt + 1)) acc[rt] = mfma32(qs[fidx(rt, s) * 64 + lane], bx, acc[rt]);
    }
    double nrm = 0.0;
#pragma unroll
    for (int rt = 0; rt < C::RT; ++rt) {
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            const float z = acc[rt][t] - cs[32 * rt + drow(t, lane)];
            acc[rt][t] = z;
            nrm = fma((double)z, (double)z, nrm);
        }
    }
    return nrm + __shfl_xor(nrm, 32, kWave);
}

// LDS written by a wave and read back by other lanes of the same wave: a
// wave-scope fence around a wave barrier (no other wave takes part).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

struct GmmHdr {
    uint32_t done;
    uint32_t pad[63];
};

// ------------------------------------------------------------------ forward
// Online log-sum-exp step: one exponential whichever side is larger (a branch
// per side runs both when the lanes disagree).  A component of weight zero (sv
// = -inf) adds nothing, also where it comes first in its range (m = -inf still,
// and sv - m is no number).
__device__ __forceinline__ void lse_step(double sv, double& m, double& ssum) {
    const bool up = sv > m;
    const double e = sv == -INFINITY ? 0.0 : exp(up ? m - sv : sv - m);
    ssum = up ? ssum * e + 1.0 : ssum + e;
    m = up ? sv : m;
}

// Sum of every thread's v over the grid (blocks of 256), by the last block in
// a fixed order, into the log-likelihood.
__device__ __forceinline__ void finish_loglik(double v, int64_t N, int D, const double* lse_alpha, double* parts,
                                              GmmHdr* hdr, double* loglik) {
    __shared__ double red[4];
    __shared__ int s_last;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, kWave);
    if (lane == 0) red[w] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        st_coherent(&parts[blockIdx.x], (red[0] + red[1]) + (red[2] + red[3]));
        const uint32_t d = __hip_atomic_fetch_add(&hdr->done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
        s_last = (d == gridDim.x - 1);
    }
    __syncthreads();
    if (!s_last) return;
    // Last block: fixed-order sum of the block partials.
    double acc = 0.0;
    for (int b = threadIdx.x; b < (int)gridDim.x; b += 256) acc += ld_coherent(&parts[b]);
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) acc += __shfl_xor(acc, d, kWave);
    __syncthreads();
    if (lane == 0) red[w] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        const double tot = (red[0] + red[1]) + (red[2] + red[3]);
        *loglik = tot - (double)N * (*lse_alpha) - 0.5 * (double)N * D * kLog2Pi;
        __hip_atomic_store(&hdr->done, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// The block's four waves share each batch of CPB components: Q_k's fragments
// and c_k are staged in LDS once per block, and each wave interleaves the
// independent MFMA chains of the batch (CPB components x the row tiles of
// each), so the matrix unit has several chains to alternate between.  Every
// chain sees the same operands in the same order as tile_znorm_lds, so z, |z|^2
// and s_ik are bit-identical to the per-component form, and the online LSE
// takes the components in index order.
template <int D>
struct GmFwd {
    static constexpr int CPB = D == 64 ? 2 : 4;                // components per batch
    static constexpr int QF = Gm<D>::NF * 64;                  // fragment floats per component
    static constexpr int STAGE = CPB * (QF + D);               // floats staged per batch
    static constexpr int PER = (STAGE + 255) / 256;            // per thread (the last round partly empty)
    static constexpr int XS = 4 * 32 * D;                      // the X tiles, staged first
    static constexpr int LDS = XS > PER * 256 ? XS : PER * 256;
};

template <int D>
__device__ __forceinline__ void fwd_fetch(const float* __restrict__ Qf, const float* __restrict__ cvec, int k0, int K,
                                          float (&r)[GmFwd<D>::PER]) {
    using F = GmFwd<D>;
#pragma unroll
    for (int u = 0; u < F::PER; ++u) {
        const int e = u * 256 + (int)threadIdx.x;  // staged float index
        const int c = e < F::CPB * F::QF ? e / F::QF : (e - F::CPB * F::QF) / D;
        const int k = k0 + c;
        float v = 0.f;
        if (e < F::STAGE && k < K) {
            if (e < F::CPB * F::QF)
                v = Qf[(int64_t)k * F::QF + (e - c * F::QF)];
            else
                v = cvec[(int64_t)k * D + (e - F::CPB * F::QF - c * D)];
        }
        r[u] = v;
    }
}

// The grid's second dimension splits the components where the points alone
// leave the chip idle: block row y takes components [y kper, (y + 1) kper) and
// leaves each point's (max, sum) to gmm_lse_merge_kernel (N = 10,007, D = 32,
// K = 50: 79 blocks in 71 us, now 1,027 in 20 and the merge's 9).  With one
// row the block finishes its points itself.
template <int D>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void gmm_fwd_kernel(const float* __restrict__ X, int64_t N, int K, int kper,
                                                      const float* __restrict__ Qf, const float* __restrict__ cvec,
                                                      const double* __restrict__ bias,
                                                      const double* __restrict__ lse_alpha, double* __restrict__ lse,
                                                      double* __restrict__ sck, double2* __restrict__ msum,
                                                      double* parts, GmmHdr* hdr, double* loglik) {
    using C = Gm<D>;
    using F = GmFwd<D>;
    __shared__ float sm[F::LDS];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t p0 = ((int64_t)blockIdx.x * 4 + w) * 32;
    float* Xs = sm + w * 32 * D;
    stage_x<D>(X, N, p0, Xs);
    __syncthreads();
    float bx[C::S];
#pragma unroll
    for (int s = 0; s < C::S; ++s) bx[s] = Xs[xs_at<D>(lane & 31, 2 * s + (lane >> 5))];
    const int64_t p = p0 + (lane & 31);
    const float* qs = sm;                       // [CPB][QF] during the batches
    const float* cs = sm + F::CPB * F::QF;      // [CPB][D]

    double m = -INFINITY, ssum = 0.0;
    const bool own = (lane < 32) && (p < N);
    const int kbeg = blockIdx.y * kper, kend = min(K, kbeg + kper);
    for (int k0 = kbeg; k0 < kend; k0 += F::CPB) {
        {
            float nxt[F::PER];
            fwd_fetch<D>(Qf, cvec, k0, kend, nxt);
            __syncthreads();  // every wave is done with the previous batch (or with X)
#pragma unroll
            for (int u = 0; u < F::PER; ++u) sm[u * 256 + threadIdx.x] = nxt[u];
            __syncthreads();
        }
        f32x16 acc[F::CPB][C::RT];
#pragma unroll
        for (int c = 0; c < F::CPB; ++c)
#pragma unroll
            for (int rt = 0; rt < C::RT; ++rt)
#pragma unroll
                for (int t = 0; t < 16; ++t) acc[c][rt][t] = 0.f;
#pragma unroll 4
        for (int s = 0; s < C::S; ++s)
#pragma unroll
            for (int rt = 0; rt < C::RT; ++rt)
#pragma unroll
                for (int c = 0; c < F::CPB; ++c)
                    if (s < 16 * (rt + 1)) acc[c][rt] = mfma32(qs[c * F::QF + fidx(rt, s) * 64 + lane], bx[s], acc[c][rt]);
#pragma unroll
        for (int c = 0; c < F::CPB; ++c) {
            const int k = k0 + c;
            if (k >= kend) break;
            double nrm = 0.0;
#pragma unroll
            for (int rt = 0; rt < C::RT; ++rt) {
#pragma unroll
                for (int t = 0; t < 16; ++t) {
                    const float z = acc[c][rt][t] - cs[c * D + 32 * rt + drow(t, lane)];
                    nrm = fma((double)z, (double)z, nrm);
                }
            }
            nrm += __shfl_xor(nrm, 32, kWave);
            const double sv = bias[k] - 0.5 * nrm;
            if (sck && own) sck[(int64_t)k * N + p] = sv;  // component-major: 32 points per wave in a row
            lse_step(sv, m, ssum);
        }
    }
    if (gridDim.y > 1) {
        if (own) msum[(int64_t)blockIdx.y * N + p] = make_double2(m, ssum);
        return;
    }
    const double l_i = m + log(ssum);
    if (own && lse) lse[p] = l_i;
    finish_loglik(own ? l_i : 0.0, N, D, lse_alpha, parts, hdr, loglik);
}

// The points' LSE from the (max, sum) of each range of components, in range
// order, and the log-likelihood.
template <int D>
__global__ __launch_bounds__(256) void gmm_lse_merge_kernel(int64_t N, int ny, const double2* __restrict__ msum,
                                                            const double* __restrict__ lse_alpha,
                                                            double* __restrict__ lse, double* parts, GmmHdr* hdr,
                                                            double* loglik) {
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    double l_i = 0.0;
    if (p < N) {
        // the maximum first: the exponentials are then independent.  A range of
        // weights zero has the sum 0 (and its maximum, -inf, gives exp(-inf) = 0).
        double m = -INFINITY, s = 0.0;
#pragma unroll 8
        for (int y = 0; y < ny; ++y) m = fmax(m, msum[(int64_t)y * N + p].x);
#pragma unroll 8
        for (int y = 0; y < ny; ++y) {
            const double2 v = msum[(int64_t)y * N + p];
            s += v.y * (v.x == m ? 1.0 : exp(v.x - m));
        }
        l_i = m + log(s);
        if (lse) lse[p] = l_i;
    }
    finish_loglik(l_i, N, D, lse_alpha, parts, hdr, loglik);
}

// ----------------------------------------------------------------- backward
// The contraction runs over y = x - mu_k on both sides: S_k = sum_i w_ik
// y_ik y_ik^T and u_k = sum_i w_ik y_ik, from the X tile in LDS and each
// point's weight (no weighted-z tile); gmm_param_kernel then forms
// G_k = Q_k S_k and v_k = Q_k u_k in FP64 (z_ik = Q_k y_ik).  The weight
// needs s_ik: recomputed from |z_ik|^2 (one MFMA pass over Q_k), or, with
// FROM_S, read from the forward's s_ik checkpoint (sck, K x N), which halves
// the MFMA work.
template <int D, bool FROM_S>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void gmm_bwd_kernel(const float* __restrict__ X, int64_t N, int K, int64_t chunk,
                                                      int nch, const float* __restrict__ Qf,
                                                      const float* __restrict__ cvec, const float* __restrict__ mu,
                                                      const double* __restrict__ bias, const double* __restrict__ lse,
                                                      const double* __restrict__ sck,
                                                      double ell_bar, float* __restrict__ gpart,
                                                      float* __restrict__ vpart, double* __restrict__ wpart) {
    using C = Gm<D>;
    // X tiles of the four waves, and room for the scratch of the cross-wave
    // reduction at the end.  Q_k's MFMA fragments live in LDS too, read at
    // each step: held in registers they would leave room for only one wave
    // per SIMD.
    __shared__ __align__(16) float smem[2 * 4 * 32 * D];
    __shared__ float qs[C::NF * 64];
    __shared__ float cs[D];
    float* const Xw = smem + (threadIdx.x >> 6) * 32 * D;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int k = blockIdx.x % K;
    const int ch = blockIdx.x / K;
    const int h = lane >> 5, j = lane & 31;

    if (!FROM_S)
        for (int e = threadIdx.x; e < C::NF * 64; e += 256) qs[e] = Qf[(int64_t)k * C::NF * 64 + e];
    // cs: c_k for the recomputing form, mu_k for the checkpointed one
    if (threadIdx.x < D) cs[threadIdx.x] = FROM_S ? mu[(int64_t)k * D + threadIdx.x] : cvec[(int64_t)k * D + threadIdx.x];
    float mub[C::RT];
#pragma unroll
    for (int ct = 0; ct < C::RT; ++ct) mub[ct] = mu[(int64_t)k * D + 32 * ct + j];
    const double bk = bias[k];

    f32x16 gacc[C::NGT];
#pragma unroll
    for (int g = 0; g < C::NGT; ++g)
#pragma unroll
        for (int t = 0; t < 16; ++t) gacc[g][t] = 0.f;
    float urow[C::RT];
#pragma unroll
    for (int t = 0; t < C::RT; ++t) urow[t] = 0.f;
    double wsum = 0.0;

    const int64_t cbeg = (int64_t)ch * chunk;
    const int iters = (int)(chunk / 128);
    __syncthreads();  // qs and cs
    // Every tile below is private to its wave (Xw), so the waves only
    // synchronise with themselves and drift apart freely: one wave's MFMA
    // phase overlaps another's loads and FP64 work.
    // The next tile's X values (and its point's LSE and s_ik) are loaded
    // while this tile computes.
    XRegs<D> xr;
    double lse_n = 0.0, s_n = 0.0;
    {
        const int64_t p0 = cbeg + (int64_t)w * 32;
        load_x<D>(X, N, p0, xr);
        if (p0 + j < N) {
            lse_n = lse[p0 + j];
            if (FROM_S) s_n = sck[(int64_t)k * N + p0 + j];
        }
    }
    for (int it = 0; it < iters; ++it) {
        const int64_t p0 = cbeg + (int64_t)(it * 4 + w) * 32;
        wave_lds_sync();
        store_x<D>(xr, Xw);
        wave_lds_sync();
        const double lse_p = lse_n, s_p = s_n;
        if (it + 1 < iters) {
            const int64_t pn = p0 + 4 * 32;
            load_x<D>(X, N, pn, xr);
            if (pn + j < N) {
                lse_n = lse[pn + j];
                if (FROM_S) s_n = sck[(int64_t)k * N + pn + j];
            }
        }
        const int64_t p = p0 + j;
        double wd = 0.0;
        if (FROM_S) {
            if (p < N) wd = ell_bar * exp(s_p - lse_p);
        } else {
            // s_ik from |z|^2: z is recomputed for its norm only (the MFMA
            // phases run at raised wave priority, so that the other wave on
            // the SIMD issues its loads and FP64 work in their gaps)
            f32x16 z[C::RT];
            __builtin_amdgcn_s_setprio(1);
            const double nrm = tile_znorm_lds<D>(qs, cs, Xw, z);
            __builtin_amdgcn_s_setprio(0);
            if (p < N) wd = ell_bar * exp((bk - 0.5 * nrm) - lse_p);
        }
        const float wf = (float)wd;  // lane (j, h): the weight of point j
        if (h == 0) wsum += wd;
        // S_k += (w Y)^T Y over this tile's 32 points, lower-triangular
        // blocks: step s contracts point 2s + h, whose weight comes from lane
        // 2s + h; u_k = sum w y accumulates from the same products.  Each step
        // loads one operand per row tile and feeds the blocks' independent
        // accumulators in turn.
        __builtin_amdgcn_s_setprio(1);
#pragma unroll 8
        for (int s = 0; s < 16; ++s) {
            const int pt = 2 * s + h;
            const float wp = __shfl(wf, pt, kWave);
            float za[C::RT], yb[C::RT];
#pragma unroll
            for (int t = 0; t < C::RT; ++t) {
                yb[t] = Xw[xs_at<D>(pt, 32 * t + j)] - mub[t];
                za[t] = wp * yb[t];
                urow[t] += za[t];
            }
            int g = 0;
#pragma unroll
            for (int rt = 0; rt < C::RT; ++rt)
#pragma unroll
                for (int ct = 0; ct <= rt; ++ct) {
                    gacc[g] = mfma32(za[rt], yb[ct], gacc[g]);
                    ++g;
                }
        }
        __builtin_amdgcn_s_setprio(0);
    }

    // u: the two half-waves hold the halves of each row sum; lane r < D takes
    // row r's (rows 32 t + j live in lane j's urow[t]).
#pragma unroll
    for (int t = 0; t < C::RT; ++t) urow[t] += __shfl_xor(urow[t], 32, kWave);
    const float uhi = __shfl(urow[C::RT - 1], lane & 31, kWave);
    float vrow = lane < 32 ? urow[0] : uhi;
#pragma unroll
    for (int d = 16; d >= 1; d >>= 1) wsum += __shfl_xor(wsum, d, kWave);

    // Combine the four waves through LDS (reusing the tiles) in a fixed order.
    __syncthreads();
    float* red = smem;
    constexpr int kRedFloats = 3 * Gm<D>::NGT * 1024 + 3 * D;
    static_assert(kRedFloats + 8 <= 2 * 4 * 32 * D, "reduction scratch");
    double* wred = reinterpret_cast<double*>(smem + ((kRedFloats + 1) & ~1));
    if (w > 0) {
#pragma unroll
        for (int g = 0; g < C::NGT; ++g)
#pragma unroll
            for (int t = 0; t < 16; ++t) red[((w - 1) * C::NGT * 16 + g * 16 + t) * 64 + lane] = gacc[g][t];
        if (lane < D) red[3 * C::NGT * 1024 + (w - 1) * D + lane] = vrow;
    }
    if (lane == 0) wred[w] = wsum;
    __syncthreads();
    if (w == 0) {
        const int64_t rec = (int64_t)k * nch + ch;
#pragma unroll
        for (int g = 0; g < C::NGT; ++g)
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                float s = gacc[g][t];
                for (int o = 0; o < 3; ++o) s += red[(o * C::NGT * 16 + g * 16 + t) * 64 + lane];
                gpart[(rec * C::NGT * 16 + g * 16 + t) * 64 + lane] = s;
            }
        if (lane < D) {
            float s = vrow;
            for (int o = 0; o < 3; ++o) s += red[3 * C::NGT * 1024 + o * D + lane];
            vpart[rec * D + lane] = s;
        }
        if (lane == 0) wpart[rec] = (wred[0] + wred[1]) + (wred[2] + wred[3]);
    }
}

// ------------------------------------------- large N: bf16 triples on MFMA
// An FP32 value is exactly the sum of three bf16 values (8 bits of its
// significand each, rounded to nearest, so the remainders have either sign):
// x = h + m + l.  A product's terms hh, hm, mh, hl, lh, mm in bf16 MFMA with
// FP32 accumulators leave out ml, lm, ll, up to 2^-24 of it (|m| <= 2^-8 |x|,
// |l| <= 2^-17 |x|: one FP32 rounding) and of either sign.  Against 64 bits, on
// standard normal points, D = 32 and 64, K = 25 to 200, N = 131,073 to 10^6, the
// worst relative L2 error of the FP32 form and of this: log-likelihood 1.2e-9 and
// 1.2e-9, alpha_bar 1.6e-7 and 1.6e-7, mu_bar 1.3e-6 and 2.8e-7, q_bar 1.2e-5 and
// 5.2e-7, l_bar 2.4e-6 and 2.2e-7.  One 32x32x16 bf16 step takes 32 cycles, the
// eight 32x32x2 FP32 steps it replaces 512, so six of them are 2.7 times faster.
// Inputs, weights, the sums over chunks, |z|^2 and the log-sum-exp keep their
// types.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x16 mfma16(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// NV values (even) into three planes of packed pairs: a pair shares the
// converting instruction, and each half is widened from the packed pair (a
// shift, a mask).
template <int NV>
__device__ __forceinline__ void split(const float (&x)[NV], uint32_t (&o)[3][NV / 2]) {
#pragma unroll
    for (int i = 0; i < NV / 2; ++i) {
        float a = x[2 * i], b = x[2 * i + 1];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            const bf16x2 v = {(__bf16)a, (__bf16)b};
            const uint32_t u = __builtin_bit_cast(uint32_t, v);
            o[q][i] = u;
            a -= __builtin_bit_cast(float, u << 16);
            b -= __builtin_bit_cast(float, u & 0xffff0000u);
        }
    }
}
__device__ __forceinline__ void split8(const float (&x)[8], bf16x8 (&p)[3]) {
    uint32_t o[3][4];
    split(x, o);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const u32x4 v = {o[q][0], o[q][1], o[q][2], o[q][3]};
        p[q] = __builtin_bit_cast(bf16x8, v);
    }
}

// The six terms in the order they are accumulated, small ones first.
__device__ constexpr int kTermA[6] = {0, 2, 1, 0, 1, 0};
__device__ constexpr int kTermB[6] = {2, 0, 1, 1, 0, 0};

template <int D>
struct Gs {
    static constexpr int RT = D / 32;        // 32-row tiles of Q_k
    static constexpr int KS = D / 16;        // 16-wide contraction steps over a full row
    static constexpr int F = RT * (RT + 1);  // steps in the lower triangle (row tile rt needs 2 (rt + 1))
    static constexpr int Q16 = F * 3 * 64;   // 16-byte fragments of a component
    static constexpr int U16 = Q16 + D / 4;  // and its c_k in FP32
};
// A fragment of step s for row tile rt: lane l holds row 32 rt + l % 32,
// columns 16 s + 8 (l / 32) + 0..7.
__host__ __device__ constexpr int sidx(int rt, int s) { return rt * (rt + 1) + s; }

// Q_k x of a wave's TL 32-point tiles.  qa(f, plane) and xb(tile, s, plane)
// give the operand fragments.  Both sweeps run this sequence and
// split_square's, so the return sweep recomputes the forward's s_ik bit for
// bit.
template <int D, int TL, class QA, class XB>
__device__ __forceinline__ void split_qx(QA qa, XB xb, f32x16 (&acc)[Gs<D>::RT][TL]) {
    using C = Gs<D>;
#pragma unroll
    for (int rt = 0; rt < C::RT; ++rt)
#pragma unroll
        for (int tl = 0; tl < TL; ++tl)
#pragma unroll
            for (int t = 0; t < 16; ++t) acc[rt][tl][t] = 0.f;
#pragma unroll
    for (int s = 0; s < C::KS; ++s) {
        bf16x8 a[C::RT][3], b[TL][3];
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) {
#pragma unroll
            for (int rt = 0; rt < C::RT; ++rt)
                if (s < 2 * (rt + 1)) a[rt][pl] = qa(sidx(rt, s), pl);
#pragma unroll
            for (int tl = 0; tl < TL; ++tl) b[tl][pl] = xb(tl, s, pl);
        }
#pragma unroll
        for (int q = 0; q < 6; ++q)
#pragma unroll
            for (int rt = 0; rt < C::RT; ++rt)
#pragma unroll
                for (int tl = 0; tl < TL; ++tl)
                    if (s < 2 * (rt + 1)) acc[rt][tl] = mfma16(a[rt][kTermA[q]], b[tl][kTermB[q]], acc[rt][tl]);
    }
}

// |z|^2, z = Q_k x - c_k, in FP64 (the difference too: started from -c_k the
// FP32 accumulators lose more than the FP32 form did) of the lane's point:
// point l % 32 of the tile, or with two tiles point l of the 64 (each half-wave
// holds half of every point's rows).
template <int D, int TL>
__device__ __forceinline__ double split_square(const f32x16 (&acc)[Gs<D>::RT][TL], const float* cs) {
    using C = Gs<D>;
    const int h = (threadIdx.x >> 5) & 1;
    double nrm[2] = {0.0, 0.0};
#pragma unroll
    for (int rt = 0; rt < C::RT; ++rt)
#pragma unroll
        for (int t4 = 0; t4 < 4; ++t4) {
            const float4 c = *reinterpret_cast<const float4*>(cs + 32 * rt + 8 * t4 + 4 * h);
            const double cv[4] = {c.x, c.y, c.z, c.w};
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int tl = 0; tl < TL; ++tl) {
                    const double z = (double)acc[rt][tl][4 * t4 + i] - cv[i];
                    nrm[tl] = fma(z, z, nrm[tl]);
                }
        }
    if (TL == 1) return nrm[0] + __shfl_xor(nrm[0], 32, kWave);
    const bool up = threadIdx.x & 32;
    return (up ? nrm[1] : nrm[0]) + __shfl_xor(up ? nrm[0] : nrm[1], 32, kWave);
}

// Q_k's fragments in three planes, followed by c_k: what a block stages per
// component.
template <int D>
__global__ __launch_bounds__(256) void gmm_split_q_kernel(const float* __restrict__ q, const float* __restrict__ l,
                                                          const float* __restrict__ cvec, bf16x8* __restrict__ Qs) {
    using C = Gs<D>;
    const int64_t k = blockIdx.x;
    const int64_t tri = (int64_t)D * (D - 1) / 2;
    for (int e = threadIdx.x; e < C::F * 64; e += 256) {
        const int f = e / 64, lane = e % 64;
        const int rt = f < 2 ? 0 : 1, s = f - sidx(rt, 0);
        const int r = 32 * rt + (lane & 31), c0 = 16 * s + 8 * (lane >> 5);
        float x[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int c = c0 + i;
            x[i] = 0.f;
            if (r == c)
                x[i] = (float)exp((double)q[k * D + r]);
            else if (r > c)
                x[i] = l[k * tri + r * (r - 1) / 2 + c];
        }
        bf16x8 p[3];
        split8(x, p);
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) Qs[k * C::U16 + (f * 3 + pl) * 64 + lane] = p[pl];
    }
    if (threadIdx.x < D)
        reinterpret_cast<float*>(Qs + k * C::U16 + C::Q16)[threadIdx.x] = cvec[k * D + threadIdx.x];
}

// Forward: a wave keeps 64 points' X fragments in registers (split once) and
// takes its block row's components one after another, their Q fragments and
// c_k staged in LDS for the block's four waves, the next component's loaded
// while this one computes.  Bound by the bf16 matrix pipe (2,304 cycles for 64
// points and a component at D = 64, 75% busy) at the 1.75 GHz the card holds
// under it: N = 10^6, D = 64, K = 200 in 5.4 ms (12.1 in FP32 MFMA), 1.35
// PFLOP/s of bf16 where a large library product of random matrices reaches
// 1.2.
template <int D>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void gmm_fwd_split_kernel(
    const float* __restrict__ X, int64_t N, int K, int kper, const bf16x8* __restrict__ Qs,
    const double* __restrict__ bias, const double* __restrict__ lse_alpha, double* __restrict__ lse,
    double* __restrict__ sck, double2* __restrict__ msum, double* parts, GmmHdr* hdr, double* loglik) {
    using C = Gs<D>;
    constexpr int TOT = C::U16;  // 16-byte units staged per component
    constexpr int PER = (TOT + 255) / 256;
    __shared__ u32x4 st[2][TOT];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t p0 = ((int64_t)blockIdx.x * 4 + w) * 64;
    const int kbeg = blockIdx.y * kper, kend = min(K, kbeg + kper);

    u32x4 nxt[PER];
    auto fetch = [&](int k) {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int e = min(u * 256 + (int)threadIdx.x, TOT - 1);
            nxt[u] = reinterpret_cast<const u32x4*>(Qs)[(int64_t)k * TOT + e];
        }
    };
    auto put = [&](int b) {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int e = u * 256 + (int)threadIdx.x;
            if (e < TOT) st[b][e] = nxt[u];
        }
    };
    fetch(kbeg);
    bf16x8 xf[2][C::KS][3];
#pragma unroll
    for (int tl = 0; tl < 2; ++tl) {
        const int64_t p = p0 + 32 * tl + (lane & 31);
#pragma unroll
        for (int s = 0; s < C::KS; ++s) {
            float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            if (p < N) {
                const float4* src = reinterpret_cast<const float4*>(X + p * D + 16 * s + 8 * (lane >> 5));
                const float4 u = src[0], v = src[1];
                x[0] = u.x, x[1] = u.y, x[2] = u.z, x[3] = u.w;
                x[4] = v.x, x[5] = v.y, x[6] = v.z, x[7] = v.w;
            }
            split8(x, xf[tl][s]);
        }
    }
    put(0);
    const int64_t p = p0 + lane;
    double m = -INFINITY, ssum = 0.0;
    for (int k = kbeg; k < kend; ++k) {
        const int b = (k - kbeg) & 1;
        if (k + 1 < kend) fetch(k + 1);
        __syncthreads();  // buffer b is filled, and the other one no longer read
        const bf16x8* qf = reinterpret_cast<const bf16x8*>(st[b]);
        f32x16 acc[C::RT][2];
        split_qx<D, 2>([&](int f, int pl) { return qf[(f * 3 + pl) * 64 + lane]; },
                       [&](int tl, int s, int pl) { return xf[tl][s][pl]; }, acc);
        const double sv = bias[k] - 0.5 * split_square<D, 2>(acc, reinterpret_cast<const float*>(&st[b][C::Q16]));
        if (k + 1 < kend) put(b ^ 1);
        if (sck && p < N) sck[(int64_t)k * N + p] = sv;
        lse_step(sv, m, ssum);
    }
    if (gridDim.y > 1) {
        if (p < N) msum[(int64_t)blockIdx.y * N + p] = make_double2(m, ssum);
        return;
    }
    const double l_i = m + log(ssum);
    if (p < N && lse) lse[p] = l_i;
    finish_loglik(p < N ? l_i : 0.0, N, D, lse_alpha, parts, hdr, loglik);
}

// 2x for the bf16 pairs of a remainder plane: one on each exponent (a zero
// becomes 2^-126, which is nothing beside the leading plane's product; where
// the value is not finite that product is not either).
__device__ __forceinline__ bf16x8 twice(bf16x8 v) {
    u32x4 u = __builtin_bit_cast(u32x4, v);
    u += 0x00800080u;
    return __builtin_bit_cast(bf16x8, u);
}

// Return sweep: a wave per component, eight to a block, all on the block's
// stream of tiles (32 points at D = 64, 64 at D = 32; loaded two tiles ahead,
// split once, kept in LDS as B fragments and as X^T).  Each wave keeps Q_k's
// leading plane and the lower blocks of S_k in registers: s_ik as in the
// forward, then S_k += V^T V with the rows v_i = sqrt(w_i) (x_i - mu_k), whose
// fragments serve as both operands (a lane holds one dimension of eight
// points either way).  On a diagonal block hm + mh and hl + lh are taken as
// h (2m) and h (2l), whose symmetric part is the same; the parameter kernel
// takes that part.  A tile's product is summed from zero and then added to
// S_k: one FP32 rounding of the long sum per tile (one per 2 points in the
// FP32 form, over at most 4,096 points against 32,768 here; accumulated in
// place over 4,096 points q_bar's error was 1.4e-6 against 1.4e-7).  A 32-point
// tile and component take 2,048 MFMA cycles and about as many of vector work
// (forming and splitting v, squares, weights).  A wave waiting to issue an MFMA
// keeps the other wave's vector instructions from issuing, so each wave
// interleaves the two itself: after every MFMA a short step of the vector work
// that does not depend on it, held in place by a scheduling barrier (left to
// itself the compiler groups them: 11.9 ms, now 11.2).  N = 10^6, D = 64, K =
// 200: 26.5 -> 11.2 ms, MFMA busy 54% of the cycles.
template <int D, bool FROM_S>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2))) void gmm_bwd_split_kernel(
    const float* __restrict__ X, int64_t N, int K, int64_t chunk, int nch, const bf16x8* __restrict__ Qs,
    const float* __restrict__ mu, const double* __restrict__ bias, const double* __restrict__ lse,
    const double* __restrict__ sck, float* __restrict__ gpart, float* __restrict__ vpart,
    double* __restrict__ wpart) {
    using C = Gs<D>;
    constexpr int RT = C::RT, NGT = Gm<D>::NGT;
    constexpr int TL = 2 / RT;  // 32-point tiles taken at once
    constexpr int NP = 32 * TL;  // points per tile: 2,048 values of X, four to a thread
    constexpr int XT = NP + 4;      // the pad spreads the 16-byte column reads over the banks
    constexpr int NV = 2 * TL;   // 16-point contraction steps per tile
    __shared__ bf16x8 xp[FROM_S ? 1 : 2][TL][C::KS][3][64];
    __shared__ bf16x8 ql[FROM_S ? 1 : 8][C::F][2][64];  // the two lower planes of each wave's Q_k
    __shared__ __align__(16) float xt[3][D][XT];
    __shared__ __align__(16) float sws[8][NP];
    __shared__ __align__(16) float cs[8][D];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int j = lane & 31, h = lane >> 5;
    const int groups = (K + 7) / 8;
    const int ch = blockIdx.x / groups;
    const int k = (blockIdx.x % groups) * 8 + w;
    const int kk = min(k, K - 1);  // the last group's spare waves repeat a component and write nothing
    const int64_t cbeg = (int64_t)ch * chunk, cend = min(N, cbeg + chunk);

    bf16x8 qa[C::F];
    if (!FROM_S) {
        const bf16x8* src = Qs + (int64_t)kk * C::U16;
#pragma unroll
        for (int f = 0; f < C::F; ++f) {
            qa[f] = src[f * 3 * 64 + lane];
#pragma unroll
            for (int pl = 1; pl < 3; ++pl) ql[w][f][pl - 1][lane] = src[(f * 3 + pl) * 64 + lane];
        }
        if (lane < D) cs[w][lane] = reinterpret_cast<const float*>(src + C::Q16)[lane];
    }
    float mub[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) mub[rt] = mu[(int64_t)kk * D + 32 * rt + j];
    const double bk = bias[kk];

    f32x16 S[NGT];
#pragma unroll
    for (int g = 0; g < NGT; ++g)
#pragma unroll
        for (int t = 0; t < 16; ++t) S[g][t] = 0.f;
    float u[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) u[rt] = 0.f;
    double wsum = 0.0;

    // A thread loads four dimensions of one point.
    const int lp = threadIdx.x % NP, lg = threadIdx.x / NP;
    const int wp = lane & (NP - 1);  // the point whose weight this lane forms
    float4 xn;
    double lse_n = 0.0, s_n = 0.0;
    auto fetch = [&](int64_t pb) {
        xn = make_float4(0.f, 0.f, 0.f, 0.f);
        if (pb + lp < N) xn = *reinterpret_cast<const float4*>(X + (pb + lp) * D + 4 * lg);
    };
    auto fetch_lse = [&](int64_t pb) {
        const int64_t p = min(pb + wp, N - 1);
        lse_n = lse[p];
        if (FROM_S) s_n = sck[(int64_t)kk * N + p];
    };
    auto put = [&](int b, int b3) {
        const float x[4] = {xn.x, xn.y, xn.z, xn.w};
        if (!FROM_S) {
            uint32_t o[3][2];
            split(x, o);
#pragma unroll
            for (int q = 0; q < 3; ++q)
                reinterpret_cast<uint2*>(&xp[b][lp >> 5][lg >> 2][q][(lp & 31) + 32 * ((lg >> 1) & 1)])[lg & 1] =
                    make_uint2(o[q][0], o[q][1]);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) xt[b3][4 * lg + i][lp] = x[i];
    };
    f32x16 acc[C::RT][TL];
    auto form_z = [&](int b) {
        split_qx<D, TL>([&](int f, int pl) { return pl == 0 ? qa[f] : ql[w][f][pl - 1][lane]; },
                        [&](int tl, int s, int pl) { return xp[b][tl][s][pl][lane]; }, acc);
    };
    // sqrt(w_i) of the lane's point of the tile at pb, for the wave's row of sws.
    auto weight_of = [&](double sv, int64_t pb) {
        const double e = exp(0.5 * (sv - lse_n));
        const double swd = pb + wp < cend ? e : 0.0;
        wsum = fma(swd, swd, wsum);
        return swd;
    };
    auto keep = [&](double swd) {
        wave_lds_sync();
        sws[w][wp] = (float)swd;  // with 32 points both half-waves write the same value
        wave_lds_sync();
    };
    const int tiles = (int)((cend - cbeg + NP - 1) / NP);
    fetch(cbeg);
    put(0, 0);
    fetch(cbeg + NP);
    put(1, 1);
    fetch_lse(cbeg);
    __syncthreads();
    if (!FROM_S) form_z(0);
    keep(weight_of(FROM_S ? s_n : bk - 0.5 * split_square<D, TL>(acc, cs[w]), cbeg));
    int b3 = 0;  // tile it is in buffer it % 3 of xt
    for (int it = 0; it < tiles; ++it) {
        const int64_t pb = cbeg + (int64_t)it * NP;
        fetch(pb + 2 * NP);
        fetch_lse(pb + NP);
        __builtin_amdgcn_sched_barrier(0);
        // the next tile's z (past the last tile the buffers hold an old one,
        // and its weights are zero), and between its MFMAs this tile's v
        bf16x8 vf[NV][RT][3];
        float us[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) us[rt] = 0.f;
        // v in 32 short steps: a chunk (16 points' step s, row tile rt) has four
        // pairs of two steps; the next chunk's operands are read half a chunk
        // ahead
        float xv[8], sq[8], xa[8], sa[8], ra, rb;
        uint32_t o[3][4];
        auto vread = [&](int c) {
            const int at = 16 * (c / RT) + 8 * h, rt = c % RT;
            const float4 s0 = *reinterpret_cast<const float4*>(&sws[w][at]);
            const float4 s1 = *reinterpret_cast<const float4*>(&sws[w][at + 4]);
            const float4 x0 = *reinterpret_cast<const float4*>(&xt[b3][32 * rt + j][at]);
            const float4 x1 = *reinterpret_cast<const float4*>(&xt[b3][32 * rt + j][at + 4]);
            sa[0] = s0.x, sa[1] = s0.y, sa[2] = s0.z, sa[3] = s0.w;
            sa[4] = s1.x, sa[5] = s1.y, sa[6] = s1.z, sa[7] = s1.w;
            xa[0] = x0.x, xa[1] = x0.y, xa[2] = x0.z, xa[3] = x0.w;
            xa[4] = x1.x, xa[5] = x1.y, xa[6] = x1.z, xa[7] = x1.w;
        };
        auto plane = [&](int q, int i) {
            const bf16x2 v = {(__bf16)ra, (__bf16)rb};
            const uint32_t u2 = __builtin_bit_cast(uint32_t, v);
            o[q][i] = u2;
            ra -= __builtin_bit_cast(float, u2 << 16);
            rb -= __builtin_bit_cast(float, u2 & 0xffff0000u);
        };
        auto vstep = [&](int n) {
            const int c = n >> 3, i = (n >> 1) & 3, rt = c % RT;
            if ((n & 7) == 0)
#pragma unroll
                for (int e = 0; e < 8; ++e) xv[e] = xa[e], sq[e] = sa[e];
            if ((n & 7) == 3 && c + 1 < NV * RT) vread(c + 1);
            if ((n & 1) == 0) {
                ra = sq[2 * i] * (xv[2 * i] - mub[rt]);
                us[rt] = fmaf(sq[2 * i], ra, us[rt]);
                rb = sq[2 * i + 1] * (xv[2 * i + 1] - mub[rt]);
                us[rt] = fmaf(sq[2 * i + 1], rb, us[rt]);
                plane(0, i);
            } else {
                plane(1, i);
                plane(2, i);
            }
            if ((n & 7) == 7)
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    const u32x4 v = {o[q][0], o[q][1], o[q][2], o[q][3]};
                    vf[c / RT][rt][q] = __builtin_bit_cast(bf16x8, v);
                }
        };
        constexpr int VS = 8 * NV * RT;
        static_assert(VS == 32, "four chunks of v");
        int vn = 0;
        vread(0);
        if (!FROM_S) {
            constexpr int NM = 6 * C::F * TL;
            const int zb = (it + 1) & 1;
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int tl = 0; tl < TL; ++tl)
#pragma unroll
                    for (int t = 0; t < 16; ++t) acc[rt][tl][t] = 0.f;
            bf16x8 qz[2][RT][3], xz[2][TL][3];
            auto zread = [&](int s, int pl) {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
                    if (s < 2 * (rt + 1))
                        qz[s & 1][rt][pl] =
                            pl == 0 ? qa[sidx(rt, s)] : ql[w][sidx(rt, s)][pl > 0 ? pl - 1 : 0][lane];
#pragma unroll
                for (int tl = 0; tl < TL; ++tl) xz[s & 1][tl][pl] = xp[zb][tl][s][pl][lane];
            };
#pragma unroll
            for (int pl = 0; pl < 3; ++pl) zread(0, pl);
            __builtin_amdgcn_sched_barrier(0);
            int mn = 0;
#pragma unroll
            for (int s = 0; s < C::KS; ++s)
#pragma unroll
                for (int q = 0; q < 6; ++q) {
                    if (q >= 2 && q < 5 && s + 1 < C::KS) zread(s + 1, 4 - q);
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                        for (int tl = 0; tl < TL; ++tl)
                            if (s < 2 * (rt + 1)) {
                                acc[rt][tl] =
                                    mfma16(qz[s & 1][rt][kTermA[q]], xz[s & 1][tl][kTermB[q]], acc[rt][tl]);
                                ++mn;
#pragma unroll
                                for (int e = 0; e < 2; ++e)
                                    if (vn * NM < mn * VS) vstep(vn++);
                                __builtin_amdgcn_sched_barrier(0);
                            }
                }
        }
#pragma unroll
        for (int e = 0; e < VS; ++e)
            if (FROM_S) vstep(e);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) u[rt] += us[rt];
        __builtin_amdgcn_sched_barrier(0);
        // its contraction, between its MFMAs the next tile's |z|^2; then its weights
        f32x16 tmp[NGT];
#pragma unroll
        for (int g = 0; g < NGT; ++g)
#pragma unroll
            for (int t = 0; t < 16; ++t) tmp[g][t] = 0.f;
        // |z|^2 in steps of two rows (split_square's order)
        double nrm[2] = {0.0, 0.0};
        float4 cq = {0.f, 0.f, 0.f, 0.f};
        auto nstep = [&](int n) {
            const int rt = n / 8, t4 = (n / 2) & 3, i0 = 2 * (n & 1);
            if (i0 == 0) cq = *reinterpret_cast<const float4*>(&cs[w][32 * rt + 8 * t4 + 4 * h]);
            const double cv[2] = {i0 == 0 ? cq.x : cq.z, i0 == 0 ? cq.y : cq.w};
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int tl = 0; tl < TL; ++tl) {
                    const double z = (double)acc[rt][tl][4 * t4 + i0 + i] - cv[i];
                    nrm[tl] = fma(z, z, nrm[tl]);
                }
        };
        constexpr int NS = 8 * RT;
        int nn = 0;
#pragma unroll
        for (int s = 0; s < NV; ++s)
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                int g = 0;
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int ct = 0; ct <= rt; ++ct, ++g) {
                        bool did = true;
                        if (ct < rt)
                            tmp[g] = mfma16(vf[s][rt][kTermA[q]], vf[s][ct][kTermB[q]], tmp[g]);
                        else if (kTermA[q] == kTermB[q])
                            tmp[g] = mfma16(vf[s][rt][kTermA[q]], vf[s][rt][kTermB[q]], tmp[g]);
                        else if (kTermA[q] == 0)
                            tmp[g] = mfma16(vf[s][rt][0], twice(vf[s][rt][kTermB[q]]), tmp[g]);
                        else
                            did = false;
                        if (!FROM_S && did && nn < NS) {
                            nstep(nn++);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
            }
#pragma unroll
        for (int e = 0; e < NS; ++e)
            if (!FROM_S && e >= nn) nstep(e);
        double sq2 = 0.0;
        if (!FROM_S) {
            if (TL == 1) {
                sq2 = nrm[0] + __shfl_xor(nrm[0], 32, kWave);
            } else {
                const bool up = threadIdx.x & 32;
                sq2 = (up ? nrm[1] : nrm[0]) + __shfl_xor(up ? nrm[0] : nrm[1], 32, kWave);
            }
        }
        const double swd = weight_of(FROM_S ? s_n : bk - 0.5 * sq2, pb + NP);
#pragma unroll
        for (int g = 0; g < NGT; ++g)
#pragma unroll
            for (int t = 0; t < 16; ++t) S[g][t] += tmp[g][t];
        __builtin_amdgcn_sched_barrier(0);
        keep(swd);
        b3 = b3 == 2 ? 0 : b3 + 1;
        put(it & 1, b3 == 2 ? 0 : b3 + 1);  // tile it + 2
        __syncthreads();
    }

#pragma unroll
    for (int rt = 0; rt < RT; ++rt) u[rt] += __shfl_xor(u[rt], 32, kWave);
    if (lane >= NP) wsum = 0.0;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) wsum += __shfl_xor(wsum, d, kWave);
    if (k >= K) return;
    const int64_t rec = (int64_t)k * nch + ch;
#pragma unroll
    for (int g = 0; g < NGT; ++g)
#pragma unroll
        for (int t = 0; t < 16; ++t) gpart[(rec * NGT * 16 + g * 16 + t) * 64 + lane] = S[g][t];
    if (lane < 32) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) vpart[rec * D + 32 * rt + j] = u[rt];
    }
    if (lane == 0) wpart[rec] = wsum;
}

// ------------------------------------------------------ reduce + parameters
// The chunks' partials of S_k (lower 32x32 blocks), u_k and W_k summed in FP64
// in chunk order, times `scale`, into sred[k][NGT * 1024 + D + 1].  A thread per entry, all
// components at once: done by the K blocks of the parameter kernel the chunk
// loop was the longest part of a small gradient (N = 10,007, D = 32, K = 50:
// 127 us for both, now 5 + 7; N = 10^6, D = 64, K = 200: 363, now 27 + 20).
template <int D>
__global__ __launch_bounds__(256) void gmm_reduce_kernel(int nch, double scale, const float* __restrict__ gpart,
                                                         const float* __restrict__ vpart,
                                                         const double* __restrict__ wpart,
                                                         double* __restrict__ sred) {
    constexpr int NG = Gm<D>::NGT * 1024;
    const int64_t k = blockIdx.y;
    const int e = blockIdx.x * 256 + threadIdx.x;
    if (e > NG + D) return;
    double s = 0.0;
    if (e < NG) {
        const float* src = gpart + k * nch * NG + e;
#pragma unroll 8
        for (int c = 0; c < nch; ++c) s += (double)src[(int64_t)c * NG];
    } else if (e < NG + D) {
        const float* src = vpart + k * nch * D + (e - NG);
#pragma unroll 8
        for (int c = 0; c < nch; ++c) s += (double)src[(int64_t)c * D];
    } else {
#pragma unroll 8
        for (int c = 0; c < nch; ++c) s += wpart[k * nch + c];
    }
    sred[k * (NG + D + 1) + e] = scale * s;
}

// G_k = Q_k S_k (the entries the adjoints read: r >= c), v_k = Q_k u_k and the
// parameter maps, a block per component.  The dot products read LDS four
// steps ahead and 16 D threads share them: with 256 threads and one step at a
// time LDS latency took 55 us at D = 64, K = 200.
template <int D>
__global__ __launch_bounds__(16 * D) void gmm_param_kernel(int64_t N, const float* __restrict__ alpha,
                                                        const float* __restrict__ q, const float* __restrict__ l,
                                                        const double* __restrict__ lse_alpha, double ell_bar,
                                                        const double* __restrict__ sred, int sym,
                                                        float* __restrict__ abar, float* __restrict__ mbar,
                                                        float* __restrict__ qbar, float* __restrict__ lbar,
                                                        int accumulate) {
    constexpr int NG = Gm<D>::NGT * 1024;
    const int k = blockIdx.x;
    const int64_t tri = (int64_t)D * (D - 1) / 2;
    __shared__ double S[D][D + 1];
    __shared__ double u[D], v[D];
    __shared__ float Q[D][D + 1];
    const double* src = sred + (int64_t)k * (NG + D + 1);
    for (int e = threadIdx.x; e < NG; e += 16 * D) {
        // block g of the lower triangle: (0,0), (1,0), (1,1); the off-diagonal
        // one is mirrored, the diagonal ones are whole (with sym their
        // symmetric part is S_k, otherwise their lower half)
        const int g = e / 1024, t = (e / 64) % 16, lane = e % 64;
        const int rt = g > 0, ct = g > 1;
        const int r = 32 * rt + drow(t, lane), c = 32 * ct + (lane & 31);
        if (g == 1 || (r >= c && !sym)) {
            S[r][c] = src[e];
            S[c][r] = src[e];
        } else if (sym) {
            S[r][c] = src[e];
        }
    }
    if (sym) {
        __syncthreads();
        for (int e = threadIdx.x; e < D * D; e += 16 * D) {
            const int r = e / D, c = e % D;
            if (r > c && (r ^ c) < 32) {
                const double s = 0.5 * (S[r][c] + S[c][r]);
                S[r][c] = s;
                S[c][r] = s;
            }
        }
    }
    if (threadIdx.x < D) u[threadIdx.x] = src[NG + threadIdx.x];
    for (int e = threadIdx.x; e < D * D; e += 16 * D) {
        const int r = e / D, c = e % D;
        float x = 0.f;
        if (r == c)
            x = (float)exp((double)q[(int64_t)k * D + r]);
        else if (r > c)
            x = l[(int64_t)k * tri + r * (r - 1) / 2 + c];
        Q[r][c] = x;
    }
    const double W = src[NG + D];
    __syncthreads();
    for (int r = threadIdx.x; r < D; r += 16 * D) {
        double s = 0.0;
#pragma unroll 4
        for (int j = 0; j <= r; ++j) s += (double)Q[r][j] * u[j];
        v[r] = s;
    }
    if (threadIdx.x == 0) {
        const double a = W - (double)N * ell_bar * exp((double)alpha[k] - *lse_alpha);
        abar[k] = accumulate ? abar[k] + (float)a : (float)a;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < D * D; e += 16 * D) {
        const int r = e / D, c = e % D;
        if (c > r) continue;
        double g = 0.0;
#pragma unroll 4
        for (int j = 0; j <= r; ++j) g += (double)Q[r][j] * S[j][c];
        if (r == c) {
            const int64_t o = (int64_t)k * D + c;
            double s = 0.0;  // (Q_k^T v_k)_c = sum_{i >= c} Q[i][c] v[i]
#pragma unroll 4
            for (int i = c; i < D; ++i) s += (double)Q[i][c] * v[i];
            mbar[o] = accumulate ? mbar[o] + (float)s : (float)s;
            const double qd = W - (double)Q[c][c] * g;
            qbar[o] = accumulate ? qbar[o] + (float)qd : (float)qd;
        } else {
            const int64_t o = (int64_t)k * tri + r * (r - 1) / 2 + c;
            const float x = (float)(-g);
            lbar[o] = accumulate ? lbar[o] + x : x;
        }
    }
}

// ------------------------------------------------------------------ host
struct GmmLayout {
    size_t Qf, Qs, cvec, bias, scal, fparts, lse, gpart, vpart, wpart, sred, msum, total;
    int64_t nch, chunk;
    unsigned fgrid;
    int kper, ny;  // components per block row of the forward, rows
    bool split;    // bf16 triples (large N) or FP32 MFMA
};

// From 2^17 points on the bf16 triples: N = 10^6, D = 64, K = 200 takes 18.6 ms
// (objective and gradient) against 38.6 in FP32 MFMA.
// Below, a call is a few hundred microseconds of which the matrix pipe is a
// part only, and the FP64 log-likelihood of few points keeps the FP32 chains'
// rounding (the two forms differ by about 5e-8 N^(-1/2) of it).  At least five
// components keep most of a block's eight waves busy.
constexpr int64_t kGmmSplitN = (int64_t)1 << 17;
static bool gmm_split(int64_t N, int K) { return N >= kGmmSplitN && K >= 5; }

static GmmLayout gmm_layout(int64_t N, int D, int K) {
    GmmLayout L{};
    const int64_t n1 = N > 0 ? N : 1;
    // Chunks, and (max, sum) entries of component ranges, of this input or any
    // shorter one, some of which have more of them: of the FP32 form first.
    int64_t nch_most = 1, sums_most = 0;
    {
        const int64_t target = std::max<int64_t>(4096 / K, 1), n = std::min(n1, gmm_split(N, K) ? kGmmSplitN : n1);
        nch_most = std::max(std::min(ceil_div(n, 128), target), ceil_div(n, 16384));
        const int64_t batches = ceil_div(K, D == 64 ? 2 : 4);
        if (batches > 1) sums_most = std::min(n * batches, 128 * (1024 + std::min<int64_t>(ceil_div(n, 128), 1024)));
    }
    const int RT = D / 32;
    const int NF = 16 * RT * (RT + 1) / 2, NGT = RT * (RT + 1) / 2;
    L.split = gmm_split(N, K);
    if (L.split) {
        // One block of eight waves fits a CU: whole rounds of 256 blocks, as
        // few of them as keep a chunk within 32,768 points (the FP32 sums).
        const int64_t groups = ceil_div(K, 8);
        for (int64_t r = 1;; ++r) {
            const int64_t per = 256 * r / groups > 0 ? 256 * r / groups : 1;
            L.chunk = ceil_div(ceil_div(N, per), 64) * 64;
            nch_most = std::max(nch_most, per);
            if (L.chunk <= 32768) break;
        }
        L.nch = ceil_div(N, L.chunk);
        // The forward's 256-point blocks, two a CU: component ranges of 16 or
        // more until there are some eight rounds of them.
        L.fgrid = (unsigned)ceil_div(N, 256);
        int64_t rows = ceil_div(4096, L.fgrid);
        if (rows > K / 16) rows = K / 16;
        if (rows < 1) rows = 1;
        L.kper = (int)ceil_div(K, rows);
        L.ny = (int)ceil_div(K, L.kper);
        if (K >= 32)
            sums_most = std::max(sums_most, std::min(N * (K / 16), 256 * (4096 + std::min<int64_t>(L.fgrid, 4096))));
    } else {
        // About 4,096 blocks of at least 128 points.  Fewer are faster for small N
        // (objective and gradient at N = 10,007, D = 32, K = 50 with 1,024, 2,048
        // and 4,096: 89, 92 and 102 us) but lengthen the FP32 accumulation: with
        // 1,024 the gradient's error there went from 1.3e-7 to 2.4e-7.
        int64_t target = 4096 / K;
        if (target < 1) target = 1;
        int64_t chunk = ceil_div(ceil_div(N > 0 ? N : 1, target), 128) * 128;
        if (chunk > 16384) chunk = 16384;
        if (chunk < 128) chunk = 128;
        L.chunk = chunk;
        L.nch = ceil_div(N > 0 ? N : 1, chunk);
        L.fgrid = (unsigned)ceil_div(N > 0 ? N : 1, 128);
        // The forward takes a 128-point block through all components; with fewer
        // than 1,024 such blocks (three fit a CU) the components are split too,
        // in whole batches.
        const int cpb = D == 64 ? 2 : 4;
        const int64_t batches = ceil_div(K, cpb);
        int64_t rows = ceil_div(1024, L.fgrid);
        if (rows > batches) rows = batches;
        L.kper = (int)(ceil_div(batches, rows) * cpb);
        L.ny = (int)ceil_div(K, L.kper);
    }
    size_t o = 0;
    auto take = [&](size_t bytes) {
        size_t at = o;
        o += align_up(bytes, 256);
        return at;
    };
    L.scal = take(sizeof(GmmHdr) + 256);  // header, lse_alpha, loglik scratch
    L.Qf = take((size_t)K * NF * 64 * 4);
    L.Qs = take(L.split ? (size_t)K * (RT * (RT + 1) * 3 * 64 + D / 4) * 16 : 0);
    L.cvec = take((size_t)K * D * 4);
    L.bias = take((size_t)K * 8);
    L.fparts = take((size_t)ceil_div(n1, 128) * 8);
    L.lse = take((size_t)(N > 0 ? N : 1) * 8);
    L.gpart = take((size_t)K * nch_most * NGT * 1024 * 4);
    L.vpart = take((size_t)K * nch_most * D * 4);
    L.wpart = take((size_t)K * nch_most * 8);
    L.sred = take((size_t)K * (NGT * 1024 + D + 1) * 8);
    L.msum = take((size_t)sums_most * 16);
    L.total = o;
    return L;
}

template <int D>
static void launch_prep(const float* alpha, const float* mu, const float* q, const float* l, int K, char* ws,
                        const GmmLayout& L, hipStream_t st) {
    double* scal = reinterpret_cast<double*>(ws + L.scal + sizeof(GmmHdr));
    hipLaunchKernelGGL(gmm_prep_kernel<D>, dim3(K), dim3(256), 0, st, alpha, mu, q, l, K, (float*)(ws + L.Qf),
                       (float*)(ws + L.cvec), (double*)(ws + L.bias), scal);
    if (L.split)
        hipLaunchKernelGGL(gmm_split_q_kernel<D>, dim3(K), dim3(256), 0, st, q, l, (const float*)(ws + L.cvec),
                           (bf16x8*)(ws + L.Qs));
}

template <int D>
static void launch_fwd(const float* X, int64_t N, int K, char* ws, const GmmLayout& L, double* lse, double* sck,
                       double* loglik, hipStream_t st) {
    double* scal = reinterpret_cast<double*>(ws + L.scal + sizeof(GmmHdr));
    if (L.split)
        hipLaunchKernelGGL(gmm_fwd_split_kernel<D>, dim3(L.fgrid, L.ny), dim3(256), 0, st, X, N, K, L.kper,
                           (const bf16x8*)(ws + L.Qs), (const double*)(ws + L.bias),
                           (const double*)scal, lse, sck, (double2*)(ws + L.msum), (double*)(ws + L.fparts),
                           (GmmHdr*)(ws + L.scal), loglik);
    else
        hipLaunchKernelGGL(gmm_fwd_kernel<D>, dim3(L.fgrid, L.ny), dim3(256), 0, st, X, N, K, L.kper,
                           (const float*)(ws + L.Qf), (const float*)(ws + L.cvec), (const double*)(ws + L.bias),
                           (const double*)scal, lse, sck, (double2*)(ws + L.msum), (double*)(ws + L.fparts),
                           (GmmHdr*)(ws + L.scal), loglik);
    if (L.ny > 1)
        hipLaunchKernelGGL(gmm_lse_merge_kernel<D>, dim3((unsigned)ceil_div(N > 0 ? N : 1, 256)), dim3(256), 0, st, N,
                           L.ny, (const double2*)(ws + L.msum), (const double*)scal, lse, (double*)(ws + L.fparts),
                           (GmmHdr*)(ws + L.scal), loglik);
}

template <int D, bool FROM_S>
static void launch_bwd_t(const float* X, int64_t N, int K, const float* alpha, const float* mu, const float* q,
                         const float* l, double ell_bar, const double* lse, const double* sck, float* ab, float* mb,
                         float* qb, float* lb, int acc, char* ws, const GmmLayout& L, hipStream_t st) {
    double* scal = reinterpret_cast<double*>(ws + L.scal + sizeof(GmmHdr));
    if (L.split)
        hipLaunchKernelGGL((gmm_bwd_split_kernel<D, FROM_S>), dim3((unsigned)(ceil_div(K, 8) * L.nch)), dim3(512), 0,
                           st, X, N, K, L.chunk, (int)L.nch, (const bf16x8*)(ws + L.Qs),
                           mu, (const double*)(ws + L.bias), lse, sck, (float*)(ws + L.gpart),
                           (float*)(ws + L.vpart), (double*)(ws + L.wpart));
    else
        hipLaunchKernelGGL((gmm_bwd_kernel<D, FROM_S>), dim3((unsigned)(K * L.nch)), dim3(256), 0, st, X, N, K,
                           L.chunk, (int)L.nch, (const float*)(ws + L.Qf), (const float*)(ws + L.cvec), mu,
                           (const double*)(ws + L.bias), lse, sck, ell_bar, (float*)(ws + L.gpart),
                           (float*)(ws + L.vpart), (double*)(ws + L.wpart));
    hipLaunchKernelGGL(gmm_reduce_kernel<D>, dim3(Gm<D>::NGT * 4 + 1, K), dim3(256), 0, st, (int)L.nch,
                       L.split ? ell_bar : 1.0, (const float*)(ws + L.gpart), (const float*)(ws + L.vpart), (const double*)(ws + L.wpart),
                       (double*)(ws + L.sred));
    hipLaunchKernelGGL(gmm_param_kernel<D>, dim3(K), dim3(16 * D), 0, st, N, alpha, q, l, (const double*)scal, ell_bar,
                       (const double*)(ws + L.sred), (int)L.split, ab, mb, qb, lb, acc);
}

template <int D>
static void launch_bwd(const float* X, int64_t N, int K, const float* alpha, const float* mu, const float* q,
                       const float* l, double ell_bar, const double* lse, const double* sck, float* ab, float* mb,
                       float* qb, float* lb, int acc, char* ws, const GmmLayout& L, hipStream_t st) {
    if (sck)
        launch_bwd_t<D, true>(X, N, K, alpha, mu, q, l, ell_bar, lse, sck, ab, mb, qb, lb, acc, ws, L, st);
    else
        launch_bwd_t<D, false>(X, N, K, alpha, mu, q, l, ell_bar, lse, sck, ab, mb, qb, lb, acc, ws, L, st);
}

static pvjp_status gmm_args(int64_t N, int D, int K, const void* X, const void* alpha, const void* mu,
                            const void* q, const void* l, const char* name) {
    if (D != 32 && D != 64) {
        set_error("%s: D = %d unsupported (the MFMA path is built for D = 32 and D = 64)", name, D);
        return PVJP_EUNSUPPORTED;
    }
    PVJP_REQUIRE(N >= 0 && N <= ((int64_t)1 << 40), "%s: N = %lld out of range", name, (long long)N);
    PVJP_REQUIRE(K >= 1 && K <= 65535, "%s: K = %d out of range [1, 65535]", name, K);
    PVJP_REQUIRE(alpha && mu && q && l && (N == 0 || X), "%s: X, alpha, mu, q and l must be non-NULL", name);
    PVJP_REQUIRE(aligned(X, 16), "%s: X must be 16-byte aligned", name);
    return PVJP_OK;
}

}  // namespace pvjp

using namespace pvjp;

extern "C" size_t pvjp_gmm_ws_bytes(int64_t N, int D, int K) {
    if (N < 0 || (D != 32 && D != 64) || K < 1) return 0;
    return gmm_layout(N, D, K).total;
}

extern "C" pvjp_status pvjp_gmm_objective(const float* X, int64_t N, int D, int K, const float* alpha,
                                          const float* mu, const float* q, const float* l, double* loglik,
                                          double* lse, double* s, void* ws, size_t ws_bytes, void* stream) {
    clear_error();
    if (pvjp_status e = gmm_args(N, D, K, X, alpha, mu, q, l, "pvjp_gmm_objective")) return e;
    PVJP_REQUIRE(loglik != nullptr, "pvjp_gmm_objective: loglik is NULL");
    PVJP_REQUIRE(ws != nullptr && aligned(ws, 256), "pvjp_gmm_objective: ws must be non-NULL and 256-byte aligned");
    const GmmLayout L = gmm_layout(N, D, K);
    if (ws_bytes < L.total) {
        set_error("pvjp_gmm_objective: workspace has %zu bytes, needs %zu", ws_bytes, L.total);
        return PVJP_ENOMEM;
    }
    char* w = reinterpret_cast<char*>(ws);
    hipStream_t st = as_stream(stream);
    if (D == 64) {
        launch_prep<64>(alpha, mu, q, l, K, w, L, st);
        launch_fwd<64>(X, N, K, w, L, lse, s, loglik, st);
    } else {
        launch_prep<32>(alpha, mu, q, l, K, w, L, st);
        launch_fwd<32>(X, N, K, w, L, lse, s, loglik, st);
    }
    PVJP_LAUNCHED("pvjp_gmm_objective");
    return PVJP_OK;
}

extern "C" pvjp_status pvjp_gmm_vjp(const float* X, int64_t N, int D, int K, const float* alpha, const float* mu,
                                    const float* q, const float* l, double ell_bar, const double* lse,
                                    const double* s, float* alpha_bar, float* mu_bar, float* q_bar, float* l_bar,
                                    int accumulate, void* ws, size_t ws_bytes, void* stream) {
    clear_error();
    if (pvjp_status e = gmm_args(N, D, K, X, alpha, mu, q, l, "pvjp_gmm_vjp")) return e;
    PVJP_REQUIRE(s == nullptr || lse != nullptr, "pvjp_gmm_vjp: the s checkpoint needs lse as well");
    PVJP_REQUIRE(alpha_bar && mu_bar && q_bar && l_bar, "pvjp_gmm_vjp: the four adjoint outputs must be non-NULL");
    PVJP_REQUIRE(ws != nullptr && aligned(ws, 256), "pvjp_gmm_vjp: ws must be non-NULL and 256-byte aligned");
    const GmmLayout L = gmm_layout(N, D, K);
    if (ws_bytes < L.total) {
        set_error("pvjp_gmm_vjp: workspace has %zu bytes, needs %zu", ws_bytes, L.total);
        return PVJP_ENOMEM;
    }
    char* w = reinterpret_cast<char*>(ws);
    hipStream_t st = as_stream(stream);
    double* ll_scratch = reinterpret_cast<double*>(w + L.scal + sizeof(GmmHdr)) + 1;
    if (D == 64) {
        launch_prep<64>(alpha, mu, q, l, K, w, L, st);
        if (lse == nullptr) {
            launch_fwd<64>(X, N, K, w, L, (double*)(w + L.lse), nullptr, ll_scratch, st);
            lse = (const double*)(w + L.lse);
        }
        launch_bwd<64>(X, N, K, alpha, mu, q, l, ell_bar, lse, s, alpha_bar, mu_bar, q_bar, l_bar, accumulate, w, L,
                       st);
    } else {
        launch_prep<32>(alpha, mu, q, l, K, w, L, st);
        if (lse == nullptr) {
            launch_fwd<32>(X, N, K, w, L, (double*)(w + L.lse), nullptr, ll_scratch, st);
            lse = (const double*)(w + L.lse);
        }
        launch_bwd<32>(X, N, K, alpha, mu, q, l, ell_bar, lse, s, alpha_bar, mu_bar, q_bar, l_bar, accumulate, w, L,
                       st);
    }
    PVJP_LAUNCHED("pvjp_gmm_vjp");
    return PVJP_OK;
}
