// Dense k-means (Sec. 7.4), the workload of the forward-over-reverse example:
//   f(C) = sum_i min_k |x_i - c_k|^2   (squared distance; X [N x D] and
//   C [K x D] row-major FP32).
// The objective's search keeps each point's nearest centre (the primal's
// auxiliary output).  With the assignments fixed the gradient is an
// accumulator of the points into their centres (Sec. 5.4 / 6):
//   C_bar_k = 2 f_bar (n_k c_k - S_k),  S_k = sum_{a_i = k} x_i,
// and the jvp of the vjp in direction C_dot (the Hessian-vector product,
// the Hessian being diagonal) is 2 f_bar n_k C_dot_k; C_dot = 1 gives the
// diagonal.  Both come from one accumulation pass, and the search is not
// repeated.
//
// Distances are formed in FP64 by the chain acc = fma(x_d - c_d, x_d - c_d,
// acc), d = 0..D-1, so every implementation of that chain (the oracle's
// included) decides the same nearest centre, ties going to the lowest k.
// Large searches form the chains of few centres only: those that FP32 sums of
// bf16 products, with a bound on their error, leave within reach of the
// nearest.
#include <math.h>

#include <algorithm>

#include "common.h"
#include "prims.h"

namespace pvjp {

constexpr int kKmChunkD = 32;        // dimensions of X staged (and held in registers) at a time
constexpr int kKmMaxD = 1024;
constexpr size_t kKmSliceBytes = 64 * 1024;  // a slice's FP64 centres: 32 centres up to D = 256
constexpr int kKmPts = 256;          // points per distance block, one per lane
constexpr int kKmSumBlocks = 1024;   // fixed partition of the objective's sum
constexpr int kKmSmallK = 16;        // register accumulators in the gradient up to this K
constexpr int kKmChunkMax = 4096;
constexpr int64_t kKmFill = 256;     // blocks that the distances want
constexpr int kKmNearPts = 128;      // points per block of the bounded search
constexpr int kKmNearSlices = 16;    // at most this many ranges of centres in it
constexpr int kKmWhole = 16;         // entries formed whole by a block of decisions, at most

// Centres per slice: as many as kKmSliceBytes of FP64 holds (>= 4), at most 32.
static int km_cps(int D, int K) {
    int c = (int)(kKmSliceBytes / ((size_t)D * 8));
    c = c >= 32 ? 32 : (c >= 16 ? 16 : (c >= 8 ? 8 : 4));
    return K < c ? K : c;
}

// The centres in FP64, once per call, laid out per slice as [d][CPS]: Cw[(s D
// + d) CPS + k'] = c_{s cps + k'}[d], zero beyond the slice's centres.  A
// chunk of dimensions of one slice is then one contiguous block that the
// distance kernel reads at wave-uniform addresses, and the chains subtract
// FP64 values without a conversion.
__global__ __launch_bounds__(256) void km_widen_kernel(const float* __restrict__ C, int K, int D, int cps, int CPS,
                                                       int64_t n, double* __restrict__ Cw) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
        const int kp = (int)(e % CPS);
        const int64_t sd = e / CPS;
        const int d = (int)(sd % D);
        const int64_t k = (sd / D) * cps + kp;
        Cw[e] = (kp < cps && k < K) ? (double)C[k * D + d] : 0.0;
    }
}

// Whether any of n flags is set (the whole block asks).
__device__ __forceinline__ bool km_any(const int32_t* __restrict__ f, int n) {
    int any = 0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) any |= f[i];
    return __syncthreads_or(any);
}

// Block (bx, s) takes points [bx 256, bx 256 + 256), one per lane, and centre
// slice s (centres [s cps, s cps + cps)).  X comes in 32-dimension chunks,
// copied into LDS with consecutive threads on consecutive addresses.  For each
// dimension d in order, a lane reads x[d] once and extends the CPS chains
// acc_k = fma(x[d] - c_k[d], x[d] - c_k[d], acc_k) (independent of each
// other, each in d order); the c_k[d] are wave-uniform reads of the widened
// centres (scalar loads, no LDS).  Every lane writes its nearest (distance,
// centre) of the slice.
template <int CPS>
__global__ __launch_bounds__(256) void km_dist_kernel(const float* __restrict__ X, int64_t N, int D,
                                                      const double* __restrict__ Cw, int K, int cps,
                                                      const int32_t* __restrict__ bad, int nbad,
                                                      const int32_t* __restrict__ open,
                                                      double* __restrict__ bd, int32_t* __restrict__ bk) {
    if (bad && !open[blockIdx.x] && !km_any(bad, nbad)) return;  // the bounded search has them
    constexpr int kStride = kKmChunkD + 1;  // odd row stride: lanes hit distinct banks
    __shared__ float xs[kKmPts * kStride];
    const int s = blockIdx.y;
    const int k0 = s * cps;
    const int kc = (K - k0) < cps ? (K - k0) : cps;
    const int64_t p0 = (int64_t)blockIdx.x * kKmPts;
    const int np = (N - p0) < kKmPts ? (int)(N - p0) : kKmPts;
    const int t = threadIdx.x;
    const bool live = t < np;
    double acc[CPS];
#pragma unroll
    for (int k = 0; k < CPS; ++k) acc[k] = 0.0;
    for (int d0 = 0; d0 < D; d0 += kKmChunkD) {
        const int dn = (D - d0) < kKmChunkD ? (D - d0) : kKmChunkD;
        if (d0 > 0) __syncthreads();  // the previous chunk has been read
        const float* xb = X + p0 * D + d0;
        if (dn == kKmChunkD && np == kKmPts) {
            // thread t copies column t % 32 of rows t / 32 + 8 u, u < 32, kU
            // loads in flight (fewer where the chains need the registers);
            // each 32-lane group reads one contiguous 128-byte row piece
            constexpr int kU = CPS >= 16 ? 8 : kKmChunkD;
            const int j = t & (kKmChunkD - 1), r0 = t / kKmChunkD;
            const uint32_t lo = (uint32_t)(r0 * D + j);  // the lane's offset from a uniform row base
#pragma unroll
            for (int u0 = 0; u0 < kKmChunkD; u0 += kU) {
                float v[kU];
#pragma unroll
                for (int u = 0; u < kU; ++u) v[u] = (xb + (int64_t)(8 * (u0 + u)) * D)[lo];
#pragma unroll
                for (int u = 0; u < kU; ++u) xs[(r0 + 8 * (u0 + u)) * kStride + j] = v[u];
            }
        } else {
            for (int e = t; e < np * dn; e += kKmPts) {
                const int pt = e / dn, j = e - pt * dn;
                xs[pt * kStride + j] = xb[(int64_t)pt * D + j];
            }
        }
        __syncthreads();
        const double* cb = Cw + ((int64_t)s * D + d0) * CPS;
        const float* xr = xs + (live ? t : 0) * kStride;
#pragma unroll 2
        for (int j = 0; j < dn; ++j) {
            const double xj = (double)xr[j];
#pragma unroll
            for (int k = 0; k < CPS; ++k) {
                const double u = xj - cb[j * CPS + k];
                acc[k] = fma(u, u, acc[k]);
            }
        }
    }
    if (!live) return;  // after the last barrier
    double best = acc[0];
    int bkk = 0;
#pragma unroll
    for (int k = 1; k < CPS; ++k)
        if (k < kc && acc[k] < best) best = acc[k], bkk = k;
    bd[(int64_t)s * N + p0 + t] = best;
    bk[(int64_t)s * N + p0 + t] = k0 + bkk;
}

// -------------------------------------------------------- bounded search
// x and c are taken relative to the first centre (a common offset of the data
// would only widen the bound).  Then
// |x - c|^2 - |x|^2 = |c|^2 - 2 x.c, with x.c as FP32 sums of bf16 products:
// x = h + m + r, each part rounded to nearest in 8 bits, so |m| <= 2^-8 |x| and
// |r| <= 2^-17 |x|.  Of a product the terms hh, hm, mh are taken; those left out
// reach 2^-16 + 2 2^-17 = 8 2^-18 of it (x = c = 1.0039139: 7.95), so each of the
// D products is off by less than 8.1 2^-18 of it, and the 3 D additions (a step
// of the matrix unit may truncate: 2^-23 each) by less than 4 (D + 16) 2^-23
// of sum |x_d c_d| <= |x| |c|.  With beta the sum of both, the FP32 value g of
// centre k is within
//   e = |c| (2 beta |x| + 2^-21 |c|) + 2^-38 |x|^2 + 2^-100
// of the exact one, up to what all centres of a point share (2^-21 and the
// slack of beta cover the rounding of the differences, of |c|^2, g and the
// bounds; the last terms that of the FP64 chain itself and underflow).  A centre
// whose g - e exceeds the smallest g + e is not the nearest.  Per point and
// range of centres the three smallest g - e are kept, two with their centre;
// then the FP64 chains of those within reach decide, of a whole range where
// its third is within reach too; points with many such ranges go to the FP64
// search after all.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void km_split8(const float (&x)[8], bf16x8 (&p)[2]) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const __bf16 hi = (__bf16)x[i];
        p[0][i] = hi;
        p[1][i] = (__bf16)(x[i] - (float)hi);
    }
}

// Eight dimensions from d0 of one row, relative to row `ref` (zero beyond D).
__device__ __forceinline__ void km_row8(const float* __restrict__ row, const float* __restrict__ ref, int d0, int D,
                                        bool vec, float (&x)[8]) {
    if (vec && d0 + 8 <= D) {
        const float4 a = *reinterpret_cast<const float4*>(row + d0), b = *reinterpret_cast<const float4*>(row + d0 + 4);
        const float4 r = *reinterpret_cast<const float4*>(ref + d0), s = *reinterpret_cast<const float4*>(ref + d0 + 4);
        x[0] = a.x - r.x, x[1] = a.y - r.y, x[2] = a.z - r.z, x[3] = a.w - r.w;
        x[4] = b.x - s.x, x[5] = b.y - s.y, x[6] = b.z - s.z, x[7] = b.w - s.w;
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = d0 + i < D ? row[d0 + i] - ref[d0 + i] : 0.f;
    }
}

// A tile of 32 centres: its fragments (lane l: centre l % 32, dimensions 16 s
// + 8 (l / 32) + 0..7, planes h and m), |c|^2, a bound of |c| and 2^-21 |c|^2
// (a row past K: |c|^2 infinite), and the flag of a |c|^2 that FP32 cannot
// work with, which sends the call to the FP64 search.
template <int KS>
__global__ __launch_bounds__(256) void km_near_prep_kernel(const float* __restrict__ C, int K, int D, bool vec,
                                                           bf16x8* __restrict__ Cf, float* __restrict__ cst,
                                                           int32_t* __restrict__ bad) {
    __shared__ double sq[256];
    const int t = threadIdx.x, tile = blockIdx.x;
    const int k = 32 * tile + (t & 31);
    double s = 0.0;
    for (int e = t; e < KS * 64; e += 256) {  // e % 64 is the thread's lane throughout
        float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (k < K) km_row8(C + (int64_t)k * D, C, 16 * (e / 64) + 8 * ((e >> 5) & 1), D, vec, x);
#pragma unroll
        for (int i = 0; i < 8; ++i) s = fma((double)x[i], (double)x[i], s);
        bf16x8 p[2];
        km_split8(x, p);
#pragma unroll
        for (int q = 0; q < 2; ++q) Cf[((int64_t)tile * KS * 2 + (e / 64) * 2 + q) * 64 + (e & 63)] = p[q];
    }
    sq[t] = s;
    __syncthreads();
    if (t < 32) {
        for (int g = 1; g < 8; ++g) s += sq[t + 32 * g];
        const float nc = (float)sqrt(s) * 1.001f;
        float* o = cst + (int64_t)tile * 96 + t;
        o[0] = k < K ? (float)s : INFINITY;
        o[32] = k < K ? nc : 0.f;
        o[64] = k < K ? nc * nc * 0x1p-21f : 0.f;
        const uint64_t b = __ballot(k < K && !(s < 1e36));
        if (t == 0) bad[tile] = b != 0;
    }
}

struct KmNear {
    float u;           // the smallest g + e
    float m1, m2, m3;  // the smallest g - e
    int32_t k1, k2;    // of the first two, the centres
};

// Block (bx, s): points [128 bx, 128 bx + 128), 32 to a wave, and centre tiles
// [s per, (s + 1) per).  A wave keeps its points' fragments in registers; the
// centre tiles pass through LDS, the next one loaded while this one is worked
// on.  Bound by LDS reads and MFMA at D = 256 (48 steps of 32 cycles per tile)
// and by the 13 vector instructions per pair at small D.
// N = 10,000, D = 256, K = 1,024: 40 us (the FP64 chains of all pairs: 231).
template <int KS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void km_near_kernel(
    const float* __restrict__ X, int64_t N, int D, const float* __restrict__ C, bool vec,
    const bf16x8* __restrict__ Cf, const float* __restrict__ cst, int ntiles, int per, KmNear* __restrict__ out,
    int32_t* __restrict__ open) {
    constexpr int U = KS * 2 * 64;  // 16-byte units per tile
    constexpr int PER = U / 256;
    static_assert(U % 256 == 0, "a tile is whole rounds of the block");
    __shared__ u32x4 ct[2][U];
    __shared__ __align__(16) float cc[2][96];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int j = lane & 31, h = lane >> 5;
    const int64_t p = (int64_t)blockIdx.x * kKmNearPts + w * 32 + j;
    const int t0 = blockIdx.y * per, t1 = min(ntiles, t0 + per);
    static_assert(kKmPts % kKmNearPts == 0, "a flag per block of the FP64 search");
    if (blockIdx.y == 0 && t == 0) open[blockIdx.x / (kKmPts / kKmNearPts)] = 0;  // the decisions set it
    u32x4 nx[PER];
    float nk = 0.f;
    auto fetch = [&](int tile) {
#pragma unroll
        for (int u = 0; u < PER; ++u) nx[u] = reinterpret_cast<const u32x4*>(Cf)[(int64_t)tile * U + u * 256 + t];
        if (t < 96) nk = cst[(int64_t)tile * 96 + t];
    };
    auto put = [&](int b) {
#pragma unroll
        for (int u = 0; u < PER; ++u) ct[b][u * 256 + t] = nx[u];
        if (t < 96) cc[b][t] = nk;
    };
    fetch(t0);
    bf16x8 xf[KS][2];
    float x2 = 0.f;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if (p < N) km_row8(X + p * D, C, 16 * s + 8 * h, D, vec, x);
#pragma unroll
        for (int i = 0; i < 8; ++i) x2 = fmaf(x[i], x[i], x2);
        km_split8(x, xf[s]);
    }
    x2 += __shfl_xor(x2, 32, kWave);
    x2 *= 1.001f;
    constexpr float kBeta = 8.1f * 0x1p-18f + 4.f * (16.f * KS + 16.f) * 0x1p-23f;
    const float ex = 2.f * kBeta * sqrtf(x2);
    put(0);
    float u = INFINITY, m1 = INFINITY, m2 = INFINITY, m3 = INFINITY;
    int k1 = 0, k2 = 0;
    for (int tile = t0; tile < t1; ++tile) {
        const int b = (tile - t0) & 1;
        if (tile + 1 < t1) fetch(tile + 1);
        __syncthreads();  // buffer b is filled, and the other one no longer read
        const bf16x8* cf = reinterpret_cast<const bf16x8*>(ct[b]);
        f32x16 acc;
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const bf16x8 ch = cf[(s * 2) * 64 + lane], cm = cf[(s * 2 + 1) * 64 + lane];
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(cm, xf[s][0], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ch, xf[s][1], acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ch, xf[s][0], acc, 0, 0, 0);
        }
        const int kb = 32 * tile + 4 * h;
#pragma unroll
        for (int t4 = 0; t4 < 4; ++t4) {
            const float4 a = *reinterpret_cast<const float4*>(&cc[b][8 * t4 + 4 * h]);
            const float4 n = *reinterpret_cast<const float4*>(&cc[b][32 + 8 * t4 + 4 * h]);
            const float4 d = *reinterpret_cast<const float4*>(&cc[b][64 + 8 * t4 + 4 * h]);
            const float c2[4] = {a.x, a.y, a.z, a.w}, nc[4] = {n.x, n.y, n.z, n.w}, dc[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float g = fmaf(-2.f, acc[4 * t4 + i], c2[i]);
                const float e = fmaf(nc[i], ex, dc[i]);
                const float lo = g - e;
                const int k = kb + 8 * t4 + i;
                u = fminf(u, g + e);
                const bool b1 = lo < m1, b2 = lo < m2;
                m3 = fminf(m3, fmaxf(m2, lo));
                m2 = fminf(m2, fmaxf(m1, lo));
                m1 = fminf(m1, lo);
                k2 = b1 ? k1 : (b2 ? k : k2);
                k1 = b1 ? k : k1;
            }
        }
        if (tile + 1 < t1) put(b ^ 1);
    }
    if (p >= N) return;
    const float e0 = fmaf(x2, 0x1p-38f, 0x1p-100f);
    KmNear r;
    r.u = x2 < 1e36f ? u + e0 : NAN;  // NaN: the FP64 search has the point
    r.m1 = m1 - e0, r.m2 = m2 - e0, r.m3 = m3 - e0;
    r.k1 = k1, r.k2 = k2;
    out[((int64_t)blockIdx.y * 2 + h) * N + p] = r;
}

// The distance chain of point row x and centre row c.
__device__ __forceinline__ double km_chain(const float* __restrict__ x, const float* __restrict__ c, int D, bool vec) {
    double acc = 0.0;
    int d = 0;
    if (vec) {
#pragma unroll 4
        for (; d + 4 <= D; d += 4) {
            const float4 a = *reinterpret_cast<const float4*>(x + d), b = *reinterpret_cast<const float4*>(c + d);
            const double u0 = (double)a.x - (double)b.x, u1 = (double)a.y - (double)b.y;
            const double u2 = (double)a.z - (double)b.z, u3 = (double)a.w - (double)b.w;
            acc = fma(u3, u3, fma(u2, u2, fma(u1, u1, fma(u0, u0, acc))));
        }
    } else {
#pragma unroll 8
        for (; d < D; ++d) {
            const double u = (double)x[d] - (double)c[d];
            acc = fma(u, u, acc);
        }
    }
    return acc;
}

// Four lanes per point: the centres within reach, their chains, the nearest
// (the lowest of equal ones).  Where an entry's third is within reach too, a
// wave afterwards forms the chains of all its centres.  With more than kKmWhole
// such entries in a block (centres that all agree to within the bound, or in
// tight groups far from the first one), or a point's norm beyond FP32, the
// block leaves its points to the FP64 search that follows (the flag open of
// their 256), which costs less.  Objective in all, with that way out, without it
// and by the FP64 search alone, us: N = 10,000, D = 256, K = 1,024, equal
// centres 278, 5,140, 226, 16 groups of 64 centres 282, 4,250, 228; N = 65,536,
// D = 16, K = 256, equal centres 58, 319, 40 (the most that it costs).
__global__ __launch_bounds__(256) void km_decide_kernel(const float* __restrict__ X, int64_t N, int D,
                                                        const float* __restrict__ C, int K, bool vec,
                                                        const KmNear* __restrict__ near, int nent, int per,
                                                        const int32_t* __restrict__ bad, int ntiles,
                                                        int32_t* __restrict__ open, double* __restrict__ bd,
                                                        int32_t* __restrict__ bk) {
    constexpr int kEnt = 2 * kKmNearSlices;
    constexpr int32_t kNone = 0x7fffffff;
    __shared__ int32_t list[64][2 * kEnt];   // single centres
    __shared__ int32_t whole[kKmWhole];      // point of the block * kEnt + entry
    __shared__ double wd[kKmWhole];          // and what they gave
    __shared__ int32_t wk[kKmWhole];
    __shared__ int32_t cnt[64], nwhole;
    if (km_any(bad, ntiles)) return;
    const int q = threadIdx.x & 3, pt = threadIdx.x >> 2;
    const int64_t p = (int64_t)blockIdx.x * 64 + pt;
    if (threadIdx.x < 64) cnt[threadIdx.x] = 0;
    if (threadIdx.x == 0) nwhole = 0;
    __syncthreads();
    if (p < N) {
        float u = INFINITY;
        bool all = false;
        for (int e = q; e < nent; e += 4) {
            const float v = near[(int64_t)e * N + p].u;
            all |= v != v;
            u = fminf(u, v);
        }
        u = fminf(u, __shfl_xor(u, 1, kWave));
        u = fminf(u, __shfl_xor(u, 2, kWave));
        all = __shfl((int)all, threadIdx.x & 60, kWave);  // entry 0 is lane 0's, and all entries agree
        if (all) {
            if (q == 0) atomicAdd(&nwhole, kKmWhole + 1);
        } else {
            for (int e = q; e < nent; e += 4) {
                const KmNear r = near[(int64_t)e * N + p];
                if (r.m3 <= u) {
                    const int at = atomicAdd(&nwhole, 1);
                    if (at < kKmWhole) whole[at] = pt * kEnt + e;
                } else {
                    if (r.m1 <= u) list[pt][atomicAdd(&cnt[pt], 1)] = r.k1;
                    if (r.m2 <= u) list[pt][atomicAdd(&cnt[pt], 1)] = r.k2;
                }
            }
        }
    }
    __syncthreads();
    if (nwhole > kKmWhole) {
        if (threadIdx.x == 0) open[(int64_t)blockIdx.x * 64 / kKmPts] = 1;
        return;
    }
    double best = INFINITY;
    int32_t bestk = kNone;
    auto take = [&](double d, int32_t k) {
        if (d < best || (d == best && k < bestk)) best = d, bestk = k;
    };
    auto meet = [&](int o) {
        const double d = __shfl_xor(best, o, kWave);
        const int32_t k = __shfl_xor(bestk, o, kWave);
        take(d, k);
    };
    for (int i = threadIdx.x / kWave; i < nwhole; i += 256 / kWave) {
        const int e = whole[i] % kEnt;
        const float* x = X + ((int64_t)blockIdx.x * 64 + whole[i] / kEnt) * D;
        const int first = (e >> 1) * per, last = min(ntiles, first + per);
        best = INFINITY, bestk = kNone;
        // the entry's centres: those with bit 2 equal to e's bit 0, 64 in 128
        for (int c0 = 32 * first; c0 < min(K, 32 * last); c0 += 2 * kWave) {
            const int l = threadIdx.x & (kWave - 1);
            const int c = c0 + ((l & ~3) << 1) + ((e & 1) << 2) + (l & 3);
            if (c < min(K, 32 * last)) take(km_chain(x, C + (int64_t)c * D, D, vec), c);
        }
#pragma unroll
        for (int o = 1; o < kWave; o *= 2) meet(o);
        if ((threadIdx.x & (kWave - 1)) == 0) wd[i] = best, wk[i] = bestk;
    }
    __syncthreads();
    best = INFINITY, bestk = kNone;
    if (p < N) {
        for (int i = q; i < cnt[pt]; i += 4)
            take(km_chain(X + p * D, C + (int64_t)list[pt][i] * D, D, vec), list[pt][i]);
        for (int i = q; i < nwhole; i += 4)
            if (whole[i] / kEnt == pt) take(wd[i], wk[i]);
    }
    meet(1);
    meet(2);
    if (q == 0 && p < N) bd[p] = best, bk[p] = bestk;
}

// Nearest centre over the slices in increasing order (strict <: ties keep
// the lower centre), and the block's share of the objective: block b takes
// points b 256 + t + r G 256 (G = gridDim.x, fixed by N), sums them per
// thread in r order and then over the block in a fixed tree.
__global__ __launch_bounds__(256) void km_combine_kernel(const double* __restrict__ bd, const int32_t* __restrict__ bk,
                                                         int64_t N, int nslice, const int32_t* __restrict__ bad,
                                                         int nbad, const int32_t* __restrict__ open,
                                                         int32_t* __restrict__ assign, double* __restrict__ part) {
    __shared__ double sh[256];
    const bool decided = bad && !km_any(bad, nbad);  // by the bounded search, but for the open points
    double acc = 0.0;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < N; p += (int64_t)gridDim.x * blockDim.x) {
        double best = bd[p];
        int32_t k = bk[p];
        const int ns = decided && !open[p / kKmPts] ? 1 : nslice;
        for (int s = 1; s < ns; ++s) {
            const double v = bd[(int64_t)s * N + p];
            if (v < best) best = v, k = bk[(int64_t)s * N + p];
        }
        assign[p] = k;
        acc += best;
    }
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int d = 128; d >= 1; d >>= 1) {
        if ((int)threadIdx.x < d) sh[threadIdx.x] += sh[threadIdx.x + d];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// f = the sum of the G block shares in a fixed tree (G <= 1024).
__global__ __launch_bounds__(1024) void km_sum_kernel(const double* __restrict__ part, int G, double* f) {
    __shared__ double sh[1024];
    sh[threadIdx.x] = (int)threadIdx.x < G ? part[threadIdx.x] : 0.0;
    __syncthreads();
    for (int d = 512; d >= 1; d >>= 1) {
        if ((int)threadIdx.x < d) sh[threadIdx.x] += sh[threadIdx.x + d];
        __syncthreads();
    }
    if (threadIdx.x == 0) *f = sh[0];
}

// Accumulators of the gradient for K <= kKmSmallK and D <= 256: block c takes
// points [c chunk, (c+1) chunk); thread t is column d = t % D of point lane
// g = t / D (G = 256 / D lanes), adds x_j[d] of points j = g, g + G, ... into
// KM FP64 registers, the one of its centre selected (the others add 0, which
// leaves them unchanged), then the G lanes are summed per column in g order.
// All of X's reads are coalesced rows.  No atomics: the order is fixed.
template <int KM>
__global__ __launch_bounds__(256) void km_acc_small_kernel(const float* __restrict__ X, int64_t N, int D, int K,
                                                           int64_t chunk, const int32_t* __restrict__ assign,
                                                           double* __restrict__ spart, int32_t* __restrict__ npart) {
    __shared__ double rs[256];
    __shared__ int32_t rc[256];
    const int G = 256 / D;
    const int t = threadIdx.x, g = t / D, d = t - g * D;
    const bool act = g < G;
    const int64_t i0 = (int64_t)blockIdx.x * chunk;
    const int64_t i1 = (i0 + chunk < N) ? i0 + chunk : N;
    double acc[KM];
    int32_t cnt[KM];
#pragma unroll
    for (int k = 0; k < KM; ++k) acc[k] = 0.0, cnt[k] = 0;
    if (act) {
        constexpr int U = 8;  // points whose loads are in flight together
        int64_t j = i0 + g;
        for (; j + (U - 1) * (int64_t)G < i1; j += U * (int64_t)G) {
            int32_t a[U];
            float x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                a[u] = assign[j + u * (int64_t)G];
                x[u] = X[(j + u * (int64_t)G) * D + d];
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int k = 0; k < KM; ++k) {
                    acc[k] += (a[u] == k) ? (double)x[u] : 0.0;
                    cnt[k] += (a[u] == k) ? 1 : 0;
                }
            }
        }
        for (; j < i1; j += G) {
            const int32_t a = assign[j];
            const double x = (double)X[j * D + d];
#pragma unroll
            for (int k = 0; k < KM; ++k) {
                acc[k] += (a == k) ? x : 0.0;
                cnt[k] += (a == k) ? 1 : 0;
            }
        }
    }
#pragma unroll
    for (int k = 0; k < KM; ++k) {
        if (k < K) {  // uniform: every thread meets the same barriers
            rs[t] = acc[k];
            rc[t] = cnt[k];
            __syncthreads();
            if (t < D) {
                double sum = 0.0;
                int32_t c = 0;
                for (int q = 0; q < G; ++q) sum += rs[q * D + t], c += rc[q * D + t];
                const int64_t o = (int64_t)blockIdx.x * K + k;
                spart[o * D + t] = sum;
                if (t == 0) npart[o] = c;
            }
            __syncthreads();
        }
    }
}

// Accumulators of the gradient for larger K: block (c, sl) takes points
// [c chunk, (c+1) chunk) and centres [sl cpb, sl cpb + cpb).  The block first
// lists, in point order, the chunk's points assigned to its centres (a stable
// compaction by ballots and a running offset); then thread (kk, d) adds x_i[d]
// of the listed points of centre sl cpb + kk in that order, in FP64 (thread
// (kk, 0) also counts them).  No atomics: the order is fixed.
__global__ __launch_bounds__(1024) void km_acc_kernel(const float* __restrict__ X, int64_t N, int D, int K, int cpb,
                                                      int64_t chunk, const int32_t* __restrict__ assign,
                                                      double* __restrict__ spart, int32_t* __restrict__ npart) {
    __shared__ int32_t lj[kKmChunkMax];  // listed point offsets within the chunk
    __shared__ int32_t lk[kKmChunkMax];  // and their centres
    __shared__ int32_t wtot[1024 / kWave];
    const int64_t i0 = (int64_t)blockIdx.x * chunk;
    const int64_t i1 = (i0 + chunk < N) ? i0 + chunk : N;
    const int cnt = (int)(i1 - i0);
    const int klo = blockIdx.y * cpb;
    const int khi = (klo + cpb < K) ? klo + cpb : K;
    const int w = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
    const int nw = (int)((blockDim.x + kWave - 1) / kWave);
    int m = 0;  // listed so far (the same in every thread)
    for (int j0 = 0; j0 < cnt; j0 += blockDim.x) {
        const int j = j0 + (int)threadIdx.x;
        const int32_t a = j < cnt ? assign[i0 + j] : -1;
        const bool f = a >= klo && a < khi;
        const uint64_t bal = __ballot(f);
        const int rank = __popcll(bal & ((1ull << lane) - 1ull));
        if (lane == 0) wtot[w] = __popcll(bal);
        __syncthreads();
        int base = m, tot = 0;
        for (int q = 0; q < nw; ++q) {
            if (q < w) base += wtot[q];
            tot += wtot[q];
        }
        if (f) lj[base + rank] = j, lk[base + rank] = a;
        m += tot;
        __syncthreads();  // wtot is rewritten next round; the list is read below
    }
    const int kk = threadIdx.x / D, d = threadIdx.x % D;
    const int k = klo + kk;
    if (kk >= cpb || k >= K) return;  // after the last barrier
    double s = 0.0;
    int32_t c = 0;
    const float* xc = X + i0 * D + d;
    for (int q = 0; q < m; ++q) {
        if (lk[q] == k) {
            s += (double)xc[(int64_t)lj[q] * D];
            ++c;
        }
    }
    const int64_t o = ((int64_t)blockIdx.x * K + k);
    spart[o * D + d] = s;
    if (d == 0) npart[o] = c;
}

// C_bar = 2 f_bar (n c - S) and, with C_dot, hvp = 2 f_bar n C_dot, from the
// chunk partials summed in chunk order.  WAVE: one wave per element, lane l
// takes the partials l, l + 64, ... and a fixed shuffle tree combines the
// lanes (many chunks); otherwise one thread per element (few chunks).
template <bool WAVE>
__global__ __launch_bounds__(256) void km_finish_kernel(int D, int K, int nchunk, const float* __restrict__ C,
                                                        double f_bar, const double* __restrict__ spart,
                                                        const int32_t* __restrict__ npart, float* __restrict__ cbar,
                                                        const float* __restrict__ cdot, float* __restrict__ hvp,
                                                        int accumulate) {
    const int64_t KD = (int64_t)K * D;
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t e = WAVE ? (int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave
                           : (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= KD) return;  // whole waves leave together when WAVE
    const int64_t k = e / D;
    double S = 0.0;
    int64_t n = 0;
    if (WAVE) {
        for (int c = lane; c < nchunk; c += kWave) {
            S += spart[(int64_t)c * KD + e];
            n += npart[(int64_t)c * K + k];
        }
#pragma unroll
        for (int o = kWave / 2; o >= 1; o >>= 1) {
            S += __shfl_down(S, o, kWave);
            n += __shfl_down(n, o, kWave);
        }
        if (lane != 0) return;
    } else {
        // eight chunks' partials in flight (49 chunks: 14.9 us one after another,
        // 6)
#pragma unroll 8
        for (int c = 0; c < nchunk; ++c) {
            S += spart[(int64_t)c * KD + e];
            n += npart[(int64_t)c * K + k];
        }
    }
    const double g = 2.0 * f_bar * ((double)n * (double)C[e] - S);
    cbar[e] = accumulate ? cbar[e] + (float)g : (float)g;
    if (hvp) {
        const double h = 2.0 * f_bar * (double)n * (double)cdot[e];
        hvp[e] = accumulate ? hvp[e] + (float)h : (float)h;
    }
}

// ------------------------------------------------------------------ host
struct KmPlan {
    int cps, cpsT, nslice, sum_blocks;  // centres per slice, and the kernel's width for them
    bool small;  // register accumulators in the gradient
    int cpb, nslices_acc;
    int64_t chunk, nchunk;
    int near_ks, near_tiles, near_per, near_slices;  // the bounded search (0: not used)
    size_t cd, bd, bk, part, spart, npart, cf, cst, bad, open, near, total;
};

// The bounded search wants enough pairs to pay for its three more launches and
// its decisions, fragments that fit the registers (D <= 256), and chains longer
// than the 13 vector instructions it spends on a pair; rows of no whole 16
// bytes load slowly and want twice the work.  Objective and gradient, FP64
// search against this one, just above the line: N = 40,000, D = 64, K = 128:
// 78 and 65 us; N = 65,536, D = 16, K = 256: 77 and 66; N = 4,099, D = 256, K =
// 256: 128 and 64; N = 70,003, D = 35, K = 1,000: 250 and 133 (but N =
// 100,003, D = 35, K = 77: 95 and 106).
static bool km_near(int64_t N, int D, int K) {
    const int64_t least = (int64_t)1 << (D % 4 ? 30 : 28);
    return D >= 16 && D <= 256 && K >= 64 && N * K >= least / D;
}

static KmPlan km_plan(int64_t N, int D, int K) {
    KmPlan p{};
    // fewer centres a slice while the blocks (256 points and a slice each) do
    // not fill the chip.  Objective and gradient, widest slices, these and twice
    // the blocks, us: N = 3,117, D = 64, K = 19 48, 38, 38; N = 5,000, D = 256, K =
    // 20 116, 82, 82; N = 30,000, D = 64, K = 50 60, 53, 53 (four times: 64).
    const int64_t n0 = N > 0 ? N : 1;
    auto width = [](int cps) { return cps <= 4 ? 4 : (cps <= 8 ? 8 : (cps <= 16 ? 16 : 32)); };
    p.cps = km_cps(D, K);
    while (p.cps > 4 && ceil_div(N, kKmPts) * ceil_div(K, p.cps) < kKmFill) p.cps = (p.cps + 1) / 2;
    p.cpsT = width(p.cps);
    p.nslice = (int)ceil_div(K, p.cps);
    // (point, slice) pairs and widened centres of any shorter input, which may
    // have more slices: those of cps centres end where the step before fills the
    // chip
    int64_t pairs = 0, wide = 0;
    for (int cps = km_cps(D, K), up = 0;; up = cps, cps = (cps + 1) / 2) {
        const int64_t most = up ? kKmPts * ((kKmFill - 1) / ceil_div(K, up)) : n0;
        pairs = std::max(pairs, std::min(n0, most) * ceil_div(K, cps));
        wide = std::max(wide, ceil_div(K, cps) * width(cps));
        if (cps <= 4) break;
    }
    {
        const int64_t b = ceil_div(N > 0 ? N : 1, 256);
        p.sum_blocks = (int)(b < kKmSumBlocks ? b : kKmSumBlocks);
    }
    const int64_t n1 = N > 0 ? N : 1;
    p.small = K <= kKmSmallK && D <= 256;
    int64_t want = 1024;  // about so many blocks
    if (p.small) {
        p.cpb = K;
        p.nslices_acc = 1;
        p.chunk = ceil_div(n1, want);
        if (p.chunk < 64) p.chunk = 64;
    } else {
        p.cpb = 1024 / D;
        if (p.cpb > K) p.cpb = K;
        if (p.cpb < 1) p.cpb = 1;
        p.nslices_acc = (int)ceil_div(K, p.cpb);
        want = ceil_div(1024, p.nslices_acc);  // enough blocks to fill the chip
        p.chunk = ceil_div(n1, want);
        if (p.chunk < 64) p.chunk = 64;
        if (p.chunk > kKmChunkMax) p.chunk = kKmChunkMax;
    }
    p.nchunk = ceil_div(n1, p.chunk);
    const int64_t chunks = std::max(std::min(ceil_div(n1, 64), want), p.nchunk);  // of any shorter input
    size_t o = 0;
    auto take = [&](size_t b) {
        const size_t at = o;
        o += align_up(b > 0 ? b : 1, 256);
        return at;
    };
    p.cd = take((size_t)wide * D * 8);
    p.bd = take((size_t)pairs * 8);
    p.bk = take((size_t)pairs * 4);
    p.part = take((size_t)kKmSumBlocks * 8);
    p.spart = take((size_t)chunks * K * D * 8);
    p.npart = take((size_t)chunks * K * 4);
    if (km_near(N, D, K)) {
        p.near_ks = D <= 32 ? 2 : D <= 64 ? 4 : D <= 128 ? 8 : 16;
        p.near_tiles = (int)ceil_div(K, 32);
        // some 512 blocks (two fit a CU; a block splits its points once), in
        // at most kKmNearSlices ranges.  N = 10,000, D = 256, K = 1,024 and
        // N = 20,001, D = 128, K = 1,001, all of a step, with 256, 512, 1,024:
        // 87, 91, 96 us and 90, 88, 94 us.
        int64_t s = ceil_div(512, ceil_div(N, kKmNearPts));
        if (s > kKmNearSlices) s = kKmNearSlices;
        if (s > p.near_tiles) s = p.near_tiles;
        p.near_per = (int)ceil_div(p.near_tiles, s);
        p.near_slices = (int)ceil_div(p.near_tiles, p.near_per);
        p.cf = take((size_t)p.near_tiles * p.near_ks * 2 * 1024);
        p.cst = take((size_t)p.near_tiles * 96 * 4);
        p.bad = take((size_t)p.near_tiles * 4);
        p.open = take((size_t)ceil_div(N, kKmPts) * 4);
        int64_t entries = N;  // of any shorter input: s slices while 512 / s blocks or fewer
        for (int64_t sl = 2; sl <= std::min(kKmNearSlices, p.near_tiles); ++sl)
            entries = std::max(entries, sl * std::min(N, kKmNearPts * (ceil_div(512, sl - 1) - 1)));
        p.near = take((size_t)entries * 2 * sizeof(KmNear));
    }
    p.total = o;
    return p;
}

template <int CPS>
static void launch_dist(const float* X, int64_t N, int D, int K, const KmPlan& p, char* ws, hipStream_t st) {
    const dim3 grid((unsigned)ceil_div(N, kKmPts), (unsigned)p.nslice);
    hipLaunchKernelGGL((km_dist_kernel<CPS>), grid, dim3(kKmPts), 0, st, X, N, D, (const double*)(ws + p.cd), K,
                       p.cps, p.near_ks ? (const int32_t*)(ws + p.bad) : nullptr, p.near_tiles,
                       (const int32_t*)(ws + p.open), (double*)(ws + p.bd), (int32_t*)(ws + p.bk));
}

template <int KS>
static void launch_near(const float* X, int64_t N, int D, const float* C, int K, const KmPlan& p, char* ws,
                        hipStream_t st) {
    const bool vec = D % 4 == 0 && aligned(X, 16) && aligned(C, 16);
    bf16x8* cf = reinterpret_cast<bf16x8*>(ws + p.cf);
    float* cst = reinterpret_cast<float*>(ws + p.cst);
    int32_t* bad = reinterpret_cast<int32_t*>(ws + p.bad);
    int32_t* open = reinterpret_cast<int32_t*>(ws + p.open);
    KmNear* near = reinterpret_cast<KmNear*>(ws + p.near);
    hipLaunchKernelGGL(km_near_prep_kernel<KS>, dim3((unsigned)p.near_tiles), dim3(256), 0, st, C, K, D, vec, cf, cst,
                       bad);
    hipLaunchKernelGGL(km_near_kernel<KS>, dim3((unsigned)ceil_div(N, kKmNearPts), (unsigned)p.near_slices), dim3(256),
                       0, st, X, N, D, C, vec, cf, cst, p.near_tiles, p.near_per, near, open);
    hipLaunchKernelGGL(km_decide_kernel, dim3((unsigned)ceil_div(N, 64)), dim3(256), 0, st, X, N, D, C, K, vec, near,
                       2 * p.near_slices, p.near_per, bad, p.near_tiles, open, (double*)(ws + p.bd), (int32_t*)(ws + p.bk));
}

template <int KM>
static void launch_acc_small(const float* X, int64_t N, int D, int K, const int32_t* assign, const KmPlan& p, char* ws,
                             hipStream_t st) {
    hipLaunchKernelGGL((km_acc_small_kernel<KM>), dim3((unsigned)p.nchunk), dim3(256), 0, st, X, N, D, K, p.chunk,
                       assign, (double*)(ws + p.spart), (int32_t*)(ws + p.npart));
}

static pvjp_status km_check(const char* name, const float* X, int64_t N, int D, const float* C, int K, void* ws,
                            size_t ws_bytes) {
    PVJP_REQUIRE(N >= 0 && N <= INT32_MAX, "%s: N = %lld out of range [0, 2^31)", name, (long long)N);
    PVJP_REQUIRE(D >= 1 && D <= kKmMaxD, "%s: D = %d out of range [1, %d]", name, D, kKmMaxD);
    PVJP_REQUIRE(K >= 1 && K <= (1 << 20), "%s: K = %d out of range [1, 2^20]", name, K);
    PVJP_REQUIRE(C != nullptr && (N == 0 || X != nullptr), "%s: X and C must be non-NULL", name);
    PVJP_REQUIRE(ws != nullptr && aligned(ws, 256), "%s: ws must be non-NULL and 256-byte aligned", name);
    const size_t need = km_plan(N, D, K).total;
    if (ws_bytes < need) {
        set_error("%s: workspace has %zu bytes, needs %zu", name, ws_bytes, need);
        return PVJP_ENOMEM;
    }
    return PVJP_OK;
}

}  // namespace pvjp

using namespace pvjp;

extern "C" size_t pvjp_kmeans_ws_bytes(int64_t N, int D, int K) {
    if (N < 0 || D < 1 || D > kKmMaxD || K < 1) return 0;
    return km_plan(N, D, K).total;
}

extern "C" pvjp_status pvjp_kmeans_objective(const float* X, int64_t N, int D, const float* C, int K, int32_t* assign,
                                             double* f, void* ws, size_t ws_bytes, void* stream) {
    clear_error();
    if (pvjp_status e = km_check("pvjp_kmeans_objective", X, N, D, C, K, ws, ws_bytes)) return e;
    PVJP_REQUIRE(f != nullptr && (N == 0 || assign != nullptr), "pvjp_kmeans_objective: assign and f are required");
    const KmPlan p = km_plan(N, D, K);
    char* w = reinterpret_cast<char*>(ws);
    hipStream_t st = as_stream(stream);
    if (N > 0) {
        const int64_t nw = (int64_t)p.nslice * D * p.cpsT;
        hipLaunchKernelGGL(km_widen_kernel, dim3(flat_grid(nw, 256, 4)), dim3(256), 0, st, C, K, D, p.cps, p.cpsT, nw,
                           (double*)(w + p.cd));
        if (p.near_ks == 2) launch_near<2>(X, N, D, C, K, p, w, st);
        else if (p.near_ks == 4) launch_near<4>(X, N, D, C, K, p, w, st);
        else if (p.near_ks == 8) launch_near<8>(X, N, D, C, K, p, w, st);
        else if (p.near_ks == 16) launch_near<16>(X, N, D, C, K, p, w, st);
        // after a bounded search the FP64 one takes the points left open, or all
        // where a centre's norm is beyond FP32 (or not a number): it asks the flags
        if (p.cpsT == 4) launch_dist<4>(X, N, D, K, p, w, st);
        else if (p.cpsT == 8) launch_dist<8>(X, N, D, K, p, w, st);
        else if (p.cpsT == 16) launch_dist<16>(X, N, D, K, p, w, st);
        else launch_dist<32>(X, N, D, K, p, w, st);
        hipLaunchKernelGGL(km_combine_kernel, dim3((unsigned)p.sum_blocks), dim3(256), 0, st,
                           (const double*)(w + p.bd), (const int32_t*)(w + p.bk), N, p.nslice,
                           p.near_ks ? (const int32_t*)(w + p.bad) : nullptr, p.near_tiles,
                           (const int32_t*)(w + p.open), assign, (double*)(w + p.part));
    }
    hipLaunchKernelGGL(km_sum_kernel, dim3(1), dim3(1024), 0, st, (const double*)(w + p.part),
                       N > 0 ? p.sum_blocks : 0, f);
    PVJP_LAUNCHED("pvjp_kmeans_objective");
    return PVJP_OK;
}

extern "C" pvjp_status pvjp_kmeans_vjp(const float* X, int64_t N, int D, const float* C, int K, const int32_t* assign,
                                       double f_bar, float* C_bar, const float* C_dot, float* hvp, int accumulate,
                                       void* ws, size_t ws_bytes, void* stream) {
    clear_error();
    if (pvjp_status e = km_check("pvjp_kmeans_vjp", X, N, D, C, K, ws, ws_bytes)) return e;
    PVJP_REQUIRE(C_bar != nullptr, "pvjp_kmeans_vjp: C_bar is NULL");
    PVJP_REQUIRE(N == 0 || assign != nullptr, "pvjp_kmeans_vjp: assign (from pvjp_kmeans_objective) is NULL");
    PVJP_REQUIRE((C_dot == nullptr) == (hvp == nullptr), "pvjp_kmeans_vjp: C_dot and hvp go together");
    const KmPlan p = km_plan(N, D, K);
    char* w = reinterpret_cast<char*>(ws);
    hipStream_t st = as_stream(stream);
    if (N > 0) {
        if (p.small) {
            if (K <= 4) launch_acc_small<4>(X, N, D, K, assign, p, w, st);
            else if (K <= 8) launch_acc_small<8>(X, N, D, K, assign, p, w, st);
            else launch_acc_small<16>(X, N, D, K, assign, p, w, st);
        } else {
            const dim3 grid((unsigned)p.nchunk, (unsigned)p.nslices_acc);
            hipLaunchKernelGGL(km_acc_kernel, grid, dim3((unsigned)(p.cpb * D)), 0, st, X, N, D, K, p.cpb, p.chunk,
                               assign, (double*)(w + p.spart), (int32_t*)(w + p.npart));
        }
    }
    const int nchunk = N > 0 ? (int)p.nchunk : 0;
    const int64_t KD = (int64_t)K * D;
    if (nchunk > kWave)
        hipLaunchKernelGGL((km_finish_kernel<true>), dim3((unsigned)ceil_div(KD, 256 / kWave)), dim3(256), 0, st, D, K,
                           nchunk, C, f_bar, (const double*)(w + p.spart), (const int32_t*)(w + p.npart), C_bar, C_dot,
                           hvp, accumulate);
    else
        hipLaunchKernelGGL((km_finish_kernel<false>), dim3((unsigned)ceil_div(KD, 256)), dim3(256), 0, st, D, K,
                           nchunk, C, f_bar, (const double*)(w + p.spart), (const int32_t*)(w + p.npart), C_bar, C_dot,
                           hvp, accumulate);
    PVJP_LAUNCHED("pvjp_kmeans_vjp");
    return PVJP_OK;
}
