// reduce_by_index with a general associative operator (Sec. 5.1.2, with the
// general rule of Sec. 5.1.1 inside every bin) and its VJP.
//
// hs[b] = the fold, in index order, of the elements i with inds[i] = b (the
// neutral element for an empty bin; indices outside [0, m) are skipped).
// The operator need not commute, so each bin's elements must meet in index
// order:
//   1. a stable sort of the in-range elements by bin: passes of up to 8 bits
//      (9 when that saves a pass; the bin's bits split evenly), low digit
//      first, each a per-chunk digit count, a digit-major scan of the counts
//      and a stable scatter staged in LDS (ranks among equal digits from wave
//      ballots, so equal bins keep their order; each digit's records leave as
//      contiguous runs).  The sort moves whole records -- bin and components
//      -- so x is read once, in index order, instead of gathered at random
//      into sorted order.  For the VJP each pass also keeps where every one of
//      its records went;
//   2. over the sorted elements, segmented exclusive scans: forward (the
//      fold of the bin's earlier elements, ls) and, for the VJP, reversed (of
//      its later ones, rs), with the usual lifted operator that restarts at a
//      flagged element (a bin's first element forward, its last one
//      reversed), over fixed tiles: tile folds, the tiles' carries (a wave per
//      64 tiles, one block over the groups, a wave per group again), then per
//      tile the in-tile scans with the tile's carry;
//   3. the primal writes each bin's fold at its last element (over the neutral
//      element, which empty bins keep); the VJP maps f(ls, x, rs, hs_bar[bin])
//      (the reduce rule, y_bar = the bin's hs_bar) over the sorted elements;
//   4. the VJP's adjoints, in sorted order, go back through the passes'
//      positions, last pass first: each step gathers in the order the pass
//      read its records, so it reads the runs that the pass wrote (a block's
//      2,048 records are some 64 bytes each from 256 places) and writes in
//      order.  Storing each adjoint at its element's index from sorted order
//      instead is K scattered words an element (2^24 elements, K = 2: 468 us;
//      the two steps back take 235).
// Folds are formed in FP64 for FP32 and FP64 data alike.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "gops.h"
#include "prims.h"

namespace pvjp {

constexpr int kHgDigits = 512;  // row length of the per-chunk digit counts
constexpr int kHgCountBlock = 256;
constexpr int kHgColChunk = 64;      // sort chunks per column-scan chunk
constexpr int kHgScanThreads = 512;  // at 1,024 the two directions' FP64 states spill
constexpr int kHgBlock = 256;
// Sorted elements per thread of the tile kernels.  Objective and VJP at 2^24
// FP32, m = 2^16 with 2, 4 and 8: linear recurrence 1.28, 1.25, 1.40 ms, 2x2
// product 2.12, 2.06, 2.30 ms; the FP64 2x2 product's 36-byte records are
// faster with 2 (n = 9,000,003, m = 300: 1.11, 1.24, 1.44 ms).
constexpr int hg_ipt(size_t rec_bytes) { return rec_bytes <= 20 ? 4 : 2; }
constexpr size_t kHgSlot = 64;       // bytes per tile for a lifted state
constexpr int64_t kHgMaxBins = (int64_t)1 << 24;  // three sort passes of 8 bits

// A sort record: word 0 the bin, from word 1 the element's K components (T
// each, as words).
template <int W>
struct HgRec {
    uint32_t w[W];
};
template <class T, int K>
constexpr int hg_words() {
    return 1 + K * (int)(sizeof(T) / 4);
}
template <class T, int W>
__device__ __forceinline__ T hg_comp(const HgRec<W>& r, int k) {
    if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, r.w[1 + k]);
    else return __builtin_bit_cast(T, ((uint64_t)r.w[2 + 2 * k] << 32) | r.w[1 + 2 * k]);
}
template <class T, int W>
__device__ __forceinline__ void hg_set_comp(HgRec<W>& r, int k, T v) {
    if constexpr (sizeof(T) == 4) r.w[1 + k] = __builtin_bit_cast(uint32_t, v);
    else {
        const uint64_t b = __builtin_bit_cast(uint64_t, v);
        r.w[1 + 2 * k] = (uint32_t)b;
        r.w[2 + 2 * k] = (uint32_t)(b >> 32);
    }
}

// One element's K adjoints, as they lie in sorted order.
template <class T, int K>
struct alignas(K * sizeof(T) < 16 ? K * sizeof(T) : 16) HgAdj {
    T c[K];
};
// Their type on the way back: the data's, or FP64 where they are added to x_bar,
// so that the sum is rounded once (8 10^6 linear-recurrence elements in FP32, m
// = 2^16: 366 us with FP32 adjoints, 443 with these).  The 2x2 product's four
// keep the data's type: in FP64 they would not fit a record's buffer.
template <class T, int K, bool ACC>
using HgBack = typename std::conditional<ACC && K <= 2, double, T>::type;

// Up to four component arrays of one dtype.
template <class T>
struct HgIn {
    const T* p[4];
};
template <class T>
struct HgOut {
    T* p[4];
};

// ------------------------------------------------------------------ sort
// Digit counts of one chunk (any order: counting needs no stability).  The
// first pass reads the indices (out-of-range ones skipped), the later ones the
// pass before's output, whose length is on the device.
template <int W>
__global__ __launch_bounds__(kHgCountBlock) void hg_count_kernel(const int32_t* __restrict__ keys,
                                                                 const HgRec<W>* __restrict__ recs, int64_t n,
                                                                 const int32_t* __restrict__ nvalid, int chunk,
                                                                 int32_t m, int shift, int dmask, int ndig,
                                                                 int32_t* __restrict__ cntb) {
    constexpr int U = 8;  // loads in flight per thread
    __shared__ int32_t cnt[kHgDigits];
    for (int d = threadIdx.x; d < ndig; d += kHgCountBlock) cnt[d] = 0;
    __syncthreads();
    const int64_t ne = nvalid ? (int64_t)*nvalid : n;
    const int64_t lo = (int64_t)blockIdx.x * chunk;
    const int64_t hi = (lo + chunk < ne) ? lo + chunk : ne;
    for (int64_t i0 = lo + threadIdx.x; i0 < hi; i0 += U * kHgCountBlock) {
        int32_t k[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = i0 + u * kHgCountBlock < hi ? i0 + u * kHgCountBlock : hi - 1;
            k[u] = keys ? keys[i] : (int32_t)recs[i].w[0];
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i0 + u * kHgCountBlock < hi && (uint32_t)k[u] < (uint32_t)m)
                atomicAdd(&cnt[(k[u] >> shift) & dmask], 1);
    }
    __syncthreads();
    for (int d = threadIdx.x; d < ndig; d += kHgCountBlock) cntb[(int64_t)blockIdx.x * kHgDigits + d] = cnt[d];
}

// Per digit (a thread) and column chunk of kHgColChunk sort chunks (grid y):
// the count of each chunk is replaced by the sum of the earlier chunks'
// counts in the column chunk, whose total goes to ctot[c][d].
__global__ __launch_bounds__(kHgCountBlock) void hg_colscan_kernel(int32_t* __restrict__ cntb, int nblk, int ndig,
                                                                   int32_t* __restrict__ ctot) {
    const int d = blockIdx.x * kHgCountBlock + (int)threadIdx.x;
    const int c = blockIdx.y;
    if (d >= ndig) return;
    int v[kHgColChunk];
#pragma unroll
    for (int j = 0; j < kHgColChunk; ++j) {
        const int b = c * kHgColChunk + j;
        v[j] = b < nblk ? cntb[(int64_t)b * kHgDigits + d] : 0;
    }
    int run = 0;
#pragma unroll
    for (int j = 0; j < kHgColChunk; ++j) {
        const int b = c * kHgColChunk + j;
        if (b < nblk) cntb[(int64_t)b * kHgDigits + d] = run;
        run += v[j];
    }
    ctot[(int64_t)c * kHgDigits + d] = run;
}

// One block, a thread per digit: ctot[c][d] becomes the start of (column chunk
// c, digit d) in the sorted output (the digit's start plus its earlier column
// chunks), and the number of sorted elements is written once.
__global__ __launch_bounds__(kHgDigits) void hg_digitscan_kernel(int32_t* __restrict__ ctot, int nchunks, int ndig,
                                                                 int32_t* __restrict__ nvalid) {
    __shared__ IntSum::S wtot[kHgDigits / kWave];
    constexpr int U = 16;  // loads in flight
    const int d = threadIdx.x;
    int sum = 0;
    if (d < ndig)
        for (int c0 = 0; c0 < nchunks; c0 += U) {
            int v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = c0 + u < nchunks ? ctot[(int64_t)(c0 + u) * kHgDigits + d] : 0;
#pragma unroll
            for (int u = 0; u < U; ++u) sum += v[u];
        }
    IntSum::S all;
    int run = block_exclusive_scan<IntSum, kHgDigits, false>(IntSum::S{sum}, all, wtot).v;
    if (d < ndig)
        for (int c0 = 0; c0 < nchunks; c0 += U) {
            int v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = c0 + u < nchunks ? ctot[(int64_t)(c0 + u) * kHgDigits + d] : 0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (c0 + u < nchunks) ctot[(int64_t)(c0 + u) * kHgDigits + d] = run;
                run += v[u];
            }
        }
    if (threadIdx.x == 0 && nvalid) *nvalid = all.v;
}

// Stable scatter of one chunk, staged in LDS so that each digit's records
// leave as contiguous runs instead of one scattered store per record.  The
// chunk is taken in sub-chunks of kHgSub records in index order (long
// enough that a digit's run in it averages a whole line); wave w of the
// block owns records [w * 64 G, (w + 1) * 64 G) of a sub-chunk, as G =
// kHgSortGroups groups of 64 taken in order.  Ranks: within a group, the lanes of equal
// digit find each other with one ballot per digit bit (rank = earlier such
// lanes); a wave's running count per digit orders its groups; the counts
// of earlier waves order the waves; earlier sub-chunks and chunks come
// before through the digit's running position.  So equal digits keep their
// index order.  Records are placed in LDS at (the digit's start in the
// sub-chunk + rank), then thread t writes slots t, t + 256, ... to the
// digit's running position in the output.  The first pass builds each
// record from the indices and x (read in order), later passes move records.
// A sub-chunk's loads are issued before the stores of the one before, and the
// stores are not under branches (a slot beyond the last repeats it): a wave's
// memory operations return in order, so loads issued after the stores waited
// for those as well.  Per pass over 2^24 linear-recurrence elements, m = 2^16:
// 225 us with neither, 16-byte records (the index with them) and 512 blocks;
// now 137 us, 3.4 TB/s.
constexpr int kHgSortThreads = 256;
constexpr int kHgSortWaves = kHgSortThreads / kWave;
constexpr int kHgSortGroups = 8;                               // groups of 64 per wave and sub-chunk
constexpr int kHgSub = kHgSortThreads * kHgSortGroups;         // 2048 records
constexpr int kHgPassBits = 8;                                 // bits per pass, one digit per thread
constexpr int kHgPassDigits = 1 << kHgPassBits;
static_assert(kHgPassDigits == kHgSortThreads, "a thread per digit in the sub-chunk scans");

// DPT: digits per thread in the per-digit steps (1: up to 256 digits, 2: up
// to 512); thread t owns digits [DPT t, DPT t + DPT).
template <class T, int K, int W, int DPT>
__global__ __launch_bounds__(kHgSortThreads) void hg_scatter_kernel(const int32_t* __restrict__ keys_in, HgIn<T> x,
                                                                    const HgRec<W>* __restrict__ recs_in, int64_t n,
                                                                    const int32_t* __restrict__ nvalid, int chunk,
                                                                    int32_t m, int shift, int dmask, int ndig,
                                                                    int nbits, const int32_t* __restrict__ cntb,
                                                                    const int32_t* __restrict__ ctot,
                                                                    HgRec<W>* __restrict__ recs_out,
                                                                    int32_t* __restrict__ keys_out,
                                                                    int32_t* __restrict__ pos) {
    constexpr int ND = kHgPassDigits * DPT;
    __shared__ HgRec<W> stage[kHgSub];
    __shared__ int32_t wcnt[kHgSortWaves][ND];  // per wave: running count, then its offset
    __shared__ int32_t lstart[ND];              // the digit's first slot in the sub-chunk
    __shared__ int32_t gpos[ND];                // the digit's running output position
    __shared__ IntSum::S wtot[kHgSortWaves];
    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = tid / kWave;
    const int blk = blockIdx.x;
    const int c = blk / kHgColChunk;
    const int64_t ne = nvalid ? (int64_t)*nvalid : n;
    const int64_t lo = (int64_t)blk * chunk;
    const int64_t hi = (lo + chunk < ne) ? lo + chunk : ne;
    if (lo >= hi) return;
#pragma unroll
    for (int u = 0; u < DPT; ++u) {
        const int d = DPT * tid + u;
        if (d < ndig) gpos[d] = ctot[(int64_t)c * kHgDigits + d] + cntb[(int64_t)blk * kHgDigits + d];
    }
    const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (kWave - lane));
    const int64_t own = wave * (kHgSortGroups * kWave) + lane;  // the thread's first element in a sub-chunk
    HgRec<W> r[kHgSortGroups];
    auto load = [&](int64_t s0) {
        if (keys_in) {
#pragma unroll
            for (int g = 0; g < kHgSortGroups; ++g) {
                const int64_t i = min(s0 + own + g * kWave, hi - 1);
                r[g].w[0] = (uint32_t)keys_in[i];
#pragma unroll
                for (int k = 0; k < K; ++k) hg_set_comp<T, W>(r[g], k, x.p[k][i]);
            }
        } else {
#pragma unroll
            for (int g = 0; g < kHgSortGroups; ++g) r[g] = recs_in[min(s0 + own + g * kWave, hi - 1)];
        }
    };
    load(lo);
    for (int64_t s0 = lo; s0 < hi; s0 += kHgSub) {
        for (int w = 0; w < kHgSortWaves; ++w)
#pragma unroll
            for (int u = 0; u < DPT; ++u) wcnt[w][DPT * tid + u] = 0;
        bool valid[kHgSortGroups];
        int dg[kHgSortGroups];
        __syncthreads();  // counters cleared; the previous sub-chunk's slots read out
        // ranks within the wave, groups in order
        int rank[kHgSortGroups];
#pragma unroll
        for (int g = 0; g < kHgSortGroups; ++g) {
            valid[g] = s0 + own + g * kWave < hi && r[g].w[0] < (uint32_t)m;
            const int d = valid[g] ? ((int32_t)r[g].w[0] >> shift) & dmask : 0;
            dg[g] = d;
            uint64_t peers = __ballot(valid[g]);
            for (int bit = 0; bit < nbits; ++bit) {
                const bool one = (d >> bit) & 1;
                const uint64_t b = __ballot(valid[g] && one);
                peers &= one ? b : ~b;
            }
            const int before = valid[g] ? wcnt[wave][d] : 0;
            rank[g] = before + __popcll(peers & below);
            // the highest lane of the group moves the wave's count on (lanes
            // of a wave run together: every lane has read it first)
            if (valid[g] && (peers >> lane) == 1ull) wcnt[wave][d] = before + __popcll(peers);
        }
        __syncthreads();
        // per digit (DPT a thread): the waves' offsets and the digit's total,
        // then the digits' starts in the sub-chunk
        int tot[DPT], sum = 0;
#pragma unroll
        for (int u = 0; u < DPT; ++u) {
            const int d = DPT * tid + u;
            tot[u] = 0;
            for (int w = 0; w < kHgSortWaves; ++w) {
                const int cw = wcnt[w][d];
                wcnt[w][d] = tot[u];
                tot[u] += cw;
            }
            sum += tot[u];
        }
        IntSum::S all;
        int st = block_exclusive_scan<IntSum, kHgSortThreads, false>(IntSum::S{sum}, all, wtot).v;
#pragma unroll
        for (int u = 0; u < DPT; ++u) {
            lstart[DPT * tid + u] = st;
            st += tot[u];
        }
        __syncthreads();
        int to[kHgSortGroups];  // where the thread's records go, or -1
#pragma unroll
        for (int g = 0; g < kHgSortGroups; ++g) {
            const int at = wcnt[wave][dg[g]] + rank[g];
            if (valid[g]) stage[lstart[dg[g]] + at] = r[g];
            to[g] = valid[g] ? gpos[dg[g]] + at : -1;
        }
        if (s0 + kHgSub < hi) load(s0 + kHgSub);
        __syncthreads();
        if (pos) {
#pragma unroll
            for (int g = 0; g < kHgSortGroups; ++g) pos[s0 + own + g * kWave] = to[g];  // padded to whole sub-chunks
        }
        if (all.v > 0) {
#pragma unroll
            for (int u = 0; u < kHgSortGroups; ++u) {
                const int sl = min(u * kHgSortThreads + tid, all.v - 1);
                const HgRec<W> q = stage[sl];
                const int d = ((int32_t)q.w[0] >> shift) & dmask;
                const int64_t o = gpos[d] + (sl - lstart[d]);
                recs_out[o] = q;
                if (keys_out) keys_out[o] = (int32_t)q.w[0];  // what the next pass counts
            }
        }
        __syncthreads();  // every slot placed before the positions move on
#pragma unroll
        for (int u = 0; u < DPT; ++u) gpos[DPT * tid + u] += tot[u];
    }
}

// --------------------------------------------------- segmented fold scans
// The lifted operator: a state remembers whether it holds a flagged element,
// and a later flagged state discards everything before it.
template <class Q>
struct SegOf {
    using QS = typename Q::S;
    struct S {
        QS v;
        uint32_t f, pad;
    };
    __device__ static __forceinline__ S id() { return S{Q::id(), 0u, 0u}; }
    __device__ static __forceinline__ S comb(S x, S y) { return y.f ? y : S{Q::comb(x.v, y.v), x.f, 0u}; }
};


// Sorted element p: its bin and its components (as FP64, from its record),
// plus whether it opens (first) and closes (last) its bin.
template <class Op, class T>
struct HgElem {
    int32_t key;
    bool first, last;
    typename Op::S a;
};

template <class Op, class T, int W>
__device__ __forceinline__ HgElem<Op, T> hg_elem(const HgRec<W>* __restrict__ recs, int64_t nv, int64_t p) {
    HgElem<Op, T> e;
    const HgRec<W> r = recs[p];
    e.key = (int32_t)r.w[0];
    e.first = p == 0 || (int32_t)recs[p - 1].w[0] != e.key;
    e.last = p + 1 == nv || (int32_t)recs[p + 1].w[0] != e.key;
    double c[Op::K];
#pragma unroll
    for (int k = 0; k < Op::K; ++k) c[k] = (double)hg_comp<T, W>(r, k);
    e.a = Op::elem(c);
    return e;
}

// Tile folds, forward (flag: the bin's first element) and, with REV, reversed
// (flag: its last element, scanned with the operands exchanged).
template <class Op, class T, int W, bool REV>
__global__ __launch_bounds__(kHgBlock) void hg_tile_fold_kernel(const HgRec<W>* __restrict__ recs,
                                                                const int32_t* __restrict__ nvalid, char* __restrict__ aggF,
                                                                char* __restrict__ aggR) {
    constexpr int kIpt = hg_ipt(sizeof(HgRec<W>));
    using F = SegOf<Op>;
    using R = SegOf<Flip<Op>>;
    __shared__ typename F::S wf[kHgBlock / kWave];
    __shared__ typename R::S wr[kHgBlock / kWave];
    const int64_t nv = *nvalid;
    const int64_t p0 = ((int64_t)blockIdx.x * kHgBlock + threadIdx.x) * kIpt;
    typename F::S sf = F::id();
    typename R::S sr = R::id();
    typename R::S re[kIpt];
#pragma unroll
    for (int j = 0; j < kIpt; ++j) {
        re[j] = R::id();
        if (p0 + j < nv) {
            const HgElem<Op, T> e = hg_elem<Op, T, W>(recs, nv, p0 + j);
            sf = F::comb(sf, typename F::S{e.a, e.first ? 1u : 0u, 0u});
            re[j] = typename R::S{e.a, e.last ? 1u : 0u, 0u};
        }
    }
    typename F::S tf;
    block_exclusive_scan<F, kHgBlock, false>(sf, tf, wf);
    if (threadIdx.x == 0) *reinterpret_cast<typename F::S*>(aggF + (size_t)blockIdx.x * kHgSlot) = tf;
    if (REV) {
#pragma unroll
        for (int j = kIpt - 1; j >= 0; --j) sr = R::comb(sr, re[j]);
        typename R::S tr;
        block_exclusive_scan<R, kHgBlock, true>(sr, tr, wr);
        if (threadIdx.x == 0) *reinterpret_cast<typename R::S*>(aggR + (size_t)blockIdx.x * kHgSlot) = tr;
    }
}

// One block: each item's carry, the lifted fold of all items before it
// (forward) and after it (reversed), for an array of tile or group folds.
// Thread t owns a contiguous run of items.
template <class Op, bool REV>
__global__ __launch_bounds__(kHgScanThreads) void hg_tile_scan_kernel(const char* __restrict__ aggF,
                                                                      const char* __restrict__ aggR, int64_t ntiles,
                                                                      char* __restrict__ carF, char* __restrict__ carR) {
    using F = SegOf<Op>;
    using R = SegOf<Flip<Op>>;
    __shared__ typename F::S wf[kHgScanThreads / kWave];
    __shared__ typename R::S wr[kHgScanThreads / kWave];
    const int64_t per = (ntiles + kHgScanThreads - 1) / kHgScanThreads;
    const int64_t t0 = (int64_t)threadIdx.x * per;
    const int64_t t1 = (t0 + per < ntiles) ? t0 + per : ntiles;
    auto getF = [&](int64_t t) { return *reinterpret_cast<const typename F::S*>(aggF + (size_t)t * kHgSlot); };
    auto getR = [&](int64_t t) { return *reinterpret_cast<const typename R::S*>(aggR + (size_t)t * kHgSlot); };
    typename F::S sf = F::id();
    typename R::S sr = R::id();
    for (int64_t t = t0; t < t1; ++t) sf = F::comb(sf, getF(t));
    if (REV)
        for (int64_t t = t1 - 1; t >= t0; --t) sr = R::comb(sr, getR(t));
    typename F::S tf;
    typename R::S tr;
    sf = block_exclusive_scan<F, kHgScanThreads, false>(sf, tf, wf);
    if (REV) sr = block_exclusive_scan<R, kHgScanThreads, true>(sr, tr, wr);
    for (int64_t t = t0; t < t1; ++t) {
        *reinterpret_cast<typename F::S*>(carF + (size_t)t * kHgSlot) = sf;
        sf = F::comb(sf, getF(t));
    }
    if (!REV) return;
    for (int64_t t = t1 - 1; t >= t0; --t) {
        *reinterpret_cast<typename R::S*>(carR + (size_t)t * kHgSlot) = sr;
        sr = R::comb(sr, getR(t));
    }
}

// Tile carries in three steps: a wave folds each group of 64 tiles, one
// block scans the group folds (hg_tile_scan_kernel over the groups), and a
// wave per group turns the group's carry into its tiles' carries.
constexpr int kHgGroup = kWave;

template <class Op, bool REV>
__global__ __launch_bounds__(kHgGroup) void hg_group_fold_kernel(const char* __restrict__ aggF,
                                                                 const char* __restrict__ aggR, int64_t ntiles,
                                                                 char* __restrict__ gF, char* __restrict__ gR) {
    using F = SegOf<Op>;
    using R = SegOf<Flip<Op>>;
    __shared__ typename F::S wf[1];
    __shared__ typename R::S wr[1];
    const int64_t t = (int64_t)blockIdx.x * kHgGroup + threadIdx.x;
    const typename F::S af = t < ntiles ? *reinterpret_cast<const typename F::S*>(aggF + (size_t)t * kHgSlot) : F::id();
    const typename R::S ar = REV && t < ntiles ? *reinterpret_cast<const typename R::S*>(aggR + (size_t)t * kHgSlot) : R::id();
    typename F::S tf;
    typename R::S tr;
    block_exclusive_scan<F, kHgGroup, false>(af, tf, wf);
    if (REV) block_exclusive_scan<R, kHgGroup, true>(ar, tr, wr);
    if (threadIdx.x == 0) {
        *reinterpret_cast<typename F::S*>(gF + (size_t)blockIdx.x * kHgSlot) = tf;
        if (REV) *reinterpret_cast<typename R::S*>(gR + (size_t)blockIdx.x * kHgSlot) = tr;
    }
}

template <class Op, bool REV>
__global__ __launch_bounds__(kHgGroup) void hg_group_carry_kernel(const char* __restrict__ aggF,
                                                                  const char* __restrict__ aggR, int64_t ntiles,
                                                                  const char* __restrict__ gcF,
                                                                  const char* __restrict__ gcR,
                                                                  char* __restrict__ carF, char* __restrict__ carR) {
    using F = SegOf<Op>;
    using R = SegOf<Flip<Op>>;
    __shared__ typename F::S wf[1];
    __shared__ typename R::S wr[1];
    const int64_t t = (int64_t)blockIdx.x * kHgGroup + threadIdx.x;
    const typename F::S af = t < ntiles ? *reinterpret_cast<const typename F::S*>(aggF + (size_t)t * kHgSlot) : F::id();
    const typename R::S ar = REV && t < ntiles ? *reinterpret_cast<const typename R::S*>(aggR + (size_t)t * kHgSlot) : R::id();
    typename F::S tf;
    typename R::S tr;
    const typename F::S xf = block_exclusive_scan<F, kHgGroup, false>(af, tf, wf);
    const typename R::S xr = REV ? block_exclusive_scan<R, kHgGroup, true>(ar, tr, wr) : ar;
    if (t < ntiles) {
        *reinterpret_cast<typename F::S*>(carF + (size_t)t * kHgSlot) =
            F::comb(*reinterpret_cast<const typename F::S*>(gcF + (size_t)blockIdx.x * kHgSlot), xf);
        if (REV) *reinterpret_cast<typename R::S*>(carR + (size_t)t * kHgSlot) =
            R::comb(*reinterpret_cast<const typename R::S*>(gcR + (size_t)blockIdx.x * kHgSlot), xr);
    }
}

// Per tile: the forward scan with the tile's carry; the primal writes each
// bin's fold at its last element.  The VJP also runs the reversed scan and
// maps f over (ls, x, rs) with y_bar = hs_bar of the element's bin.
template <class Op, class T, int W, bool VJP, class A>
__global__ __launch_bounds__(kHgBlock) void hg_apply_kernel(const HgRec<W>* __restrict__ recs,
                                                            const int32_t* __restrict__ nvalid,
                                                            const char* __restrict__ carF,
                                                            const char* __restrict__ carR, HgOut<T> hs,
                                                            HgIn<T> hs_bar, HgAdj<A, Op::K>* __restrict__ adj) {
    constexpr int kIpt = hg_ipt(sizeof(HgRec<W>));
    using F = SegOf<Op>;
    using R = SegOf<Flip<Op>>;
    using QS = typename Op::S;
    __shared__ typename F::S wf[kHgBlock / kWave];
    __shared__ typename R::S wr[kHgBlock / kWave];
    const int64_t nv = *nvalid;
    const int64_t p0 = ((int64_t)blockIdx.x * kHgBlock + threadIdx.x) * kIpt;
    HgElem<Op, T> e[kIpt];
    bool in[kIpt];
    typename F::S sf = F::id();
#pragma unroll
    for (int j = 0; j < kIpt; ++j) {
        in[j] = p0 + j < nv;
        if (in[j]) {
            e[j] = hg_elem<Op, T, W>(recs, nv, p0 + j);
            sf = F::comb(sf, typename F::S{e[j].a, e[j].first ? 1u : 0u, 0u});
        }
    }
    typename F::S tf;
    typename F::S xf = block_exclusive_scan<F, kHgBlock, false>(sf, tf, wf);
    xf = F::comb(*reinterpret_cast<const typename F::S*>(carF + (size_t)blockIdx.x * kHgSlot), xf);
    if (!VJP) {
#pragma unroll
        for (int j = 0; j < kIpt; ++j) {
            if (!in[j]) continue;
            xf = F::comb(xf, typename F::S{e[j].a, e[j].first ? 1u : 0u, 0u});
            if (e[j].last) {
                double out[Op::K];
                Op::value(xf.v, out);
#pragma unroll
                for (int k = 0; k < Op::K; ++k) hs.p[k][e[j].key] = (T)out[k];
            }
        }
        return;
    }
    QS ls[kIpt], la[kIpt];
#pragma unroll
    for (int j = 0; j < kIpt; ++j) {
        if (!in[j]) continue;
        ls[j] = e[j].first ? Op::id() : xf.v;
        la[j] = Op::comb(ls[j], e[j].a);
        xf = F::comb(xf, typename F::S{e[j].a, e[j].first ? 1u : 0u, 0u});
    }
    typename R::S sr = R::id();
#pragma unroll
    for (int j = kIpt - 1; j >= 0; --j)
        if (in[j]) sr = R::comb(sr, typename R::S{e[j].a, e[j].last ? 1u : 0u, 0u});
    typename R::S tr;
    typename R::S xr = block_exclusive_scan<R, kHgBlock, true>(sr, tr, wr);
    xr = R::comb(*reinterpret_cast<const typename R::S*>(carR + (size_t)blockIdx.x * kHgSlot), xr);
#pragma unroll
    for (int j = kIpt - 1; j >= 0; --j) {
        if (!in[j]) continue;
        const QS rs = e[j].last ? Op::id() : xr.v;
        double yb[Op::K], out[Op::K];
#pragma unroll
        for (int k = 0; k < Op::K; ++k) yb[k] = (double)hs_bar.p[k][e[j].key];
        Op::vjp(ls[j], e[j].a, rs, la[j], yb, out);
        HgAdj<A, Op::K> q;
#pragma unroll
        for (int k = 0; k < Op::K; ++k) q.c[k] = (A)out[k];
        adj[p0 + j] = q;
        xr = R::comb(xr, typename R::S{e[j].a, e[j].last ? 1u : 0u, 0u});
    }
}

// Every bin the neutral element, before the folds are written.
template <class Op, class T>
__global__ __launch_bounds__(256) void hg_empty_kernel(int32_t m, HgOut<T> hs) {
    const int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (b >= m) return;
    double out[Op::K];
    Op::value(Op::id(), out);
#pragma unroll
    for (int k = 0; k < Op::K; ++k) hs.p[k][b] = (T)out[k];
}

// One step back through a sort pass: dst[j] = src[pos[j]], j in the order the
// pass read its records; a thread takes eight, the block a sub-chunk.
constexpr int kHgBackU = kHgSub / 256;
template <class A, int K>
__global__ __launch_bounds__(256) void hg_back_kernel(const int32_t* __restrict__ pos,
                                                      const int32_t* __restrict__ nvalid,
                                                      const HgAdj<A, K>* __restrict__ src,
                                                      HgAdj<A, K>* __restrict__ dst) {
    const int64_t nv = *nvalid;
    const int64_t at = (int64_t)blockIdx.x * kHgSub;
    if (at >= nv) return;
    const int64_t j0 = at + threadIdx.x;
    int p[kHgBackU];
    HgAdj<A, K> v[kHgBackU];
#pragma unroll
    for (int u = 0; u < kHgBackU; ++u) p[u] = pos[min(j0 + u * 256, nv - 1)];
#pragma unroll
    for (int u = 0; u < kHgBackU; ++u) v[u] = src[p[u]];
#pragma unroll
    for (int u = 0; u < kHgBackU; ++u)
        if (j0 + u * 256 < nv) dst[j0 + u * 256] = v[u];
}

// The last step, through the first pass: x_bar in index order (0, or what was
// there, where the index is out of range).
template <class T, int K, bool ACC, class A>
__global__ __launch_bounds__(256) void hg_back_write_kernel(const int32_t* __restrict__ pos, int64_t n,
                                                            const int32_t* __restrict__ nvalid,
                                                            const HgAdj<A, K>* __restrict__ src, HgOut<T> x_bar) {
    const int64_t j0 = (int64_t)blockIdx.x * kHgSub + threadIdx.x;
    const bool any = *nvalid > 0;
    int p[kHgBackU];
    HgAdj<A, K> v[kHgBackU];
#pragma unroll
    for (int u = 0; u < kHgBackU; ++u) p[u] = pos[min(j0 + u * 256, n - 1)];
#pragma unroll
    for (int u = 0; u < kHgBackU; ++u)
        if (any) v[u] = src[max(p[u], 0)];
#pragma unroll
    for (int u = 0; u < kHgBackU; ++u) {
        const int64_t j = j0 + u * 256;
        if (j >= n || (ACC && p[u] < 0)) continue;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            T* d = x_bar.p[k] + j;
            const A a = p[u] < 0 ? A(0) : v[u].c[k];
            *d = ACC ? (T)((double)*d + (double)a) : (T)a;
        }
    }
}

// ------------------------------------------------------------------ host
static int hg_components(pvjp_gop op) {
    return op == PVJP_GOP_LOGADDEXP ? 1 : op == PVJP_GOP_LINREC ? 2 : op == PVJP_GOP_MAT2 ? 4 : 0;
}

struct HgLayout {
    int64_t chunk, nblk, nchunks, ntiles, npad;
    int64_t ngroups;
    int passes, bits;  // sort passes, bits per pass
    size_t cntb, ctot, nvalid, recA, recB, keyA, keyB, pos, aggF, aggR, carF, carR, gF, gR, gcF, gcR, total;
};

// Records of 32 bytes or more: each pass but the last also writes its output's
// keys compactly, which the next pass counts instead of reading whole records
// (a shorter one costs the count about as much to read).
static bool hg_compact_keys(size_t rec_bytes) { return rec_bytes >= 32; }

// K components of es bytes each.  A record is 4 + K es bytes; its buffers also
// take the adjoints (HgBack).
static HgLayout hg_layout(int64_t n, int64_t m, int K, size_t es) {
    HgLayout L{};
    const size_t rec_bytes = 4 + K * es;
    const size_t buf_bytes = std::max(rec_bytes, K <= 2 ? K * sizeof(double) : 0);
    const int64_t nn = n > 0 ? n : 1;
    // A block's chunk: whole sub-chunks, 32,768 elements or, so that short
    // inputs fill the chip, as many as leave some 2,048 blocks (eight a CU;
    // 2^24 16-byte records in 512 blocks of 32,768: 225 us a pass, at 2^26,
    // with 2,048 blocks, 178 us per 2^24).
    L.chunk = kHgSub;
    while (L.chunk < 32768 && L.chunk * 2048 < nn) L.chunk *= 2;
    L.nblk = ceil_div(nn, L.chunk);
    L.nchunks = ceil_div(L.nblk, kHgColChunk);
    L.ntiles = ceil_div(nn, (int64_t)kHgBlock * hg_ipt(rec_bytes));
    L.npad = ceil_div(nn, kHgSub) * kHgSub;
    int b = 0;
    while (((int64_t)1 << b) < m) ++b;
    // As few passes as 9 bits each allow, the bits split evenly.
    L.passes = std::max(1, (b + kHgPassBits) / (kHgPassBits + 1));
    L.bits = std::max(1, (b + L.passes - 1) / L.passes);
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o += align_up(bytes, 256);
        return at;
    };
    // chunks grow with the length: a shorter input may have more blocks, up to 2,048
    const int64_t most = std::max(std::min<int64_t>(ceil_div(nn, kHgSub), 2048), L.nblk);
    L.cntb = take((size_t)most * kHgDigits * 4);
    L.ctot = take((size_t)ceil_div(most, kHgColChunk) * kHgDigits * 4);
    L.nvalid = take(4);
    L.recA = take((size_t)nn * buf_bytes);
    L.recB = take((size_t)nn * buf_bytes);
    const bool ck = hg_compact_keys(rec_bytes);
    L.keyA = take(ck ? (size_t)nn * 4 : 0);
    L.keyB = take(ck ? (size_t)nn * 4 : 0);
    L.pos = take((size_t)L.passes * L.npad * 4);
    L.aggF = take((size_t)L.ntiles * kHgSlot);
    L.aggR = take((size_t)L.ntiles * kHgSlot);
    L.carF = take((size_t)L.ntiles * kHgSlot);
    L.carR = take((size_t)L.ntiles * kHgSlot);
    L.ngroups = ceil_div(L.ntiles, kHgGroup);
    L.gF = take((size_t)L.ngroups * kHgSlot);
    L.gR = take((size_t)L.ngroups * kHgSlot);
    L.gcF = take((size_t)L.ngroups * kHgSlot);
    L.gcR = take((size_t)L.ngroups * kHgSlot);
    L.total = o;
    return L;
}

// The stable sort by bin; records ping-pong between the two buffers.  Returns
// the sorted ones.  keep: the passes' positions go to the workspace.
template <class T, int K, int W>
static HgRec<W>* hg_sort(const int32_t* keys, const HgIn<T>& x, int64_t n, int64_t m, bool keep, char* w,
                         const HgLayout& L, hipStream_t st) {
    int32_t* cntb = reinterpret_cast<int32_t*>(w + L.cntb);
    int32_t* ctot = reinterpret_cast<int32_t*>(w + L.ctot);
    int32_t* nvalid = reinterpret_cast<int32_t*>(w + L.nvalid);
    HgRec<W>* rin = nullptr;
    const int32_t* kcount = keys;
    for (int pass = 0; pass < L.passes; ++pass) {
        const int shift = pass * L.bits;
        const int dmask = (1 << L.bits) - 1;
        const int ndig = (int)std::min<int64_t>((int64_t)1 << L.bits, ceil_div(m, (int64_t)1 << shift));
        int nbits = 0;
        while ((1 << nbits) < ndig) ++nbits;
        HgRec<W>* rout = reinterpret_cast<HgRec<W>*>(w + ((pass & 1) ? L.recB : L.recA));
        int32_t* kout = nullptr;
        if (hg_compact_keys(sizeof(HgRec<W>)) && pass + 1 < L.passes)
            kout = reinterpret_cast<int32_t*>(w + ((pass & 1) ? L.keyB : L.keyA));
        int32_t* pos = keep ? reinterpret_cast<int32_t*>(w + L.pos) + (int64_t)pass * L.npad : nullptr;
        const int32_t* kin = pass == 0 ? keys : nullptr;
        const int32_t* nv = pass == 0 ? nullptr : nvalid;
        hipLaunchKernelGGL(hg_count_kernel<W>, dim3((unsigned)L.nblk), dim3(kHgCountBlock), 0, st, kcount, rin, n,
                           nv, (int)L.chunk, (int32_t)m, shift, dmask, ndig, cntb);
        hipLaunchKernelGGL(hg_colscan_kernel, dim3((unsigned)ceil_div(ndig, kHgCountBlock), (unsigned)L.nchunks),
                           dim3(kHgCountBlock), 0, st, cntb, (int)L.nblk, ndig, ctot);
        hipLaunchKernelGGL(hg_digitscan_kernel, dim3(1), dim3(kHgDigits), 0, st, ctot, (int)L.nchunks, ndig,
                           pass == 0 ? nvalid : nullptr);
        if (ndig > kHgPassDigits)
            hipLaunchKernelGGL((hg_scatter_kernel<T, K, W, 2>), dim3((unsigned)L.nblk), dim3(kHgSortThreads), 0, st,
                               kin, x, rin, n, nv, (int)L.chunk, (int32_t)m, shift, dmask, ndig, nbits, cntb, ctot,
                               rout, kout, pos);
        else
            hipLaunchKernelGGL((hg_scatter_kernel<T, K, W, 1>), dim3((unsigned)L.nblk), dim3(kHgSortThreads), 0, st,
                               kin, x, rin, n, nv, (int)L.chunk, (int32_t)m, shift, dmask, ndig, nbits, cntb, ctot,
                               rout, kout, pos);
        rin = rout;
        kcount = kout;
    }
    return rin;
}

// The sort and the tile carries, shared by both entry points (REV: the
// reversed carries too, and the passes' positions kept).
template <class Op, class T, bool REV>
static HgRec<hg_words<T, Op::K>()>* hg_prepare(const int32_t* inds, int64_t n, int32_t m, const HgIn<T>& x, char* w,
                                               const HgLayout& L, hipStream_t st) {
    constexpr int W = hg_words<T, Op::K>();
    int32_t* nvalid = reinterpret_cast<int32_t*>(w + L.nvalid);
    HgRec<W>* rin = hg_sort<T, Op::K, W>(inds, x, n, m, REV, w, L, st);
    hipLaunchKernelGGL((hg_tile_fold_kernel<Op, T, W, REV>), dim3((unsigned)L.ntiles), dim3(kHgBlock), 0, st, rin,
                       nvalid, w + L.aggF, w + L.aggR);
    hipLaunchKernelGGL((hg_group_fold_kernel<Op, REV>), dim3((unsigned)L.ngroups), dim3(kHgGroup), 0, st, w + L.aggF,
                       w + L.aggR, L.ntiles, w + L.gF, w + L.gR);
    hipLaunchKernelGGL((hg_tile_scan_kernel<Op, REV>), dim3(1), dim3(kHgScanThreads), 0, st, w + L.gF, w + L.gR,
                       L.ngroups, w + L.gcF, w + L.gcR);
    hipLaunchKernelGGL((hg_group_carry_kernel<Op, REV>), dim3((unsigned)L.ngroups), dim3(kHgGroup), 0, st, w + L.aggF,
                       w + L.aggR, L.ntiles, w + L.gcF, w + L.gcR, w + L.carF, w + L.carR);
    return rin;
}

template <class Op, class T>
static void hg_primal(const int32_t* inds, int64_t n, int32_t m, const void* const* x, void* const* hs, char* w,
                      hipStream_t st) {
    constexpr int W = hg_words<T, Op::K>();
    const HgLayout L = hg_layout(n, m, Op::K, sizeof(T));
    HgIn<T> xi{};
    HgOut<T> ho{};
    for (int k = 0; k < Op::K; ++k) {
        xi.p[k] = n > 0 ? (const T*)x[k] : nullptr;
        ho.p[k] = (T*)hs[k];
    }
    const HgRec<W>* recs = hg_prepare<Op, T, false>(inds, n, m, xi, w, L, st);
    int32_t* nvalid = reinterpret_cast<int32_t*>(w + L.nvalid);
    hipLaunchKernelGGL((hg_empty_kernel<Op, T>), dim3((unsigned)ceil_div(m, 256)), dim3(256), 0, st, m, ho);
    hipLaunchKernelGGL((hg_apply_kernel<Op, T, W, false, T>), dim3((unsigned)L.ntiles), dim3(kHgBlock), 0, st, recs,
                       nvalid, w + L.carF, w + L.carR, ho, HgIn<T>{}, (HgAdj<T, Op::K>*)nullptr);
}

template <class Op, class T, bool ACC>
static void hg_vjp_t(const int32_t* inds, int64_t n, int32_t m, const void* const* x, const void* const* hs_bar,
                     void* const* x_bar, char* w, hipStream_t st) {
    constexpr int W = hg_words<T, Op::K>();
    using A = HgBack<T, Op::K, ACC>;
    using Adj = HgAdj<A, Op::K>;
    static_assert(sizeof(Adj) <= sizeof(HgRec<W>) || (Op::K <= 2 && sizeof(Adj) <= Op::K * sizeof(double)),
                  "adjoints fit a record buffer");
    const HgLayout L = hg_layout(n, m, Op::K, sizeof(T));
    HgIn<T> xi{}, hb{};
    HgOut<T> xb{};
    for (int k = 0; k < Op::K; ++k) {
        xi.p[k] = (const T*)x[k];
        hb.p[k] = (const T*)hs_bar[k];
        xb.p[k] = (T*)x_bar[k];
    }
    const HgRec<W>* recs = hg_prepare<Op, T, true>(inds, n, m, xi, w, L, st);
    const int32_t* nvalid = reinterpret_cast<const int32_t*>(w + L.nvalid);
    const int32_t* pos = reinterpret_cast<const int32_t*>(w + L.pos);
    Adj* from = reinterpret_cast<Adj*>(w + ((const char*)recs == w + L.recA ? L.recB : L.recA));
    Adj* to = reinterpret_cast<Adj*>(const_cast<HgRec<W>*>(recs));  // free once the adjoints are formed
    hipLaunchKernelGGL((hg_apply_kernel<Op, T, W, true, A>), dim3((unsigned)L.ntiles), dim3(kHgBlock), 0, st, recs,
                       nvalid, w + L.carF, w + L.carR, HgOut<T>{}, hb, from);
    const dim3 grid((unsigned)(L.npad / kHgSub));
    for (int pass = L.passes - 1; pass > 0; --pass) {
        hipLaunchKernelGGL((hg_back_kernel<A, Op::K>), grid, dim3(256), 0, st, pos + (int64_t)pass * L.npad, nvalid,
                           from, to);
        std::swap(from, to);
    }
    hipLaunchKernelGGL((hg_back_write_kernel<T, Op::K, ACC, A>), grid, dim3(256), 0, st, pos, n, nvalid, from, xb);
}

template <class Op, class T>
static void hg_vjp(const int32_t* inds, int64_t n, int32_t m, const void* const* x, const void* const* hs_bar,
                   void* const* x_bar, bool acc, char* w, hipStream_t st) {
    if (acc)
        hg_vjp_t<Op, T, true>(inds, n, m, x, hs_bar, x_bar, w, st);
    else
        hg_vjp_t<Op, T, false>(inds, n, m, x, hs_bar, x_bar, w, st);
}

static pvjp_status hg_check(const char* name, pvjp_gop op, pvjp_dtype dtype, const int32_t* inds,
                            const void* const* x, int64_t n, int64_t m, void* ws, size_t ws_bytes) {
    const int K = hg_components(op);
    PVJP_REQUIRE(K > 0, "%s: unknown operator %d", name, (int)op);
    PVJP_REQUIRE(valid_dtype(dtype), "%s: unknown dtype %d", name, (int)dtype);
    PVJP_REQUIRE(n >= 0 && n <= INT32_MAX, "%s: n = %lld out of range [0, 2^31)", name, (long long)n);
    PVJP_REQUIRE(m >= 1 && m <= kHgMaxBins, "%s: m = %lld out of range [1, 2^24]", name, (long long)m);
    PVJP_REQUIRE(ws != nullptr && aligned(ws, 256), "%s: workspace must be non-NULL and 256-byte aligned", name);
    const size_t need = pvjp_hist_generic_ws_bytes(op, dtype, n, m);
    if (ws_bytes < need) {
        set_error("%s: workspace of %zu bytes, need %zu", name, ws_bytes, need);
        return PVJP_ENOMEM;
    }
    if (n > 0) {
        PVJP_REQUIRE(inds != nullptr && x != nullptr, "%s: inds and x must be non-NULL", name);
        for (int c = 0; c < K; ++c) {
            PVJP_REQUIRE(x[c] != nullptr, "%s: component %d of x is NULL", name, c);
            PVJP_REQUIRE(aligned(x[c], dsize(dtype)), "%s: component %d of x is misaligned", name, c);
        }
    }
    return PVJP_OK;
}

}  // namespace pvjp

using namespace pvjp;

extern "C" size_t pvjp_hist_generic_ws_bytes(pvjp_gop op, pvjp_dtype dtype, int64_t n, int64_t m) {
    if (hg_components(op) == 0 || !valid_dtype(dtype) || n < 0 || m < 1 || m > kHgMaxBins) return 0;
    return hg_layout(n, m, hg_components(op), dsize(dtype)).total;
}

extern "C" pvjp_status pvjp_hist_generic(pvjp_gop op, pvjp_dtype dtype, const int32_t* inds, const void* const* x,
                                         int64_t n, int64_t m, void* const* hs, void* ws, size_t ws_bytes,
                                         void* stream) {
    clear_error();
    const pvjp_status s = hg_check("pvjp_hist_generic", op, dtype, inds, x, n, m, ws, ws_bytes);
    if (s != PVJP_OK) return s;
    const int K = hg_components(op);
    PVJP_REQUIRE(hs != nullptr, "pvjp_hist_generic: hs is NULL");
    for (int c = 0; c < K; ++c) PVJP_REQUIRE(hs[c] != nullptr, "pvjp_hist_generic: component %d of hs is NULL", c);
    const hipStream_t st = as_stream(stream);
    char* w = reinterpret_cast<char*>(ws);
    const int32_t mm = (int32_t)m;
    if (dtype == PVJP_F64) {
        if (op == PVJP_GOP_LOGADDEXP) hg_primal<GLogAddExp<double>, double>(inds, n, mm, x, hs, w, st);
        else if (op == PVJP_GOP_LINREC) hg_primal<GLinRec<double>, double>(inds, n, mm, x, hs, w, st);
        else hg_primal<GMat2<double>, double>(inds, n, mm, x, hs, w, st);
    } else {
        if (op == PVJP_GOP_LOGADDEXP) hg_primal<GLogAddExp<double>, float>(inds, n, mm, x, hs, w, st);
        else if (op == PVJP_GOP_LINREC) hg_primal<GLinRec<double>, float>(inds, n, mm, x, hs, w, st);
        else hg_primal<GMat2<double>, float>(inds, n, mm, x, hs, w, st);
    }
    PVJP_LAUNCHED("pvjp_hist_generic");
    return PVJP_OK;
}

extern "C" pvjp_status pvjp_hist_generic_vjp(pvjp_gop op, pvjp_dtype dtype, const int32_t* inds,
                                             const void* const* x, int64_t n, int64_t m, const void* const* hs_bar,
                                             void* const* x_bar, int accumulate, void* ws, size_t ws_bytes,
                                             void* stream) {
    clear_error();
    const pvjp_status s = hg_check("pvjp_hist_generic_vjp", op, dtype, inds, x, n, m, ws, ws_bytes);
    if (s != PVJP_OK) return s;
    if (n == 0) return PVJP_OK;
    const int K = hg_components(op);
    PVJP_REQUIRE(hs_bar != nullptr && x_bar != nullptr, "pvjp_hist_generic_vjp: hs_bar and x_bar must be non-NULL");
    for (int c = 0; c < K; ++c) {
        PVJP_REQUIRE(hs_bar[c] != nullptr, "pvjp_hist_generic_vjp: component %d of hs_bar is NULL", c);
        PVJP_REQUIRE(x_bar[c] != nullptr, "pvjp_hist_generic_vjp: component %d of x_bar is NULL", c);
        PVJP_REQUIRE(aligned(x_bar[c], dsize(dtype)), "pvjp_hist_generic_vjp: component %d of x_bar is misaligned",
                     c);
    }
    const hipStream_t st = as_stream(stream);
    char* w = reinterpret_cast<char*>(ws);
    const int32_t mm = (int32_t)m;
    const bool acc = accumulate != 0;
    if (dtype == PVJP_F64) {
        if (op == PVJP_GOP_LOGADDEXP) hg_vjp<GLogAddExp<double>, double>(inds, n, mm, x, hs_bar, x_bar, acc, w, st);
        else if (op == PVJP_GOP_LINREC) hg_vjp<GLinRec<double>, double>(inds, n, mm, x, hs_bar, x_bar, acc, w, st);
        else hg_vjp<GMat2<double>, double>(inds, n, mm, x, hs_bar, x_bar, acc, w, st);
    } else {
        if (op == PVJP_GOP_LOGADDEXP) hg_vjp<GLogAddExp<double>, float>(inds, n, mm, x, hs_bar, x_bar, acc, w, st);
        else if (op == PVJP_GOP_LINREC) hg_vjp<GLinRec<double>, float>(inds, n, mm, x, hs_bar, x_bar, acc, w, st);
        else hg_vjp<GMat2<double>, float>(inds, n, mm, x, hs_bar, x_bar, acc, w, st);
    }
    PVJP_LAUNCHED("pvjp_hist_generic_vjp");
    return PVJP_OK;
}
