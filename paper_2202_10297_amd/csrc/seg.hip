// Segmented batches: many linear-recurrence scans (and their VJPs) and many
// sum-reduce VJPs of uneven lengths, stored back to back, processed as ONE
// segmented operation per launch (the segmented-scan idea of Sec. 5.2's
// vectorised-operator rule, generalised to irregular segments).
//
//  - Return sweep (seg_batch_vjp): one persistent launch over a queue of
//    work items: first the scan's tile chains, longest first, then every
//    sum-reduce tile.  The lin_o reversed scan needs no flag: the last
//    element of each segment has no successor in its segment, so its c_i is
//    0, which cuts the carry exactly as the end of the array does.  So a
//    tile holding a segment end (a "cut tile") passes to its left a carry
//    that is its own aggregate, whatever lies to its right.  The tiles split
//    into chains: from just left of one cut tile down to the previous cut
//    tile included (the segment table fixes them when the batch is
//    prepared).  A chain's block first folds the cut tile at its right end
//    into its carry (one read of that tile's a and y_bar), then walks the
//    chain right to left, handing the carry from tile to tile in registers:
//    no tile ever waits on another block.  The
//    primal prefixes are recomputed from the checkpoint with the segmented
//    operator.  A sum-reduce tile writes x_bar_i = y_bar[segment of i]
//    (reduce(+)'s adjoint, Sec. 5.1.1).
//  - Primal (seg_linrec_fwd): the same left to right, with the segmented
//    operator (a flag restarts the recurrence at each segment head): a tile
//    holding a head passes on its own aggregate.  It writes per-segment
//    results and checkpoints every PVJP_LINREC_CKPT_INTERVAL global elements.
//  - Where a few long segments would leave most of the chip waiting for their
//    chains, long chains are cut into pieces (when the batch is prepared): a
//    launch before each sweep folds what lies before a chain's last piece in
//    short runs of tiles, and a piece starts from the folds before it.
//
// Segment heads of a tile come from the tile's first segment (a table written
// once by pvjp_seg_prepare) and the segment offsets.
#include <algorithm>
#include <utility>
#include <vector>

#include "common.h"
#include "prims.h"

namespace pvjp {

constexpr int kSegBlock = 256;
constexpr int kSegCk = PVJP_LINREC_CKPT_INTERVAL;
constexpr int64_t kSumGroup = 16;  // sum tiles per work item of the return sweep
constexpr int64_t kSegGrid = 2048;  // persistent blocks of the primal and of the folds (the most)
constexpr int64_t kSegResident = 1024;  // blocks that work at once, four a CU
constexpr int64_t kSegWhole = 8;  // chains of so many tiles are never cut, so smaller batches need no fold launch

constexpr size_t kSegSlot = 32;  // bytes of a fold's state
static_assert(sizeof(SegLinRec<double>::S) <= kSegSlot && sizeof(LinO<double>::S) <= kSegSlot,
              "a slot holds either sweep's state");

// A sweep's tables.  Walk entries, longest first: first tile in walking order,
// number of tiles, and where the carry comes from: x >= 0 the aggregate of tile
// x, x = -1 the neutral element, x <= -2 the y folds from slot -2 - x on.
// Fold entries (runs of tiles of cut chains; entry i fills slot i): first tile,
// number of tiles, tile whose aggregate comes before them or -1.
struct SegWalk {
    int32_t first, len, x, y;
};
struct SegFold {
    int32_t first, len, x;
};

// Workspace: [LookbackHdr | tile_seg0 int32[ntiles+1] | offsets int64[nseg+1] |
//             counts int32[4] (primal walks and folds, return sweep's) |
//             walks and folds of the primal, of the return sweep | fold states]
struct SegLayout {
    size_t seg0, offs, counts, walks[2], folds[2], states, total;
    int64_t ntiles;
};

static SegLayout seg_layout(int64_t total, int64_t nseg, int ts) {
    SegLayout L{};
    L.ntiles = ceil_div(total > 0 ? total : 1, ts);
    size_t o = align_up(sizeof(LookbackHdr), 256);
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o += align_up(bytes, 256);
        return at;
    };
    const size_t nt = (size_t)(L.ntiles + 1);
    L.seg0 = take(nt * 4);
    L.offs = take((size_t)(nseg + 1) * 8);
    L.counts = take(16);
    for (int d = 0; d < 2; ++d) {
        L.walks[d] = take(nt * sizeof(SegWalk));
        L.folds[d] = take(nt * sizeof(SegFold));
    }
    L.states = take(nt * kSegSlot);
    L.total = o;
    return L;
}


// Bitmap of segment heads over tile positions 0..TS (position TS is the first
// element of the next tile): bit j set iff base + j starts a segment (or is
// the end of the data).  Segments are non-empty, so a position holds at most
// one head.
template <int TS>
__device__ __forceinline__ void build_heads(uint32_t* bits, const int32_t* __restrict__ seg0,
                                            const int64_t* __restrict__ offs, int64_t nseg, int64_t tile,
                                            int64_t base) {
    constexpr int NW = (TS + 1 + 31) / 32;
    for (int w = threadIdx.x; w < NW; w += kSegBlock) bits[w] = 0u;
    __syncthreads();
    const int64_t s_lo = seg0[tile], s_hi = seg0[tile + 1] + 1;
    for (int64_t s = s_lo + threadIdx.x; s <= s_hi && s <= nseg; s += kSegBlock) {
        const int64_t j = offs[s] - base;
        if (j >= 0 && j <= TS) atomicOr(&bits[j >> 5], 1u << (j & 31));
    }
    __syncthreads();
}

__device__ __forceinline__ bool bit_at(const uint32_t* bits, int j) { return (bits[j >> 5] >> (j & 31)) & 1u; }

// The head bits of positions first .. first + IPT (a thread's run, which lies
// in one word, and the position after it) as one register.  A tile of few
// segments needs no bitmap: every thread looks at each offset (scalar loads
// in a uniform loop, no barrier).  Every thread of the block calls this.
constexpr int kFewHeads = 8;

template <int IPT>
__device__ __forceinline__ uint32_t run_heads(uint32_t* bits, const int32_t* __restrict__ seg0,
                                              const int64_t* __restrict__ offs, int64_t nseg, int64_t tile) {
    static_assert(32 % IPT == 0, "a run lies in one word");
    constexpr int TS = kSegBlock * IPT;
    const int64_t base = tile * TS;
    const int first = (int)threadIdx.x * IPT;
    const int s_lo = seg0[tile];
    const int64_t end = (int64_t)seg0[tile + 1] + 1;
    const int n = (int)((end < nseg ? end : nseg) - s_lo) + 1;
    if (n <= kFewHeads) {
        uint32_t m = 0;
        for (int i = 0; i < n; ++i) {
            const int64_t j = offs[s_lo + i] - base;  // negative: the tile starts inside its first segment
            const uint32_t d = (uint32_t)((j >= 0 && j <= TS ? (int)j : 2 * TS) - first);
            m |= d <= (uint32_t)IPT ? 1u << (d & 31) : 0u;
        }
        return m;
    }
    __syncthreads();  // the last tile's bits are no longer read
    build_heads<TS>(bits, seg0, offs, nseg, tile, base);
    return ((bits[first >> 5] >> (first & 31)) & ((1u << IPT) - 1u)) | ((uint32_t)bit_at(bits, first + IPT) << IPT);
}

// Waits for every load (and store) in flight.
__device__ __forceinline__ void seg_wait_memory() { __builtin_amdgcn_s_waitcnt(0x0f70); }  // vmcnt(0)

// The carry a walk entry starts from, besides a tile's aggregate: the block
// combines the folds before it (valid in every thread).
template <class Op>
__device__ __forceinline__ typename Op::S seg_piece_carry(const char* __restrict__ states, int32_t x, int32_t y,
                                                          typename Op::S* wtot) {
    typename Op::S c = Op::id(), tot;
    if (y == 0) return c;
    const int per = (y + kSegBlock - 1) / kSegBlock, i0 = (int)threadIdx.x * per;
    for (int i = i0; i < i0 + per && i < y; ++i)
        c = Op::comb(c, *reinterpret_cast<const typename Op::S*>(states + (size_t)(-2 - x + i) * kSegSlot));
    (void)block_exclusive_scan<Op, kSegBlock, false>(c, tot, wtot);
    __syncthreads();
    return tot;
}

// ------------------------------------------------------------------ primal
template <class T, int IPT>
struct SegFwdIn {  // a tile's inputs, striped over the block
    T a[IPT], b[IPT];
    __device__ __forceinline__ void load(const T* __restrict__ pa, const T* __restrict__ pb, int64_t total,
                                         int64_t tile) {
        constexpr int TS = kSegBlock * IPT;
        const int64_t base = tile * TS;
        const int cnt = (int)((total - base) < TS ? (total - base) : TS);
        load_striped<T, kSegBlock, IPT>(pa + base, cnt, a, T(1));
        load_striped<T, kSegBlock, IPT>(pb + base, cnt, b, T(0));
    }
};

// A thread's run of IPT elements of one tile with their head flags, and their
// fold.
template <class T, int IPT>
__device__ __forceinline__ typename SegLinRec<T>::S seg_fwd_run(const SegFwdIn<T, IPT>& in, uint32_t heads, T* lds,
                                                                typename SegLinRec<T>::S (&e)[IPT]) {
    using Op = SegLinRec<T>;
    using S = typename Op::S;
    T ra[IPT], rb[IPT];
    striped_to_blocked<T, kSegBlock, IPT>(in.a, ra, lds);
    __syncthreads();
    striped_to_blocked<T, kSegBlock, IPT>(in.b, rb, lds);
#pragma unroll
    for (int j = 0; j < IPT; ++j) e[j] = S{ra[j], rb[j], (heads >> j) & 1u, 0u};
    S agg = e[0];
#pragma unroll
    for (int j = 1; j < IPT; ++j) agg = Op::comb(agg, e[j]);
    return agg;
}

template <class T, int IPT>
__device__ __forceinline__ typename SegLinRec<T>::S seg_fwd_agg(const T* __restrict__ a, const T* __restrict__ b,
                                                                int64_t total, int64_t nseg,
                                                                const int64_t* __restrict__ offs,
                                                                const int32_t* __restrict__ seg0, int64_t tile,
                                                                T* lds, uint32_t* bits,
                                                                typename SegLinRec<T>::S* wtot) {
    using Op = SegLinRec<T>;
    constexpr int TS = kSegBlock * IPT;
    typename Op::S e[IPT], tot;
    // The elements after the tile's last head: few of them need no tile (20,000
    // segments of 64 .. 600 elements, FP32, a chain per tile: 38.6 us, now 35.8).
    const int64_t head = offs[seg0[tile + 1]], left = (tile + 1) * TS - head;
    if (left <= 4 * kSegBlock) {
        if (left <= 0) return Op::id();  // the next tile starts at a head
        const int64_t i0 = head + 4 * (int64_t)threadIdx.x, end = min((tile + 1) * TS, total);
        typename Op::S agg = Op::id();
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (i0 + j < end) agg = Op::comb(agg, typename Op::S{a[i0 + j], b[i0 + j], 0u, 0u});
        (void)block_exclusive_scan<Op, kSegBlock, false>(agg, tot, wtot);
        __syncthreads();
        return tot;
    }
    SegFwdIn<T, IPT> in;
    in.load(a, b, total, tile);
    const auto agg = seg_fwd_run<T, IPT>(in, run_heads<IPT>(bits, seg0, offs, nseg, tile), lds, e);
    (void)block_exclusive_scan<Op, kSegBlock, false>(agg, tot, wtot);
    __syncthreads();  // the tile's LDS is free
    return tot;
}

// A block per fold entry.
template <class T, int IPT>
__global__ __launch_bounds__(kSegBlock) void seg_fwd_fold_kernel(const T* __restrict__ a, const T* __restrict__ b,
                                                                 int64_t total, int64_t nseg,
                                                                 const int64_t* __restrict__ offs,
                                                                 const int32_t* __restrict__ seg0,
                                                                 const SegFold* __restrict__ folds,
                                                                 const int32_t* __restrict__ nfold,
                                                                 char* __restrict__ states) {
    using Op = SegLinRec<T>;
    constexpr int TS = kSegBlock * IPT;
    __shared__ T lds[lds_elems<T, TS>()];
    __shared__ typename Op::S wtot[kSegBlock / kWave];
    __shared__ uint32_t bits[(TS + 1 + 31) / 32];
    for (int i = blockIdx.x; i < *nfold; i += gridDim.x) {
        const SegFold f = folds[i];
        typename Op::S c = Op::id();
        if (f.x >= 0) c = seg_fwd_agg<T, IPT>(a, b, total, nseg, offs, seg0, f.x, lds, bits, wtot);
        for (int t = 0; t < f.len; ++t)
            c = Op::comb(c, seg_fwd_agg<T, IPT>(a, b, total, nseg, offs, seg0, f.first + t, lds, bits, wtot));
        if (threadIdx.x == 0) *reinterpret_cast<typename Op::S*>(states + (size_t)i * kSegSlot) = c;
    }
}

// Persistent blocks draw walk entries.  Bound by HBM and by the longest chain:
// the next tile's loads are issued before the scan of this one and waited for
// before its stores, so neither's latency is in the chain.  As one
// decoupled-lookback launch over the tiles, 4,096 segments of 64 .. 2^20 FP32
// elements (431 M) took 2,457 us, 2.8 TB/s; by chains 1,760; with the loads
// ahead and head bits without a bitmap 1,536, 4.5 TB/s.  64 segments, 5 M
// elements, take 32 us with the folds (31 in one launch), 2,048 (longest chain
// cut) 980 (1,190).
template <class T, int IPT>
__global__ __launch_bounds__(kSegBlock) void seg_linrec_fwd_kernel(
    const T* __restrict__ a, const T* __restrict__ b, int64_t total, int64_t nseg, const int64_t* __restrict__ offs,
    const int32_t* __restrict__ seg0, T* __restrict__ A, T* __restrict__ B, T* __restrict__ ckpt, LookbackHdr* hdr,
    const SegWalk* __restrict__ walks, const int32_t* __restrict__ nwalk, const char* __restrict__ states) {
    using Op = SegLinRec<T>;
    using S = typename Op::S;
    constexpr int TS = kSegBlock * IPT;
    __shared__ T lds[lds_elems<T, TS>()];
    __shared__ S wtot[kSegBlock / kWave];
    __shared__ uint32_t bits[(TS + 1 + 31) / 32];
    __shared__ uint32_t s_ticket;

    const int first = (int)threadIdx.x * IPT;
    // every block makes one final, empty draw: the launch's last ticket
    const uint32_t nw = (uint32_t)*nwalk, last = nw + gridDim.x - 1;
    while (true) {
        if (threadIdx.x == 0) {
            s_ticket = lookback_draw(hdr, last, nullptr);
            if (s_ticket > last) lookback_error(hdr, kErrTicket);
        }
        __syncthreads();
        const uint32_t item = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_ticket);
        if (item >= nw) return;  // done (or the workspace was not in its rest state)
        const SegWalk wk = walks[item];
        S carry = wk.x >= 0 ? seg_fwd_agg<T, IPT>(a, b, total, nseg, offs, seg0, wk.x, lds, bits, wtot)
                            : seg_piece_carry<Op>(states, wk.x, wk.y, wtot);
        SegFwdIn<T, IPT> in;
        in.load(a, b, total, wk.first);
        for (int64_t tile = wk.first, end = tile + wk.len; tile < end; ++tile) {
            const int64_t base = tile * TS;
            const int cnt = (int)((total - base) < TS ? (total - base) : TS);
            S e[IPT];
            const S agg = seg_fwd_run<T, IPT>(in, run_heads<IPT>(bits, seg0, offs, nseg, tile), lds, e);
            if (tile + 1 < end) in.load(a, b, total, tile + 1);
            S tot;
            const S excl = block_exclusive_scan<Op, kSegBlock, false>(agg, tot, wtot);
            S run = Op::comb(carry, excl);
            seg_wait_memory();
            if (ckpt != nullptr && (first % kSegCk) == 0 && first < cnt) {
                const int64_t c = (base + first) / kSegCk;
                ckpt[2 * c] = run.a;
                ckpt[2 * c + 1] = run.b;
            }
            if (A != nullptr) {
                T ra[IPT], rb[IPT];
#pragma unroll
                for (int j = 0; j < IPT; ++j) {
                    run = Op::comb(run, e[j]);
                    ra[j] = run.a;
                    rb[j] = run.b;
                }
                store_blocked<T, kSegBlock, IPT, false>(A + base, cnt, ra, lds);
                store_blocked<T, kSegBlock, IPT, false>(B + base, cnt, rb, lds);
            }
            carry = Op::comb(carry, tot);
            __syncthreads();
        }
    }
}

// ----------------------------------------------------------- return sweep
template <class T, int IPT>
struct SegVjpIn {  // a tile's inputs, striped over the block, and a's first element after it
    T a[IPT], b[IPT], ya[IPT], yb[IPT], after;
    template <bool B>
    __device__ __forceinline__ void load(const T* __restrict__ pa, const T* __restrict__ pb,
                                         const T* __restrict__ pya, const T* __restrict__ pyb, int64_t total,
                                         int64_t tile) {
        constexpr int TS = kSegBlock * IPT;
        const int64_t base = tile * TS;
        const int cnt = (int)((total - base) < TS ? (total - base) : TS);
        load_striped<T, kSegBlock, IPT>(pa + base, cnt, a, T(1));
        if constexpr (B) load_striped<T, kSegBlock, IPT>(pb + base, cnt, b, T(0));
        load_striped<T, kSegBlock, IPT>(pya + base, cnt, ya, T(0));
        load_striped<T, kSegBlock, IPT>(pyb + base, cnt, yb, T(0));
        after = ((int)threadIdx.x == kSegBlock - 1 && base + TS < total) ? pa[base + TS] : T(1);
    }
    // a_i and a_{i+1} of the thread's run
    __device__ __forceinline__ void run_a(T (&ra)[IPT], T (&rc)[IPT], T* lds) const {
        striped_to_blocked<T, kSegBlock, IPT>(a, ra, lds);
        const T nxt =
            ((int)threadIdx.x < kSegBlock - 1) ? lds[lds_pad<T>(((int)threadIdx.x + 1) * IPT)] : after;
#pragma unroll
        for (int j = 0; j < IPT - 1; ++j) rc[j] = ra[j + 1];
        rc[IPT - 1] = nxt;
        __syncthreads();
    }
};

// One scan tile of a chain: `carry` is the inclusive lin_o state of the tile
// to its right (the neutral element at the chain's right end); returns this
// tile's inclusive state (valid in every thread), the next tile's carry.
// `in` holds the tile's inputs, then those of tile `next` (if not negative).
template <class T, int IPT, bool ACC>
__device__ __forceinline__ typename LinO<T>::S seg_scan_vjp_tile(const T* __restrict__ a, const T* __restrict__ b,
                                                                 const T* __restrict__ ya, const T* __restrict__ yb,
                                                                 int64_t total, const T* __restrict__ ckpt,
                                                                 T* __restrict__ abar, T* __restrict__ bbar,
                                                                 int64_t tile, int64_t next, SegVjpIn<T, IPT>& in,
                                                                 typename LinO<T>::S carry, T* lds, uint32_t heads,
                                                                 typename SegLinRec<T>::S* wtot_p,
                                                                 typename LinO<T>::S* wtot_l) {
    using P = SegLinRec<T>;
    using L = LinO<T>;
    using PS = typename P::S;
    using LS = typename L::S;
    constexpr int TS = kSegBlock * IPT;
    const int64_t base = tile * TS;
    const int cnt = (int)((total - base) < TS ? (total - base) : TS);

    T ra[IPT], rc[IPT], rb[IPT], rya[IPT], ryb[IPT];
    in.run_a(ra, rc, lds);
    striped_to_blocked<T, kSegBlock, IPT>(in.b, rb, lds);
    __syncthreads();
    striped_to_blocked<T, kSegBlock, IPT>(in.ya, rya, lds);
    __syncthreads();
    striped_to_blocked<T, kSegBlock, IPT>(in.yb, ryb, lds);
    if (next >= 0) in.template load<true>(a, b, ya, yb, total, next);

    // 1. primal prefixes (A_{i-1}, B_{i-1}) within each segment
    T pA[IPT], pB[IPT];
    {
        PS pe[IPT];
#pragma unroll
        for (int j = 0; j < IPT; ++j) pe[j] = PS{ra[j], rb[j], (heads >> j) & 1u, 0u};
        PS pagg = pe[0];
#pragma unroll
        for (int j = 1; j < IPT; ++j) pagg = P::comb(pagg, pe[j]);
        PS ptot;
        PS pexcl = block_exclusive_scan<P, kSegBlock, false>(pagg, ptot, wtot_p);
        const int64_t c = base / kSegCk;
        PS run = P::comb(PS{ckpt[2 * c], ckpt[2 * c + 1], 0u, 0u}, pexcl);
#pragma unroll
        for (int j = 0; j < IPT; ++j) {
            const bool head = pe[j].f != 0u;
            pA[j] = head ? T(1) : run.a;
            pB[j] = head ? T(0) : run.b;
            run = P::comb(run, pe[j]);
        }
    }
    // 2. lin_o elements: c_i = a_{i+1}, or 0 when i ends its segment
    LS e[IPT];
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        const bool last = (heads >> (j + 1)) & 1u;
        e[j] = LS{last ? T(0) : rc[j], rya[j], ryb[j]};
    }
    // 3. reversed scan inside the tile, after the carry from the right
    LS agg = L::id();
#pragma unroll
    for (int j = IPT - 1; j >= 0; --j) agg = L::comb(agg, e[j]);
    LS tot;
    LS excl = block_exclusive_scan<L, kSegBlock, true>(agg, tot, wtot_l);
    // 4. input adjoints
    LS run = L::comb(carry, excl);
#pragma unroll
    for (int j = IPT - 1; j >= 0; --j) {
        run = L::comb(run, e[j]);
        ra[j] = pA[j] * run.dA + pB[j] * run.dB;
        rb[j] = run.dB;
    }
    seg_wait_memory();
    store_blocked<T, kSegBlock, IPT, ACC>(abar + base, cnt, ra, lds);
    store_blocked<T, kSegBlock, IPT, ACC>(bbar + base, cnt, rb, lds);
    return L::comb(carry, tot);
}

template <class T, int IPT, bool ACC>
__device__ __forceinline__ void seg_sum_vjp_tile(int64_t total, const int32_t* __restrict__ seg0,
                                                 const T* __restrict__ ybar, T* __restrict__ xbar, int64_t tile,
                                                 uint32_t heads, T* lds, IntSum::S* wtot_i) {
    constexpr int TS = kSegBlock * IPT;
    const int64_t base = tile * TS;
    const int cnt = (int)((total - base) < TS ? (total - base) : TS);
    const int first = (int)threadIdx.x * IPT;
    // The segment of tile position j is seg0[tile] plus the number of heads at
    // positions 1..j: a block exclusive scan of per-thread head counts, then a
    // walk over the thread's own items.
    if (first == 0) heads &= ~1u;
    const int mine = __popc(heads & ((1u << IPT) - 1u));
    IntSum::S tot;
    int seg = seg0[tile] + block_exclusive_scan<IntSum, kSegBlock, false>(IntSum::S{mine}, tot, wtot_i).v;
    T out[IPT];
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        seg += (int)((heads >> j) & 1u);
        out[j] = (first + j < cnt) ? ybar[seg] : T(0);
    }
    store_blocked<T, kSegBlock, IPT, ACC>(xbar + base, cnt, out, lds);
}

// The lin_o aggregate of one tile (c_i = a_{i+1}, 0 at segment ends; d_i =
// y_bar_i), folded right to left; valid in every thread.
template <class T, int IPT>
__device__ __forceinline__ typename LinO<T>::S seg_tile_linagg(const T* __restrict__ a, const T* __restrict__ ya,
                                                               const T* __restrict__ yb, int64_t total, int64_t tile,
                                                               T* lds, uint32_t heads,
                                                               typename LinO<T>::S* wtot_l) {
    using L = LinO<T>;
    using LS = typename L::S;
    T ra[IPT], rc[IPT], rya[IPT], ryb[IPT];
    SegVjpIn<T, IPT> in;
    in.template load<false>(a, nullptr, ya, yb, total, tile);
    in.run_a(ra, rc, lds);
    striped_to_blocked<T, kSegBlock, IPT>(in.ya, rya, lds);
    __syncthreads();
    striped_to_blocked<T, kSegBlock, IPT>(in.yb, ryb, lds);
    LS agg = L::id();
#pragma unroll
    for (int j = IPT - 1; j >= 0; --j) {
        const bool last = (heads >> (j + 1)) & 1u;
        agg = L::comb(agg, LS{last ? T(0) : rc[j], rya[j], ryb[j]});
    }
    LS tot;
    (void)block_exclusive_scan<L, kSegBlock, true>(agg, tot, wtot_l);
    return tot;
}

// A block per fold entry.
template <class T, int IPT>
__global__ __launch_bounds__(kSegBlock) void seg_vjp_fold_kernel(const T* __restrict__ a, const T* __restrict__ ya,
                                                                 const T* __restrict__ yb, int64_t total,
                                                                 int64_t nseg, const int64_t* __restrict__ offs,
                                                                 const int32_t* __restrict__ seg0,
                                                                 const SegFold* __restrict__ folds,
                                                                 const int32_t* __restrict__ nfold,
                                                                 char* __restrict__ states) {
    using L = LinO<T>;
    constexpr int TS = kSegBlock * IPT;
    __shared__ T lds[lds_elems<T, TS>()];
    __shared__ typename L::S wtot_l[kSegBlock / kWave];
    __shared__ uint32_t bits[(TS + 1 + 31) / 32];
    for (int i = blockIdx.x; i < *nfold; i += gridDim.x) {
        const SegFold f = folds[i];
        typename L::S c = L::id();
        for (int t = f.x >= 0 ? -1 : 0; t < f.len; ++t) {
            const int64_t tile = t < 0 ? f.x : f.first - t;
            c = L::comb(c, seg_tile_linagg<T, IPT>(a, ya, yb, total, tile, lds,
                                                   run_heads<IPT>(bits, seg0, offs, nseg, tile), wtot_l));
            __syncthreads();
        }
        if (threadIdx.x == 0) *reinterpret_cast<typename L::S*>(states + (size_t)i * kSegSlot) = c;
    }
}

// Bound by HBM: the 4,096 segments above take 2,472 us, with the sum-reduce
// tiles 5.2 TB/s (2,818 with each tile's loads behind the stores of the last and
// the heads from a bitmap).  64 segments, 5 M elements, take 55 us with the folds
// (1,150 while their chains were not cut), 2,048 1,480 (2,020).
// Sixteen FP64 elements a thread fill the registers: with the next tile's inputs
// among them the kernel takes 396, one wave a SIMD; without, held to two waves,
// 2,000 segments of 64 .. 2^19 elements take 1,286 us (1,549 with them, 1,420 as
// one launch over the tiles), 4,096 of 64 .. 2^14 141 (185, 183).
template <class T, int IPT>
constexpr bool seg_ahead() {
    return sizeof(T) * IPT <= 64;
}

template <class T, int IPT, bool ACC>
__global__ __launch_bounds__(kSegBlock, (seg_ahead<T, IPT>() ? 1 : 2)) void seg_batch_vjp_kernel(
    const T* __restrict__ a, const T* __restrict__ b, const T* __restrict__ ya, const T* __restrict__ yb,
    int64_t total, int64_t nseg, const int64_t* __restrict__ offs, const int32_t* __restrict__ seg0,
    const T* __restrict__ ckpt, T* __restrict__ abar, T* __restrict__ bbar, const T* __restrict__ sum_ybar,
    T* __restrict__ sum_xbar, LookbackHdr* hdr, const int32_t* __restrict__ nwalk,
    const SegWalk* __restrict__ walks, const char* __restrict__ states, int64_t ntiles, int scan, int64_t nsum) {
    constexpr int TS = kSegBlock * IPT;
    __shared__ T lds[lds_elems<T, TS>()];
    __shared__ typename SegLinRec<T>::S wtot_p[kSegBlock / kWave];
    __shared__ typename LinO<T>::S wtot_l[kSegBlock / kWave];
    __shared__ IntSum::S wtot_i[kSegBlock / kWave];
    __shared__ uint32_t bits[(TS + 1 + 31) / 32];
    __shared__ uint32_t s_ticket;

    const int64_t nscan = scan ? (int64_t)*nwalk : 0;
    // every block makes one final, empty draw: the launch's last ticket
    const uint32_t last = (uint32_t)(nscan + nsum + gridDim.x - 1);
    if (threadIdx.x == 0) {
        s_ticket = lookback_draw(hdr, last, nullptr);
        if (s_ticket > last) lookback_error(hdr, kErrTicket);
    }
    __syncthreads();
    if (s_ticket > last) return;  // the workspace was not in its rest state: do nothing
    // Queue: items [0, nscan) are the scan's tile chains (longest first),
    // items [nscan, nscan + nsum) runs of kSumGroup sum tiles.  No item waits
    // on another.
    while (true) {
        const int64_t item = (uint32_t)__builtin_amdgcn_readfirstlane((int)s_ticket);
        if (item >= nscan + nsum) break;
        if (item < nscan) {
            const SegWalk wk = walks[item];
            typename LinO<T>::S carry;
            if (wk.x >= 0) {  // the cut tile right of the chain: its aggregate is the carry
                carry = seg_tile_linagg<T, IPT>(a, ya, yb, total, wk.x, lds,
                                                run_heads<IPT>(bits, seg0, offs, nseg, wk.x), wtot_l);
                __syncthreads();
            } else {
                carry = seg_piece_carry<LinO<T>>(states, wk.x, wk.y, wtot_l);
            }
            SegVjpIn<T, IPT> in;
            constexpr bool kAhead = seg_ahead<T, IPT>();
            if (kAhead) in.template load<true>(a, b, ya, yb, total, wk.first);
            for (int64_t t = wk.first, end = t - wk.len; t > end; --t) {
                if (!kAhead) in.template load<true>(a, b, ya, yb, total, t);
                carry = seg_scan_vjp_tile<T, IPT, ACC>(a, b, ya, yb, total, ckpt, abar, bbar, t,
                                                       kAhead && t - 1 > end ? t - 1 : -1, in, carry, lds,
                                                       run_heads<IPT>(bits, seg0, offs, nseg, t), wtot_p, wtot_l);
                __syncthreads();
            }
        } else {
            // a sum item is a run of kSumGroup tiles: one ticket per run keeps
            // the queue's counter (one device-scope atomic per draw, serialised
            // on one address) off the critical path
            const int64_t t0 = (item - nscan) * kSumGroup;
            const int64_t t1 = (t0 + kSumGroup < ntiles) ? t0 + kSumGroup : ntiles;
            for (int64_t tile = t0; tile < t1; ++tile) {
                seg_sum_vjp_tile<T, IPT, ACC>(total, seg0, sum_ybar, sum_xbar, tile,
                                              run_heads<IPT>(bits, seg0, offs, nseg, tile), lds, wtot_i);
                __syncthreads();
            }
        }
        __syncthreads();
        if (threadIdx.x == 0) s_ticket = lookback_draw(hdr, last, nullptr);
        __syncthreads();
    }
}

// ------------------------------------------------------------------ host
static bool valid_tile(int ts) { return ts == 1024 || ts == 2048 || ts == 4096; }

template <class T, int IPT>
static void launch_fwd(const void* a, const void* b, int64_t total, int64_t nseg, void* A, void* B, void* ckpt,
                       char* ws, const SegLayout& L, hipStream_t st) {
    const int32_t* counts = (const int32_t*)(ws + L.counts);
    const unsigned grid = (unsigned)(L.ntiles < kSegGrid ? L.ntiles : kSegGrid);
    if (L.ntiles > kSegWhole)
            hipLaunchKernelGGL((seg_fwd_fold_kernel<T, IPT>), dim3(grid), dim3(kSegBlock), 0, st, (const T*)a,
                           (const T*)b, total, nseg, (const int64_t*)(ws + L.offs), (const int32_t*)(ws + L.seg0),
                           (const SegFold*)(ws + L.folds[0]), counts + 1, ws + L.states);
    hipLaunchKernelGGL((seg_linrec_fwd_kernel<T, IPT>), dim3(grid), dim3(kSegBlock), 0, st, (const T*)a, (const T*)b,
                       total, nseg, (const int64_t*)(ws + L.offs), (const int32_t*)(ws + L.seg0), (T*)A, (T*)B,
                       (T*)ckpt, (LookbackHdr*)ws, (const SegWalk*)(ws + L.walks[0]), counts, ws + L.states);
}

template <class T, int IPT, bool ACC>
static void launch_batch(const void* a, const void* b, const void* ya, const void* yb, int64_t total, int64_t nseg,
                         const void* ckpt, void* abar, void* bbar, const void* sy, void* sx, int grid, char* ws,
                         const SegLayout& L, hipStream_t st) {
    const int32_t* counts = (const int32_t*)(ws + L.counts);
    if (a && L.ntiles > kSegWhole)
        hipLaunchKernelGGL((seg_vjp_fold_kernel<T, IPT>), dim3((unsigned)(L.ntiles < kSegGrid ? L.ntiles : kSegGrid)),
                           dim3(kSegBlock), 0, st, (const T*)a, (const T*)ya, (const T*)yb, total, nseg,
                           (const int64_t*)(ws + L.offs), (const int32_t*)(ws + L.seg0),
                           (const SegFold*)(ws + L.folds[1]), counts + 3, ws + L.states);
    hipLaunchKernelGGL((seg_batch_vjp_kernel<T, IPT, ACC>), dim3((unsigned)grid), dim3(kSegBlock), 0, st, (const T*)a,
                       (const T*)b, (const T*)ya, (const T*)yb, total, nseg, (const int64_t*)(ws + L.offs),
                       (const int32_t*)(ws + L.seg0), (const T*)ckpt, (T*)abar, (T*)bbar, (const T*)sy, (T*)sx,
                       (LookbackHdr*)ws, counts + 2, (const SegWalk*)(ws + L.walks[1]), ws + L.states, L.ntiles,
                       a ? 1 : 0, sy ? ceil_div(L.ntiles, kSumGroup) : 0);
}

template <class T, bool ACC>
static void dispatch_batch(int ts, const void* a, const void* b, const void* ya, const void* yb, int64_t total,
                           int64_t nseg, const void* ckpt, void* abar, void* bbar, const void* sy, void* sx, int grid,
                           char* ws, const SegLayout& L, hipStream_t st) {
    if (ts == 1024)
        launch_batch<T, 1024 / kSegBlock, ACC>(a, b, ya, yb, total, nseg, ckpt, abar, bbar, sy, sx, grid, ws, L, st);
    else if (ts == 2048)
        launch_batch<T, 2048 / kSegBlock, ACC>(a, b, ya, yb, total, nseg, ckpt, abar, bbar, sy, sx, grid, ws, L, st);
    else
        launch_batch<T, 4096 / kSegBlock, ACC>(a, b, ya, yb, total, nseg, ckpt, abar, bbar, sy, sx, grid, ws, L, st);
}

}  // namespace pvjp

using namespace pvjp;

extern "C" size_t pvjp_seg_ws_bytes(int64_t total, int64_t nseg, int tile_elems) {
    if (total < 1 || nseg < 1 || !valid_tile(tile_elems)) return 0;
    return seg_layout(total, nseg, tile_elems).total;
}

extern "C" pvjp_status pvjp_seg_prepare(const int64_t* host_offsets, int64_t nseg, int tile_elems, void* ws,
                                        size_t ws_bytes, void* stream) {
    clear_error();
    PVJP_REQUIRE(host_offsets != nullptr && nseg >= 1, "pvjp_seg_prepare: need host offsets of nseg >= 1 segments");
    PVJP_REQUIRE(valid_tile(tile_elems), "pvjp_seg_prepare: tile_elems must be 1024, 2048 or 4096");
    PVJP_REQUIRE(host_offsets[0] == 0, "pvjp_seg_prepare: offsets[0] must be 0");
    for (int64_t s = 0; s < nseg; ++s)
        PVJP_REQUIRE(host_offsets[s + 1] > host_offsets[s], "pvjp_seg_prepare: segment %lld is empty or offsets decrease",
                     (long long)s);
    const int64_t total = host_offsets[nseg];
    PVJP_REQUIRE(total <= ((int64_t)1 << 40), "pvjp_seg_prepare: total length out of range");
    PVJP_REQUIRE(ws != nullptr && aligned(ws, 256), "pvjp_seg_prepare: ws must be non-NULL and 256-byte aligned");
    const SegLayout L = seg_layout(total, nseg, tile_elems);
    if (ws_bytes < L.total) {
        set_error("pvjp_seg_prepare: workspace has %zu bytes, needs %zu", ws_bytes, L.total);
        return PVJP_ENOMEM;
    }
    std::vector<int32_t> seg0((size_t)L.ntiles + 1);
    int64_t s = 0;
    for (int64_t t = 0; t < L.ntiles; ++t) {
        const int64_t base = t * tile_elems;
        while (host_offsets[s + 1] <= base) ++s;
        seg0[(size_t)t] = (int32_t)s;
    }
    seg0[(size_t)L.ntiles] = (int32_t)nseg;
    // A sweep's chains.  stop[t] (t in walking order): the tile passes on its
    // own aggregate (return sweep: it holds a segment end; primal: a head).
    // With such tiles c_0 < ... < c_K, a chain covers the tiles after c_k up to
    // c_{k+1} (or the end), from the carry of c_k's aggregate; the tiles up to
    // c_0 start neutral.  Longest first, so the queue's tail holds short work.
    // Chains are cut into pieces where the longest is more than three times a
    // block's share of the tiles: a tile of a chain takes a block about four
    // times as long as the busy chip takes per tile and block, so a chain of up
    // to four shares ends with the queue.  The folds read the inputs once more:
    // forward and return sweep of 2,000 segments of 64 .. 2^20 elements (longest
    // chain 4.8 shares) take 2.64 ms in pieces of four shares, 2.47 of three,
    // 2.33 of two, 2.47 of one; 4,096 segments (2.5 shares) 4.0 uncut and 4.4 in
    // pieces of two.  A piece is folded in several parts, because a fold of a
    // whole piece by one block is itself a chain (200 segments, 24 M elements:
    // the two fold launches take 96 us in parts of four tiles, 82 in parts of a
    // quarter of a share, here one).
    std::vector<SegWalk> walks[2];
    std::vector<SegFold> folds[2];
    const int64_t share = ceil_div(L.ntiles, kSegResident);
    for (int d = 0; d < 2; ++d) {
        std::vector<char> stop((size_t)L.ntiles, 0);
        const int64_t nt = L.ntiles;
        for (int64_t s2 = 0; s2 < nseg; ++s2) {
            if (d == 0)
                stop[(size_t)(host_offsets[s2] / tile_elems)] = 1;
            else
                stop[(size_t)(nt - 1 - (host_offsets[s2 + 1] - 1) / tile_elems)] = 1;
        }
        auto tile_of = [&](int64_t t) { return (int32_t)(d == 0 ? t : nt - 1 - t); };
        std::vector<std::pair<int64_t, int64_t>> chains;  // tiles (after, to] in walking order, after = -1: neutral
        int64_t after = -1, longest = 0;
        for (int64_t t = 0; t < nt; ++t) {
            if (!stop[(size_t)t] && t + 1 < nt) continue;
            chains.push_back({after, t});
            longest = std::max(longest, t - after);
            after = t;
        }
        const bool cut = longest > std::max(3 * share, kSegWhole);
        const int64_t unit = cut ? std::max<int64_t>(share / 4, 1) : longest;  // tiles a fold
        const int64_t per = cut ? 2 * share / unit : 1;  // folds a piece
        for (const auto& c : chains) {
            const int32_t x = c.first < 0 ? -1 : tile_of(c.first);
            const int32_t slot = (int32_t)folds[d].size();
            int32_t before = 0;  // folds before the piece
            for (int64_t t = c.first + 1; t <= c.second; t += per * unit) {
                const int64_t len = std::min(per * unit, c.second + 1 - t);
                walks[d].push_back(SegWalk{tile_of(t), (int32_t)len, before ? -2 - slot : x, before});
                if (t + len > c.second) break;
                for (int64_t u = t; u < t + len; u += unit, ++before)
                    folds[d].push_back(SegFold{tile_of(u), (int32_t)unit, before ? -1 : x});
            }
        }
        std::stable_sort(walks[d].begin(), walks[d].end(),
                         [](const SegWalk& x, const SegWalk& y) { return x.len > y.len; });
    }
    const int32_t counts[4] = {(int32_t)walks[0].size(), (int32_t)folds[0].size(), (int32_t)walks[1].size(),
                               (int32_t)folds[1].size()};
    auto upload = [&](size_t at, const void* src, size_t bytes, hipStream_t s3) {
        return bytes == 0 || hipMemcpyAsync(reinterpret_cast<char*>(ws) + at, src, bytes, hipMemcpyHostToDevice, s3) ==
                                 hipSuccess;
    };
    hipStream_t st = as_stream(stream);
    bool ok = upload(L.seg0, seg0.data(), seg0.size() * 4, st) &&
              upload(L.offs, host_offsets, (size_t)(nseg + 1) * 8, st) && upload(L.counts, counts, sizeof(counts), st);
    for (int d = 0; d < 2; ++d)
        ok = ok && upload(L.walks[d], walks[d].data(), walks[d].size() * sizeof(SegWalk), st) &&
             upload(L.folds[d], folds[d].data(), folds[d].size() * sizeof(SegFold), st);
    if (!ok || hipStreamSynchronize(st) != hipSuccess) {
        set_error("pvjp_seg_prepare: uploading the segment tables failed");
        return PVJP_EDEVICE;
    }
    return PVJP_OK;
}

extern "C" pvjp_status pvjp_seg_linrec_scan(pvjp_dtype dtype, const void* a, const void* b, int64_t total, int64_t nseg,
                                            int tile_elems, void* A, void* B, void* ckpt, void* ws, size_t ws_bytes,
                                            void* stream) {
    clear_error();
    PVJP_REQUIRE(valid_dtype(dtype), "pvjp_seg_linrec_scan: unknown dtype %d", (int)dtype);
    PVJP_REQUIRE(total >= 1 && nseg >= 1, "pvjp_seg_linrec_scan: total and nseg must be >= 1");
    PVJP_REQUIRE(valid_tile(tile_elems), "pvjp_seg_linrec_scan: tile_elems must be 1024, 2048 or 4096");
    PVJP_REQUIRE(a && b, "pvjp_seg_linrec_scan: a and b must be non-NULL");
    PVJP_REQUIRE((A == nullptr) == (B == nullptr) && (A || ckpt), "pvjp_seg_linrec_scan: need A and B, or ckpt");
    PVJP_REQUIRE(ws != nullptr && aligned(ws, 256), "pvjp_seg_linrec_scan: ws must be non-NULL and 256-byte aligned");
    const SegLayout L = seg_layout(total, nseg, tile_elems);
    if (ws_bytes < L.total) {
        set_error("pvjp_seg_linrec_scan: workspace has %zu bytes, needs %zu", ws_bytes, L.total);
        return PVJP_ENOMEM;
    }
    char* w = reinterpret_cast<char*>(ws);
    hipStream_t st = as_stream(stream);
    if (dtype == PVJP_F64) {
        if (tile_elems == 1024) launch_fwd<double, 4>(a, b, total, nseg, A, B, ckpt, w, L, st);
        else if (tile_elems == 2048) launch_fwd<double, 8>(a, b, total, nseg, A, B, ckpt, w, L, st);
        else launch_fwd<double, 16>(a, b, total, nseg, A, B, ckpt, w, L, st);
    } else {
        if (tile_elems == 1024) launch_fwd<float, 4>(a, b, total, nseg, A, B, ckpt, w, L, st);
        else if (tile_elems == 2048) launch_fwd<float, 8>(a, b, total, nseg, A, B, ckpt, w, L, st);
        else launch_fwd<float, 16>(a, b, total, nseg, A, B, ckpt, w, L, st);
    }
    PVJP_LAUNCHED("pvjp_seg_linrec_scan");
    return PVJP_OK;
}

extern "C" pvjp_status pvjp_seg_batch_vjp(pvjp_dtype dtype, const void* a, const void* b, const void* yA_bar,
                                          const void* yB_bar, int64_t total, int64_t nseg, int tile_elems,
                                          const void* ckpt, void* a_bar, void* b_bar, const void* sum_ybar,
                                          void* sum_xbar, int accumulate, int grid_blocks, void* ws, size_t ws_bytes,
                                          void* stream) {
    clear_error();
    PVJP_REQUIRE(valid_dtype(dtype), "pvjp_seg_batch_vjp: unknown dtype %d", (int)dtype);
    PVJP_REQUIRE(total >= 1 && nseg >= 1, "pvjp_seg_batch_vjp: total and nseg must be >= 1");
    PVJP_REQUIRE(valid_tile(tile_elems), "pvjp_seg_batch_vjp: tile_elems must be 1024, 2048 or 4096");
    const bool scan = a != nullptr;
    PVJP_REQUIRE(!scan || (b && yA_bar && yB_bar && ckpt && a_bar && b_bar),
                 "pvjp_seg_batch_vjp: the scan part needs b, yA_bar, yB_bar, ckpt, a_bar and b_bar");
    PVJP_REQUIRE((sum_ybar == nullptr) == (sum_xbar == nullptr), "pvjp_seg_batch_vjp: sum_ybar and sum_xbar go together");
    PVJP_REQUIRE(scan || sum_ybar, "pvjp_seg_batch_vjp: nothing to compute");
    PVJP_REQUIRE(grid_blocks >= 1 && grid_blocks <= 65536, "pvjp_seg_batch_vjp: grid_blocks out of range [1, 65536]");
    PVJP_REQUIRE(ws != nullptr && aligned(ws, 256), "pvjp_seg_batch_vjp: ws must be non-NULL and 256-byte aligned");
    const SegLayout L = seg_layout(total, nseg, tile_elems);
    if (ws_bytes < L.total) {
        set_error("pvjp_seg_batch_vjp: workspace has %zu bytes, needs %zu", ws_bytes, L.total);
        return PVJP_ENOMEM;
    }
    char* w = reinterpret_cast<char*>(ws);
    hipStream_t st = as_stream(stream);
    if (dtype == PVJP_F64) {
        if (accumulate)
            dispatch_batch<double, true>(tile_elems, a, b, yA_bar, yB_bar, total, nseg, ckpt, a_bar, b_bar, sum_ybar,
                                         sum_xbar, grid_blocks, w, L, st);
        else
            dispatch_batch<double, false>(tile_elems, a, b, yA_bar, yB_bar, total, nseg, ckpt, a_bar, b_bar, sum_ybar,
                                          sum_xbar, grid_blocks, w, L, st);
    } else {
        if (accumulate)
            dispatch_batch<float, true>(tile_elems, a, b, yA_bar, yB_bar, total, nseg, ckpt, a_bar, b_bar, sum_ybar,
                                        sum_xbar, grid_blocks, w, L, st);
        else
            dispatch_batch<float, false>(tile_elems, a, b, yA_bar, yB_bar, total, nseg, ckpt, a_bar, b_bar, sum_ybar,
                                         sum_xbar, grid_blocks, w, L, st);
    }
    PVJP_LAUNCHED("pvjp_seg_batch_vjp");
    return PVJP_OK;
}
