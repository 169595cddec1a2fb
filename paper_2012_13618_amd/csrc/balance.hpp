// Balance step of Algorithm 5 (and the rounds of Algorithm 3) for small
// segments, every round in one launch - and, for the levels at the coarse end
// whose segments are all small, projection, initial bisection, swaps and
// balance of all these levels in one launch (k_seg_levels).
//
// One workgroup per segment keeps the segment's gains and sides in LDS and
// runs the rounds itself: the over-weight side, the ceil(sqrt n) best nodes
// of that side in (gain desc, id asc) order, the shortest prefix covering the
// excess cut back to what the other side can take, the moves, and the gain
// changes they cause, until the segment is balanced or no node can move.
// The gains start from a full computation (Algorithm 4) and follow the moves
// exactly: after a round, every hyperedge with a moved pin is recounted and
// each of its pins' gains changes by the difference of its contributions
// (integer sums, so equal to a recomputation).  Segments are independent, so
// each runs only the rounds it needs; no launch and no host check per round.
//
// Selection inside a round, with each thread's gains in registers: radix
// passes over u = gmax - gain (8-bit digits from the top) narrow the r-th
// node down to a bin; a bin of at most kFuseCand nodes is ranked directly by
// (u, id), a larger one whose nodes share one u by id with one scan.  The
// chosen set is the one the multi-launch path chooses.
#pragma once
#include "uncoarsen.hpp"

namespace bp {

constexpr int kFuseThreads = 1024;
constexpr int32_t kFuseNodes = 8192;                 // nodes of a segment (LDS gains, sides, weights)
constexpr int kFuseItems = kFuseNodes / kFuseThreads;  // per thread, strided
constexpr int32_t kFuseWords = kBins;                // hyperedge bitmap words (shares the histogram)
constexpr int32_t kFuseHedges = kFuseWords * 32;     // hyperedges of a segment
constexpr int kFuseKeys = 128;                       // >= ceil(sqrt(kFuseNodes))
constexpr int kFuseDigit = 8;                        // radix digit of the selection
constexpr int kFuseBins = 1 << kFuseDigit;
constexpr int kFuseSmallDeg = 16;                    // hyperedges up to this degree: a thread each
constexpr int kFuseMidDeg = 64;                      // up to this: 16 lanes each; larger: a wavefront each
constexpr int kFuseQueue = 4096;
constexpr int kFuseCand = 256;                       // bins this small are ranked directly

// Level arrays the rounds read, and the per-segment state they change.
struct FuseArgs {
    const int32_t *off, *pins, *hw, *noff, *inc, *nw, *nbase, *hbase;
    uint8_t *side;
    const int64_t *max0, *max1;
    unsigned long long *segw;
    uint8_t *done;
    int32_t *stuck;
    int32_t *rounds;    // atomicMax of the rounds any segment ran (may be null)
    int32_t max_pins;   // segments with more pins are left to the multi-launch rounds
    // initial bisection only: segments whose coarsest level is `level`, their
    // part counts and total weight
    const int32_t *coarsest, *k0, *k1;
    const int64_t *W;
    int32_t level;
};

// LDS the selection of a list's best nodes works in.
struct PickLds {
    uint32_t *hist;         // kFuseBins
    uint64_t *cand;         // kFuseCand
    int32_t *tcnt;          // ITEMS * TH / 64
    int32_t *ncand;         // zero on entry
    int32_t *sbin;          // [3]
};

// Chooses the r nodes of smallest (u, id) among a list's c nodes, u = gmax -
// gain.  uat(j, u) tells whether item j of this thread (node id j * TH +
// threadIdx.x) is in the list and sets its u; T is the bit length of the
// largest u.  emit(take, u, id) is called with every chosen node once (take
// set), by all lanes of a wavefront together.  Every thread calls; what emit
// writes is complete after the caller's next barrier.
//
// Nodes with u < ulo are chosen, and the rem smallest of "the bin", u in
// [ulo, ulo + 2^lo): by rank when the bin is small (bmode 1), by id when its
// u are all equal (bmode 2).  Radix passes over u (8-bit digits from the top)
// narrow the bin down.
template <int TH, int ITEMS, typename UAt, typename Emit>
__device__ __forceinline__ void pick_best(UAt uat, int32_t r, int32_t c, int T, const PickLds &pl, Emit emit)
{
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    uint64_t ulo = r == c ? ~0ull : 0ull;
    int lo = 0, bmode = 0;
    int32_t rem = 0;
    if (r > 0 && r < c) {
        uint32_t pre = 0;
        rem = r;
        for (int p = 0;; p++) {
            int hi = T - kFuseDigit * p;
            lo = hi - kFuseDigit > 0 ? hi - kFuseDigit : 0;
            if (tid < kFuseBins) pl.hist[tid] = 0;
            __syncthreads();
#pragma unroll
            for (int j = 0; j < ITEMS; j++) {
                uint32_t u = 0;
                bool in = uat(j, u);  // hi <= 24 when p > 0
                bool act = in && (p == 0 || ((u ^ pre) >> hi) == 0);
                lds_hist_add(act, (u >> lo) & ((1u << (hi - lo)) - 1u), pl.hist);
            }
            __syncthreads();
            if (wv == 0) {  // the bin holding the rem-th key: one wavefront
                constexpr int per = kFuseBins / 64;
                int32_t x[per], loc = 0;
#pragma unroll
                for (int j = 0; j < per; j++) {
                    x[j] = (int32_t)pl.hist[lane * per + j];
                    loc += x[j];
                }
                int32_t ex = wave_incl_scan(loc) - loc;
                if (ex < rem && rem <= ex + loc) {
                    int32_t acc = ex;
#pragma unroll
                    for (int j = 0; j < per; j++) {
                        if (acc < rem && rem <= acc + x[j]) {
                            pl.sbin[0] = lane * per + j;
                            pl.sbin[1] = acc;
                            pl.sbin[2] = x[j];
                        }
                        acc += x[j];
                    }
                }
            }
            __syncthreads();
            int32_t bin = pl.sbin[0], left = rem - pl.sbin[1], inb = pl.sbin[2];
            pre |= (uint32_t)bin << lo;
            rem = left;
            ulo = pre;
            if (left == inb) {  // the whole bin
                ulo = (uint64_t)pre + (1ull << lo);
                break;
            }
            if (inb <= kFuseCand) {
                bmode = 1;
                break;
            }
            if (lo == 0) {
                bmode = 2;
                break;
            }
        }
    }

    if (bmode == 1) {
        // the bin's nodes as (u, id) keys; each chosen iff fewer than rem of
        // them are smaller (TH / kFuseCand threads per key)
#pragma unroll
        for (int j = 0; j < ITEMS; j++) {
            uint32_t u = 0;
            bool in = uat(j, u);
            int32_t k = lds_wave_slot(in && (u >> lo) == (uint32_t)(ulo >> lo), pl.ncand);
            if (k >= 0) pl.cand[k] = ((uint64_t)u << 32) | (uint32_t)(j * TH + tid);
        }
        __syncthreads();
        constexpr int tpc = TH / kFuseCand;
        int32_t nc = *pl.ncand, ci = tid / tpc, part = tid % tpc;
        uint64_t x = ci < nc ? pl.cand[ci] : 0ull;
        int32_t rk = 0;
        if (ci < nc) {
#pragma unroll 8
            for (int32_t q = part; q < nc; q += tpc) rk += pl.cand[q] < x;
        }
#pragma unroll
        for (int o = 1; o < tpc; o <<= 1) rk += __shfl_xor(rk, o, 64);
        emit(ci < nc && part == 0 && rk < rem, (uint32_t)(x >> 32), (int32_t)(x & 0xffffffffu));
    } else if (bmode == 2) {
        // the bin's nodes all have u == ulo: the first rem by id (ids ascend
        // with (item j, wavefront, lane))
#pragma unroll
        for (int j = 0; j < ITEMS; j++) {
            uint32_t u = 0;
            bool t = uat(j, u) && u == (uint32_t)ulo;
            unsigned long long b = __ballot(t);
            if (lane == 0) pl.tcnt[j * (TH / 64) + wv] = __popcll(b);
        }
        __syncthreads();
        if (wv == 0) {
            constexpr int nc = ITEMS * (TH / 64), per = nc / 64;
            int32_t v[per], sum = 0;
#pragma unroll
            for (int q = 0; q < per; q++) {
                v[q] = pl.tcnt[lane * per + q];
                sum += v[q];
            }
            int32_t base = wave_incl_scan(sum) - sum;
#pragma unroll
            for (int q = 0; q < per; q++) {
                pl.tcnt[lane * per + q] = base;
                base += v[q];
            }
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < ITEMS; j++) {
            uint32_t u = 0;
            bool t = uat(j, u) && u == (uint32_t)ulo;
            unsigned long long b = __ballot(t);
            emit(t && pl.tcnt[j * (TH / 64) + wv] + __popcll(b & ((1ull << lane) - 1ull)) < rem, u, j * TH + tid);
        }
    }
    // and the nodes below the bin
    if (r > 0) {
#pragma unroll
        for (int j = 0; j < ITEMS; j++) {
            uint32_t u = 0;
            bool in = uat(j, u);
            emit(in && (uint64_t)u < ulo, u, j * TH + tid);
        }
    }
}

// Whether segment s is balanced here (nodes, hyperedges and pins in range).
__device__ __forceinline__ bool fuse_fits(const FuseArgs &fa, int32_t s)
{
    int32_t n = fa.nbase[s + 1] - fa.nbase[s];
    int32_t e0 = fa.hbase[s], ne = fa.hbase[s + 1] - e0;
    int32_t np = fa.off[e0 + ne] - fa.off[e0];
    return n <= kFuseNodes && ne <= kFuseHedges && np <= fa.max_pins;
}

// Gain contributions of hyperedge e to its pins.  full: add the hyperedge's
// contribution (gains start at 0).  Otherwise the pins flagged in mv moved
// from side h to 1 - h in the last round: add new minus old contribution.
// Lanes lane, lane + stride, ... of the hyperedge's pins (stride 1: a thread
// alone, 64: a wavefront).
// The same for d <= R * stride: the pins are loaded once, all in flight
// together, and kept in registers for both the count and the deltas.
template <int R>
__device__ __forceinline__ void fuse_hedge_regs(int32_t e, int32_t b, int32_t d, bool full, int h, int lane,
                                                int stride, int32_t a0, const FuseArgs &fa, const uint8_t *sd,
                                                const uint32_t *mv, int32_t *g)
{
    int32_t u[R];
#pragma unroll
    for (int k = 0; k < R; k++) u[k] = fa.pins[b + min(lane + k * stride, d - 1)] - a0;
    int32_t n1 = 0, km = 0;
#pragma unroll
    for (int k = 0; k < R; k++)
        if (lane + k * stride < d) {
            n1 += sd[u[k]];
            if (!full) km += (mv[u[k] >> 5] >> (u[k] & 31)) & 1;
        }
    if (stride > 1) {
        n1 = wave_sum(n1);
        km = wave_sum(km);
    }
    int32_t w = fa.hw[e];
    int2 cn = hedge_contrib_value(w, d, n1);
    int2 co = make_int2(0, 0);
    if (!full) {
        if (km == 0) return;
        co = hedge_contrib_value(w, d, h ? n1 + km : n1 - km);
    }
#pragma unroll
    for (int k = 0; k < R; k++) {
        if (lane + k * stride >= d) continue;
        int sn = sd[u[k]];
        int so = full ? sn : (sn ^ (int)((mv[u[k] >> 5] >> (u[k] & 31)) & 1));
        int32_t delta = (sn ? cn.y : cn.x) - (full ? 0 : (so ? co.y : co.x));
        if (delta) atomicAdd(&g[u[k]], delta);
    }
}

__device__ __forceinline__ void fuse_hedge(int32_t e, bool full, int h, int lane, int stride, int32_t a0,
                                           const FuseArgs &fa, const uint8_t *sd, const uint32_t *mv,
                                           int32_t *g)
{
    int32_t b = fa.off[e], d = fa.off[e + 1] - b;
    // pins in registers when few (a thread: up to 4, or up to kFuseSmallDeg;
    // a wavefront: up to 512)
    if (stride == 1 && d <= kFuseSmallDeg) {
        if (__ballot(d > 4) == 0) fuse_hedge_regs<4>(e, b, d, full, h, lane, 1, a0, fa, sd, mv, g);
        else fuse_hedge_regs<kFuseSmallDeg>(e, b, d, full, h, lane, 1, a0, fa, sd, mv, g);
        return;
    }
    if (stride == 64 && d <= 512) {
        fuse_hedge_regs<8>(e, b, d, full, h, lane, 64, a0, fa, sd, mv, g);
        return;
    }
    int32_t n1 = 0, km = 0;
#pragma unroll 4
    for (int32_t i = lane; i < d; i += stride) {
        int32_t u = fa.pins[b + i] - a0;
        n1 += sd[u];
        if (!full) km += (mv[u >> 5] >> (u & 31)) & 1;
    }
    if (stride > 1) {
        n1 = wave_sum(n1);
        km = wave_sum(km);
    }
    int32_t w = fa.hw[e];
    int2 cn = hedge_contrib_value(w, d, n1);
    int2 co = make_int2(0, 0);
    if (!full) {
        if (km == 0) return;
        co = hedge_contrib_value(w, d, h ? n1 + km : n1 - km);
    }
#pragma unroll 4
    for (int32_t i = lane; i < d; i += stride) {
        int32_t u = fa.pins[b + i] - a0;
        int sn = sd[u];
        int so = full ? sn : (sn ^ (int)((mv[u >> 5] >> (u & 31)) & 1));
        int32_t delta = (sn ? cn.y : cn.x) - (full ? 0 : (so ? co.y : co.x));
        if (delta) atomicAdd(&g[u], delta);
    }
}

// The same for d <= kFuseMidDeg by 16 lanes (sub: the lane's place among them,
// 4 pins each); on: whether these lanes have a hyperedge.
__device__ __forceinline__ void fuse_hedge16(bool on, int32_t e, bool full, int h, int sub, int32_t a0,
                                             const FuseArgs &fa, const uint8_t *sd, const uint32_t *mv, int32_t *g)
{
    constexpr int R = kFuseMidDeg / 16;
    int32_t b = 0, d = 0, w = 0, u[R], n1 = 0, km = 0;
    if (on) {
        b = fa.off[e];
        d = fa.off[e + 1] - b;
        w = fa.hw[e];
#pragma unroll
        for (int k = 0; k < R; k++) u[k] = fa.pins[b + min(sub + 16 * k, d - 1)] - a0;
#pragma unroll
        for (int k = 0; k < R; k++)
            if (sub + 16 * k < d) {
                n1 += sd[u[k]];
                if (!full) km += (mv[u[k] >> 5] >> (u[k] & 31)) & 1;
            }
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) {
        n1 += __shfl_xor(n1, o, 64);
        if (!full) km += __shfl_xor(km, o, 64);
    }
    if (!on || (!full && km == 0)) return;
    const int2 cn = hedge_contrib_value(w, d, n1);
    const int2 co = full ? make_int2(0, 0) : hedge_contrib_value(w, d, h ? n1 + km : n1 - km);
#pragma unroll
    for (int k = 0; k < R; k++) {
        if (sub + 16 * k >= d) continue;
        const int sn = sd[u[k]], so = full ? sn : (sn ^ (int)((mv[u[k] >> 5] >> (u[k] & 31)) & 1));
        const int32_t delta = (sn ? cn.y : cn.x) - (so ? co.y : co.x);
        if (delta) atomicAdd(&g[u[k]], delta);
    }
}

// LDS of the kernels below: one segment's state.
struct FuseShared {
    int32_t g[kFuseNodes], nwl[kFuseNodes], noffl[kFuseNodes + 1];
    uint8_t sd[kFuseNodes];
    uint32_t mv[kFuseNodes / 32];
    uint32_t work[kFuseWords];  // radix histogram, then the hyperedge bitmap
    uint64_t keys[kFuseKeys], sorted[kFuseKeys];
    int32_t dpre[kFuseKeys + 1];
    int32_t queue[kFuseQueue];
    int32_t tcnt[kFuseItems * (kFuseThreads / 64)];
    int32_t red[kFuseThreads / 64][6];
    int64_t lds64[16], w01[2];
    uint64_t cand[kFuseCand];
    int32_t qt, qn, qh, nkeys, ncand, sbin[3], np_s;  // queue: entries, mid ones (from the front), large ones (from the back)
};

// A segment of one level: its nodes a0 .. a0 + n and hyperedges e0 .. e0 + ne.
struct FuseSeg {
    int32_t a0, n, e0, ne;
};

// A thread's hyperedge in flight: its bounds and weight, and up to
// kFuseSmallDeg pins (as many as the wavefront's largest such hyperedge has, in
// steps of 4, 8 and 16).
struct FuseHedge {
    int32_t b, d, w, u[kFuseSmallDeg];
    int steps;  // the same in every lane of a wavefront

    __device__ __forceinline__ void bounds(const FuseArgs &fa, const FuseSeg &q, int32_t i)
    {
        b = d = w = 0;
        if (i >= q.ne) return;
        const int32_t e = q.e0 + i;
        b = fa.off[e];
        d = fa.off[e + 1] - b;
        w = fa.hw[e];
    }
    template <int K0, int K1> __device__ __forceinline__ void load(const FuseArgs &fa)
    {
#pragma unroll
        for (int k = K0; k < K1; k++) u[k] = fa.pins[b + min(k, d - 1)];
    }
    __device__ __forceinline__ void pins(const FuseArgs &fa)
    {
        const bool in = d > 0 && d <= kFuseSmallDeg;
        steps = __ballot(in && d > 8) ? 16 : (__ballot(in && d > 4) ? 8 : 4);
        if (!in) return;
        load<0, 4>(fa);
        if (steps > 4) load<4, 8>(fa);
        if (steps > 8) load<8, 16>(fa);
    }
    template <int R> __device__ __forceinline__ void add(int32_t a0, FuseShared &sh) const
    {
        uint32_t s = 0;  // bit k: pin k's side
#pragma unroll
        for (int k = 0; k < R; k++)
            if (k < d) s |= (uint32_t)sh.sd[u[k] - a0] << k;
        const int2 c = hedge_contrib_value(w, d, __popc(s));
        if (c.x == 0 && c.y == 0) return;
#pragma unroll
        for (int k = 0; k < R; k++) {
            const int32_t delta = (s >> k) & 1 ? c.y : c.x;
            if (k < d && delta) atomicAdd(&sh.g[u[k] - a0], delta);
        }
    }
};

__device__ __forceinline__ void fuse_queue_reset(FuseShared &sh)
{
    sh.qt = 0;
    sh.qn = 0;
    sh.qh = 0;
}

// Queues hyperedge e of d > kFuseSmallDeg pins; false when the queue is full.
__device__ __forceinline__ bool fuse_queue(int32_t e, int32_t d, FuseShared &sh)
{
    if (atomicAdd(&sh.qt, 1) >= kFuseQueue) return false;
    const int32_t k = d <= kFuseMidDeg ? atomicAdd(&sh.qn, 1) : kFuseQueue - 1 - atomicAdd(&sh.qh, 1);
    sh.queue[k] = e;
    return true;
}

// The queued hyperedges (a barrier before and after).
__device__ __forceinline__ void fuse_queue_run(bool full, int h, int32_t a0, const FuseArgs &fa, FuseShared &sh)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int32_t n = sh.qn;
    for (int32_t k = 4 * wv; k < n; k += kFuseThreads / 16) {
        const int32_t i = k + (lane >> 4);
        fuse_hedge16(i < n, sh.queue[min(i, n - 1)], full, h, lane & 15, a0, fa, sh.sd, sh.mv, sh.g);
    }
    for (int32_t k = wv; k < sh.qh; k += kFuseThreads / 64)
        fuse_hedge(sh.queue[kFuseQueue - 1 - k], full, h, lane, 64, a0, fa, sh.sd, sh.mv, sh.g);
}

// Every gain of the segment, hyperedge by hyperedge (large ones 16 lanes or one
// wavefront each).  A thread's next hyperedge's pins and the bounds of the one after are
// loaded while it works on one, so that an iteration waits for one memory
// round trip and not three.  (One that a full queue left to its thread held all
// others up: netlist segments of 126 K pins spent 200 us a pass that way.)  Ends
// with a barrier.
__device__ __forceinline__ void fuse_gains(const FuseArgs &fa, const FuseSeg &q, FuseShared &sh)
{
    const int tid = threadIdx.x;
    FuseHedge cur, nxt;
    cur.bounds(fa, q, tid);
    nxt.bounds(fa, q, tid + kFuseThreads);
    for (int32_t i = tid; i < q.n; i += kFuseThreads) sh.g[i] = 0;
    if (tid == 0) fuse_queue_reset(sh);
    cur.pins(fa);
    __syncthreads();
    for (int32_t base = 0; base < q.ne; base += kFuseThreads) {
        FuseHedge nn;
        nn.bounds(fa, q, base + 2 * kFuseThreads + tid);
        nxt.pins(fa);
        if (cur.d > kFuseSmallDeg) {
            const int32_t e = q.e0 + base + tid;
            if (!fuse_queue(e, cur.d, sh)) fuse_hedge(e, true, 0, 0, 1, q.a0, fa, sh.sd, sh.mv, sh.g);
        } else if (cur.d > 0) {
            if (cur.steps == 4) cur.add<4>(q.a0, sh);
            else if (cur.steps == 8) cur.add<8>(q.a0, sh);
            else cur.add<16>(q.a0, sh);
        }
        cur = nxt;
        nxt.b = nn.b;
        nxt.d = nn.d;
        nxt.w = nn.w;
    }
    __syncthreads();
    fuse_queue_run(true, 0, q.a0, fa, sh);
    __syncthreads();
}

// The rounds of a balance step on the gains in sh.g, which they keep up to
// date; w01 holds the side weights.  fa.side (nullable) receives the moves.
// INIT: the rounds of Algorithm 3 instead (segments at their coarsest level,
// all nodes starting on side 1): while side 0 is below its share W k0 / (k0 +
// k1) and side 1 has nodes, move the ceil(sqrt n) best nodes of side 1 to side
// 0 (all of them, no prefix).  Returns the rounds run.
template <bool INIT>
__device__ __forceinline__ int32_t fuse_rounds(int32_t s, const FuseArgs &fa, const FuseSeg &sg, FuseShared &sh)
{
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int32_t a0 = sg.a0, n = sg.n, e0 = sg.e0, ne = sg.ne;
    const int32_t m = (int32_t)ceil_sqrt_i64(n);
    const int64_t mx0 = INIT ? 0 : fa.max0[s], mx1 = INIT ? 0 : fa.max1[s];
    const int64_t ks = INIT ? (int64_t)fa.k0[s] + fa.k1[s] : 0, Wk0 = INIT ? fa.W[s] * (int64_t)fa.k0[s] : 0;
    int32_t *g = sh.g, *nwl = sh.nwl, *noffl = sh.noffl, *queue = sh.queue, *dpre = sh.dpre;
    uint8_t *sd = sh.sd;
    uint32_t *mv = sh.mv, *work = sh.work;
    uint64_t *keys = sh.keys, *sorted = sh.sorted;
    int32_t rounds = 0;
    for (;;) {
        // the side over its bound, the excess and the room
        int64_t w0 = sh.w01[0], w1 = sh.w01[1];
        int h = INIT ? 1 : (w0 > mx0 ? 0 : (w1 > mx1 ? 1 : -1));
        if (h < 0) break;
        if (rounds > n) {  // never: each round moves a node for good, so <= n rounds
            if (tid == 0 && !INIT) fa.stuck[s] = 1;
            break;
        }

        // this thread's nodes (ids j * kFuseThreads + tid): gains in registers,
        // bit j of `on` = node on side h
        int32_t gi[kFuseItems];
        uint32_t on = 0;
#pragma unroll
        for (int j = 0; j < kFuseItems; j++) {
            int32_t i = j * kFuseThreads + tid;
            gi[j] = 0;
            if (i < n) {
                gi[j] = g[i];
                if (sd[i] == h) on |= 1u << j;
            }
        }
        // list h: size and gain extremes
        int32_t c = __popc(on), gmax = INT32_MIN, gmin = INT32_MAX;
#pragma unroll
        for (int j = 0; j < kFuseItems; j++)
            if ((on >> j) & 1) {
                gmax = max(gmax, gi[j]);
                gmin = min(gmin, gi[j]);
            }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            c += __shfl_xor(c, o, 64);
            gmax = max(gmax, __shfl_xor(gmax, o, 64));
            gmin = min(gmin, __shfl_xor(gmin, o, 64));
        }
        if (lane == 0) {
            sh.red[wv][0] = c;
            sh.red[wv][1] = gmax;
            sh.red[wv][2] = gmin;
        }
        if (tid == 0) {
            fuse_queue_reset(sh);
            sh.nkeys = 0;
            sh.ncand = 0;
        }
        __syncthreads();
        c = 0;
        gmax = INT32_MIN;
        gmin = INT32_MAX;
#pragma unroll
        for (int w = 0; w < kFuseThreads / 64; w++) {
            c += sh.red[w][0];
            gmax = max(gmax, sh.red[w][1]);
            gmin = min(gmin, sh.red[w][2]);
        }
        if (INIT && !(w0 * ks < Wk0 && c > 0)) break;  // Algorithm 3's loop test
        rounds++;
        int32_t r = c < m ? c : m;
        // from here on the registers hold u = gmax - gain
#pragma unroll
        for (int j = 0; j < kFuseItems; j++) gi[j] = (int32_t)(uint32_t)((int64_t)gmax - gi[j]);

        PickLds pl{work, sh.cand, sh.tcnt, &sh.ncand, sh.sbin};
        pick_best<kFuseThreads, kFuseItems>(
            [=](int j, uint32_t &u) -> bool {
                u = (uint32_t)gi[j];
                return (on >> j) & 1;
            },
            r, c, bitlen_u32((uint32_t)((int64_t)gmax - gmin)), pl, [&](bool take, uint32_t u, int32_t id) {
                int32_t k = lds_wave_slot(take, &sh.nkeys);
                if (k >= 0)
                    keys[k & (kFuseKeys - 1)] = gain_order_key((int32_t)((int64_t)gmax - u), (uint32_t)(a0 + id));
            });
        __syncthreads();
        int32_t cnt = min(sh.nkeys, kFuseKeys);  // r of them
        // the moving nodes: all chosen ones (INIT), else a prefix in order
        const uint64_t *mlist = INIT ? keys : sorted;
        if (!INIT) block_rank_sort(keys, sorted, cnt);

        // prefix, moves and side weights (one wavefront)
        if (wv == 0) {
            int64_t need = h ? w1 - mx1 : w0 - mx0, room = h ? mx0 - w0 : mx1 - w1;
            int32_t p1 = cnt, fit = INIT ? cnt : 0;
            int64_t carry = 0;
            for (int32_t base = 0; !INIT && base < cnt; base += 64) {
                int32_t i = base + lane;
                int64_t w = i < cnt ? (int64_t)nwl[(uint32_t)(sorted[i] & 0xffffffffu) - a0] : 0;
                int64_t incl = wave_incl_scan(w) + carry;
                unsigned long long hit = __ballot(i < cnt && incl >= need);
                fit += __popcll(__ballot(i < cnt && incl <= room));
                if (hit) {
                    p1 = base + __ffsll((long long)hit);
                    break;
                }
                carry = __shfl(incl, 63, 64);
            }
            int32_t p = fit < p1 ? fit : p1;
            int64_t moved = 0;
            int32_t dcarry = 0;
            for (int32_t base = 0; base < p; base += 64) {
                int32_t i = base + lane;
                int32_t deg = 0;
                if (i < p) {
                    int32_t v = (int32_t)(uint32_t)(mlist[i] & 0xffffffffu), u = v - a0;
                    sd[u] = (uint8_t)(1 - h);
                    if (fa.side) fa.side[v] = (uint8_t)(1 - h);
                    atomicOr(&mv[u >> 5], 1u << (u & 31));
                    moved += nwl[u];
                    deg = noffl[u + 1] - noffl[u];
                }
                int32_t incl = wave_incl_scan(deg) + dcarry;
                if (i < p) dpre[i + 1] = incl;
                dcarry = __shfl(incl, 63, 64);
            }
            moved = wave_sum(moved);
            if (lane == 0) {
                dpre[0] = 0;
                sh.np_s = p;
                if (p > 0) {
                    sh.w01[h] -= moved;
                    sh.w01[1 - h] += moved;
                }
            }
        }
        __syncthreads();
        int32_t p = sh.np_s;
        if (p == 0) {
            if (tid == 0 && !INIT) fa.stuck[s] = 1;
            break;
        }

        int32_t D = dpre[p];
        if (D >= ne / 2) {
            // the moved nodes touch so many hyperedges that all gains again cost
            // less: 1024 hyperedges a memory round trip against 1024 incidences
            // in four
            for (int32_t i = tid; i < p; i += kFuseThreads) {
                int32_t u = (int32_t)(uint32_t)(mlist[i] & 0xffffffffu) - a0;
                atomicAnd(&mv[u >> 5], ~(1u << (u & 31)));
            }
            fuse_gains(fa, sg, sh);
            continue;
        }
        // mark the moved nodes' hyperedges, then update their pins' gains
        int32_t nwords = (ne + 31) >> 5;
        for (int32_t i = tid; i < nwords; i += kFuseThreads) work[i] = 0;
        __syncthreads();
        // one thread per incidence of a moved node; the thread that marks a
        // hyperedge first updates it (the moves are all made, so its counts
        // are final), large ones queued for a wavefront
        for (int32_t t = tid; t < D; t += kFuseThreads) {
            int32_t lo = 0, hi = p;  // dpre[lo] <= t < dpre[hi]
            while (hi - lo > 1) {
                int32_t mid = (lo + hi) >> 1;
                if (dpre[mid] <= t) lo = mid;
                else hi = mid;
            }
            int32_t u = (int32_t)(uint32_t)(mlist[lo] & 0xffffffffu) - a0;
            int32_t x = fa.inc[noffl[u] + (t - dpre[lo])] - e0;
            uint32_t bit = 1u << (x & 31);
            if (atomicOr(&work[x >> 5], bit) & bit) continue;
            int32_t e = e0 + x;
            const int32_t d = fa.off[e + 1] - fa.off[e];
            if (d > kFuseSmallDeg && fuse_queue(e, d, sh)) continue;
            fuse_hedge(e, false, h, 0, 1, a0, fa, sd, mv, g);
        }
        __syncthreads();
        fuse_queue_run(false, h, a0, fa, sh);
        __syncthreads();
        // the move marks are spent
        for (int32_t i = tid; i < p; i += kFuseThreads) {
            int32_t u = (int32_t)(uint32_t)(mlist[i] & 0xffffffffu) - a0;
            atomicAnd(&mv[u >> 5], ~(1u << (u & 31)));
        }
        __syncthreads();
    }
    return rounds;
}

template <bool INIT>
__global__ __launch_bounds__(kFuseThreads) void k_seg_fused(int32_t S, FuseArgs fa)
{
    __shared__ FuseShared sh;
    int32_t s = blockIdx.x;
    if (s >= S || (INIT ? fa.coarsest[s] != fa.level : fa.done[s] != 0) || !fuse_fits(fa, s)) return;
    const int tid = threadIdx.x;
    const FuseSeg q{fa.nbase[s], fa.nbase[s + 1] - fa.nbase[s], fa.hbase[s], fa.hbase[s + 1] - fa.hbase[s]};
    for (int32_t i = tid; i < q.n; i += kFuseThreads) {
        sh.sd[i] = fa.side[q.a0 + i];
        sh.nwl[i] = fa.nw[q.a0 + i];
        sh.noffl[i] = fa.noff[q.a0 + i];
    }
    if (tid == 0) sh.noffl[q.n] = fa.noff[q.a0 + q.n];
    for (int32_t i = tid; i < kFuseNodes / 32; i += kFuseThreads) sh.mv[i] = 0;
    if (tid == 0) {
        sh.w01[0] = (int64_t)fa.segw[2 * s];
        sh.w01[1] = (int64_t)fa.segw[2 * s + 1];
    }
    __syncthreads();
    // (a balanced segment needs no gains)
    const int64_t w0 = sh.w01[0], w1 = sh.w01[1];
    int32_t rounds = 0;
    if (INIT || w0 > fa.max0[s] || w1 > fa.max1[s]) {
        fuse_gains(fa, q, sh);
        rounds = fuse_rounds<INIT>(s, fa, q, sh);
    }
    if (tid == 0) {
        fa.segw[2 * s] = (unsigned long long)sh.w01[0];
        fa.segw[2 * s + 1] = (unsigned long long)sh.w01[1];
        if (!INIT) fa.done[s] = 1;
        if (fa.rounds) atomicMax(fa.rounds, rounds);
    }
}

// One swap of Algorithm 5 on the gains in sh.g: the best min(|L0|, |L1|) nodes
// of non-negative gain of each side change sides.  The gains are spent.
__device__ __forceinline__ void fuse_swap(const FuseSeg &q, FuseShared &sh)
{
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    int32_t gi[kFuseItems];
    uint32_t on[2] = {0, 0};
    int32_t x[6] = {0, 0, INT32_MIN, INT32_MIN, INT32_MAX, INT32_MAX};  // per list: size, largest, smallest gain
#pragma unroll
    for (int j = 0; j < kFuseItems; j++) {
        int32_t i = j * kFuseThreads + tid;
        gi[j] = i < q.n ? sh.g[i] : -1;
        if (gi[j] < 0) continue;
        int h = sh.sd[i];
        if (h) {
            on[1] |= 1u << j;
            x[1]++;
            x[3] = max(x[3], gi[j]);
            x[5] = min(x[5], gi[j]);
        } else {
            on[0] |= 1u << j;
            x[0]++;
            x[2] = max(x[2], gi[j]);
            x[4] = min(x[4], gi[j]);
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        x[0] += __shfl_xor(x[0], o, 64);
        x[1] += __shfl_xor(x[1], o, 64);
        x[2] = max(x[2], __shfl_xor(x[2], o, 64));
        x[3] = max(x[3], __shfl_xor(x[3], o, 64));
        x[4] = min(x[4], __shfl_xor(x[4], o, 64));
        x[5] = min(x[5], __shfl_xor(x[5], o, 64));
    }
    if (lane == 0)
        for (int k = 0; k < 6; k++) sh.red[wv][k] = x[k];
    __syncthreads();
    for (int k = 0; k < 6; k++) {
        x[k] = sh.red[0][k];
        for (int w = 1; w < kFuseThreads / 64; w++)
            x[k] = k < 2 ? x[k] + sh.red[w][k] : (k < 4 ? max(x[k], sh.red[w][k]) : min(x[k], sh.red[w][k]));
    }
    const int32_t r = min(x[0], x[1]);
    if (r == 0) return;  // (the same in every thread)
    int64_t d01 = 0;     // weight moving from side 0 to side 1
    for (int h = 0; h < 2; h++) {
        __syncthreads();
        if (tid == 0) sh.ncand = 0;
        __syncthreads();
        const int32_t gmax = h ? x[3] : x[2], gmin = h ? x[5] : x[4], c = h ? x[1] : x[0];
        const uint32_t mine = h ? on[1] : on[0];
        PickLds pl{sh.work, sh.cand, sh.tcnt, &sh.ncand, sh.sbin};
        pick_best<kFuseThreads, kFuseItems>(
            [=](int j, uint32_t &u) -> bool {
                u = (uint32_t)gmax - (uint32_t)gi[j];
                return (mine >> j) & 1;
            },
            r, c, bitlen_u32((uint32_t)gmax - (uint32_t)gmin), pl, [&](bool take, uint32_t, int32_t id) {
                if (!take) return;
                sh.sd[id] = (uint8_t)(1 - h);
                d01 += h ? -(int64_t)sh.nwl[id] : (int64_t)sh.nwl[id];
            });
    }
    d01 = block_sum(d01, sh.lds64);
    if (tid == 0) {
        sh.w01[0] -= d01;
        sh.w01[1] += d01;
    }
    __syncthreads();
}

// Levels `top` down to `bottom` of every segment that starts at one of them
// (the levels' segments all fit), one workgroup a segment: at its coarsest
// level the initial bisection, at the finer ones the projection, then the swaps
// and the balance step.  The sides stay in LDS; the bottom level's are written
// out.  Launch after launch over such levels costs their latency a dozen times
// per level: 1 K nodes of 10 K pins, 4 levels, a whole bisection 1.03 ms by
// launches and 0.90 this way.  Up to kFuseLevelPins pins a segment, as one
// workgroup takes the full gain passes slower than the whole chip does: limits
// of 0, 49152, 65536, 98304 and 131072 gave 12 K nodes k=5 4.48, 4.45, 4.40,
// 4.52, 4.51 ms, a 41 K-node netlist 4.63, 4.61, 4.60, 4.69, 4.79.
constexpr int kFuseLevels = 8;  // levels of a launch
constexpr int32_t kFuseLevelPins = 65536;
struct FuseLevel {
    const int32_t *off, *pins, *hw, *noff, *inc, *nw, *nbase, *hbase, *parent;
};
struct FuseLevelsArgs {
    FuseLevel lv[kFuseLevels];  // lv[j - bottom]
    int32_t S, top, bottom, iters;
    uint8_t *side;              // of the bottom level
    const uint8_t *side_in;     // of level top + 1, for segments that started above (or null)
    const int32_t *nbase_in;    // that level's
    FuseArgs fa;                // the segments' state
};

__global__ __launch_bounds__(kFuseThreads) void k_seg_levels(FuseLevelsArgs a)
{
    __shared__ FuseShared sh;
    __shared__ uint8_t above[kFuseNodes];  // the coarser level's sides
    const int32_t s = blockIdx.x;
    const int tid = threadIdx.x;
    const int32_t c = a.fa.coarsest[s];
    if (c < a.bottom) return;
    int32_t rounds = 0, ca0 = 0;
    for (int32_t i = tid; i < kFuseNodes / 32; i += kFuseThreads) sh.mv[i] = 0;
    if (c > a.top) {
        ca0 = a.nbase_in[s];
        const int32_t n = a.nbase_in[s + 1] - ca0;
        for (int32_t i = tid; i < n; i += kFuseThreads) sh.sd[i] = a.side_in[ca0 + i];
    }
    for (int32_t j = min(c, a.top); j >= a.bottom; j--) {
        const FuseLevel &L = a.lv[j - a.bottom];
        FuseArgs fa = a.fa;
        fa.off = L.off;
        fa.pins = L.pins;
        fa.hw = L.hw;
        fa.noff = L.noff;
        fa.inc = L.inc;
        fa.side = nullptr;
        const FuseSeg q{L.nbase[s], L.nbase[s + 1] - L.nbase[s], L.hbase[s], L.hbase[s + 1] - L.hbase[s]};
        __syncthreads();
        for (int32_t i = tid; i < kFuseNodes; i += kFuseThreads) above[i] = sh.sd[i];
        __syncthreads();
        int64_t w0 = 0, w1 = 0;
        for (int32_t i = tid; i < q.n; i += kFuseThreads) {
            const int32_t w = L.nw[q.a0 + i];
            const uint8_t sd = j == c ? 1 : above[L.parent[q.a0 + i] - ca0];
            sh.sd[i] = sd;
            sh.nwl[i] = w;
            sh.noffl[i] = L.noff[q.a0 + i];
            if (sd) w1 += w;
            else w0 += w;
        }
        if (tid == 0) sh.noffl[q.n] = L.noff[q.a0 + q.n];
        w0 = block_sum(w0, sh.lds64);
        w1 = block_sum(w1, sh.lds64);
        if (tid == 0) {
            sh.w01[0] = w0;
            sh.w01[1] = w1;
        }
        __syncthreads();
        bool fresh = false;  // the gains in sh.g are those of the sides
        if (j == c) {
            fuse_gains(fa, q, sh);
            rounds = max(rounds, fuse_rounds<true>(s, fa, q, sh));
            __syncthreads();
            fresh = true;
        }
        for (int it = 0; it < a.iters; it++) {
            if (!fresh) fuse_gains(fa, q, sh);
            fuse_swap(q, sh);
            fresh = false;
        }
        __syncthreads();
        if (sh.w01[0] > fa.max0[s] || sh.w01[1] > fa.max1[s]) {
            if (!fresh) fuse_gains(fa, q, sh);
            rounds = max(rounds, fuse_rounds<false>(s, fa, q, sh));
        }
        ca0 = q.a0;
        __syncthreads();
        if (j == a.bottom)
            for (int32_t i = tid; i < q.n; i += kFuseThreads) a.side[q.a0 + i] = sh.sd[i];
    }
    if (tid == 0) {
        a.fa.segw[2 * s] = (unsigned long long)sh.w01[0];
        a.fa.segw[2 * s + 1] = (unsigned long long)sh.w01[1];
        if (a.fa.rounds) atomicMax(a.fa.rounds, rounds);
    }
}

}  // namespace bp
