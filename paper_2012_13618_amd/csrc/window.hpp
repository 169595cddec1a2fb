// Balance rounds (Algorithm 5) of segments too large for one workgroup, without
// sorting or gathering candidates.
//
// A round moves the shortest prefix, in (gain desc, id asc) order, of the heavy
// side's nodes that removes the excess, at most ceil(sqrt n) nodes and no more
// than the other side can take.  Whether the node at position i moves depends
// only on the count and the weight before it: i <= ceil(sqrt n), weight before
// < excess, weight through it <= room.  So it is enough to know, per gain
// value, how many nodes and how much weight stand before:
//
//  k_win_hist  every chunk of a segment counts its heavy side's nodes and
//              weight per bin of a window of gain values, for itself (rows)
//              and for the segment (tot).
//  k_win_take  every chunk finds the one bin that moves in part: the bins before
//              it move whole, the ones after it not at all.  In that bin the
//              chunk starts from the earlier chunks' rows and takes its nodes
//              in id order.  Each chunk moves and logs its own nodes.
//
// The window is kWinBins - 2 bins of 2^shift gain values below `top`, one bin
// for all gains above and one for all below.  A bin taken in part has to hold
// one gain value; when it does not, the round moves nothing but the window
// (towards that bin, finer or further out) and the next round counts again.
// Gains change little from round to round, so at one value per bin the window
// nearly always holds the bin sought: the two launches are the selection.
//
// What bounds a round is the latency of its four dependent launches (test and
// marking, gain update, and these two); the selection that this replaces kept
// ceil(n / 16384) workgroups at 31 us a round (chunk lists sorted and merged)
// on segments of 133 K nodes, these two launches take 5.5 and 9.3 us (a round of
// such a segment 45 -> 31 us with tiles of 2048 nodes, 28 with tiles of 1024).
#pragma once
#include "uncoarsen.hpp"

namespace bp {

constexpr int kWinBins = 1024;
constexpr int kWinAbove = 0, kWinBelow = kWinBins - 1;
constexpr int kWinItems = 4;  // (nodes a thread: 8, 4 and 2 gave 4 M column-nets k=8 92.5, 86.7 and 87.2 ms)
constexpr int32_t kWinTile = kBlock * kWinItems;  // nodes a workgroup takes at a time
constexpr int32_t kWinChunks = 512;               // chunks of a segment at most (same-bin atomics: 11 ns each)
constexpr int64_t kWinTotal = 2048;               // chunks of a level, about
constexpr int32_t kWinStart = 511;                // top of the first window
constexpr int32_t kWinBig = 64;                   // moved nodes logged by the whole workgroup

// nodes a chunk holds: whole tiles
inline int32_t win_chunk_nodes(int64_t maxseg, int64_t N)
{
    int64_t t = std::max(ceil_div(maxseg, (int64_t)kWinTile * kWinChunks), ceil_div(N, (int64_t)kWinTile * kWinTotal));
    return (int32_t)(std::max<int64_t>(t, 1) * kWinTile);
}

// chunks of a level at most
inline int64_t win_chunks(const Level &L)
{
    return ceil_div(L.N, win_chunk_nodes(L.maxseg_nodes, L.N)) + L.S;
}

struct WinArgs {
    int32_t S, N;  // segments, nodes of the level
    const int4 *tab;
    const int32_t *gain, *nw, *m;
    const uint8_t *mode;
    uint8_t *side;
    const int64_t *need, *room;
    unsigned long long *segw;
    WinState win;
    MoveLog ml;
    int32_t cur, nxt;  // window and histogram slots of this round and the next
    const int32_t *go;
};

__device__ __forceinline__ int win_bin(int32_t gain, int32_t top, int32_t shift)
{
    if (gain > top) return kWinAbove;
    uint32_t q = ((uint32_t)top - (uint32_t)gain) >> shift;
    return q >= (uint32_t)(kWinBins - 2) ? kWinBelow : 1 + (int)q;
}

// The chunk table of a level - segment, first node, nodes, the segment's first
// chunk; up to `bound` entries, the ones past the last chunk without nodes -
// and its first window, the last one of the level before.  The entries are
// shared out over the threads, kWinTabSegs segments at a time: written by a
// thread a segment they took 20 us for one of 1 M nodes (2 now).
constexpr int kWinTabSegs = 1024;
__global__ __launch_bounds__(kWinTabSegs) void k_win_table(int32_t S, int32_t cn, const int32_t *nbase, int64_t bound,
                                                           WinState win)
{
    __shared__ int32_t lds[16], first[kWinTabSegs], node[kWinTabSegs];  // of each segment: its first chunk, its first node
    const int tid = threadIdx.x;
    int32_t carry = 0;
    for (int32_t base = 0; base < S; base += kWinTabSegs) {
        const int32_t s = base + tid, a = s < S ? nbase[s] : 0, n = s < S ? nbase[s + 1] - a : 0;
        int32_t tot;
        const int32_t at = block_excl_scan((n + cn - 1) / cn, lds, &tot) + carry;
        first[tid] = at;
        node[tid] = a;
        if (s < S) {
            win.top[s] = win.top[3 * S + s];
            win.shift[s] = win.shift[3 * S + s];
        }
        __syncthreads();
        for (int32_t i = carry + tid; i < carry + tot; i += kWinTabSegs) {
            int lo = 0, hi = kWinTabSegs;  // the last segment that starts at chunk i or before (empty ones start where the next does)
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (first[mid] <= i) lo = mid;
                else hi = mid;
            }
            const int32_t b = node[lo] + (i - first[lo]) * cn;
            win.tab[i] = make_int4(base + lo, b, min(nbase[base + lo + 1] - b, cn), first[lo]);
        }
        carry += tot;
        __syncthreads();
    }
    for (int64_t i = carry + tid; i < bound; i += kWinTabSegs) win.tab[i] = make_int4(0, 0, 0, 0);
}

// A thread's nodes of a tile: gains, sides and weights, loaded together (past
// the level's end: its last node).  STRIDED: one node in kBlock, else
// kWinItems consecutive ones.
struct WinNodes {
    int32_t g[kWinItems], w[kWinItems];
    uint8_t sd[kWinItems];
    template <bool STRIDED> __device__ __forceinline__ void load(const WinArgs &a, int32_t first)
    {
#pragma unroll
        for (int j = 0; j < kWinItems; j++) {
            const int32_t i = STRIDED ? j * kBlock + (int32_t)threadIdx.x : (int32_t)threadIdx.x * kWinItems + j;
            const int32_t v = min(first + i, a.N - 1);
            g[j] = a.gain[v];
            sd[j] = a.side[v];
            w[j] = a.nw[v];
        }
    }
};

__global__ __launch_bounds__(kBlock) void k_win_hist(WinArgs a)
{
    __shared__ unsigned long long h[kWinBins];  // nodes << 32 | weight (a weight sum stays below 2^31)
    const int32_t ci = blockIdx.x;
    const int32_t gv = *a.go;
    const int4 t = a.tab[ci];
    const int32_t s = t.x, a0 = t.y, n = t.z;
    if (gv == 0 || n == 0) return;
    // the segment's state and the first tile's nodes, loaded together
    const uint8_t md = a.mode[s];
    const int32_t top = a.win.top[a.cur * a.S + s], shift = a.win.shift[a.cur * a.S + s];
    WinNodes x;
    x.load<true>(a, a0);
    if (!md) return;
    const int hs = (md & kList1) ? 1 : 0, lane = threadIdx.x & 63;
    for (int i = threadIdx.x; i < kWinBins; i += kBlock) h[i] = 0;
    __syncthreads();
    int32_t below = 0;
    for (int32_t t0 = 0; t0 < n; t0 += kWinTile) {
        if (t0 > 0) x.load<true>(a, a0 + t0);
#pragma unroll
        for (int j = 0; j < kWinItems; j++) {
            const bool in = t0 + j * kBlock + (int32_t)threadIdx.x < n && x.sd[j] == hs;
            const int b = win_bin(x.g[j], top, shift);
            below += in && b == kWinBelow;
            bool act = in && b != kWinBelow;
            const unsigned long long am = __ballot(act);
            if (!am) continue;
            // gains crowd into few bins: the lanes of the first one's bin add once
            const int leader = __ffsll((long long)am) - 1;
            const int lb = __builtin_amdgcn_readlane(b, leader);
            const unsigned long long eq = __ballot(act && b == lb);
            const int c = __popcll(eq);
            if (c >= 8) {
                const int32_t ws = wave_sum((eq >> lane) & 1 ? x.w[j] : 0);
                if (lane == leader) atomicAdd(&h[lb], ((unsigned long long)c << 32) | (uint32_t)ws);
                act = act && b != lb;
            }
            if (act) atomicAdd(&h[b], (1ull << 32) | (uint32_t)x.w[j]);
        }
    }
    below = wave_sum(below);
    if (lane == 0 && below) atomicAdd(&h[kWinBelow], (unsigned long long)below << 32);
    __syncthreads();
    unsigned long long *row = a.win.rows + (int64_t)ci * kWinBins;
    unsigned long long *tot = a.win.tot + ((int64_t)a.cur * a.S + s) * kWinBins;
    for (int i = threadIdx.x; i < kWinBins; i += kBlock) {
        const unsigned long long y = h[i];
        row[i] = y;
        if (y) atomicAdd(&tot[i], y);
    }
}

__global__ __launch_bounds__(kBlock) void k_win_take(WinArgs a)
{
    static_assert(kWinBins == 4 * kBlock, "four bins a thread");
    __shared__ unsigned long long lds[16], bef_s, tot_s;
    __shared__ int32_t part_s, ldsi[16], log_s, nbig;
    __shared__ int4 big[kWinBig];  // moved nodes of many log entries: node, first incidence, last, place
    __shared__ int64_t lds64[16];
    const int32_t ci = blockIdx.x, tid = threadIdx.x;
    const int32_t gv = *a.go;
    const int4 ct = a.tab[ci];
    const int32_t s = ct.x, a0 = ct.y, n = ct.z, cfirst = ct.w;
    if (gv == 0 || n == 0) return;
    // the segment's state, its histogram and the first tile's nodes, loaded together
    const uint8_t md = a.mode[s];
    const int32_t top = a.win.top[a.cur * a.S + s], shift = a.win.shift[a.cur * a.S + s], m = a.m[s];
    const int64_t need = a.need[s], room = a.room[s];
    unsigned long long x[4];
    const unsigned long long *tot = a.win.tot + ((int64_t)a.cur * a.S + s) * kWinBins;
#pragma unroll
    for (int k = 0; k < 4; k++) x[k] = tot[4 * tid + k];
    WinNodes y;
    y.load<false>(a, a0);
    if (!md) return;
    const int hs = (md & kList1) ? 1 : 0;
    if (tid == 0) {
        part_s = kWinBins;
        nbig = 0;
    }
    // (the next round's histogram starts cleared)
    if (ci == cfirst)
        for (int i = tid; i < kWinBins; i += kBlock) a.win.tot[((int64_t)a.nxt * a.S + s) * kWinBins + i] = 0;
    unsigned long long all;
    const unsigned long long ex = block_excl_scan(x[0] + x[1] + x[2] + x[3], lds, &all);
    // the first bin that does not move whole (the weight below the window is
    // not known, so that bin never does)
    unsigned long long acc = ex;
    int mine = kWinBins;
    unsigned long long mbef = 0, mtot = 0;
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const unsigned long long inc = acc + x[k];
        const int64_t C = (int64_t)(inc >> 32), W = (int64_t)(inc & 0xffffffffu);
        const bool whole = C <= m && W < need && W <= room && 4 * tid + k != kWinBelow;
        if (x[k] && !whole && mine == kWinBins) {
            mine = 4 * tid + k;
            mbef = acc;
            mtot = x[k];
        }
        acc = inc;
    }
    if (mine < kWinBins) atomicMin(&part_s, mine);
    __syncthreads();
    const int b = part_s;
    if (mine == b && b < kWinBins) {
        bef_s = mbef;
        tot_s = mtot;
    }
    __syncthreads();
    const unsigned long long bef = b < kWinBins ? bef_s : 0;
    const int64_t inbin = b < kWinBins ? (int64_t)(tot_s >> 32) : 0;
    const bool zoom = b == kWinBelow || ((b == kWinAbove || shift > 0) && inbin > 1);
    if (ci == cfirst && tid == 0) {
        // the next round's window
        int64_t t = top;
        int32_t sh = shift;
        if (zoom) {
            if (b == kWinAbove) {
                sh = min(shift + 6, 22);
                t = (int64_t)top + ((int64_t)(kWinBins - 2) << sh);
            } else if (b == kWinBelow) {
                t = (int64_t)top - ((int64_t)(kWinBins - 2) << shift);
                sh = min(shift + 6, 22);
            } else {
                t = (int64_t)top - ((int64_t)(b - 1) << shift);
                sh = max(shift - 9, 0);
            }
            a.win.zoom[s] = 1;
        } else if (b > kWinAbove && b < kWinBelow && shift == 0) {
            t = (int64_t)top - (b - 1) + 255;
        }
        const int32_t tt = (int32_t)min(max(t, (int64_t)INT32_MIN), (int64_t)INT32_MAX);
        a.win.top[a.nxt * a.S + s] = tt;
        a.win.shift[a.nxt * a.S + s] = sh;
        a.win.top[3 * a.S + s] = tt;
        a.win.shift[3 * a.S + s] = sh;
    }
    if (zoom) return;
    // what stands before this chunk's first node of bin b
    unsigned long long pre = 0;
    if (b < kWinBins) {
        const unsigned long long *rows = a.win.rows + b;
        for (int32_t c = cfirst + tid; c < ci; c += kBlock) pre += rows[(int64_t)c * kWinBins];
    }
    int64_t moved = 0;  // weight
    const bool logm = a.ml.cnode != nullptr;
    bool any = false;
    for (int32_t t0 = 0; t0 < n; t0 += kWinTile) {
        // consecutive nodes a thread, so that one scan gives every node's prefix
        if (t0 > 0) y.load<false>(a, a0 + t0);
        const int32_t i0 = t0 + tid * kWinItems;
        uint32_t go = 0, eq = 0;
        unsigned long long sum = 0;
        int32_t beg[kWinItems], end[kWinItems];
#pragma unroll
        for (int j = 0; j < kWinItems; j++) {
            const int q = win_bin(y.g[j], top, shift);
            beg[j] = 0;
            end[j] = 0;
            if (i0 + j >= n || y.sd[j] != hs || q > b) continue;
            if (q < b) {
                go |= 1u << j;
            } else {
                eq |= 1u << j;
                sum += (1ull << 32) | (uint32_t)y.w[j];
            }
            if (logm) {  // (in flight with the rows)
                beg[j] = a.ml.noff[a0 + i0 + j];
                end[j] = a.ml.noff[a0 + i0 + j + 1];
            }
        }
        if (t0 == 0) pre = block_sum(pre, lds) + bef;
        unsigned long long tsum;
        unsigned long long p = block_excl_scan(sum, lds, &tsum) + pre;
        pre += tsum;
        int32_t nc = 0;
#pragma unroll
        for (int j = 0; j < kWinItems; j++) {
            if ((eq >> j) & 1) {
                const int64_t C = (int64_t)(p >> 32), W = (int64_t)(p & 0xffffffffu);
                if (C < m && W < need && W + y.w[j] <= room) go |= 1u << j;
                p += (1ull << 32) | (uint32_t)y.w[j];
            }
            if ((go >> j) & 1) {
                a.side[a0 + i0 + j] = (uint8_t)(1 - hs);
                moved += y.w[j];
                nc += (int32_t)ceil_div(end[j] - beg[j], kLogChunk);
            }
        }
        if (!__syncthreads_or(go != 0)) continue;
        any = true;
        if (!logm) continue;
        int32_t nct, at = block_excl_scan(nc, ldsi, &nct);
        if (tid == 0) log_s = nct ? atomicAdd(&a.ml.count[0], nct) : 0;
        __syncthreads();
        at += log_s;
#pragma unroll
        for (int j = 0; j < kWinItems; j++) {
            if (!((go >> j) & 1)) continue;
            const int32_t v = a0 + i0 + j, c = (int32_t)ceil_div(end[j] - beg[j], kLogChunk);
            int32_t k = c > 4 ? atomicAdd(&nbig, 1) : kWinBig;
            if (k < kWinBig) {
                big[k] = make_int4(v, beg[j], c, at);
            } else {
                for (int32_t o = 0; o < c; o++) {
                    a.ml.cnode[at + o] = v;
                    a.ml.cbeg[at + o] = beg[j] + o * kLogChunk;
                }
            }
            at += c;
        }
        __syncthreads();
        // nodes of many entries by the whole workgroup
        const int32_t nb = min(nbig, kWinBig);
        for (int32_t k = 0; k < nb; k++) {
            const int4 r = big[k];
            for (int32_t o = tid; o < r.z; o += kBlock) {
                a.ml.cnode[r.w + o] = r.x;
                a.ml.cbeg[r.w + o] = r.y + o * kLogChunk;
            }
        }
        __syncthreads();
        if (tid == 0) nbig = 0;
    }
    if (!any) return;
    moved = block_sum(moved, lds64);
    if (tid == 0) {
        a.win.moved[s] = 1;
        if (moved) {
            atomicAdd(&a.segw[2 * s + hs], (unsigned long long)(-moved));
            atomicAdd(&a.segw[2 * s + 1 - hs], (unsigned long long)moved);
        }
    }
}

// After the last round of a chunk of rounds: settles it and estimates the
// rounds still needed if they move what the level's rounds moved on average
// (go[3], zeroed by the round's test).
__global__ __launch_bounds__(kBlock) void k_win_check(RoundBal rb, int32_t *go)
{
    const int32_t s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= rb.S || !rb.mode[s]) return;
    const bool zoomed = rb.win.pend[s] && rb.win.zoom[s];
    win_settle(s, rb);
    if (rb.done[s]) return;
    const int64_t w0 = (int64_t)rb.segw[2 * s], w1 = (int64_t)rb.segw[2 * s + 1];
    const int64_t rest = w0 > rb.max0[s] ? w0 - rb.max0[s] : w1 - rb.max1[s];
    if (rest <= 0) return;
    const int64_t mw = rb.bal_moved[2 * s], mr = rb.bal_moved[2 * s + 1];
    int64_t est = mw > 0 ? (rest * mr + mw - 1) / mw : 1;
    if (zoomed) est++;
    atomicMax(&go[3], (int32_t)(est < (1 << 20) ? est : (1 << 20)));
}

}  // namespace bp
