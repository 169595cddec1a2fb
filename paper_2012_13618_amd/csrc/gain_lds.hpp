// Gains of a whole level (Algorithm 4) with each segment's gains in LDS.
//
// A level whose segments have at most kGlNodes nodes and many pins per node
// (coarse levels: few nodes, nearly all pins still there) computes its gains
// hyperedge by hyperedge: a workgroup keeps one segment's gains and sides in
// LDS, streams a slab of the segment's hyperedges, counts each one's sides
// from LDS and adds what it contributes to its pins by LDS atomics - only
// where it contributes at all, an uncut hyperedge to every pin and one with a
// lone pin to that pin.  The slabs' sums are added up by a second launch.
// Integer sums, so the result is that of the hyperedge and node passes.
//
// Against those two passes this drops the node pass's gather of one
// contribution per pin from an array of all hyperedges (bound by the lines it
// pulls through the fabric: 60 G gathers/s measured over 40 MB) and the pins'
// side gathers from memory.  What bounds it is the stream of pins, 4 P bytes,
// and for small levels the slabs' sums written and read back, so the number
// of slabs balances the two (gl_slabs).  Measured on 103 M pins over 14,637
// nodes (8.0 M hyperedges of 13 pins): 3.2 ms in two passes, 0.23 ms this way
// (1.8 TB/s of pins); 10 M pins over 8,000 nodes: 139 us against 41.
#pragma once
#include "uncoarsen.hpp"

namespace bp {

constexpr int kGlThreads = 1024;
constexpr int32_t kGlNodesHalf = 16384;  // up to here two workgroups share a CU's LDS
constexpr int32_t kGlNodes = 36864;      // gains and side bits of one segment: 149 KiB of LDS
constexpr int kGlQueue = 1024;           // hyperedges of a slab taken by wavefronts
constexpr int kGlHuge = 64;              // ... and by the whole workgroup
constexpr int32_t kGlHugeMin = 4096;     // pins from which the whole workgroup takes one

// The slabs of up to kBoundLevels levels, one workgroup per level (grid y):
// segment s gets max(1, ceil(its pins / pps)) of them, cut at equal pin counts.
struct GlTableArgs {
    const int32_t *off[kBoundLevels], *nbase[kBoundLevels], *hbase[kBoundLevels];
    GainSlabs gs[kBoundLevels];
    int32_t S;
};

__global__ __launch_bounds__(1024) void k_gain_slabs(GlTableArgs a)
{
    __shared__ int32_t lds[16];
    __shared__ int64_t lds64[16];
    const int j = blockIdx.y;
    const GainSlabs gs = a.gs[j];
    const int32_t *off = a.off[j], *nbase = a.nbase[j], *hbase = a.hbase[j];
    const int32_t S = a.S;
    int32_t carry = 0;
    int64_t pcarry = 0;
    for (int32_t base = 0; base < S; base += blockDim.x) {
        int32_t s = base + (int32_t)threadIdx.x, c = 0, n = 0;
        if (s < S) {
            int32_t p = off[hbase[s + 1]] - off[hbase[s]];
            n = nbase[s + 1] - nbase[s];
            c = max(1, (int32_t)ceil_div(p, gs.pps));
        }
        int32_t tot;
        int64_t ptot;
        int32_t at = block_excl_scan(c, lds, &tot) + carry;
        int64_t pat = block_excl_scan((int64_t)c * n, lds64, &ptot) + pcarry;
        if (s < S) {
            gs.slab0[s] = at;
            gs.pbase[s] = pat;
        }
        carry += tot;
        pcarry += ptot;
    }
    if (threadIdx.x == 0) gs.slab0[S] = carry;
    __syncthreads();
    for (int32_t i = threadIdx.x; i < carry; i += blockDim.x) {
        int32_t lo = 0, hi = S;  // slab0[lo] <= i < slab0[hi]
        while (hi - lo > 1) {
            int32_t mid = (lo + hi) >> 1;
            if (gs.slab0[mid] <= i) lo = mid;
            else hi = mid;
        }
        const int32_t q = i - gs.slab0[lo], nq = gs.slab0[lo + 1] - gs.slab0[lo];
        const int32_t hb = hbase[lo], he = hbase[lo + 1];
        int32_t cut[2];
        for (int k = 0; k < 2; k++) {
            int64_t target = (int64_t)off[hb] + (int64_t)(q + k) * gs.pps;
            int32_t x = hb, y = he;
            if (q + k == nq) x = he;
            else
                while (x < y) {
                    int32_t mid = (x + y) >> 1;
                    if (off[mid] < target) x = mid + 1;
                    else y = mid;
                }
            cut[k] = x;
        }
        gs.rec[i] = make_int4(lo, cut[0], cut[1], q);
    }
}

struct GainLdsArgs {
    GainSlabs gs;
    int32_t S;
    const int32_t *off, *pins, *hw, *nbase;
    const uint8_t *gmask, *side;
    void *cc;  // contributions and counts of pins on side 1, for incremental rounds, or null
    int pk;
    int32_t *n1;
    const int32_t *go;
};

// One hyperedge by lanes lane, lane + stride, ... (stride 1: a thread alone):
// its pins' sides counted, then its contributions added.  The pins are read
// again for the second part, from cache, and only when there is something to
// add; a thread keeps the first eight.
template <int STRIDE>
__device__ __forceinline__ void gl_hedge(int32_t e, int32_t b, int32_t d, int32_t w, int lane, int32_t a0,
                                         const GainLdsArgs &a, const uint32_t *sb, int32_t *g, int32_t *lds)
{
    constexpr int R = 8;
    const int32_t stride = STRIDE == kGlThreads ? kGlThreads : STRIDE;
    int32_t n1 = 0, u[R];
#pragma unroll
    for (int k = 0; k < R; k++) u[k] = a.pins[b + min(lane + k * stride, d - 1)] - a0;
#pragma unroll
    for (int k = 0; k < R; k++)
        if (lane + k * stride < d) n1 += (sb[u[k] >> 5] >> (u[k] & 31)) & 1;
    for (int32_t i0 = R * stride; i0 < d; i0 += R * stride) {
        int32_t x[R];
#pragma unroll
        for (int k = 0; k < R; k++) x[k] = a.pins[b + min(i0 + lane + k * stride, d - 1)] - a0;
#pragma unroll
        for (int k = 0; k < R; k++)
            if (i0 + lane + k * stride < d) n1 += (sb[x[k] >> 5] >> (x[k] & 31)) & 1;
    }
    if (STRIDE == 64) n1 = wave_sum(n1);
    if (STRIDE == kGlThreads) n1 = block_sum(n1, lds);
    int2 c = hedge_contrib_value(w, d, n1);
    if (a.cc && lane == 0) {
        cc_put(a.cc, a.pk, e, c);
        a.n1[e] = n1;
    }
    if (c.x == 0 && c.y == 0) return;
#pragma unroll
    for (int k = 0; k < R; k++) {
        if (lane + k * stride >= d) continue;
        int32_t delta = ((sb[u[k] >> 5] >> (u[k] & 31)) & 1) ? c.y : c.x;
        if (delta) atomicAdd(&g[u[k]], delta);
    }
    for (int32_t i = R * stride + lane; i < d; i += stride) {
        int32_t x = a.pins[b + i] - a0;
        int32_t delta = ((sb[x >> 5] >> (x & 31)) & 1) ? c.y : c.x;
        if (delta) atomicAdd(&g[x], delta);
    }
}

template <int CAP>
__global__ __launch_bounds__(kGlThreads) void k_gain_lds(GainLdsArgs a)
{
    static_assert(CAP % 64 == 0, "side words are written in pairs");
    __shared__ int32_t g[CAP];
    __shared__ uint32_t sb[CAP / 32];
    __shared__ int32_t queue[kGlQueue], huge[kGlHuge];
    __shared__ int32_t nq, nh, lds[16];
    const int32_t gv = a.go ? *a.go : 1, cnt = a.gs.slab0[a.S];
    if (gv == 0 || (int32_t)blockIdx.x >= cnt) return;
    const int4 r = a.gs.rec[blockIdx.x];
    const int32_t s = r.x, e0 = r.y, e1 = r.z;
    if (!a.gmask[s]) return;
    const int32_t a0 = a.nbase[s], n = a.nbase[s + 1] - a0;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    if (tid == 0) {
        nq = 0;
        nh = 0;
    }
    for (int32_t i = tid; i < ((n + 63) & ~63); i += kGlThreads) {
        unsigned long long m = __ballot(i < n && a.side[a0 + min(i, n - 1)]);
        g[i] = 0;
        if (lane == 0) {
            sb[i >> 5] = (uint32_t)m;
            sb[(i >> 5) + 1] = (uint32_t)(m >> 32);
        }
    }
    __syncthreads();
    // hyperedges of up to kHedgeThreadMax pins one a thread; larger ones are
    // queued (past a full queue: a thread takes them all the same)
    int32_t nb = 0, ne = 0, nw = 0;
    if (e0 + tid < e1) {
        nb = a.off[e0 + tid];
        ne = a.off[e0 + tid + 1];
        nw = a.hw[e0 + tid];
    }
    for (int32_t e = e0 + tid; e < e1; e += kGlThreads) {
        const int32_t b = nb, d = ne - nb, w = nw;
        if (e + kGlThreads < e1) {  // the next one's bounds, ahead of this one's pins
            nb = a.off[e + kGlThreads];
            ne = a.off[e + kGlThreads + 1];
            nw = a.hw[e + kGlThreads];
        }
        if (d > kHedgeThreadMax) {
            if (d >= kGlHugeMin) {
                int32_t k = atomicAdd(&nh, 1);
                if (k < kGlHuge) {
                    huge[k] = e;
                    continue;
                }
            }
            int32_t k = atomicAdd(&nq, 1);
            if (k < kGlQueue) {
                queue[k] = e;
                continue;
            }
        }
        if (d > 0) gl_hedge<1>(e, b, d, w, 0, a0, a, sb, g, nullptr);
    }
    __syncthreads();
    for (int32_t k = wv; k < min(nq, kGlQueue); k += kGlThreads / 64) {
        const int32_t e = queue[k], b = a.off[e], d = a.off[e + 1] - b;
        gl_hedge<64>(e, b, d, a.hw[e], lane, a0, a, sb, g, nullptr);
    }
    for (int32_t k = 0; k < min(nh, kGlHuge); k++) {
        const int32_t e = huge[k], b = a.off[e], d = a.off[e + 1] - b;
        gl_hedge<kGlThreads>(e, b, d, a.hw[e], tid, a0, a, sb, g, lds);
    }
    __syncthreads();
    int32_t *part = a.gs.part + a.gs.pbase[s] + (int64_t)r.w * n;
    for (int32_t i = tid; i < n; i += kGlThreads) part[i] = g[i];
}

// Sums of the slabs' gains: 32 nodes at a time, eight threads a node, each
// over every eighth slab.  With stats also what the selection needs: per list
// the eligible nodes and their gain extremes; a workgroup then takes 64
// nodes (per) and ends in one atomic a list.
__global__ __launch_bounds__(kBlock) void k_gain_reduce(int32_t N, int32_t per, GainSlabs gs, const int32_t *nseg,
                                                        const int32_t *nbase, const uint8_t *gmask,
                                                        const uint8_t *side, int32_t *gain, const uint8_t *mode,
                                                        int32_t *tot, int32_t *gmax, int32_t *gmin,
                                                        const int32_t *go)
{
    __shared__ int32_t acc[8][33];
    __shared__ int32_t at[kAggLists], amax[kAggLists], amin[kAggLists];
    if (go && *go == 0) return;
    const bool stats = tot != nullptr;
    const int x = threadIdx.x & 31, y = threadIdx.x >> 5;
    const int64_t v0 = (int64_t)blockIdx.x * per, v1 = min(v0 + per, (int64_t)N);
    if (v0 >= v1) return;
    const int32_t c0 = 2 * nseg[v0], nl = 2 * nseg[v1 - 1] + 2 - c0;
    const bool local = nl <= kAggLists;
    for (int i = threadIdx.x; i < kAggLists; i += blockDim.x) {
        at[i] = 0;
        amax[i] = INT32_MIN;
        amin[i] = INT32_MAX;
    }
    for (int64_t vb = v0; vb < v1; vb += 32) {
        const int64_t v = vb + x;
        int32_t sum = 0, s = 0;
        bool on = false;
        if (v < v1) {
            s = nseg[v];
            on = gmask[s];
        }
        if (on) {
            const int32_t nb = nbase[s], n = nbase[s + 1] - nb, nsl = gs.slab0[s + 1] - gs.slab0[s];
            const int32_t *p = gs.part + gs.pbase[s] + (v - nb);
#pragma unroll 8
            for (int32_t i = y; i < nsl; i += 8) sum += p[(int64_t)i * n];
        }
        __syncthreads();
        acc[y][x] = sum;
        __syncthreads();
        if (y != 0 || !on) continue;
#pragma unroll
        for (int k = 1; k < 8; k++) sum += acc[k][x];
        gain[v] = sum;
        const int sd = stats ? side[v] : 0;
        if (!stats || !sel_list(s, sd, sum, mode)) continue;
        const int32_t c = 2 * s + sd;
        if (local) {
            atomicAdd(&at[c - c0], 1);
            atomicMax(&amax[c - c0], sum);
            atomicMin(&amin[c - c0], sum);
        } else {
            atomicAdd(&tot[c], 1);
            atomicMax(&gmax[c], sum);
            atomicMin(&gmin[c], sum);
        }
    }
    __syncthreads();
    if (stats && local)
        for (int i = threadIdx.x; i < nl; i += blockDim.x)
            if (at[i]) {
                atomicAdd(&tot[c0 + i], at[i]);
                atomicMax(&gmax[c0 + i], amax[i]);
                atomicMin(&gmin[c0 + i], amin[i]);
            }
}

// Whether a level's gains go through LDS: every segment fits, and the pins
// are many.  Below about 2^20 pins both ways take launches' time (n = 8000
// nodes: 0.3 M pins 18 against 18 us, 1 M 26 against 22, 3 M 49 against 31,
// 10 M 139 against 41); below 64 pins a node of the largest segment the slabs'
// sums outweigh the stream (n = 36,000: 1 M pins 25 against 34 us, 3 M 70
// against 38); and each segment has at least a slab of its own.
inline bool gl_ok(const Level &L)
{
    return L.maxseg_nodes <= kGlNodes && L.P >= (1 << 20) && (int64_t)L.P >= 64 * (int64_t)L.maxseg_nodes &&
           (int64_t)L.P >= 8 * (int64_t)L.N && (int64_t)L.P >= (int64_t)L.S * 4096;
}

// Slabs of a level: x workgroups stream the pins in about P / (2600 x) us and
// cost n x 8 / 4.5e6 us in sums (both rates measured), least at the x below; no
// more than the workgroups the LDS holds at once.
inline int32_t gl_slabs(const Level &L)
{
    double n = std::max(L.maxseg_nodes, 1);
    int64_t x = (int64_t)std::sqrt((double)L.P * 216.0 / n);
    int64_t cap = L.maxseg_nodes <= kGlNodesHalf ? 512 : 256;
    return (int32_t)std::max<int64_t>(1, std::min(x, cap));
}

// pins a slab, and partial sums of a level: over the segments, (1 + pins / pps)
// times their nodes
inline int32_t gl_pps(const Level &L) { return (int32_t)ceil_div(L.P, gl_slabs(L)); }
inline int64_t gl_parts(const Level &L) { return (int64_t)L.N + ceil_div(L.P, gl_pps(L)) * L.maxseg_nodes; }

}  // namespace bp
