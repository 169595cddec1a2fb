// Algorithm 1 of a level with each segment's minima in LDS.
//
// On coarse levels (few nodes, nearly all pins still there) the node side
// gathers one 8-byte key per pin from an array of all hyperedges, bound by the
// lines that it pulls through the fabric.  Here a workgroup streams a run of
// hyperedges of equal pin counts and keeps the smallest key of each node of one
// segment in LDS: a pin costs a coalesced read, a look at LDS and, while the
// minimum still falls, an LDS atomic.  What it found goes to memory with a
// 64-bit minimum where it is below what is there, the workgroups starting at
// different nodes so that most find the others' results already in place.
// Minima of the same keys, so the result is that of the node side.
//
// What bounds it is the stream of pins and, for few of them, the results' way
// to memory.  103 M pins over 14,637 nodes 1.72 ms by node and 0.20 here
// (2.0 TB/s of pins), over 262 nodes (81 M) 414 us and 150; 3.8 M pins over
// 1614 nodes 39 us and 27.  Half the LDS and two workgroups a CU: the same for
// 100 M pins, and a third slower for 4 M, whose results are looked at twice as
// often.
#pragma once
#include "gain_lds.hpp"

namespace bp {

constexpr int kMlThreads = 1024;
constexpr int32_t kMlNodes = 16384;  // minima of one range of a segment's nodes: 128 KiB of LDS

struct MatchLdsArgs {
    int32_t E, slabs;
    int64_t ntiles;
    const int32_t *off, *pins, *hseg, *nbase, *hbase, *tfirst;
    const uint8_t *sact;
    const uint64_t *hkey;
    unsigned long long *key;
};

// Key k offered to the pins [b, b + d) by lanes lane, lane + STRIDE, ...
template <int STRIDE>
__device__ __forceinline__ void ml_hedge(unsigned long long k, int32_t b, int32_t d, int lane, int32_t a0, int32_t n,
                                         const int32_t *pins, unsigned long long *m)
{
    constexpr int R = 8;
    for (int32_t i0 = lane; i0 < d; i0 += R * STRIDE) {
        uint32_t u[R];
#pragma unroll
        for (int j = 0; j < R; j++) u[j] = (uint32_t)(pins[b + min(i0 + j * STRIDE, d - 1)] - a0);
#pragma unroll
        for (int j = 0; j < R; j++)
            if (i0 + j * STRIDE < d && u[j] < (uint32_t)n && k < m[u[j]]) atomicMin(&m[u[j]], k);
    }
}

// Grid: runs of hyperedges (x) by ranges of kMlNodes nodes of a segment (y).
// A run that spans segments takes them one after the other.
__global__ __launch_bounds__(kMlThreads) void k_match_lds(MatchLdsArgs a)
{
    __shared__ unsigned long long m[kMlNodes];
    __shared__ int32_t queue[kGlQueue], huge[kGlHuge];
    __shared__ int32_t nq, nh;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int32_t x = blockIdx.x;
    const int32_t c0 = x == 0 ? 0 : a.tfirst[a.ntiles * x / a.slabs];
    const int32_t c1 = x + 1 == a.slabs ? a.E : a.tfirst[a.ntiles * (x + 1) / a.slabs];
    for (int32_t e0 = c0, e1; e0 < c1; e0 = e1) {
        const int32_t s = a.hseg[e0], a0 = a.nbase[s] + (int32_t)blockIdx.y * kMlNodes;
        const int32_t n = min(kMlNodes, a.nbase[s + 1] - a0);
        e1 = min(c1, a.hbase[s + 1]);
        if (!a.sact[s] || n <= 0) continue;
        for (int32_t i = tid; i < n; i += kMlThreads) m[i] = kNoKey;
        if (tid == 0) {
            nq = 0;
            nh = 0;
        }
        __syncthreads();
        // (hyperedges by size as in the gains' LDS pass)
        int32_t nb = 0, ne = 0;
        unsigned long long nk = 0;
        if (e0 + tid < e1) {
            nb = a.off[e0 + tid];
            ne = a.off[e0 + tid + 1];
            nk = a.hkey[e0 + tid];
        }
        for (int32_t e = e0 + tid; e < e1; e += kMlThreads) {
            const int32_t b = nb, d = ne - nb;
            const unsigned long long k = nk;
            if (e1 - e > kMlThreads) {
                nb = a.off[e + kMlThreads];
                ne = a.off[e + kMlThreads + 1];
                nk = a.hkey[e + kMlThreads];
            }
            if (d > kHedgeThreadMax) {
                if (d >= kGlHugeMin) {
                    const int32_t q = atomicAdd(&nh, 1);
                    if (q < kGlHuge) {
                        huge[q] = e;
                        continue;
                    }
                }
                const int32_t q = atomicAdd(&nq, 1);
                if (q < kGlQueue) {
                    queue[q] = e;
                    continue;
                }
            }
            ml_hedge<1>(k, b, d, 0, a0, n, a.pins, m);
        }
        __syncthreads();
        for (int32_t q = wv; q < min(nq, kGlQueue); q += kMlThreads / 64) {
            const int32_t e = queue[q], b = a.off[e];
            ml_hedge<64>(a.hkey[e], b, a.off[e + 1] - b, lane, a0, n, a.pins, m);
        }
        for (int32_t q = 0; q < min(nh, kGlHuge); q++) {
            const int32_t e = huge[q], b = a.off[e];
            ml_hedge<kMlThreads>(a.hkey[e], b, a.off[e + 1] - b, tid, a0, n, a.pins, m);
        }
        __syncthreads();
        const int32_t rot = (int32_t)((int64_t)n * x / a.slabs);
        constexpr int R = 4;
        for (int32_t i0 = tid; i0 < n; i0 += R * kMlThreads) {
            unsigned long long old[R];
            int32_t at[R];
#pragma unroll
            for (int j = 0; j < R; j++) {
                const int32_t i = min(i0 + j * kMlThreads, n - 1) + rot;
                at[j] = i < n ? i : i - n;
                old[j] = __hip_atomic_load(&a.key[a0 + at[j]], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
#pragma unroll
            for (int j = 0; j < R; j++)
                if (i0 + j * kMlThreads < n && m[at[j]] < old[j]) atomicMin(&a.key[a0 + at[j]], m[at[j]]);
        }
        __syncthreads();
    }
}

inline int32_t ml_ranges(const Level &L) { return (int32_t)ceil_div(std::max(L.maxseg_nodes, 1), kMlNodes); }

// Whether a level's minima go through LDS.  Segments of up to kMlFew nodes: from
// 2^18 pins (below, both ways are a launch's time).  Larger segments only with
// many pins, 24 a node and 2^24 in all, as each range reads all of them and
// every workgroup looks over its range's results: 25,750 nodes in each of 256
// segments, 39 M pins, 521 us by node and 328 here; 94,094 nodes and 103 M pins
// 1720 and 900; but 13,323 nodes and 4.7 M pins 41 and 51, 24,156 and 4.9 M 39
// and 49, 36,933 (256 segments) and 19 M, 11 a node, 303 and 310.
constexpr int32_t kMlFew = 10240;
inline bool ml_ok(const Level &L)
{
    if (!L.tfirst || L.maxseg_nodes <= 0 || L.P < (1 << 18) || (int64_t)L.P < (int64_t)L.S * 4096) return false;
    return L.maxseg_nodes <= kMlFew || (L.P >= (1 << 24) && (int64_t)L.P >= 24 * (int64_t)L.N && ml_ranges(L) <= 6);
}

// Runs of hyperedges: one workgroup a CU over the ranges of a segment (a
// multiple of 8, so that the ranges that read the same pins share an L2), of
// two radix tiles at least.
inline int32_t ml_slabs(const Level &L)
{
    const int64_t x = 256 / ml_ranges(L) / 8 * 8;
    return (int32_t)std::max<int64_t>(1, std::min(x, ceil_div(L.P, kRsTile) / 2));
}

}  // namespace bp
