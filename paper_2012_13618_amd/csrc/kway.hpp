// Input normalisation, nested k-way subgraph extraction (Algorithm 6), the
// connectivity-1 cut (problem statement) and device-side input validation.
#pragma once
#include "level.hpp"
#include "scan.hpp"

namespace bp {

// ---- validation -----------------------------------------------------------------

struct ValidateOut {
    int32_t bad_offsets;
    int32_t bad_pins;
    int32_t bad_weights;
    int32_t pad;
    unsigned long long sum_nw, sum_hw;
};

// One workgroup a CU with eight pins a thread in flight: the sums end in one
// atomic a workgroup and array, 11 ns each on one address (2048 workgroups of
// 256 threads spent 45 of 59 us there at 5.4 M pins, now 16 in all).
constexpr int kValThreads = 1024;
__global__ __launch_bounds__(kValThreads) void k_validate(int32_t N, int32_t E, const int32_t *off,
                                                          const int32_t *pins, const int32_t *nw,
                                                          const int32_t *hw, ValidateOut *out)
{
    __shared__ int64_t lds[16];
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t P = off[E];
    int64_t snw = 0, shw = 0;
    int bo = 0, bp_ = 0, bw = 0;
#pragma unroll 4
    for (int64_t e = tid; e < E; e += stride) {
        const int32_t w = hw ? hw[e] : 0;
        if (off[e + 1] < off[e]) bo = 1;
        if (w < 0) bw = 1;
        shw += w;
    }
    if (tid == 0 && (off[0] != 0 || P < 0)) bo = 1;
    if (!bo) {
#pragma unroll 8
        for (int64_t i = tid; i < P; i += stride)
            if ((uint32_t)pins[i] >= (uint32_t)N) bp_ = 1;
    }
    if (nw) {
#pragma unroll 4
        for (int64_t v = tid; v < N; v += stride) {
            const int32_t w = nw[v];
            if (w < 0) bw = 1;
            snw += w;
        }
    }
    if (bo) atomicOr(&out->bad_offsets, 1);
    if (bp_) atomicOr(&out->bad_pins, 1);
    if (bw) atomicOr(&out->bad_weights, 1);
    if (nw) snw = block_sum(snw, lds);
    if (hw) shw = block_sum(shw, lds);
    if (threadIdx.x == 0) {
        if (nw) atomicAdd(&out->sum_nw, (unsigned long long)snw);
        if (hw) atomicAdd(&out->sum_hw, (unsigned long long)shw);
    }
}

// ---- level 0: drop hyperedges that cannot be cut --------------------------------

// copy the kept hyperedges' pins (degree >= 2) to their compacted place
constexpr int kNormShort = 16;

__global__ __launch_bounds__(kBlock) void k_norm_copy(int32_t E, const int32_t *off,
                                                      const int32_t *pins, const int32_t *dst,
                                                      int32_t *cpins)
{
    // a thread per hyperedge of at most kNormShort pins (its loads all in
    // flight before the stores); longer ones are copied by the whole
    // wavefront, one after another, 8 loads a lane in flight.  Every lane
    // reaches the ballot: lanes past E carry an empty hyperedge.
    const int lane = threadIdx.x & 63;
    int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int32_t b = 0, d = 0, o = 0;
    if (e < E) {
        b = off[e];
        d = off[e + 1] - b;
        if (d >= 2) o = dst[e];
        else d = 0;
    }
    if (d <= kNormShort) {
        int32_t v[kNormShort];
#pragma unroll
        for (int i = 0; i < kNormShort; i++)
            if (i < d) v[i] = pins[b + i];
#pragma unroll
        for (int i = 0; i < kNormShort; i++)
            if (i < d) cpins[o + i] = v[i];
    }
    unsigned long long lm = __ballot(d > kNormShort);
    while (lm) {
        int l = __ffsll((long long)lm) - 1;
        lm &= lm - 1;
        int32_t lb = __shfl(b, l, 64), ld = __shfl(d, l, 64), lo = __shfl(o, l, 64);
        for (int32_t i0 = 0; i0 < ld; i0 += 8 * 64) {
            int32_t v[8];
#pragma unroll
            for (int u = 0; u < 8; u++) {
                int32_t i = i0 + u * 64 + lane;
                v[u] = i < ld ? pins[lb + i] : 0;
            }
#pragma unroll
            for (int u = 0; u < 8; u++) {
                int32_t i = i0 + u * 64 + lane;
                if (i < ld) cpins[lo + i] = v[u];
            }
        }
    }
}

__global__ void k_iota(int64_t n, int32_t *p)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = (int32_t)i;
}

__global__ void k_copy_weights(int64_t n, const int32_t *src, int32_t *dst)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        dst[i] = src ? src[i] : 1;
}

// Schedule lists of a freshly built level: each workgroup stages the
// hyperedges of its kClsItems ids in LDS and reserves room in each list with
// one atomic (same-address atomics from many workgroups serialise).  With
// tot (a level just compacted) the count and the pin total come from the
// device: E is then only a bound.  List order is arbitrary; every consumer
// treats its items independently.
constexpr int kClsItems = 2048;

// Block vb of the classification.
__device__ __forceinline__ void classify_block(int64_t vb, int32_t E, const int32_t *off, const uint64_t *tot,
                                               int32_t *lmid, int32_t *lbig, int32_t *lhuge, int32_t *counters)
{
    __shared__ int32_t items[3][kClsItems];
    __shared__ int32_t cnt[3], base[3];
    int32_t P = 0;
    if (tot) {
        E = (int32_t)(*tot >> 32);
        P = (int32_t)(*tot & 0xffffffffu);
    }
    int64_t first = vb * kClsItems;
    if (first >= E) return;
    if (!tot) P = off[E];
    if (threadIdx.x < 3) cnt[threadIdx.x] = 0;
    __syncthreads();
    for (int r = 0; r < kClsItems / kBlock; r++) {
        int64_t e = first + r * kBlock + threadIdx.x;
        int32_t d = 0;
        if (e < E) d = (e + 1 < E ? off[e + 1] : P) - off[e];
        lds_append(d > kHedgeThreadMax && d <= kMidMax, (int32_t)e, items[0], &cnt[0]);
        lds_append(d > kMidMax, (int32_t)e, items[1], &cnt[1]);
        lds_append(d > kBigMax, (int32_t)e, items[2], &cnt[2]);
    }
    __syncthreads();
    if (threadIdx.x < 3) base[threadIdx.x] = cnt[threadIdx.x] ? atomicAdd(&counters[1 + threadIdx.x], cnt[threadIdx.x]) : 0;
    __syncthreads();
    for (int i = threadIdx.x; i < cnt[0]; i += blockDim.x) lmid[base[0] + i] = items[0][i];
    for (int i = threadIdx.x; i < cnt[1]; i += blockDim.x) lbig[base[1] + i] = items[1][i];
    for (int i = threadIdx.x; i < cnt[2]; i += blockDim.x) lhuge[base[2] + i] = items[2][i];
}

__global__ __launch_bounds__(kBlock) void k_classify(int32_t E, const int32_t *off, const uint64_t *tot,
                                                     int32_t *lmid, int32_t *lbig, int32_t *lhuge,
                                                     int32_t *counters)
{
    classify_block(blockIdx.x, E, off, tot, lmid, lbig, lhuge, counters);
}

template <int S>
__global__ __launch_bounds__(kBlock) void k_count_side1(int32_t count, const int32_t *list,
                                                        const int32_t *off, const int32_t *pins,
                                                        const uint8_t *side, int32_t *n1out)
{
    __shared__ int32_t lds[16];
    int lane, stride;
    int32_t e = sched_hedge<S>(count, list, lane, stride);
    if (e < 0) return;
    int32_t b = off[e], d = off[e + 1] - b;
    if (!thread_split<S>(d)) return;
    int32_t n1 = 0;
    for (int i = lane; i < d; i += stride) n1 += side[pins[b + i]];
    n1 = group_sum<S>(n1, lds);
    if (lane == 0) n1out[e] = n1;
}

// Child table: child (s, side) continues when it still has >= 2 parts.
struct ChildTable {
    int32_t *idx;     // [2S] child segment index or -1 (final part)
    int32_t *nbase;   // [C+1]
    int32_t *hbase;   // [C+1]
    int32_t *pbase;   // [C+1]
    int32_t *k;       // [C] parts of each child
    int32_t *lo;      // [C]
    uint64_t *F;      // [C] per-bisection factor, inherited from the parent
};

// One workgroup, a side of a segment a thread (one thread for all of them took
// 0.29 ms over 256 segments, now 8 us).
constexpr int kChildThreads = 512;
__global__ __launch_bounds__(kChildThreads) void k_child_table(
    int32_t S, int32_t N, int32_t E, const int32_t *nbase, const int32_t *hbase, const int32_t *k0, const int32_t *k1,
    const int32_t *lo, const uint64_t *F, const uint64_t *nscan, const uint64_t *hscan0, const uint64_t *hscan1,
    const uint64_t *ntot, const uint64_t *htot0, const uint64_t *htot1, ChildTable ct, LevelInfo *info)
{
    __shared__ int32_t lds[16];
    int32_t c = 0, nb = 0, hb = 0, pb = 0;
    auto at = [&](const uint64_t *scan, const uint64_t *tot, int32_t i, int32_t n) -> uint64_t {
        return i < n ? scan[i] : *tot;
    };
    for (int32_t i0 = 0; i0 < 2 * S; i0 += kChildThreads) {
        const int32_t i = i0 + (int32_t)threadIdx.x, s = i >> 1, sd = i & 1;
        int32_t kk = 0, nn = 0, ne = 0, np = 0;
        if (i < 2 * S) {
            kk = sd ? k1[s] : k0[s];
            if (kk >= 2) {
                const uint64_t na = at(nscan, ntot, nbase[s], N), nz = at(nscan, ntot, nbase[s + 1], N);
                const uint64_t *hs = sd ? hscan1 : hscan0, *ht = sd ? htot1 : htot0;
                const uint64_t ha = at(hs, ht, hbase[s], E), hz = at(hs, ht, hbase[s + 1], E);
                nn = sd ? (int32_t)((nz >> 32) - (na >> 32)) : (int32_t)((nz & 0xffffffffu) - (na & 0xffffffffu));
                ne = (int32_t)((hz >> 32) - (ha >> 32));
                np = (int32_t)((hz & 0xffffffffu) - (ha & 0xffffffffu));
            }
        }
        int32_t tc, tn, te, tp;
        const int32_t ci = c + block_excl_scan(kk >= 2 ? 1 : 0, lds, &tc);
        const int32_t ni = nb + block_excl_scan(nn, lds, &tn);
        const int32_t hi = hb + block_excl_scan(ne, lds, &te);
        const int32_t pi = pb + block_excl_scan(np, lds, &tp);
        if (i < 2 * S) ct.idx[i] = kk >= 2 ? ci : -1;
        if (kk >= 2) {
            ct.nbase[ci] = ni;
            ct.hbase[ci] = hi;
            ct.pbase[ci] = pi;
            ct.k[ci] = kk;
            ct.lo[ci] = lo[s] + (sd ? k0[s] : 0);
            ct.F[ci] = F[s];
        }
        c += tc;
        nb += tn;
        hb += te;
        pb += tp;
    }
    if (threadIdx.x != 0) return;
    ct.nbase[c] = nb;
    ct.hbase[c] = hb;
    ct.pbase[c] = pb;
    info->N = nb;
    info->E = hb;
    info->P = pb;
    info->active = c;
}

// Part ids of a tree level whose children are all single parts.
__global__ __launch_bounds__(kBlock) void k_last_parts(int32_t N, const int32_t *nseg, const uint8_t *side,
                                                       const int32_t *orig, const int32_t *k0, const int32_t *lo,
                                                       int32_t *part)
{
    int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= N) return;
    const int32_t s = nseg[v];
    part[orig[v]] = lo[s] + (side[v] ? k0[s] : 0);
}

// nodes: renumber into their child, or write the final part id
__global__ __launch_bounds__(kBlock) void k_extract_nodes(
    int32_t N, const int32_t *nseg, const int32_t *nbase, const uint8_t *side,
    const uint64_t *nscan, const int32_t *orig, const int32_t *nw, const int32_t *k0,
    const int32_t *lo, ChildTable ct, int32_t *map, int32_t *c_orig, int32_t *c_nw,
    int32_t *c_nseg, int32_t *part)
{
    int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= N) return;
    int32_t s = nseg[v], sd = side[v];
    int32_t ci = ct.idx[2 * s + sd];
    if (ci < 0) {
        part[orig[v]] = lo[s] + (sd ? k0[s] : 0);
        map[v] = -1;
        return;
    }
    uint64_t a = nscan[v], z = nscan[nbase[s]];
    int32_t rank = sd ? (int32_t)((a >> 32) - (z >> 32)) : (int32_t)((a & 0xffffffffu) - (z & 0xffffffffu));
    int32_t id = ct.nbase[ci] + rank;
    map[v] = id;
    c_orig[id] = orig[v];
    c_nw[id] = nw[v];
    c_nseg[id] = ci;
}

// hyperedges: emit each side's part when it keeps >= 2 pins
template <int S>
__global__ __launch_bounds__(kBlock) void k_extract_hedges(
    int32_t count, const int32_t *list, const int32_t *off, const int32_t *pins,
    const int32_t *hw, const int32_t *hseg, const int32_t *hbase, const uint8_t *side,
    const int32_t *n1, const uint64_t *hscan0, const uint64_t *hscan1, const int32_t *map,
    ChildTable ct, int32_t *c_off, int32_t *c_pins, int32_t *c_hw, int32_t *c_hseg)
{
    __shared__ int32_t lds[16];
    __shared__ int32_t carry;
    int lane, stride;
    int32_t e = sched_hedge<S>(count, list, lane, stride);
    if (e < 0) return;
    int32_t b = off[e], d = off[e + 1] - b;
    if (!thread_split<S>(d)) return;
    int32_t s = hseg[e];
    int32_t cnt1 = n1[e];
    for (int sd = 0; sd < 2; sd++) {
        int32_t ci = ct.idx[2 * s + sd];
        int32_t ns = sd ? cnt1 : d - cnt1;
        if (ci < 0 || ns < 2) continue;  // uniform over the group
        const uint64_t *hs = sd ? hscan1 : hscan0;
        uint64_t a = hs[e], z = hs[hbase[s]];
        int32_t id = ct.hbase[ci] + (int32_t)((a >> 32) - (z >> 32));
        int32_t po = ct.pbase[ci] + (int32_t)((a & 0xffffffffu) - (z & 0xffffffffu));
        if (lane == 0) {
            c_off[id] = po;
            c_hw[id] = hw[e];
            c_hseg[id] = ci;
        }
        if (S == SMALL) {
            int32_t k = 0;
            for (int i = 0; i < d; i++) {
                int32_t v = pins[b + i];
                if (side[v] == sd) c_pins[po + k++] = map[v];
            }
        } else if (S == WAVE) {
            int32_t base = 0;
            for (int i0 = 0; i0 < d; i0 += 64) {
                int i = i0 + lane;
                int32_t v = i < d ? pins[b + i] : 0;
                bool in = i < d && side[v] == sd;
                unsigned long long m = __ballot(in);
                if (in) c_pins[po + base + __popcll(m & ((1ull << lane) - 1))] = map[v];
                base += __popcll(m);
            }
        } else {
            if (threadIdx.x == 0) carry = 0;
            __syncthreads();
            for (int i0 = 0; i0 < d; i0 += blockDim.x) {
                int i = i0 + threadIdx.x;
                int32_t v = i < d ? pins[b + i] : 0;
                int32_t in = (i < d && side[v] == sd) ? 1 : 0;
                int32_t tot;
                int32_t ex = block_excl_scan(in, lds, &tot);
                if (in) c_pins[po + carry + ex] = map[v];
                __syncthreads();
                if (threadIdx.x == 0) carry += tot;
                __syncthreads();
            }
        }
    }
}

// ---- connectivity-1 cut of the final partition ----------------------------------

// Connectivity (number of distinct parts) of a hyperedge by lanes lane, lane +
// STRIDE, ... (1: a thread alone, 64: a wavefront, else the workgroup): a part
// bitmask when every part id is below 64, else a count of parts not seen at an
// earlier pin (O(d^2), rare large hyperedges).
template <int STRIDE, typename PART>
__device__ __forceinline__ int32_t cut_lambda(int32_t b, int32_t d, int lane, const int32_t *pins, const PART *part,
                                              bool mask64, unsigned long long *orl, int32_t *lds)
{
    constexpr int R = 8;
    if (mask64) {
        unsigned long long m = 0;
        for (int32_t i0 = lane; i0 < d; i0 += R * STRIDE) {
            int32_t v[R];
            PART p[R];
#pragma unroll
            for (int j = 0; j < R; j++) v[j] = pins[b + min(i0 + j * STRIDE, d - 1)];
#pragma unroll
            for (int j = 0; j < R; j++) p[j] = part[v[j]];
#pragma unroll
            for (int j = 0; j < R; j++) m |= 1ull << (p[j] & 63);
        }
        if (STRIDE > 1)
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) m |= __shfl_xor(m, o, 64);
        if (STRIDE > 64) {
            __syncthreads();
            if ((threadIdx.x & 63) == 0) orl[threadIdx.x >> 6] = m;
            __syncthreads();
            m = 0;
            for (int i = 0; i < STRIDE / 64; i++) m |= orl[i];
        }
        return __popcll(m);
    }
    int32_t lam = 0;
    for (int32_t i = lane; i < d; i += STRIDE) {
        const int32_t p = part[pins[b + i]];
        bool first = true;
        for (int32_t j = 0; j < i && first; j++) first = part[pins[b + j]] != p;
        lam += first ? 1 : 0;
    }
    if (STRIDE == 64) lam = wave_sum(lam);
    if (STRIDE > 64) lam = block_sum(lam, lds);
    return lam;
}

// Launch sizes of the batch's cut (k_cut_seg).  SMALL: contiguous chunks of
// about two hyperedges a thread; WAVE: the listed hyperedges, one a wavefront
// (at most kCutBlocks workgroups).
constexpr int64_t kCutBlocks = 16384;

template <int S> inline int64_t cut_grid(int64_t count)
{
    int64_t g = S == SMALL ? ceil_div(count, (int64_t)2 * kBlock) : sched_grid<WAVE>(count);
    return g < kCutBlocks ? g : kCutBlocks;
}

// Connectivity-1 cut of all hyperedges, added to acc[0], and the largest of the
// k part weights pw, to acc[1].  A workgroup takes tiles of kCutThreads
// hyperedges: those of up to kHedgeThreadMax pins a thread each, with eight
// gathers in flight; larger ones are queued and taken by wavefronts, and from
// kCutHuge pins by the whole workgroup.  One barrier a tile: queue and counters
// of a tile are not those of the next.
//
// The gathers of the pins' parts bound it, so they are bytes where the parts of
// a level would not stay in the L2s (PART uint8_t).  5.4 M pins over 1 M nodes:
// three launches by lists 82 us, and the lists' 12 and a readback; now 58 by
// ints and 47 by bytes.  115 M pins over 10 M nodes: 2.73 ms, now 1.34.  Four
// gathers in flight: 43 us and 1.45 ms.
//
// Large hyperedges that stand together would be one workgroup's work, so a tile
// is made of runs of 2^lg hyperedges, one run of each 2^lg * gridDim.x (the
// column-net of 617 K hyperedges sorted by size, k=16: tiles of consecutive ones
// 636 us a call, now 229; unsorted 87 both ways).
//
// Above 64 parts a large hyperedge's work is its degree times the pins looked at
// for each, which no fixed share evens out: there the larger ones go to a list
// (those of up to kMidMax pins from its front, the others from its back; large
// counts both) that k_cut_large takes (unsorted, k=128: 11.5 ms a call with the
// tiles' own wavefronts, now 2.3; 1 M nodes of small hyperedges 171 and 183 us,
// 291 by three launches and a readback).
//
// ok: nothing is read through the pins if it says that they are not valid.
constexpr int kCutThreads = 512;
constexpr int kCutMaxBlocks = 1024;  // (512 threads: two waves' worth of them fill the card)
constexpr int32_t kCutHuge = 4096;

template <typename PART>
__global__ __launch_bounds__(kCutThreads) void k_cut(int32_t E, int lg, const int32_t *off, const int32_t *pins,
                                                     const int32_t *hw, const PART *part, int32_t k,
                                                     const unsigned long long *pw, unsigned long long *acc,
                                                     int32_t *list, int32_t *large, const ValidateOut *ok)
{
    __shared__ int32_t queue[2][kCutThreads];  // wavefronts' from the front, the workgroup's from the back
    __shared__ int32_t nq[3], nh[3], base[2];
    __shared__ unsigned long long orl[16];
    __shared__ int32_t lds[16];
    __shared__ int64_t lds64[16];
    if (ok && (ok->bad_offsets || ok->bad_pins)) return;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const bool mask64 = sizeof(PART) == 1 || list == nullptr;  // (bytes: up to 64 parts)
    const int32_t huge = mask64 ? kCutHuge : kMidMax + 1;
    if ((int64_t)blockIdx.x * kCutThreads < k) {
        unsigned long long m = 0;
#pragma unroll 4
        for (int64_t i = (int64_t)blockIdx.x * kCutThreads + tid; i < k; i += (int64_t)gridDim.x * kCutThreads)
            m = pw[i] > m ? pw[i] : m;
        m = wave_max(m);
        if (lane == 0 && m) atomicMax(&acc[1], m);
    }
    if (tid < 3) {
        nq[tid] = 0;
        nh[tid] = 0;
    }
    __syncthreads();
    int64_t contrib = 0;
    int t = 0, t3 = 0;
    const int64_t runs = kCutThreads >> lg;  // of a tile
    for (int64_t r0 = 0; ((r0 * gridDim.x + blockIdx.x) << lg) < E; r0 += runs) {
        const int64_t e = (((r0 + (tid >> lg)) * gridDim.x + blockIdx.x) << lg) + (tid & ((1 << lg) - 1));
        if (e < E) {
            const int32_t b = off[e], d = off[e + 1] - b;
            if (d >= huge) {
                queue[t][kCutThreads - 1 - atomicAdd(&nh[t3], 1)] = (int32_t)e;
            } else if (d > kHedgeThreadMax) {
                queue[t][atomicAdd(&nq[t3], 1)] = (int32_t)e;
            } else if (d >= 2) {
                const int32_t lam = cut_lambda<1>(b, d, 0, pins, part, mask64, orl, lds);
                if (lam > 1) contrib += (int64_t)(hw ? hw[e] : 1) * (lam - 1);
            }
        }
        __syncthreads();
        const int32_t n = nq[t3], m = nh[t3], free3 = t3 == 0 ? 2 : t3 - 1;
        if (tid == 0) {  // (the counters of the tile after the next, last read before this barrier)
            nq[free3] = 0;
            nh[free3] = 0;
        }
        if (!mask64) {
            if (n + m > 0) {
                if (tid == 0) {
                    base[0] = n ? atomicAdd(&large[0], n) : 0;
                    base[1] = m ? atomicAdd(&large[1], m) : 0;
                }
                __syncthreads();
                if (tid < n) list[base[0] + tid] = queue[t][tid];
                if (tid < m) list[E - 1 - base[1] - tid] = queue[t][kCutThreads - 1 - tid];
            }
        } else {
            for (int32_t q = wv; q < n; q += kCutThreads / 64) {
                const int32_t x = queue[t][q], b = off[x];
                const int32_t lam = cut_lambda<64>(b, off[x + 1] - b, lane, pins, part, true, orl, lds);
                if (lane == 0 && lam > 1) contrib += (int64_t)(hw ? hw[x] : 1) * (lam - 1);
            }
            for (int32_t q = 0; q < m; q++) {
                const int32_t x = queue[t][kCutThreads - 1 - q], b = off[x];
                const int32_t lam = cut_lambda<kCutThreads>(b, off[x + 1] - b, tid, pins, part, true, orl, lds);
                if (tid == 0 && lam > 1) contrib += (int64_t)(hw ? hw[x] : 1) * (lam - 1);
            }
        }
        t ^= 1;
        t3 = t3 == 2 ? 0 : t3 + 1;
    }
    contrib = block_sum(contrib, lds64);
    if (tid == 0 && contrib) atomicAdd(&acc[0], (unsigned long long)contrib);
}

// The listed hyperedges of a cut of more than 64 parts: a workgroup each from
// the back of the list, then a wavefront each from its front.
constexpr int64_t kCutLargeBlocks = 2048;
__global__ __launch_bounds__(kBlock) void k_cut_large(int32_t E, const int32_t *off, const int32_t *pins,
                                                      const int32_t *hw, const int32_t *part, const int32_t *list,
                                                      const int32_t *large, unsigned long long *acc)
{
    __shared__ int32_t lds[16];
    __shared__ int64_t lds64[16];
    const int tid = threadIdx.x, lane = tid & 63;
    const int32_t n = large[0], m = large[1];
    int64_t contrib = 0;
    for (int64_t q = blockIdx.x; q < m; q += gridDim.x) {
        const int32_t x = list[E - 1 - q], b = off[x];
        const int32_t lam = cut_lambda<kBlock>(b, off[x + 1] - b, tid, pins, part, false, nullptr, lds);
        if (tid == 0 && lam > 1) contrib += (int64_t)(hw ? hw[x] : 1) * (lam - 1);
    }
    for (int64_t q = (int64_t)blockIdx.x * (kBlock / 64) + (tid >> 6); q < n; q += (int64_t)gridDim.x * (kBlock / 64)) {
        const int32_t x = list[q], b = off[x];
        const int32_t lam = cut_lambda<64>(b, off[x + 1] - b, lane, pins, part, false, nullptr, lds);
        if (lane == 0 && lam > 1) contrib += (int64_t)(hw ? hw[x] : 1) * (lam - 1);
    }
    contrib = block_sum(contrib, lds64);
    if (tid == 0 && contrib) atomicAdd(&acc[0], (unsigned long long)contrib);
}

// Workgroups of k_cut: as many as give each the same number of whole tiles (of
// the hyperedges or, with very many parts, of the part weights); for few
// hyperedges up to kCutSpread of eight each, as many as there are wavefronts,
// should they be large (a call with 512 of 2000 pins: by one workgroup 574 us, now
// 45; by a list and a workgroup each 139).
constexpr int64_t kCutSpread = 256;
inline int64_t cut_blocks(int64_t E, int32_t k)
{
    const int64_t tiles = std::max<int64_t>(ceil_div(std::max<int64_t>(E, k), kCutThreads), 1);
    if (tiles >= kCutSpread) return ceil_div(tiles, ceil_div(tiles, kCutMaxBlocks));
    return std::max(tiles, std::min(ceil_div(E, 8), kCutSpread));
}

// log2 of k_cut's runs: a wavefront's hyperedges, shorter where that would leave
// a workgroup without a run.
inline int cut_run_bits(int64_t E, int64_t blocks)
{
    int lg = 0;
    while (lg < 6 && (E >> (lg + 1)) >= blocks) lg++;
    return lg;
}

// Part weights: registers for k <= 8, an LDS histogram for k <= 4096, else
// global atomics; one global atomic per part per workgroup otherwise.  With
// bytes also the parts' low bytes.
__global__ __launch_bounds__(kBlock) void k_part_weights(int32_t N, int32_t k, const int32_t *part,
                                                         const int32_t *nw, uint8_t *bytes,
                                                         unsigned long long *pw)
{
    __shared__ unsigned long long acc[4096];
    __shared__ int64_t lds[16];
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    if (k <= 8) {
        int64_t r[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < N; v += stride) {
            int32_t p = part[v];
            int64_t w = nw ? nw[v] : 1;
            if (bytes) bytes[v] = (uint8_t)p;
#pragma unroll
            for (int j = 0; j < 8; j++) r[j] += p == j ? w : 0;
        }
#pragma unroll
        for (int j = 0; j < 8; j++) {
            int64_t t = block_sum(r[j], lds);
            if (threadIdx.x == 0 && j < k && t) atomicAdd(&pw[j], (unsigned long long)t);
        }
        return;
    }
    bool in_lds = k <= 4096;
    if (in_lds) {
        for (int i = threadIdx.x; i < k; i += blockDim.x) acc[i] = 0;
        __syncthreads();
    }
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < N; v += stride) {
        int32_t p = part[v];
        if (bytes) bytes[v] = (uint8_t)p;
        if (p < 0 || p >= k) continue;  // range is the caller's contract; never write outside
        unsigned long long w = (unsigned long long)(nw ? nw[v] : 1);
        if (in_lds) atomicAdd(&acc[p], w);
        else atomicAdd(&pw[p], w);
    }
    if (in_lds) {
        __syncthreads();
        for (int i = threadIdx.x; i < k; i += blockDim.x)
            if (acc[i]) atomicAdd(&pw[i], acc[i]);
    }
}

}  // namespace bp
