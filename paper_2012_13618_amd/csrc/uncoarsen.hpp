// Uncoarsening kernels with few launches per round (Algorithms 3-5).
//
// Gains (Algorithm 4) take two launches: a hyperedge pass computing what a pin
// on each side gains from its hyperedge (+w when alone on its side, -w when
// the hyperedge is uncut), and a node pass summing that over the node's
// hyperedges.  The hyperedge pass takes a tile of pins a workgroup.  The node
// pass's first blocks take 256 nodes at a time (those of degree <= 32, staged
// 64), the next ones one listed larger node per wavefront, the last ones a chunk
// of a big node.  The node pass also records, per list (one side of one segment),
// how many nodes are eligible and their largest and smallest gain.
//
// Selection of the first r nodes in (gain desc, id asc) order per list is an
// exact radix select over the pair (u, lid), u = max gain - gain (so ascending
// u = descending gain) and lid = node id within its segment: 12-bit digits,
// first over the significant bits of u (1 digit when the list's gains span
// < 4096 values), then over the bits of lid - each list follows its own digit
// schedule and stops as soon as the remaining count equals a bin's count.
// In balance rounds a list also stops at the bin holding its r-th key when
// the keys through that bin fit the candidate buffer: the balance finish
// orders what it gathers and keeps the first r.
// Each pass is one launch: blocks build their histograms and the workgroup
// that finishes last (atomic ticket) picks the digit of every list.
#pragma once
#include "level.hpp"
#include "refine.hpp"
#include "transpose.hpp"

namespace bp {

constexpr int kDigit = 12;
constexpr int kBins = 1 << kDigit;        // 4096
constexpr int kSelNodes = 1024;           // nodes per workgroup in histogram passes

__device__ __forceinline__ int bitlen_u32(uint32_t x) { return x ? 32 - __clz((int)x) : 0; }

// Per-hyperedge gain contributions (what a pin on side 0 / side 1 gains from
// the hyperedge: +w, -w or 0).  When every hyperedge weight of the level is
// below 2^15 (pk) the pair is stored as two 16-bit halves of one word, which
// halves the bytes of the node pass's random gathers; else as an int2.
__device__ __forceinline__ int2 cc_get(const void *cc, int pk, int32_t e)
{
    if (pk) {
        uint32_t v = ((const uint32_t *)cc)[e];
        return make_int2((int32_t)(int16_t)(v & 0xffffu), (int32_t)(int16_t)(v >> 16));
    }
    return ((const int2 *)cc)[e];
}
__device__ __forceinline__ void cc_put(void *cc, int pk, int32_t e, int2 c)
{
    if (pk) ((uint32_t *)cc)[e] = (uint32_t)(uint16_t)(int16_t)c.x | ((uint32_t)(uint16_t)(int16_t)c.y << 16);
    else ((int2 *)cc)[e] = c;
}

// ---- gains -------------------------------------------------------------------------

__device__ __forceinline__ int2 hedge_contrib_value(int32_t w, int32_t d, int32_t n1)
{
    int32_t n0 = d - n1;
    int2 c;
    c.x = n0 == 1 ? w : (n0 == d ? -w : 0);
    c.y = n1 == 1 ? w : (n1 == d ? -w : 0);
    return c;
}

// Bits of positions [b, e) of a bit string, b < e.
__device__ __forceinline__ int32_t count_bits(const unsigned long long *bits, int32_t b, int32_t e)
{
    const int32_t w0 = b >> 6, w1 = (e - 1) >> 6;
    const unsigned long long m0 = ~0ull << (b & 63), m1 = ~0ull >> (63 - ((e - 1) & 63));
    if (w0 == w1) return __popcll(bits[w0] & m0 & m1);
    int32_t n = __popcll(bits[w0] & m0) + __popcll(bits[w1] & m1);
    for (int32_t w = w0 + 1; w < w1; w++) n += __popcll(bits[w]);
    return n;
}

// The sides as one bit a node: 1/8 of the bytes, so that the side gathers of
// levels of very many nodes stay in an L2 (from kSideBitsMin nodes on; below,
// the bytes are as fast and this pass is saved.  115 M gathers over 10 M
// nodes: 1.22 ms from bytes, 0.49 from bits; over 1 M: 0.49 and 0.39).
constexpr int32_t kSideBitsMin = 2 << 20;

__global__ __launch_bounds__(kBlock) void k_side_bits(int32_t N, const uint8_t *side, unsigned long long *bits,
                                                      const int32_t *go)
{
    if (go && *go == 0) return;
    const int64_t v = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const unsigned long long m = __ballot(v < N && side[v]);
    if ((threadIdx.x & 63) == 0 && v < N) bits[v >> 6] = m;
}

// Hyperedge pass of Algorithm 4, a tile of kBlock * R pins a workgroup (the
// hyperedges that start in it): the pins are loaded in order, R a thread, their
// sides gathered and left as one bit a pin in LDS, and a thread a hyperedge
// counts the bits of its pins.  Three memory round trips, whatever the
// degrees; one thread walking each hyperedge took two for every eight pins of
// the wavefront's largest.  Only the last hyperedge can end past the tile's
// bits: the whole workgroup counts the rest of it.  n1out (nullable): the
// counts, for incremental rounds.  Bound by the side gathers (sbits or side):
// 115 M pins over 10 M nodes 2.3 ms, now 0.57; 5.4 M over 1 M 61 us, now 38.
// Up to 2^22 pins quarter tiles (R = 4), as whole ones do not fill the card (pins
// near / far apart, R = 16 and R = 4: 93 K pins 7.6 and 4.9 us, 1.5 M 13, 16 and
// 11.4, 14.3; 5 M 18.2, 28.8 and 19.3, 28.1; 16 M 25.7, 42 and 28.8, 42.8).
// The rest of a hyperedge longer than its tile is 16 pins a thread at a time,
// with the next ones' ids loaded meanwhile: one of 500 K pins 474 us with 8 and
// nothing ahead, now 94.
constexpr int64_t kGhSmall = 1 << 22;
template <int R>
__global__ __launch_bounds__(kBlock) void k_gain_hedges(int32_t E, int32_t P, int64_t ntiles, const int32_t *off,
                                                        const int32_t *pins, const int32_t *hw,
                                                        const int32_t *hseg, const int2 *tnext,
                                                        const uint8_t *gmask, const uint8_t *side,
                                                        const uint32_t *sbits, void *cc, int pk, int32_t *n1out,
                                                        const int32_t *go, const int32_t *lnbig,
                                                        const int32_t *ncount, int32_t *gain, int32_t *big_done)
{
    constexpr int32_t kTile = kBlock * R;
    static_assert(kTile % kGhTile == 0, "whole quarter tiles");
    __shared__ unsigned long long bits[kTile / 64];
    __shared__ int32_t lds[16];
    if (go && *go == 0) return;
    // big nodes are summed chunk by chunk in the node pass: start them at 0
    const int64_t z = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (z < ncount[1]) {
        gain[lnbig[z]] = 0;
        big_done[z] = 0;
    }
    if ((int64_t)blockIdx.x >= ntiles) return;
    const int64_t t = xcd_block(blockIdx.x, ntiles);
    const int2 first = tnext[t * (kTile / kGhTile)];
    const int2 past = t + 1 < ntiles ? tnext[(t + 1) * (kTile / kGhTile)] : make_int2(E, P);
    const int32_t es = first.x, ee = past.x;
    const int32_t p0 = first.y, np = past.y - p0, n = min(np, kTile);
    if (np <= 0) return;  // (inside one hyperedge, or only empty ones start here)
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    int32_t u[R];
    uint32_t x[R];
#pragma unroll
    for (int r = 0; r < R; r++) u[r] = pins[p0 + min(w * (R * 64) + r * 64 + lane, n - 1)];
    // the thread's first hyperedge, in flight with the pins
    int32_t hb = 0, he = 0, hs = 0, ww = 0;
    if (es + (int32_t)threadIdx.x < ee) {
        hb = off[es + threadIdx.x];
        he = off[es + threadIdx.x + 1];
        hs = hseg[es + threadIdx.x];
        ww = hw[es + threadIdx.x];
    }
    if (sbits) {
#pragma unroll
        for (int r = 0; r < R; r++) x[r] = (sbits[u[r] >> 5] >> (u[r] & 31)) & 1;
    } else {
#pragma unroll
        for (int r = 0; r < R; r++) x[r] = side[u[r]];
    }
#pragma unroll
    for (int r = 0; r < R; r++) {
        const unsigned long long m = __ballot(x[r] != 0 && w * (R * 64) + r * 64 + lane < n);
        if (lane == 0) bits[w * R + r] = m;
    }
    bool on = gmask[hs];
    __syncthreads();
    for (int32_t e = es + (int32_t)threadIdx.x; e < ee; e += kBlock) {
        const int32_t b = hb - p0, d = he - hb;
        if (d > 0 && b + d <= kTile && on) {
            const int32_t n1 = count_bits(bits, b, b + d);
            cc_put(cc, pk, e, hedge_contrib_value(ww, d, n1));
            if (n1out) n1out[e] = n1;
        }
        if (e + kBlock < ee) {
            hb = off[e + kBlock];
            he = off[e + kBlock + 1];
            on = gmask[hseg[e + kBlock]];
            ww = hw[e + kBlock];
        }
    }
    if (np <= kTile) return;
    // the one that holds the next tile's first pin
    const int32_t el = ee - 1, b = off[el] - p0, d = past.y - p0 - b;
    if (!gmask[hseg[el]]) return;
    constexpr int T = 16;
    const int32_t end = b + d;
    int32_t n1 = 0, q[T], nq[T];
    auto load = [&](int32_t i0, int32_t (&id)[T]) {
#pragma unroll
        for (int k = 0; k < T; k++) id[k] = pins[p0 + min(i0 + (int32_t)threadIdx.x + k * kBlock, end - 1)];
    };
    load(kTile, q);
    for (int32_t i0 = kTile; i0 < end; i0 += T * kBlock) {
        const bool more = end - i0 > T * kBlock;
        if (more) load(i0 + T * kBlock, nq);
#pragma unroll
        for (int k = 0; k < T; k++) q[k] = side[q[k]];
#pragma unroll
        for (int k = 0; k < T; k++)
            if (i0 + (int32_t)threadIdx.x + k * kBlock < end) n1 += q[k];
        if (more)
#pragma unroll
            for (int k = 0; k < T; k++) q[k] = nq[k];
    }
    n1 = block_sum(n1, lds) + count_bits(bits, b, kTile);
    if (threadIdx.x == 0) {
        cc_put(cc, pk, el, hedge_contrib_value(hw[el], d, n1));
        if (n1out) n1out[el] = n1;
    }
}

// ---- gains after a balance round: updated from what it moved -------------------------

// One wavefront per logged chunk of a moved node's incidences: marks each
// hyperedge in the bitmap.  Of adjacent lanes that share a bitmap word the first
// sets the bits of all with one atomic (none when they are all set already).
// The radix passes leave a node's hyperedges ascending, so a word is one run;
// k_incidence_one's small levels do not, and may take a few atomics for a word,
// with the same bits.  Here: blocks b of nb
// (kBlock threads each) of the marking of the n logged chunks.
//
// Each hyperedge's count of pins on side 1 (n1) follows the move, one atomic an
// incidence; the gain update reads the counts and not the pins.
//
// It also settles the moved node's side change in its gain.  The gain update
// that follows treats every pin as unmoved (new contribution minus old, both
// for the pin's side now); a node that moved from side o to side s had gained
// the old contribution for o, so it is owed old[s] - old[o] per hyperedge,
// added here while the contributions are still the old ones.  That way the
// update reads one side byte per pin and no move flags.
__device__ __forceinline__ void log_hedges_blocks(int64_t b, int64_t nb, int32_t n, const int32_t *cnode,
                                                  const int32_t *cbeg, const int32_t *noff, const int32_t *inc,
                                                  uint32_t *bits, const void *cc, int pk, int32_t *n1,
                                                  const uint8_t *side, int32_t *gain)
{
    int lane = threadIdx.x & 63;
    const int64_t wpb = kBlock / 64;
    for (int64_t i = b * wpb + (threadIdx.x >> 6); i < n; i += nb * wpb) {
        int32_t v = cnode[i];
        int32_t j = cbeg[i] + lane, end = noff[v + 1];
        bool valid = j < end;
        int32_t e = valid ? inc[j] : 0;
        int sv = side[v];
        int32_t corr = 0;
        if (valid) {
            atomicAdd(&n1[e], sv ? 1 : -1);
            int2 oc = cc_get(cc, pk, e);
            corr = sv ? oc.y - oc.x : oc.x - oc.y;
        }
        corr = wave_sum(corr);
        if (lane == 0 && corr) atomicAdd(&gain[v], corr);
        int32_t w = valid ? (e >> 5) : -1;
        uint32_t bit = valid ? 1u << (e & 31) : 0u;
        int32_t pw = __shfl_up(w, 1, 64);
        bool head = valid && (lane == 0 || pw != w);
        unsigned long long heads = __ballot(head);
        int lead = 63 - __clzll((long long)(heads & ((2ull << lane) - 1ull)));
        uint32_t run = bit;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            uint32_t t = __shfl_down(run, o, 64);
            int tl = __shfl_down(lead, o, 64);
            if (lane + o < 64 && tl == lead) run |= t;
        }
        if (head) {
            uint32_t old = __hip_atomic_load(&bits[w], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if ((old & run) != run) atomicOr(&bits[w], run);
        }
    }
}

constexpr int kUpdSlots = 1024;  // big nodes whose gain changes gather in LDS first

// adds delta to gain[u]: in the workgroup's LDS slot when u is one of the
// first kUpdSlots big nodes (many hyperedges, so many updates), else globally
__device__ __forceinline__ void add_gain(int32_t u, int32_t delta, const int32_t *bigslot, int32_t *slot,
                                        int32_t *gain)
{
    int32_t k = bigslot[u];
    if (k >= 0 && k < kUpdSlots) atomicAdd(&slot[k], delta);
    else atomicAdd(&gain[u], delta);
}

constexpr int kUpdWords = 64;                // bitmap words a workgroup sweeps per step
constexpr int kUpdChunk = 8;                 // ... as 8 chunks of this many words
constexpr int kUpdQueue = kUpdWords * 32;  // hyperedges those words can hold
constexpr int kUpdWaveMax = 2048;          // larger changed hyperedges: the whole workgroup

// The change dc of a hyperedge's contribution to a pin on side 0 / side 1 added
// to its pins' gains by one thread, eight pins' loads in flight at a time.
__device__ __forceinline__ void spread_thread(int32_t b, int32_t d, int2 dc, const int32_t *pins,
                                              const uint8_t *side, const int32_t *bigslot, int32_t *slot,
                                              int32_t *gain)
{
    for (int32_t i0 = 0; i0 < d; i0 += 8) {
        // straight-line loads (past the degree: the last pin again)
        int32_t u[8];
        uint32_t sn[8];
#pragma unroll
        for (int j = 0; j < 8; j++) u[j] = pins[b + min(i0 + j, d - 1)];
#pragma unroll
        for (int j = 0; j < 8; j++) sn[j] = side[u[j]];
#pragma unroll
        for (int j = 0; j < 8; j++) {
            int32_t delta = sn[j] ? dc.y : dc.x;
            if (i0 + j < d && delta) add_gain(u[j], delta, bigslot, slot, gain);
        }
    }
}

// The same by lanes lane, lane + stride, ... of a wavefront or workgroup.
__device__ __forceinline__ void spread_lanes(int32_t b, int32_t d, int2 dc, int lane, int stride,
                                             const int32_t *pins, const uint8_t *side, const int32_t *bigslot,
                                             int32_t *slot, int32_t *gain)
{
    for (int32_t i0 = 0; i0 < d; i0 += 8 * stride) {
        int32_t u[8];
        uint32_t sn[8];
#pragma unroll
        for (int k = 0; k < 8; k++) u[k] = pins[b + min(i0 + lane + k * stride, d - 1)];
#pragma unroll
        for (int k = 0; k < 8; k++) sn[k] = side[u[k]];
#pragma unroll
        for (int k = 0; k < 8; k++) {
            int32_t delta = sn[k] ? dc.y : dc.x;
            if (i0 + lane + k * stride < d && delta) add_gain(u[k], delta, bigslot, slot, gain);
        }
    }
}

// Marked hyperedges, found by sweeping the bitmap: the contribution from the
// count of pins on side 1 that the marking kept, and where it changed, the
// change added to every pin's gain, as if no pin had moved (the marking launch
// has already settled what the moved nodes are owed for changing sides).
// Integer sums, so the result equals a recomputation.  The sweep clears the
// bitmap.  A hyperedge whose contribution stays - most of those with several
// pins on both sides - is done without reading a pin, which is what a recount
// of every marked hyperedge spent its time on (column-net of 617 K rows,
// k = 32: 29 us a launch, now 16).
//
// The bitmap is dealt out in chunks of 8 words (256 hyperedges, in id order),
// chunk c to workgroup c mod G: a moved node's hyperedges crowd into a few
// chunks (ids follow locality), and consecutive chunks go to different
// workgroups.  Each step a workgroup takes 8 of its chunks; one wavefront
// lists their marked hyperedges in LDS (popcount scan), then changed ones of
// degree <= 32 go one per thread, up to 2048 one per wavefront, larger ones to
// the whole workgroup.  When abytes is set (profiling), adds the algorithmic
// bytes it moved: 4 per bitmap word, per hyperedge 16 (offsets, weight, count)
// plus the contribution in and out, 9 per pin of a changed one (id, side, gain).
__global__ __launch_bounds__(kBlock) void k_gain_update(int64_t nwords, uint32_t *bits, const int32_t *off,
                                                        const int32_t *pins, const int32_t *hw,
                                                        const uint8_t *side, void *cc, int pk, const int32_t *n1,
                                                        int32_t *gain, const int32_t *bigslot,
                                                        const int32_t *lnbig, const int32_t *ncount,
                                                        const int32_t *go, int32_t *logcount,
                                                        unsigned long long *abytes)
{
    __shared__ int32_t slot[kUpdSlots];
    __shared__ int32_t queue[kUpdQueue], bigq[kUpdQueue];  // bigq: wavefront ones from the front, workgroup ones from the back
    __shared__ int2 bigd[kUpdQueue];                       // their changes
    __shared__ int32_t nq, nbq, nhq, npins;
    const int32_t gv = go ? *go : 1, nbig = ncount[1];  // loaded together
    if (gv == 0) return;
    // the move log was read by the previous launch: empty it for this round's moves
    if (logcount && blockIdx.x == 0 && threadIdx.x == 0) *logcount = 0;
    int32_t nb = min(nbig, kUpdSlots);
    for (int i = threadIdx.x; i < nb; i += blockDim.x) slot[i] = 0;
    int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int64_t G = gridDim.x;
    int64_t words_done = 0, hedges_done = 0, pins_done = 0;  // thread 0's tally (profiling)
    for (int64_t step = 0; step * 8 * G * kUpdChunk < nwords; step++) {
        if (wv == 0) {
            int64_t chunk = step * 8 * G + (lane / kUpdChunk) * G + blockIdx.x;
            int64_t wi = chunk * kUpdChunk + (lane % kUpdChunk);
            uint32_t word = wi < nwords ? bits[wi] : 0u;
            if (word) bits[wi] = 0;
            int32_t c = __popc(word);
            int32_t at = wave_incl_scan(c) - c;
            while (word) {
                int k = __ffs((int)word) - 1;
                word &= word - 1;
                queue[at++] = (int32_t)(wi * 32 + k);
            }
            if (lane == 63) nq = at;
            if (lane == 0) {
                nbq = 0;
                nhq = 0;
                npins = 0;
            }
        }
        __syncthreads();
        int32_t n = nq;
        for (int32_t q = threadIdx.x; q < n; q += blockDim.x) {
            const int32_t e = queue[q], b = off[e], d = off[e + 1] - b;
            const int2 oc = cc_get(cc, pk, e), nc = hedge_contrib_value(hw[e], d, n1[e]);
            const int2 dc = make_int2(nc.x - oc.x, nc.y - oc.y);
            if (dc.x == 0 && dc.y == 0) continue;
            cc_put(cc, pk, e, nc);
            if (abytes) atomicAdd(&npins, d);
            if (d <= kHedgeThreadMax) {
                spread_thread(b, d, dc, pins, side, bigslot, slot, gain);
                continue;
            }
            // front and back never meet
            int32_t k = d <= kUpdWaveMax ? atomicAdd(&nbq, 1) : kUpdQueue - 1 - atomicAdd(&nhq, 1);
            bigq[k] = e;
            bigd[k] = dc;
        }
        __syncthreads();
        int32_t nmid = nbq, nhuge = nhq;
        for (int32_t q = wv; q < nmid; q += blockDim.x >> 6) {
            const int32_t e = bigq[q], b = off[e], d = off[e + 1] - b;
            spread_lanes(b, d, bigd[q], lane, 64, pins, side, bigslot, slot, gain);
        }
        // the largest ones by the whole workgroup, one after another
        for (int32_t q = 0; q < nhuge; q++) {
            const int32_t e = bigq[kUpdQueue - 1 - q], b = off[e], d = off[e + 1] - b;
            spread_lanes(b, d, bigd[kUpdQueue - 1 - q], threadIdx.x, kBlock, pins, side, bigslot, slot, gain);
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            words_done += 64;
            hedges_done += n;
            pins_done += npins;
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < nb; i += blockDim.x)
        if (slot[i]) atomicAdd(&gain[lnbig[i]], slot[i]);
    if (abytes && threadIdx.x == 0 && words_done)
        atomicAdd(abytes, (unsigned long long)(4 * words_done + (pk ? 24 : 32) * hedges_done + 9 * pins_done));
}

// eligibility of a node for its list under the segment's selection mode
__device__ __forceinline__ bool sel_list(int32_t s, int sd, int32_t g, const uint8_t *mode)
{
    uint8_t md = mode[s];
    if (!((md >> sd) & 1)) return false;
    return !((md & kGainNonNeg) && g < 0);
}

// Which contributions are not zero, one bit a hyperedge (E > kNzBitsMin): the
// node pass then gathers the contributions of those only.
constexpr int32_t kNzBitsMin = 1 << 20;

__global__ __launch_bounds__(kBlock) void k_nz_bits(int32_t E, const void *cc, int pk, unsigned long long *bits,
                                                    const int32_t *go)
{
    if (go && *go == 0) return;
    const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    bool nz = false;
    if (e < E) {
        const int2 c = cc_get(cc, pk, (int32_t)e);
        nz = c.x != 0 || c.y != 0;
    }
    const unsigned long long m = __ballot(nz);
    if ((threadIdx.x & 63) == 0 && e < E) bits[e >> 6] = m;
}

// A lane's share (lane, lane + stride, ...) of the contributions to a node on
// side sd over its incidences b .. b + d, eight loads in flight at a time: the
// sums stand apart from them, as each would wait for its own (60 K nodes of ten
// incidences 12.0 us, now 10.2), and there is none for the places past the
// degree (1 M nodes of two, ids far apart: 33 us with the last one's again, now 25).
__device__ __forceinline__ int32_t gather_sum(int32_t b, int32_t d, int lane, int stride, const int32_t *inc,
                                              const void *cc, int pk, const uint32_t *nzb, int sd)
{
    int32_t g = 0;
    for (int32_t i0 = lane; i0 < d; i0 += 8 * stride) {
        int32_t e[8];
        int2 c[8];
        bool in[8];
#pragma unroll
        for (int k = 0; k < 8; k++) {
            in[k] = i0 + k * stride < d;
            e[k] = inc[b + min(i0 + k * stride, d - 1)];
        }
        if (nzb) {
#pragma unroll
            for (int k = 0; k < 8; k++) in[k] = in[k] && ((nzb[e[k] >> 5] >> (e[k] & 31)) & 1);
        }
#pragma unroll
        for (int k = 0; k < 8; k++) c[k] = in[k] ? cc_get(cc, pk, e[k]) : make_int2(0, 0);
#pragma unroll
        for (int k = 0; k < 8; k++) g += sd ? c[k].y : c[k].x;
    }
    return g;
}

constexpr int32_t kGnThread = 64;    // node degree: staged and summed by a thread; above: a wavefront

// Node pass.  Besides gain[v], per-list counts and gain extremes for the
// selection that follows (block-aggregated when a block is in one segment).
//
// The first ns blocks take runs of nodes, 256 at a time.  A thread gathers its
// node's contributions itself, two memory round trips for every eight
// incidences of the wavefront's largest node.  STAGED: the incidences of those
// of degree <= kGnThread are loaded in order, 16 a thread, their contributions
// gathered and staged in LDS, and a thread a node sums its own.  nzb (nullable):
// the contributions that are not zero.  Bound by the gathers: 115 M incidences
// of 10 M hyperedges 1.9 ms, now 0.92 (staged).
template <bool STAGED>
__global__ __launch_bounds__(kBlock) void k_gain_nodes(int32_t N, int64_t ns, const int32_t *lnmid,
                                                       const int32_t *lnbig, const int32_t *ncount,
                                                       const int32_t *noff, const int32_t *inc,
                                                       const int32_t *nseg, const uint8_t *gmask,
                                                       const uint8_t *side, const void *cc, int pk,
                                                       const uint32_t *nzb,
                                                       int32_t *gain, const uint8_t *mode,
                                                       int32_t *tot, int32_t *gmax, int32_t *gmin,
                                                       const int32_t *go, const int32_t *chunk_node,
                                                       const int32_t *chunk_beg,
                                                       const int32_t *chunk_big,
                                                       const int32_t *big_chunks, int32_t *big_done,
                                                       int32_t S, int32_t nw)
{
    __shared__ int32_t lds[16];
    __shared__ int32_t at[kAggLists], amax[kAggLists], amin[kAggLists];
    if (go && *go == 0) return;
    bool stats = tot != nullptr;
    int32_t cm = ncount[0], ck = ncount[2];
    const int32_t thread_max = STAGED ? kGnThread : kNodeSmallMax;
    int64_t vb = blockIdx.x;
    if (vb < ns) {
        __shared__ int32_t val[kRsTile];  // where a node's incidences start, then the gathered contributions
        __shared__ TileLds tl;
        __shared__ int32_t carry;
        // whole 256-node steps, shared out evenly
        const int64_t per = ceil_div(ceil_div(N, kBlock), ns) * kBlock, lo = xcd_block(vb, ns) * per,
                      hi = min(lo + per, (int64_t)N);
        if (lo >= hi) return;
        int32_t c0 = 2 * nseg[lo], nl = 2 * nseg[hi - 1] + 2 - c0;
        bool local = nl <= kAggLists;
        if (stats)
            for (int i = threadIdx.x; i < kAggLists; i += blockDim.x) {
                at[i] = 0;
                amax[i] = INT32_MIN;
                amin[i] = INT32_MAX;
            }
        __syncthreads();  // (not staged, no other barrier stands before the atomics on these)
        const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
        for (int64_t base = lo; base < hi; base += kBlock) {
            const int64_t v = base + threadIdx.x;
            int32_t b = 0, d = 0, s = 0;
            int sd = 0;
            bool on = v < hi;
            if (on) {
                b = noff[v];
                d = noff[v + 1] - b;
                s = nseg[v];
                sd = side[v];
                on = d <= thread_max && gmask[s];
            }
            if (!on) d = 0;
            int32_t T = 0, st = 0, g = 0;
            if (STAGED) st = block_excl_scan(d, lds, &T);
            else if (d > 0) g = gather_sum(b, d, 0, 1, inc, cc, pk, nzb, sd);
            for (int32_t t0 = 0; STAGED && t0 < T; t0 += kRsTile) {
                // each staged position's incidence: st + (b - st)
                if (threadIdx.x < 64) tl.bits[threadIdx.x] = 0;
                if (threadIdx.x == 0) carry = 0;
                __syncthreads();
                if (d > 0 && st >= t0 && st < t0 + kRsTile) {
                    atomicOr(&tl.bits[(st - t0) >> 6], 1ull << ((st - t0) & 63));
                    val[st - t0] = b - st;
                } else if (st < t0 && st + d > t0) {
                    carry = b - st;
                }
                __syncthreads();
                tile_last(tl);
                __syncthreads();
                int32_t e[kRsItems];
                bool in[kRsItems];
#pragma unroll
                for (int r = 0; r < kRsItems; r++) {
                    const int32_t q = t0 + (r * (kBlock / 64) + w) * 64 + lane;
                    in[r] = q < T;
                    e[r] = in[r] ? q + tile_val(r * (kBlock / 64) + w, lane, val, tl, carry) : 0;
                }
#pragma unroll
                for (int r = 0; r < kRsItems; r++) e[r] = in[r] ? inc[e[r]] : 0;
                if (nzb) {
#pragma unroll
                    for (int r = 0; r < kRsItems; r++) in[r] = in[r] && ((nzb[e[r] >> 5] >> (e[r] & 31)) & 1);
                }
                __syncthreads();
                if (pk) {
                    uint32_t c[kRsItems];
#pragma unroll
                    for (int r = 0; r < kRsItems; r++) c[r] = in[r] ? ((const uint32_t *)cc)[e[r]] : 0u;
#pragma unroll
                    for (int r = 0; r < kRsItems; r++) val[(r * (kBlock / 64) + w) * 64 + lane] = (int32_t)c[r];
                    __syncthreads();
                    const int32_t q1 = min(st + d, t0 + kRsTile) - t0;
                    for (int32_t q = max(st, t0) - t0; q < q1; q++) {
                        const uint32_t x = (uint32_t)val[q];
                        g += sd ? (int32_t)(int16_t)(x >> 16) : (int32_t)(int16_t)(x & 0xffffu);
                    }
                    __syncthreads();
                } else {
                    // a pair of words each: one side's contributions at a time
                    int2 c[kRsItems];
#pragma unroll
                    for (int r = 0; r < kRsItems; r++) c[r] = in[r] ? ((const int2 *)cc)[e[r]] : make_int2(0, 0);
#pragma unroll 1
                    for (int h = 0; h < 2; h++) {
#pragma unroll
                        for (int r = 0; r < kRsItems; r++)
                            val[(r * (kBlock / 64) + w) * 64 + lane] = h ? c[r].y : c[r].x;
                        __syncthreads();
                        const int32_t q1 = min(st + d, t0 + kRsTile) - t0;
                        if (sd == h)
                            for (int32_t q = max(st, t0) - t0; q < q1; q++) g += val[q];
                        __syncthreads();
                    }
                }
            }
            if (!on) continue;
            gain[v] = g;
            if (!stats || !sel_list(s, sd, g, mode)) continue;
            int32_t c = 2 * s + sd;
            if (local) {
                atomicAdd(&at[c - c0], 1);
                atomicMax(&amax[c - c0], g);
                atomicMin(&amin[c - c0], g);
            } else {
                atomicAdd(&tot[c], 1);
                atomicMax(&gmax[c], g);
                atomicMin(&gmin[c], g);
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
    } else if (vb < ns + nw) {
        // nodes of degree thread_max + 1 .. 2048, one per wavefront, nw workgroups striding
        // over the list; with few segments the lists aggregate in LDS
        bool local = 2 * S <= kAggLists;
        for (int i = threadIdx.x; i < kAggLists; i += blockDim.x) {
            at[i] = 0;
            amax[i] = INT32_MIN;
            amin[i] = INT32_MAX;
        }
        __syncthreads();
        int lane = threadIdx.x & 63;
        for (int64_t i = (vb - ns) * (kBlock / 64) + (threadIdx.x >> 6); i < cm; i += (int64_t)nw * (kBlock / 64)) {
            int32_t v = lnmid[i];
            int32_t s = nseg[v];
            if (!gmask[s]) continue;
            int32_t b = noff[v], d = noff[v + 1] - b;
            if (d <= thread_max) continue;  // (listed from degree 33 on)
            int sd = side[v];
            int32_t g = gather_sum(b, d, lane, 64, inc, cc, pk, nzb, sd);
            g = wave_sum(g);
            if (lane != 0) continue;
            gain[v] = g;
            if (!stats || !sel_list(s, sd, g, mode)) continue;
            int32_t c = 2 * s + sd;
            if (local) {
                atomicAdd(&at[c], 1);
                atomicMax(&amax[c], g);
                atomicMin(&amin[c], g);
            } else {
                atomicAdd(&tot[c], 1);
                atomicMax(&gmax[c], g);
                atomicMin(&gmin[c], g);
            }
        }
        __syncthreads();
        if (stats && local)
            for (int i = threadIdx.x; i < 2 * S; i += blockDim.x)
                if (at[i]) {
                    atomicAdd(&tot[i], at[i]);
                    atomicMax(&gmax[i], amax[i]);
                    atomicMin(&gmin[i], amin[i]);
                }
    } else if (vb - ns - nw < ck) {
        // one chunk of a big node: partial sum, then the last chunk of the
        // node records its statistics
        int32_t q = (int32_t)(vb - ns - nw);
        int32_t v = chunk_node[q];
        int32_t s = nseg[v];
        if (!gmask[s]) return;
        int sd = side[v];
        int32_t b = chunk_beg[q], e = min(b + kNodeChunk, noff[v + 1]);
        int32_t g = gather_sum(b, e - b, threadIdx.x, kBlock, inc, cc, pk, nzb, sd);
        g = block_sum(g, lds);
        if (threadIdx.x == 0) {
            atomicAdd(&gain[v], g);
            if (!stats) return;
            atomics_done();
            int32_t bi = chunk_big[q];
            if (atomicAdd(&big_done[bi], 1) == big_chunks[bi] - 1) {
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                int32_t gv = __hip_atomic_load(&gain[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (sel_list(s, sd, gv, mode)) {
                    int32_t c = 2 * s + sd;
                    atomicAdd(&tot[c], 1);
                    atomicMax(&gmax[c], gv);
                    atomicMin(&gmin[c], gv);
                }
            }
        }
    }
}

// Whether the node pass stages: on levels of many pins, five a node at least.  By
// a thread each / staged, ids near / far apart, on sides that cut few hyperedges:
// 1 M nodes of 4 incidences 27, 42 / 39, 47 us; 2 M of 4 31, 58 / 37, 58, of 6 43,
// 90 / 43, 86; 5 M of 6 102, 217 / 95, 221, of 8 138, 306 / 116, 302; 256 netlists of
// 5.4 (9.9 M nodes) 435 / 372; coarse levels of 0.3 M nodes and 104 M pins, degrees
// from a few to thousands, 794 / 623 and 1214 / 919.
inline bool gn_staged(const Level &L)
{
    return L.N >= (1 << 18) && (int64_t)L.P >= std::max<int64_t>(5 * (int64_t)L.N, 1 << 23);
}

// Blocks of the node pass that end in the lists' atomics, at most: each costs
// some 9 ns there, so fewer where they have little else to do.  At 512, 1024 and
// 2048: 300 K nodes of no incidence 11, 13, 18 us, of 4 16, 17, 22; 600 K of none
// 13, 16, 19, of 4 21, 22, 30; 1 M of none 16, 18, 27, of 4 30, 27, 37; 3 M of 4
// 56, 41, 42.
inline int64_t gn_blocks(const Level &L)
{
    if (gn_staged(L)) return 2048;
    return L.N >= (3 << 18) && (int64_t)L.P >= L.N / 16 ? 1024 : 512;
}

// The same of its blocks of listed nodes, four at a time.  At 512, 1024 and 2048:
// 17 K nodes of 40 incidences 19, 20, 24 us, 60 K 54, 39, 45, 150 K of 100 92, 66, 74.
inline int64_t gn_wave_blocks(const Level &L) { return L.N >= (1 << 15) ? 1024 : 512; }

// Per-list counts and gain extremes after a gain update (what the node pass
// records otherwise); empties the move log.  Chunked: the lists of a chunk
// aggregate in LDS and end in one atomic each.
__global__ __launch_bounds__(kBlock) void k_gain_stats(int32_t N, const int32_t *nseg, const uint8_t *gmask,
                                                       const uint8_t *side, const int32_t *gain,
                                                       const uint8_t *mode, int32_t *tot, int32_t *gmax,
                                                       int32_t *gmin, int32_t *counts,
                                                       const int32_t *go)
{
    __shared__ int32_t at[kAggLists], amax[kAggLists], amin[kAggLists];
    if (go && *go == 0) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) counts[0] = 0;
    int64_t lo, hi;
    reduce_chunk(N, gridDim.x, blockIdx.x, lo, hi);
    if (lo >= hi) return;
    int32_t c0 = 2 * nseg[lo], nl = 2 * nseg[hi - 1] + 2 - c0;
    bool local = nl <= kAggLists;
    for (int i = threadIdx.x; i < kAggLists; i += blockDim.x) {
        at[i] = 0;
        amax[i] = INT32_MIN;
        amin[i] = INT32_MAX;
    }
    __syncthreads();
    for (int64_t v = lo + threadIdx.x; v < hi; v += blockDim.x) {
        int32_t s = nseg[v];
        if (!gmask[s]) continue;
        int sd = side[v];
        int32_t g = gain[v];
        if (!sel_list(s, sd, g, mode)) continue;
        int32_t c = 2 * s + sd;
        if (local) {
            atomicAdd(&at[c - c0], 1);
            atomicMax(&amax[c - c0], g);
            atomicMin(&amin[c - c0], g);
        } else {
            atomicAdd(&tot[c], 1);
            atomicMax(&gmax[c], g);
            atomicMin(&gmin[c], g);
        }
    }
    __syncthreads();
    if (local)
        for (int i = threadIdx.x; i < nl; i += blockDim.x)
            if (at[i]) {
                atomicAdd(&tot[c0 + i], at[i]);
                atomicMax(&gmax[c0 + i], amax[i]);
                atomicMin(&gmin[c0 + i], amin[i]);
            }
}

// ---- radix select ----------------------------------------------------------------------

struct SelView {
    const int32_t *gain, *nseg, *nbase;
    const uint8_t *side, *mode;
    const int32_t *m;
    int idbits;  // bits of the largest local node id of the level
};

// Selection key of a node in its list: u = gmax - gain (ascending u is
// descending gain) above the node's local id, so ascending keys are the
// (gain desc, id asc) order and every key of a list is distinct.
__device__ __forceinline__ uint64_t sel_key(int32_t gmax, int32_t g, uint32_t lid, int idbits)
{
    return ((uint64_t)(uint32_t)((int64_t)gmax - g) << idbits) | lid;
}

// Width in bits of a list's keys, from its gain extremes.
__device__ __forceinline__ int sel_kbits(int32_t gmax, int32_t gmin, int idbits)
{
    return bitlen_u32((uint32_t)((int64_t)gmax - gmin)) + idbits;
}

// Digit (12 bits, from the top of the T-bit key) of key k at pass p, or -1
// when k does not carry the prefix fixed by the earlier passes.
__device__ __forceinline__ int sel_digit_k(uint64_t k, int T, int p, uint64_t pre)
{
    int hi = T - kDigit * p;
    if (hi <= 0) return (p == 0 && T == 0) ? 0 : -1;  // a 0-bit key: one bin
    int lo = hi - kDigit > 0 ? hi - kDigit : 0;
    if (p > 0 && hi < 64 && ((k ^ pre) >> hi) != 0) return -1;
    return (int)((k >> lo) & ((1ull << (hi - lo)) - 1ull));
}

// Pick of list c after pass p: the digit holding the rem-th key.  One
// workgroup.  Clears the bins it read.  clip > 0 (balance rounds): the list
// may also stop at a whole bin once the keys up to its end are at most clip;
// the balance finish then orders them and keeps the first rsel.
__device__ void sel_pick_list(const SelState &st, int32_t c, int p, int idbits, const uint8_t *mode,
                              const int32_t *m, int64_t *lds, int32_t clip)
{
    __shared__ int sbin;
    __shared__ int32_t sbefore, sin_;
    uint32_t *hc = st.hist + (int64_t)c * kBins;
    if (p == 0) {
        // the number to choose: Algorithm 5 takes min(|L0|, |L1|) from both
        // lists, Algorithm 3 and the balance step at most ceil(sqrt n)
        if (threadIdx.x == 0) {
            int32_t s = c >> 1, sd = c & 1;
            uint8_t md = mode[s];
            int64_t r = 0;
            if ((md >> sd) & 1) {
                int64_t t = st.tot[c];
                if (md & kMinPair) {
                    int64_t o = st.tot[c ^ 1];
                    r = t < o ? t : o;
                } else {
                    r = t < (int64_t)m[s] ? t : (int64_t)m[s];
                }
            }
            st.rsel[c] = (int32_t)r;
            st.rem[c] = (int32_t)r;
            st.kpre[c] = 0;
            bool whole = r > 0 && r == st.tot[c];  // the whole list: no digit needed
            st.kthr[c] = whole ? ~0ull : 0ull;
            st.kbits[c] = r > 0 ? sel_kbits(st.gmax[c], st.gmin[c], idbits) : 0;
            st.done[c] = r == 0 || whole;
            if (r == 0 || whole) atomicSub(&st.ctl[0], 1);
        }
        __syncthreads();
    }
    int per = kBins / kBlock;
    if (st.done[c]) {
        // nothing to choose: still clear what pass 0 counted for this list
        if (p == 0)
            for (int j = 0; j < per; j++) hc[threadIdx.x * per + j] = 0;
        __syncthreads();
        return;
    }
    int32_t r = st.rem[c];
    int64_t loc = 0;
    for (int j = 0; j < per; j++) loc += hc[threadIdx.x * per + j];
    int64_t tot;
    int64_t ex = block_excl_scan(loc, lds, &tot);
    if (threadIdx.x == 0) sbin = -1;
    __syncthreads();
    if (ex < r && r <= ex + loc) {
        int64_t acc = ex;
        for (int j = 0; j < per; j++) {
            int64_t x = hc[threadIdx.x * per + j];
            if (acc + x >= r) {
                sbin = threadIdx.x * per + j;
                sbefore = (int32_t)acc;
                sin_ = (int32_t)x;
                break;
            }
            acc += x;
        }
    }
    __syncthreads();
    for (int j = 0; j < per; j++) hc[threadIdx.x * per + j] = 0;
    if (threadIdx.x == 0 && sbin >= 0) {
        int T = st.kbits[c];
        int hi = T - kDigit * p, lo = hi - kDigit > 0 ? hi - kDigit : 0;
        int32_t left = r - sbefore;
        uint64_t pre = st.kpre[c] | ((uint64_t)sbin << lo);
        st.kpre[c] = pre;
        st.rem[c] = left;
        // done when the whole bin is taken or the bin is a single key, or
        // (clip) when the keys through the end of the bin fit the finish
        if (left == sin_ || lo == 0 || (clip > 0 && (int64_t)st.rsel[c] - left + sin_ <= clip)) {
            st.kthr[c] = pre | (lo ? ((1ull << lo) - 1ull) : 0ull);
            st.done[c] = 1;
            atomicSub(&st.ctl[0], 1);
        }
    }
    __syncthreads();
}

// A list of a segment without nodes chooses nothing.
__device__ __forceinline__ void empty_segment_done(const SelState &st, int32_t s)
{
    for (int sd = 0; sd < 2; sd++) {
        int32_t c = 2 * s + sd;
        st.rsel[c] = 0;
        st.rem[c] = 0;
        st.done[c] = 1;
        atomicSub(&st.ctl[0], 1);
    }
}

// Per-segment tickets: every workgroup whose node range meets segment s
// counts itself in tick[s] after its histogram is flushed; the last one does
// the picks of the segment's two lists.  Segments without nodes are settled
// in pass 0 by the workgroup holding their position.
__device__ void seg_tickets_pick(int32_t N, int p, int32_t nlists, int idbits, const SelView &sv,
                                 const SelState &st, int64_t v0, int64_t *lds, int32_t clip)
{
    __shared__ int32_t picks[kBlock];
    __shared__ int npick;
    int64_t v1 = v0 + kSelNodes < N ? v0 + kSelNodes : N;
    int32_t S = nlists / 2;
    if (p == 0) {
        for (int64_t v = v0 + threadIdx.x; v < v1; v += blockDim.x) {
            int32_t lo = v == 0 ? -1 : sv.nseg[v - 1], hi = sv.nseg[v];
            for (int32_t s = lo + 1; s < hi; s++) empty_segment_done(st, s);
        }
        if (v1 == N)
            for (int32_t s = sv.nseg[N - 1] + 1 + (int32_t)threadIdx.x; s < S; s += blockDim.x)
                empty_segment_done(st, s);
    }
    atomics_done();  // (the histograms are written by atomics alone)
    __syncthreads();
    if (threadIdx.x == 0) npick = 0;
    __syncthreads();
    int32_t sf = sv.nseg[v0], sl = sv.nseg[v1 - 1];
    for (int32_t base = sf; base <= sl; base += blockDim.x) {
        int32_t s = base + (int32_t)threadIdx.x;
        if (s <= sl) {
            int32_t a = sv.nbase[s], b = sv.nbase[s + 1];
            if (b > a) {
                int32_t nb = (b - 1) / kSelNodes - a / kSelNodes + 1;
                if (atomicAdd(&st.tick[s], 1) == nb - 1) {
                    st.tick[s] = 0;
                    picks[atomicAdd(&npick, 1)] = s;
                }
            }
        }
        __syncthreads();
        int np = npick;
        if (np > 0) {
            if (threadIdx.x == 0) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            __syncthreads();
            for (int i = 0; i < np; i++) {
                sel_pick_list(st, 2 * picks[i], p, idbits, sv.mode, sv.m, lds, clip);
                sel_pick_list(st, 2 * picks[i] + 1, p, idbits, sv.mode, sv.m, lds, clip);
            }
        }
        __syncthreads();
        if (threadIdx.x == 0) npick = 0;
        __syncthreads();
    }
}

// Histogram of global pass p; the last workgroup to finish does the picks
// when there are few lists, the last one of each segment when there are many.
__global__ __launch_bounds__(kBlock) void k_select_pass(int32_t N, int p, int32_t nlists, int idbits,
                                                        SelView sv, SelState st, int fused,
                                                        const int32_t *go, int32_t clip)
{
    __shared__ uint32_t h[2 * kBins];
    __shared__ int64_t lds[16];
    __shared__ int last;
    const int32_t gv = go ? *go : 1, ctl = st.ctl[0];  // loaded together
    if (gv == 0) return;
    if (p > 0 && ctl <= 0) return;
    int64_t v0 = (int64_t)blockIdx.x * kSelNodes;
    if (v0 < N) {
        int64_t v1 = v0 + kSelNodes < N ? v0 + kSelNodes : N;
        int32_t cbase = 2 * sv.nseg[v0];
        bool use_lds = 2 * sv.nseg[v1 - 1] + 1 - cbase < 2;
        if (use_lds) {
            for (int i = threadIdx.x; i < 2 * kBins; i += blockDim.x) h[i] = 0;
            __syncthreads();
            // one segment: its two lists' state once per workgroup, then only
            // each node's side and gain
            int32_t s = cbase / 2, nb0 = sv.nbase[s];
            uint8_t md = sv.mode[s];
            bool on0 = md & 1, on1 = (md >> 1) & 1;
            if (p > 0) {
                on0 = on0 && !st.done[cbase];
                on1 = on1 && !st.done[cbase + 1];
            } else {  // a list taken whole needs no histogram
                int64_t t0 = st.tot[cbase], t1 = st.tot[cbase + 1], ms = sv.m[s];
                bool pair = md & kMinPair;
                on0 = on0 && (pair ? min(t0, t1) : min(t0, ms)) != t0;
                on1 = on1 && (pair ? min(t1, t0) : min(t1, ms)) != t1;
            }
            int32_t gx0 = st.gmax[cbase], gx1 = st.gmax[cbase + 1];
            int T0 = p == 0 ? sel_kbits(gx0, st.gmin[cbase], idbits) : st.kbits[cbase];
            int T1 = p == 0 ? sel_kbits(gx1, st.gmin[cbase + 1], idbits) : st.kbits[cbase + 1];
            uint64_t pr0 = p == 0 ? 0ull : st.kpre[cbase], pr1 = p == 0 ? 0ull : st.kpre[cbase + 1];
            bool nonneg = md & kGainNonNeg;
            if (on0 || on1) {
#pragma unroll 4
                for (int64_t v = v0 + threadIdx.x; v < v1; v += blockDim.x) {
                    int sd = sv.side[v];
                    int32_t g = sv.gain[v];
                    if (!(sd ? on1 : on0) || (nonneg && g < 0)) continue;
                    uint64_t k = sel_key(sd ? gx1 : gx0, g, (uint32_t)(v - nb0), idbits);
                    int dig = sel_digit_k(k, sd ? T1 : T0, p, sd ? pr1 : pr0);
                    if (dig >= 0) atomicAdd(&h[sd * kBins + dig], 1u);
                }
            }
        }
        for (int64_t v = v0 + threadIdx.x; !use_lds && v < v1; v += blockDim.x) {
            int32_t s = sv.nseg[v];
            int sd = sv.side[v];
            int32_t g = sv.gain[v];
            if (!sel_list(s, sd, g, sv.mode)) continue;
            int32_t c = 2 * s + sd;
            if (p > 0 && st.done[c]) continue;
            if (p == 0) {  // a list taken whole needs no histogram
                int64_t t = st.tot[c];
                int64_t r = (sv.mode[s] & kMinPair) ? min(t, (int64_t)st.tot[c ^ 1]) : min(t, (int64_t)sv.m[s]);
                if (r == t) continue;
            }
            uint64_t k = sel_key(st.gmax[c], g, (uint32_t)(v - sv.nbase[s]), idbits);
            // pass 0 runs before the pick has fixed the key width: from the
            // extremes the node pass recorded
            int T = p == 0 ? sel_kbits(st.gmax[c], st.gmin[c], idbits) : st.kbits[c];
            int dig = sel_digit_k(k, T, p, p == 0 ? 0ull : st.kpre[c]);
            if (dig < 0) continue;
            atomicAdd(&st.hist[(int64_t)c * kBins + dig], 1u);
        }
        if (use_lds) {
            __syncthreads();
            for (int i = threadIdx.x; i < 2 * kBins; i += blockDim.x) {
                uint32_t x = h[i];
                if (x) atomicAdd(&st.hist[(int64_t)(cbase + i / kBins) * kBins + (i % kBins)], x);
            }
        }
    }
    if (!fused) return;
    if (fused == 2) {
        seg_tickets_pick(N, p, nlists, idbits, sv, st, v0, lds, clip);
        return;
    }
    // ticket: the last workgroup sees every histogram
    atomics_done();  // (written by atomics alone)
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = atomicAdd(&st.ctl[1], 1);
        last = t == (int)gridDim.x - 1;
        if (last) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
    if (!last) return;
    for (int32_t c = 0; c < nlists; c++) sel_pick_list(st, c, p, idbits, sv.mode, sv.m, lds, clip);
    if (threadIdx.x == 0) st.ctl[1] = 0;
}

__global__ __launch_bounds__(kBlock) void k_select_pick(int32_t nlists, int p, int idbits, SelView sv,
                                                        SelState st, const int32_t *go, int32_t clip)
{
    __shared__ int64_t lds[16];
    const int32_t gv = go ? *go : 1, ctl = st.ctl[0];  // loaded together
    if (gv == 0) return;
    if (p > 0 && ctl <= 0) return;
    int32_t c = blockIdx.x;
    if (c >= nlists) return;
    sel_pick_list(st, c, p, idbits, sv.mode, sv.m, lds, clip);
}

__device__ __forceinline__ bool sel_chosen(int64_t v, const SelView &sv, const SelState &st)
{
    int32_t s = sv.nseg[v];
    int sd = sv.side[v];
    int32_t g = sv.gain[v];
    if (!sel_list(s, sd, g, sv.mode)) return false;
    int32_t c = 2 * s + sd;
    if (st.rsel[c] <= 0) return false;
    return sel_key(st.gmax[c], g, (uint32_t)(v - sv.nbase[s]), sv.idbits) <= st.kthr[c];
}

// ---- small segments: the whole selection and the moves in one workgroup --------------------

// Workgroups of a selection: threads, and nodes per thread, kept in registers
// (the flipping kind holds both lists' thresholds as well; past 128 registers a
// thread a workgroup of 1024 would spill).  The smallest that holds the level's
// largest segment: items past a segment's end cost loads and compares all the
// same (balance on up to 2048 nodes: 256 threads of 32 nodes 13 us, of 8 10.7;
// up to 8192: 256 of 32 18.9 us, 512 of 16 15.0, 1024 of 8 15.1; up to 16384:
// 768 of 32 19.6, 1024 of 16 16.4).
constexpr int32_t kSegSelectMax = 16384;
constexpr int kSegKeys = 128;  // balance candidates: ceil(sqrt(kSegSelectMax))

// One workgroup per segment of at most TH * ITEMS nodes: each list's
// r-th key by the same 12-bit radix select as the multi-workgroup passes,
// with the segment's gains in registers and the histogram in LDS, then the
// moves (bf.side is written): kind 0 flips the chosen nodes of both lists
// (Algorithm 3 and the swap of Algorithm 5); kind 1 orders the chosen nodes
// of the over-weight side (by counting, their weights and incidence ranges
// gathered meanwhile) and the workgroup takes the balance prefix (Algorithm
// 5).  The chosen set is the one the multi-workgroup path chooses: the same
// keys, the same r.
template <int KIND, int TH, int ITEMS>
__global__ __launch_bounds__(TH) void k_seg_select(int32_t S, SelView sv, SelState st, int idbits_lv,
                                                           const int32_t *nw,
                                                           unsigned long long *segw, BalFinish bf,
                                                           const int32_t *go)
{
    constexpr int kSegItems = ITEMS;
    constexpr int32_t kCap = TH * kSegItems;
    constexpr int kKeys = kSegKeys;
    __shared__ uint32_t hist[kBins];
    __shared__ int64_t lds64[16];
    __shared__ int32_t sbin, sbefore, sin_;
    __shared__ uint64_t keys[kKeys], sorted[KIND == 1 ? kKeys : 1];
    __shared__ uint8_t sdl[kCap];  // the segment's sides
    __shared__ int32_t nkeys;
    // the round's flag is loaded together with what the block reads next
    const int32_t gv = go ? *go : 1;
    const int32_t s = blockIdx.x, a0 = sv.nbase[s], n = sv.nbase[s + 1] - a0;
    const uint8_t md = sv.mode[s];
    int64_t bnd = 0, brm = 0, bm0 = 0, bm1 = 0;  // balance: the segment's state, loaded early
    if (KIND == 1) {
        bnd = bf.need[s];
        brm = bf.room[s];
        bm0 = bf.bal_moved[2 * s];
        bm1 = bf.bal_moved[2 * s + 1];
    }
    if (gv == 0) return;
    const int idbits = idbits_lv;
    int32_t g[kSegItems];
    uint64_t sbits = 0, ebits = 0;  // bit j: item j's side, item j eligible for its side's list
    // per list: size and gain extremes, from the gains just loaded
    int32_t lc[2] = {0, 0}, lmax[2] = {INT32_MIN, INT32_MIN}, lmin[2] = {INT32_MAX, INT32_MAX};
    // the segment's sides by aligned 4-byte words (a word never leaves the
    // memory page of the bytes it covers) and its gains (indices past the
    // segment read its node 0): loads in flight together
    const uint8_t *sp = sv.side + a0;
    int32_t off0 = (int32_t)((uintptr_t)sp & 3), nwd = (off0 + n + 3) >> 2;
    const uint32_t *wp = (const uint32_t *)(sp - off0);
    constexpr int kW = kCap / 4 / TH + 1;
    uint32_t xw[kW];
    if (md && n > 0) {
#pragma unroll
        for (int q = 0; q < kW; q++) xw[q] = wp[min(q * TH + (int32_t)threadIdx.x, nwd - 1)];
#pragma unroll
        for (int j = 0; j < kSegItems; j++) {
            int32_t i = j * TH + (int32_t)threadIdx.x;
            g[j] = sv.gain[a0 + (i < n ? i : 0)];
        }
    }
    if (!md) return;
    // the histogram starts cleared (each radix pass clears the bins it read),
    // the balance key list empty
    for (int i = threadIdx.x; i < kBins; i += TH) hist[i] = 0;
    if (threadIdx.x == 0) nkeys = 0;
    if (n > 0) {
        // the sides staged in LDS
#pragma unroll
        for (int q = 0; q < kW; q++) {
            int32_t w = q * TH + (int32_t)threadIdx.x;
#pragma unroll
            for (int b = 0; b < 4; b++) {
                int32_t i = 4 * w + b - off0;
                if (w < nwd && i >= 0 && i < n) sdl[i] = (uint8_t)(xw[q] >> (8 * b));
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSegItems; j++) {
        int32_t i = j * TH + (int32_t)threadIdx.x;
        int sd = i < n ? sdl[i] : 0;
        sbits |= (uint64_t)sd << j;
        if (i < n && ((md >> sd) & 1) && !((md & kGainNonNeg) && g[j] < 0)) {  // sel_list
            ebits |= 1ull << j;
            lc[sd]++;
            lmax[sd] = max(lmax[sd], g[j]);
            lmin[sd] = min(lmin[sd], g[j]);
        }
    }
    {
        __shared__ int32_t red[TH / 64][6];
        int32_t x[6] = {lc[0], lc[1], lmax[0], lmax[1], lmin[0], lmin[1]};
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            x[0] += __shfl_xor(x[0], o, 64);
            x[1] += __shfl_xor(x[1], o, 64);
            x[2] = max(x[2], __shfl_xor(x[2], o, 64));
            x[3] = max(x[3], __shfl_xor(x[3], o, 64));
            x[4] = min(x[4], __shfl_xor(x[4], o, 64));
            x[5] = min(x[5], __shfl_xor(x[5], o, 64));
        }
        if ((threadIdx.x & 63) == 0)
            for (int q = 0; q < 6; q++) red[threadIdx.x >> 6][q] = x[q];
        __syncthreads();
        lc[0] = red[0][0];
        lc[1] = red[0][1];
        lmax[0] = red[0][2];
        lmax[1] = red[0][3];
        lmin[0] = red[0][4];
        lmin[1] = red[0][5];
#pragma unroll 1
        for (int w = 1; w < TH / 64; w++) {
            lc[0] += red[w][0];
            lc[1] += red[w][1];
            lmax[0] = max(lmax[0], red[w][2]);
            lmax[1] = max(lmax[1], red[w][3]);
            lmin[0] = min(lmin[0], red[w][4]);
            lmin[1] = min(lmin[1], red[w][5]);
        }
        // (red is not written again: no barrier before what follows)
    }
    uint64_t thr[2] = {0, 0};
    int32_t rr[2] = {0, 0};
    constexpr int per = (kBins + TH - 1) / TH;  // bins per thread (the last ones may run past kBins)
    for (int sd = 0; sd < 2; sd++) {
        int32_t c = 2 * s + sd;
        int64_t r = 0;
        if ((md >> sd) & 1) {
            int64_t t = lc[sd];
            if (md & kMinPair) {
                int64_t o = lc[sd ^ 1];
                r = t < o ? t : o;
            } else {
                r = t < (int64_t)sv.m[s] ? t : (int64_t)sv.m[s];
            }
        }
        rr[sd] = (int32_t)r;
        if (r == 0) continue;
        if (r == lc[sd]) {  // the whole list: no pass needed
            thr[sd] = ~0ull;
            continue;
        }
        int32_t gmax = lmax[sd];
        int T = bitlen_u32((uint32_t)((int64_t)gmax - lmin[sd])) + idbits;
        uint64_t pre = 0;
        int32_t rem = (int32_t)r;
        for (int p = 0;; p++) {
            int hi = T - kDigit * p, lo = hi - kDigit > 0 ? hi - kDigit : 0;
            uint64_t mine = ebits & (sd ? sbits : ~sbits);
#pragma unroll
            for (int j = 0; j < kSegItems; j++) {
                if (!((mine >> j) & 1)) continue;
                uint64_t k = sel_key(gmax, g[j], (uint32_t)(j * TH + threadIdx.x), idbits);
                if (p > 0 && ((k ^ pre) >> hi) != 0) continue;
                int dig = hi > 0 ? (int)((k >> lo) & ((1ull << (hi - lo)) - 1ull)) : 0;
                atomicAdd(&hist[dig], 1u);
            }
            __syncthreads();
            int64_t loc = 0;
            for (int j = 0; j < per; j++)
                if (threadIdx.x * per + j < kBins) loc += hist[threadIdx.x * per + j];
            // exclusive scan of the bin sums over the workgroup: the barrier
            // above already separates these LDS writes from the last pass's
            // reads, and the one below the bin pick from the next pass's writes
            int64_t ex = wave_incl_scan(loc);
            if ((threadIdx.x & 63) == 63) lds64[threadIdx.x >> 6] = ex;
            __syncthreads();
            for (int w = 0; w < (int)(threadIdx.x >> 6); w++) ex += lds64[w];
            ex -= loc;
            if (ex < rem && rem <= ex + loc) {
                int64_t acc = ex;
                for (int j = 0; j < per; j++) {
                    int64_t x = threadIdx.x * per + j < kBins ? hist[threadIdx.x * per + j] : 0;
                    if (acc + x >= rem) {
                        sbin = threadIdx.x * per + j;
                        sbefore = (int32_t)acc;
                        sin_ = (int32_t)x;
                        break;
                    }
                    acc += x;
                }
            }
            // only this thread reads its bins: clear them for the next pass
            for (int j = 0; j < per; j++)
                if (threadIdx.x * per + j < kBins) hist[threadIdx.x * per + j] = 0;
            __syncthreads();
            // (the next pass writes the pick only after two more barriers)
            int32_t bin = sbin, left = rem - sbefore, inb = sin_;
            pre |= (uint64_t)bin << lo;
            rem = left;
            if (left == inb || lo == 0) {
                thr[sd] = pre | (lo ? ((1ull << lo) - 1ull) : 0ull);
                break;
            }
        }
    }
    if (threadIdx.x == 0) {
        st.rsel[2 * s] = rr[0];
        st.rsel[2 * s + 1] = rr[1];
    }
    if (KIND == 0) {
        // flip the chosen nodes of both lists
        int64_t d01 = 0;  // weight moving from side 0 to side 1
#pragma unroll
        for (int j = 0; j < kSegItems; j++) {
            if (!((ebits >> j) & 1)) continue;
            int sd = (sbits >> j) & 1;
            if (rr[sd] == 0) continue;
            uint32_t lid = (uint32_t)(j * TH + threadIdx.x);
            if (sel_key(lmax[sd], g[j], lid, idbits) > thr[sd]) continue;
            int32_t v = a0 + (int32_t)lid;
            int64_t w = nw[v];
            bf.side[v] = (uint8_t)(1 - sd);
            d01 += sd ? -w : w;
        }
        d01 = block_sum(d01, lds64);
        if (threadIdx.x == 0 && d01 != 0) {
            atomicAdd(&segw[2 * s], (unsigned long long)(-d01));
            atomicAdd(&segw[2 * s + 1], (unsigned long long)d01);
        }
        return;
    }
    // balance: the chosen nodes of the over-weight side, sorted, then the prefix
    int h = (md & kList1) ? 1 : 0;
    if (rr[h] > 0) {
        uint64_t mine = ebits & (h ? sbits : ~sbits);
#pragma unroll
        for (int j = 0; j < kSegItems; j++) {
            if (!((mine >> j) & 1)) continue;
            uint32_t lid = (uint32_t)(j * TH + threadIdx.x);
            if (sel_key(lmax[h], g[j], lid, idbits) > thr[h]) continue;
            keys[atomicAdd(&nkeys, 1)] = gain_order_key(g[j], (uint32_t)(a0 + (int32_t)lid));
        }
    }
    __syncthreads();
    int32_t cnt = nkeys;
    // counting order (as block_rank_sort), each chosen node's weight and
    // incidence range loaded while its rank is counted (for the finish)
    __shared__ int32_t pw[kKeys], pnb[kKeys], pne[kKeys];
    const bool logm = bf.ml.cnode != nullptr;
    int tpc = 1;
    while (tpc < 16 && cnt * 2 * tpc <= TH) tpc <<= 1;
    for (int base = 0; base < cnt * tpc; base += TH) {
        int t = base + (int)threadIdx.x, i = t / tpc, part = t & (tpc - 1);
        uint64_t x = keys[i < cnt ? i : 0];
        int32_t v = (int32_t)(uint32_t)(x & 0xffffffffu), xw = 0, xb = 0, xe = 0;
        if (i < cnt && part == 0) {
            xw = nw[v];
            if (logm) {
                xb = bf.ml.noff[v];
                xe = bf.ml.noff[v + 1];
            }
        }
        int r = 0;
        if (i < cnt) {
#pragma unroll 8
            for (int j = part; j < cnt; j += tpc) r += keys[j] < x;
        }
        for (int o = 1; o < tpc; o <<= 1) r += __shfl_xor(r, o, 64);
        if (i < cnt && part == 0) {
            sorted[r] = x;
            pw[r] = xw;
            pnb[r] = xb;
            pne[r] = xe;
        }
    }
    __syncthreads();
    bal_finish_block(s, sorted, cnt, bf, h, bnd, brm, bm0, bm1, BalPre{pw, pnb, pne});
}

// ---- moves ---------------------------------------------------------------------------------

__global__ __launch_bounds__(kBlock) void k_flip(int32_t N, SelView sv, SelState st, uint8_t *side,
                                                 const int32_t *nw, unsigned long long *segw,
                                                 const int32_t *go)
{
    __shared__ unsigned long long dw[kAggLists / 2];  // two's complement sums
    if (go && *go == 0) return;
    int64_t lo, hi;
    reduce_chunk(N, gridDim.x, blockIdx.x, lo, hi);
    if (lo >= hi) return;
    int32_t s0 = sv.nseg[lo], ns = sv.nseg[hi - 1] + 1 - s0;
    bool local = 2 * ns <= kAggLists;
    for (int i = threadIdx.x; i < kAggLists / 2; i += blockDim.x) dw[i] = 0;
    __syncthreads();
    for (int64_t v = lo + threadIdx.x; v < hi; v += blockDim.x) {
        if (!sel_chosen(v, sv, st)) continue;
        int32_t sd = side[v];
        int64_t w = nw[v];
        side[v] = (uint8_t)(1 - sd);
        int32_t s = sv.nseg[v];
        // weight moving from side 0 to side 1 (negative: the other way)
        if (local) {
            atomicAdd(&dw[s - s0], (unsigned long long)(sd ? -w : w));
        } else {
            atomicAdd(&segw[2 * s + sd], (unsigned long long)(-w));
            atomicAdd(&segw[2 * s + 1 - sd], (unsigned long long)w);
        }
    }
    __syncthreads();
    if (local)
        for (int i = threadIdx.x; i < ns; i += blockDim.x)
            if (dw[i]) {
                atomicAdd(&segw[2 * (s0 + i)], 0ull - dw[i]);
                atomicAdd(&segw[2 * (s0 + i) + 1], dw[i]);
            }
}

__global__ __launch_bounds__(kBlock) void k_gather(int32_t N, SelView sv, SelState st, int32_t *ccount,
                                                   uint64_t *cand, int32_t stride, const int32_t *go)
{
    if (go && *go == 0) return;
    int64_t v0 = (int64_t)blockIdx.x * blockDim.x, v = v0 + threadIdx.x;
    int64_t vl = min(v0 + (int64_t)blockDim.x, (int64_t)N) - 1;
    int32_t s0 = sv.nseg[v0];
    if (s0 != sv.nseg[vl]) {  // workgroup over several segments: node by node
        if (v >= N || !sel_chosen(v, sv, st)) return;
        int32_t s = sv.nseg[v];
        int32_t at = atomicAdd(&ccount[s], 1);
        if (at < stride) cand[(int64_t)s * stride + at] = gain_order_key(sv.gain[v], (uint32_t)v);
        return;
    }
    // one segment: its lists' state once, one append atomic per wavefront
    uint8_t md = sv.mode[s0];
    int32_t nb0 = sv.nbase[s0];
    bool chosen = false;
    int32_t g = 0;
    if (v < N) {
        int sd = sv.side[v];
        g = sv.gain[v];
        int32_t c = 2 * s0 + sd;
        chosen = ((md >> sd) & 1) && !((md & kGainNonNeg) && g < 0) && st.rsel[c] > 0 &&
                 sel_key(st.gmax[c], g, (uint32_t)(v - nb0), sv.idbits) <= st.kthr[c];
    }
    int32_t at = lds_wave_slot(chosen, &ccount[s0]);
    if (at >= 0 && at < stride) cand[(int64_t)s0 * stride + at] = gain_order_key(g, (uint32_t)v);
}

// ---- per-round modes: also reset the selection state of the lists --------------------------

__device__ __forceinline__ void reset_lists(SelState st, int32_t s)
{
    for (int sd = 0; sd < 2; sd++) {
        int32_t c = 2 * s + sd;
        st.tot[c] = 0;
        st.gmax[c] = INT32_MIN;
        st.gmin[c] = INT32_MAX;
        st.done[c] = 0;
    }
    st.tick[s] = 0;
}

// Algorithm 3 loop test per segment: P0 below its share and P1 non-empty.
// Round counters without a launch of their own: round ri counts its active
// segments in slot ri % 3, reads the previous round's count from slot
// (ri - 1) % 3 (complete) and clears slot (ri + 1) % 3 for the next round.
__device__ __forceinline__ int32_t round_counters(int32_t *go, int32_t ri, int32_t s)
{
    int32_t prev = ri > 0 ? go[4 + (ri + 2) % 3] : 0;
    if (s == 0) {
        go[4 + (ri + 1) % 3] = 0;
        go[1] = prev;
        if (prev) go[2] += 1;
        go[3] = 0;
    }
    return prev;
}

__global__ void k_round_initial(int32_t S, int32_t j, const int32_t *nbase, const int32_t *coarsest,
                                const int32_t *k0, const int32_t *k1, const int64_t *W,
                                const unsigned long long *segw, int32_t *cnt1, int32_t ri,
                                uint8_t *mode, uint8_t *gmask, int32_t *m, SelState st, int32_t *go)
{
    int32_t s = blockIdx.x * blockDim.x + threadIdx.x;
    bool first = ri == 0;
    if (s == 0) st.ctl[0] = 2 * S;
    int32_t prev = round_counters(go, ri, s);
    int32_t *cur = go + 4 + ri % 3;
    if (s >= S) return;
    if (prev == 0 && !first) {  // the previous round found nothing to do
        mode[s] = 0;
        gmask[s] = 0;
        return;
    }
    uint8_t md = 0;
    if (coarsest[s] == j) {
        int32_t n = nbase[s + 1] - nbase[s];
        if (first) cnt1[s] = n;
        else cnt1[s] -= st.rsel[2 * s + 1];
        int64_t ks = (int64_t)k0[s] + k1[s];
        bool run = (int64_t)segw[2 * s] * ks < W[s] * (int64_t)k0[s] && cnt1[s] > 0;
        if (run) {
            md = kList1;
            m[s] = (int32_t)ceil_sqrt_i64(n);
            atomicAdd(cur, 1);
        }
    }
    mode[s] = md;
    gmask[s] = md ? 1 : 0;
    reset_lists(st, s);
    st.rsel[2 * s] = 0;
    st.rsel[2 * s + 1] = 0;
}

__global__ void k_round_refine(int32_t S, int32_t j, const int32_t *coarsest, uint8_t *mode,
                               uint8_t *gmask, uint8_t *done, SelState st, int32_t *go)
{
    int32_t s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s == 0) st.ctl[0] = 2 * S;
    if (s >= S) return;
    bool present = coarsest[s] >= j;
    mode[s] = present ? (kList0 | kList1 | kGainNonNeg | kMinPair) : 0;
    gmask[s] = present ? 1 : 0;
    done[s] = present ? 0 : 1;
    reset_lists(st, s);
}

// Balance test per segment: the side over its bound, the excess, the room.
struct RoundBal {
    int32_t S;
    const int32_t *nbase;
    const unsigned long long *segw;
    const int64_t *max0, *max1;
    uint8_t *done, *mode, *gmask;
    int32_t *m;
    int64_t *need, *room;
    int32_t *ccount;
    int32_t *stuck;
    int64_t *bal_moved;
    WinState win;  // windowed selection: its rounds are settled by the next test
};

// A windowed round of segment s after the fact: stuck when it moved nothing
// (and not merely its window), else its share of the level's moved weight.
__device__ __forceinline__ void win_settle(int32_t s, const RoundBal &rb)
{
    const WinState &w = rb.win;
    if (!w.pend[s]) return;
    w.pend[s] = 0;
    if (w.zoom[s]) {
        w.zoom[s] = 0;
        return;
    }
    if (!w.moved[s]) {
        rb.stuck[s] = 1;
        rb.done[s] = 1;
        return;
    }
    w.moved[s] = 0;
    const int h = (rb.mode[s] & kList1) ? 1 : 0;
    rb.bal_moved[2 * s] += w.before[s] - (int64_t)rb.segw[2 * s + h];
    rb.bal_moved[2 * s + 1] += 1;
}

__device__ __forceinline__ void round_balance_seg(int32_t s, const RoundBal &rb, SelState st, int32_t *go,
                                                  int32_t ri)
{
    int32_t S = rb.S;
    const int32_t *nbase = rb.nbase;
    const unsigned long long *segw = rb.segw;
    const int64_t *max0 = rb.max0, *max1 = rb.max1;
    uint8_t *done = rb.done, *mode = rb.mode, *gmask = rb.gmask;
    int32_t *m = rb.m, *ccount = rb.ccount;
    int64_t *need = rb.need, *room = rb.room;
    if (s == 0) st.ctl[0] = 2 * S;
    round_counters(go, ri, s);
    int32_t *cur = go + 4 + ri % 3;
    if (s >= S) return;
    uint8_t md = 0;
    ccount[s] = 0;
    if (rb.win.pend) win_settle(s, rb);
    if (!done[s]) {
        int64_t w0 = (int64_t)segw[2 * s], w1 = (int64_t)segw[2 * s + 1];
        int h = -1;
        if (w0 > max0[s]) h = 0;
        else if (w1 > max1[s]) h = 1;
        if (h < 0) {
            done[s] = 1;
        } else {
            md = h ? kList1 : kList0;
            need[s] = h ? w1 - max1[s] : w0 - max0[s];
            room[s] = h ? max0[s] - w0 : max1[s] - w1;
            m[s] = (int32_t)ceil_sqrt_i64(nbase[s + 1] - nbase[s]);
            atomicAdd(cur, 1);
            if (rb.win.pend) {
                rb.win.pend[s] = 1;
                rb.win.before[s] = h ? w1 : w0;
            }
        }
    }
    mode[s] = md;
    gmask[s] = md ? 1 : 0;
    reset_lists(st, s);
}

__global__ void k_round_balance(RoundBal rb, SelState st, int32_t *go, int32_t ri)
{
    round_balance_seg(blockIdx.x * blockDim.x + threadIdx.x, rb, st, go, ri);
}

// A later balance round's test and the marking of the hyperedges of the nodes
// the previous round moved, in one launch: they are independent (the test
// reads the side weights, the marking the move log, both left by the previous
// round).  Blocks [0, gs) test, the others mark, when the previous round had
// anything to do.
__global__ __launch_bounds__(kBlock) void k_round_balance_log(int64_t gs, RoundBal rb, SelState st, int32_t *go,
                                                              int32_t ri, const int32_t *count,
                                                              const int32_t *cnode, const int32_t *cbeg,
                                                              const int32_t *noff, const int32_t *inc,
                                                              uint32_t *bits, const void *cc, int pk, int32_t *n1,
                                                              const uint8_t *side, int32_t *gain)
{
    if ((int64_t)blockIdx.x < gs) {
        round_balance_seg(blockIdx.x * blockDim.x + threadIdx.x, rb, st, go, ri);
        return;
    }
    // the previous round's counter and its log size, loaded together
    const int32_t prev = go[4 + (ri + 2) % 3], n = count[0];
    if (prev == 0) return;  // the previous round moved nothing
    log_hedges_blocks((int64_t)blockIdx.x - gs, (int64_t)gridDim.x - gs, n, cnode, cbeg, noff, inc, bits, cc, pk,
                      n1, side, gain);
}


}  // namespace bp
