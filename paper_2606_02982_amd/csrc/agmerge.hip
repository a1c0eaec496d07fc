// Aging Priority above the sample-sort limit as a merge of sorted runs
// (Sec. "Aging Priority Scheduling"; internal to the library).
//
// The aged score max(floor, p - rate * max(0, t_now - arrival)) is, for a
// fixed priority p, a non-decreasing function of the arrival: every
// operation (subtraction from t_now, the clamp at 0, the product, the
// subtraction from p, the clamp at the floor) is monotone and IEEE rounding
// keeps it so. Along the FIFO sequence the requests of one priority class
// (the tiers sharing a priority) are therefore already in Aging order, by
// (score, FIFO rank). The Aging order is the merge of those K <= 16 runs,
// with no sort:
//   k_am_count  per tile of 4096 FIFO positions: each class's count
//   k_am_scan   one block: each tile's offset inside each class's run and
//               the runs' starts
//   k_am_place  per tile: each position's aged score (ordered bits) and FIFO
//               position go to its class run, stably
//   k_am_rank   each entry's place: its index in its run plus the entries below
//               it in every other run; writes the permutation and the key (many
//               classes: merges groups of runs first)
// Results are identical to sorting by (score, arrival, index): the scores
// are computed with the same operations as the other paths, and FIFO
// position order is (arrival, index) order.
#include <string.h>

#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace ds {
namespace {

constexpr int kAmTPB = 1024;
constexpr uint32_t kAmTile = 4096;                 // FIFO positions per count/place block
constexpr uint32_t kAmRounds = kAmTile / kAmTPB;   // 4 positions per thread
constexpr uint32_t kAmCls = 16;

struct AmArgs {
    SortInput in;            // arrival, tier, cls, prio, aging parameters; fifo = the FIFO permutation
    uint32_t n, tiles, K;
    uint32_t *cnt;           // [16][tiles]: counts, then each tile's offset in its class's run
    uint8_t *tier;           // [n] each FIFO position's tier (the count writes it, the place reads it)
    uint32_t *cstart;        // [17]: run starts (cstart[K..16] = n)
    uint64_t *rk;            // run keys
    uint32_t *rp;            // run FIFO positions
    uint64_t *hk;            // every kAmStep-th entry of each run (am_step_at), or null
    uint32_t *hp;
    // k_am_rank: K runs, run c from cstart[c * stride] on, in groups of `per`;
    // a group is merged into the output, or into a run of ok, op, ohk, ohp at
    // the same place where these are not null
    uint32_t stride, per;
    uint64_t *ok;
    uint32_t *op;
    uint64_t *ohk;
    uint32_t *ohp;
    uint32_t *perm;
    double *key_out;         // per request, or null
    uint32_t *wait_status;   // zeroed by the first kernel (no waits here), or null
};

__device__ __forceinline__ uint32_t am_tier(const SortInput &in, uint32_t i)
{
    const uint32_t q = in.tier[i];
    return q < kAmCls ? q : kAmCls - 1u;
}

// The aged score, each operation rounded separately (no fused multiply-add).
__device__ __forceinline__ double am_aged(const SortInput &in, uint32_t i, uint32_t q)
{
    double w = in.t_now - in.arrival[i];
    if (w < 0.0) w = 0.0;
    const double d = in.aging_rate * w;
    double e = in.prio[q] - d;
    if (e < in.aging_floor) e = in.aging_floor;
    return e;
}

// Lanes of the wave holding the same 4-bit class (ok lanes only).
__device__ __forceinline__ uint64_t class_peers(uint32_t c, bool ok)
{
    return match_bits<4>(c, __ballot(ok));
}

__global__ __launch_bounds__(kAmTPB) void k_am_count(AmArgs a)
{
    __shared__ uint32_t c[kAmCls];
    const uint32_t t = threadIdx.x, tile = blockIdx.x;
    if (a.wait_status && tile == 0 && t == 0) *a.wait_status = 0;
    if (t < kAmCls) c[t] = 0;
    __syncthreads();
    const uint32_t base = tile * kAmTile;
    uint32_t cl[kAmRounds];
#pragma unroll
    for (uint32_t r = 0; r < kAmRounds; r++) {
        const uint32_t j = base + r * kAmTPB + t;
        uint32_t i = j < a.n ? a.in.fifo[j] : 0u;
        i = i < a.n ? i : 0u;
        const uint32_t q = am_tier(a.in, i);
        if (j < a.n) a.tier[j] = (uint8_t)q;
        cl[r] = j < a.n ? a.in.cls[q] : kAmCls;
    }
#pragma unroll
    for (uint32_t r = 0; r < kAmRounds; r++) {
        const bool ok = cl[r] < kAmCls;
        const uint64_t peers = class_peers(cl[r], ok);
        if (ok && (peers & lanemask_lt()) == 0) atomicAdd(&c[cl[r]], (uint32_t)__popcll(peers));
    }
    __syncthreads();
    if (t < kAmCls) a.cnt[t * a.tiles + tile] = c[t];
}

// Wave w handles class w: its total over the tiles first, then (with every
// class's total known, so with the class's start) the exclusive scan over
// the tiles. Each lane takes contiguous runs of 16 tiles, all their loads in
// flight together, and the first 1024 tiles stay in registers for the scan.
__global__ __launch_bounds__(1024) void k_am_scan(AmArgs a)
{
    constexpr uint32_t kPer = 16;   // tiles per lane and step
    __shared__ uint32_t tot[kAmCls];
    const uint32_t w = threadIdx.x >> 6;
    const int lane = lane_id();
    uint32_t *row = a.cnt + w * a.tiles;
    uint32_t x[kPer], sum = 0;
#pragma unroll
    for (uint32_t k = 0; k < kPer; k++) {
        const uint32_t tl = (uint32_t)lane * kPer + k;
        x[k] = tl < a.tiles ? row[tl] : 0u;
    }
#pragma unroll
    for (uint32_t k = 0; k < kPer; k++) sum += x[k];
    for (uint32_t tl = 64 * kPer + (uint32_t)lane; tl < a.tiles; tl += 64) sum += row[tl];
    sum = readlane32(wave_incl_scan_dpp(sum), 63);
    if (lane == 0) tot[w] = sum;
    __syncthreads();
    uint32_t run = 0;
    for (uint32_t k = 0; k < w; k++) run += tot[k];
    if (lane == 0) a.cstart[w] = run;
    if (threadIdx.x == 0) a.cstart[kAmCls] = a.n;
    for (uint32_t t0 = 0; t0 < a.tiles; t0 += 64 * kPer) {
        const uint32_t tl0 = t0 + (uint32_t)lane * kPer;
        if (t0) {
#pragma unroll
            for (uint32_t k = 0; k < kPer; k++) x[k] = tl0 + k < a.tiles ? row[tl0 + k] : 0u;
        }
        uint32_t part = 0;
#pragma unroll
        for (uint32_t k = 0; k < kPer; k++) part += x[k];
        const uint32_t incl = wave_incl_scan_dpp(part);
        uint32_t ex = run + incl - part;
#pragma unroll
        for (uint32_t k = 0; k < kPer; k++) {
            if (tl0 + k < a.tiles) row[tl0 + k] = ex;
            ex += x[k];
        }
        run += readlane32(incl, 63);
    }
}

__global__ __launch_bounds__(kAmTPB) void k_am_place(AmArgs a)
{
    constexpr int kWaves = kAmTPB / 64;
    // per round and wave, each class's count; then each one's offset in
    // its class's run (the tile's offset plus everything before it)
    __shared__ uint32_t pre[kAmRounds][kWaves][kAmCls], start[kAmCls];
    const uint32_t t = threadIdx.x, tile = blockIdx.x;
    const int w = (int)(t >> 6), lane = lane_id();
    const uint32_t base = tile * kAmTile;
    // the loads of all rounds first
    uint32_t cl[kAmRounds];
    uint64_t key[kAmRounds];
#pragma unroll
    for (uint32_t r = 0; r < kAmRounds; r++) {
        const uint32_t j = base + r * kAmTPB + t;
        uint32_t i = j < a.n ? a.in.fifo[j] : 0u;
        i = i < a.n ? i : 0u;
        const uint32_t q = j < a.n ? a.tier[j] : 0u;
        cl[r] = j < a.n ? a.in.cls[q] : kAmCls;
        key[r] = ordered_bits(am_aged(a.in, i, q));
    }
    uint32_t below[kAmRounds];
#pragma unroll
    for (uint32_t r = 0; r < kAmRounds; r++) {
        const bool ok = cl[r] < kAmCls;
        below[r] = (uint32_t)__popcll(class_peers(cl[r], ok) & lanemask_lt());
        uint32_t mine = 0;
#pragma unroll
        for (uint32_t k = 0; k < kAmCls; k++) {
            const uint32_t c = (uint32_t)__popcll(__ballot(cl[r] == k));
            mine = (uint32_t)lane == k ? c : mine;
        }
        if (lane < (int)kAmCls) pre[r][w][lane] = mine;
    }
    __syncthreads();
    if (t < kAmCls) {
        start[t] = a.cstart[t];
        uint32_t s = a.cnt[t * a.tiles + tile];
        for (uint32_t r = 0; r < kAmRounds; r++)
            for (int v = 0; v < kWaves; v++) {
                const uint32_t x = pre[r][v][t];
                pre[r][v][t] = s;
                s += x;
            }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < kAmRounds; r++) {
        if (cl[r] < kAmCls) {
            const uint32_t pos = pre[r][w][cl[r]] + below[r];
            a.rk[pos] = key[r];
            a.rp[pos] = base + r * kAmTPB + t;
            const uint32_t at = pos - start[cl[r]];
            if (a.hk && at % kAmStep == 0) {
                const uint32_t h = am_step_at(start[cl[r]], cl[r]) + at / kAmStep;
                a.hk[h] = key[r];
                a.hp[h] = base + r * kAmTPB + t;
            }
        }
    }
}

__device__ __forceinline__ bool am_less(uint64_t ka, uint32_t pa, uint64_t kb, uint32_t pb)
{
    return ka < kb || (ka == kb && pa < pb);
}

// Each entry's place at once: its index in its own run plus, for every other
// run, the entries below it there. A block takes 1024 entries of one run;
// sixteen lanes per other run and end of the tile find where the tile's first
// and last entries fall (16-way probing), the stretch between is staged in LDS
// piece by piece (2048 entries, the next one's loads in flight) and each entry
// searched in it. Of a stretch of many pieces the first and the last are staged,
// and what falls between them is searched in memory. A run much shorter than
// the longest one takes smaller tiles, whose stretches there are shorter and
// which spread over more of the chip; a run of a few entries searches the others
// in memory without staging.
// Many classes are merged in two steps, groups of four into one run each and
// then these: three searches per entry and step (16 classes) in place of
// fifteen. The line lies where classes that overlap gain what the second pass
// over the entries costs those that do not: 1,048,576 requests, 10 classes 96
// (one step) and 86 us (two) overlapping, 56 and 68 apart; 12 classes 108 and 84,
// 56 and 70; 16 classes 129 and 85, 58 and 71.
// What bounds it: latency and LDS (six blocks per CU, each a chain of about
// eight dependent reads and a piece per other run, 12 dependent LDS reads each).
// The whole Aging order over a given FIFO order, against ceil(log2 K) rounds of
// pairwise merges, which read and wrote every entry each round: 2,097,152
// requests, 3 classes 132 and 91 us, 8 classes 162 and 108, 16 classes 190 and
// 133; 1,048,576 with 99% in one of two classes 61 and 53, 99.9% 60 and 46, 16
// classes of which one holds 90% 108 and 90. Slower than the rounds where the
// floor cuts every class inside the sequence (few tiles, each with long stretches
// in every other run): 8 classes 99.5 and 100.7, 16 classes 118 and 127.
constexpr uint32_t kRkT = 256, kRkPer = 4, kRkTile = kRkT * kRkPer;
constexpr uint32_t kRkPiece = 2048, kRkPieces = 4;
constexpr uint32_t kRkGroups = 11, kRkGroup = 4;   // two steps from this many classes on, groups of
constexpr uint32_t kRkFew = 512;   // runs of at most n / kRkFew entries are placed without staging the others

// The entries of a run (k, p)[0, n) below (x, y), found by kL lanes (64, or 16
// where a wave does four such searches side by side; n == 0 where it has
// fewer): among the run's every kAmStep-th entries first (hk, hp: few pages,
// near each other), then among the 64 entries behind the last of those below.
static_assert(kAmStep == 64, "64 / kL probes per lane");
template <uint32_t kL>
__device__ inline uint32_t run_below(const uint64_t *k, const uint32_t *p, uint32_t n, const uint64_t *hk,
                                     const uint32_t *hp, uint64_t x, uint32_t y)
{
    const uint32_t l = (uint32_t)lane_id() & (kL - 1u), row = (uint32_t)lane_id() & ~(kL - 1u);
    auto count = [&](bool b) { return (uint32_t)__popcll((__ballot(b) >> row) & (~0ull >> (64u - kL))); };
    uint32_t lo = 0, hi = (n + kAmStep - 1u) / kAmStep;
    while (__any(hi > lo)) {
        const bool open = hi > lo;
        const uint32_t span = hi - lo;
        const uint32_t m = lo + span * l / kL;   // lo <= m < hi where open; n / 64 * 64 < 2^32
        const uint64_t km = open ? hk[m] : 0;
        const uint32_t pm = open ? hp[m] : 0;
        const uint32_t f = count(am_less(km, pm, x, y));   // probes 0..f-1 are below, f.. are not
        if (open) {
            const uint32_t nlo = f ? lo + span * (f - 1u) / kL + 1u : lo;
            hi = f < kL ? lo + span * f / kL : hi;
            lo = nlo;
        }
    }
    const uint32_t base = lo ? (lo - 1u) * kAmStep : 0u;
    uint64_t km[kAmStep / kL];
    uint32_t pm[kAmStep / kL], c = 0;
#pragma unroll
    for (uint32_t e = 0; e < kAmStep / kL; e++) {
        const uint32_t m = base + e * kL + l;
        km[e] = lo && m < n ? k[m] : ~0ull;
        pm[e] = lo && m < n ? p[m] : ~0u;
    }
#pragma unroll
    for (uint32_t e = 0; e < kAmStep / kL; e++) c += count(am_less(km[e], pm[e], x, y));
    return base + c;
}

// The start of run c, and of the one behind it.
__device__ __forceinline__ uint32_t rk_start(const AmArgs &a, uint32_t c)
{
    return c < a.K ? a.cstart[c * a.stride] : a.n;
}

// The entry (k, p) has place `at` in its group, which starts at `base`.
__device__ __forceinline__ void rk_emit(const AmArgs &a, uint32_t group, uint32_t base, uint32_t at, uint64_t k,
                                        uint32_t p)
{
    if (base + at >= a.n) return;
    if (a.ok) {
        a.ok[base + at] = k;
        a.op[base + at] = p;
        if (at % kAmStep == 0) {
            const uint32_t h = am_step_at(base, group) + at / kAmStep;   // < am_steps(n)
            a.ohk[h] = k;
            a.ohp[h] = p;
        }
        return;
    }
    uint32_t i = a.in.fifo[p];
    i = i < a.n ? i : 0u;
    a.perm[base + at] = i;
    if (a.key_out) a.key_out[i] = am_aged(a.in, i, am_tier(a.in, i));
}

// The entries of a run (k, p)[0, n) below (x, y), found by one thread: seven
// probes in flight per round, an eighth of what is left after it. The positions
// are read behind the keys that tie; once a lane of the wave has met a tie
// (clamped scores tie with all their neighbours), beside them.
__device__ __forceinline__ uint32_t lane_below(const uint64_t *k, const uint32_t *p, uint32_t n, uint64_t x, uint32_t y)
{
    uint32_t lo = 0, hi = n;
    bool ties = false;
    while (lo < hi) {
        const uint32_t span = hi - lo, from = lo;
        uint64_t km[8];
        uint32_t pm[8];
#pragma unroll
        for (uint32_t e = 1; e < 8; e++) km[e] = k[from + span * e / 8u];   // (span * 7 < 2^27)
        if (ties) {
#pragma unroll
            for (uint32_t e = 1; e < 8; e++) pm[e] = p[from + span * e / 8u];
        }
        bool tie = false;
#pragma unroll
        for (uint32_t e = 1; e < 8; e++) tie |= km[e] == x;
        if (!ties && __any(tie)) {
            ties = true;
#pragma unroll
            for (uint32_t e = 1; e < 8; e++) pm[e] = p[from + span * e / 8u];
        }
        uint32_t f = 0;
#pragma unroll
        for (uint32_t e = 1; e < 8; e++) f += km[e] < x || (ties && km[e] == x && pm[e] < y) ? 1u : 0u;
        if (f < 7u) hi = from + span * (f + 1u) / 8u;
        if (f) lo = from + span * f / 8u + 1u;
    }
    return lo;
}

struct RkShared {
    uint64_t k[kRkPiece];
    uint32_t p[kRkPiece];
    uint32_t from[kAmCls], to[kAmCls];   // where the tile's first and last entries fall in each run
};

// The places of entries [i0, i0 + cnt) of run c, kR per thread, in its group
// grp of runs [qb, qe).
template <uint32_t kR>
__device__ __forceinline__ void rank_tile(const AmArgs &a, RkShared &S, uint32_t c, uint32_t i0, uint32_t cnt,
                                          uint32_t grp, uint32_t qb, uint32_t qe)
{
    const uint32_t t = threadIdx.x, r0 = rk_start(a, c);
    const uint64_t *rk = a.rk;
    const uint32_t *rp = a.rp;
    uint64_t k[kR];
    uint32_t p[kR], rank[kR];
#pragma unroll
    for (uint32_t r = 0; r < kR; r++) {
        const uint32_t i = r * kRkT + t, g = r0 + i0 + (i < cnt ? i : 0u);
        k[r] = rk[g];
        p[r] = rp[g];
        rank[r] = i0 + i;
    }
    // search x (the x / 2-th other run, first or last entry), by a wave each or,
    // where there are more than four, by sixteen lanes
    const uint32_t searches = 2u * (qe - qb - 1u);
    auto ends = [&](auto lanes) {
        constexpr uint32_t kL = decltype(lanes)::value;
        for (uint32_t x0 = 0; x0 < searches; x0 += kRkT / kL) {
            const uint32_t x = x0 + t / kL, o = qb + (x >> 1), q = o < c ? o : o + 1u;
            const uint32_t e = r0 + i0 + (x & 1u ? cnt - 1u : 0u);
            const bool live = x < searches;
            const uint32_t q0 = live ? rk_start(a, q) : 0u, qn = live ? rk_start(a, q + 1u) - q0 : 0u;
            const uint32_t h0 = live ? am_step_at(q0, q) : 0u;
            const uint32_t f = run_below<kL>(rk + q0, rp + q0, qn, a.hk + h0, a.hp + h0, rk[e], rp[e]);
            if (live && t % kL == 0) (x & 1u ? S.to : S.from)[q] = f;
        }
    };
    if (searches <= kRkT / 64) ends(std::integral_constant<uint32_t, 64>());
    else ends(std::integral_constant<uint32_t, 16>());
    __syncthreads();
    // The pieces of all stretches one after another: one staged in LDS and
    // searched while the next one's loads are in flight. Of a stretch of more
    // than kRkPieces the first and the last.
    auto length = [&](uint32_t q) {   // (empty where the inputs break the contract and the run is not sorted)
        return q != c && S.to[q] > S.from[q] ? S.to[q] - S.from[q] : 0u;
    };
    auto advance = [&](uint32_t &q, uint32_t &part) {
        part++;
        for (; q < qe; q++, part = 0) {
            const uint32_t n = length(q), parts = (n + kRkPiece - 1u) / kRkPiece;
            if (part < (parts > kRkPieces ? 2u : parts)) return;
        }
    };
    uint64_t pk[kRkPiece / kRkT];
    uint32_t pp[kRkPiece / kRkT];
    auto fetch = [&](uint32_t q, uint32_t part) {
        const uint32_t n = length(q), x0 = n > kRkPiece * kRkPieces && part ? n - kRkPiece : part * kRkPiece;
        const uint64_t *qk = rk + rk_start(a, q) + S.from[q] + x0;
        const uint32_t *qp = rp + rk_start(a, q) + S.from[q] + x0;
#pragma unroll
        for (uint32_t e = 0; e < kRkPiece / kRkT; e++) {
            const uint32_t x = e * kRkT + t;
            const bool in = x0 + x < n;
            pk[e] = in ? qk[x] : ~0ull;   // (past the end: above every entry)
            pp[e] = in ? qp[x] : ~0u;
        }
    };
    for (uint32_t q = qb; q < qe; q++)
        if (q != c)
            for (uint32_t r = 0; r < kR; r++) rank[r] += S.from[q];
    uint32_t q = qb, part = ~0u;
    advance(q, part);
    if (q < qe) fetch(q, part);
    bool open[kR] = {};
    while (q < qe) {
        __syncthreads();
#pragma unroll
        for (uint32_t e = 0; e < kRkPiece / kRkT; e++) {
            S.k[e * kRkT + t] = pk[e];
            S.p[e * kRkT + t] = pp[e];
        }
        __syncthreads();
        const uint32_t n = length(q), cq = q, cpart = part;
        const bool longer = n > kRkPiece * kRkPieces;
        advance(q, part);
        if (q < qe) fetch(q, part);
        // how many of the piece's entries are below each of the thread's: steps
        // of 1024 .. 1, the entries of a thread side by side, then the last
        uint32_t pos[kR];
#pragma unroll
        for (uint32_t r = 0; r < kR; r++) pos[r] = 0;
#pragma unroll
        for (uint32_t st = kRkPiece / 2; st > 0; st >>= 1) {
#pragma unroll
            for (uint32_t r = 0; r < kR; r++) {
                const uint32_t y = pos[r] + st - 1u;
                if (am_less(S.k[y], S.p[y], k[r], p[r])) pos[r] += st;
            }
        }
#pragma unroll
        for (uint32_t r = 0; r < kR; r++)
            if (am_less(S.k[pos[r]], S.p[pos[r]], k[r], p[r])) pos[r]++;   // (pos < kRkPiece before)
        if (!longer || !cpart) {
#pragma unroll
            for (uint32_t r = 0; r < kR; r++) {
                open[r] = pos[r] == kRkPiece;
                rank[r] += pos[r];
            }
            continue;
        }
        // a long stretch: most entries fall into its first piece or its last
        // one (where the floor cuts the tile: the clamped entries tie with
        // their neighbours in time, the others follow every clamped one), the
        // others are searched in memory side by side
        const uint64_t *qk = rk + rk_start(a, cq) + S.from[cq];
        const uint32_t *qp = rp + rk_start(a, cq) + S.from[cq];
        uint32_t lo[kR], hi[kR];
#pragma unroll
        for (uint32_t r = 0; r < kR; r++) {
            lo[r] = hi[r] = n - kRkPiece + pos[r];
            if (!open[r]) lo[r] = hi[r] = kRkPiece;
            else if (!pos[r]) lo[r] = kRkPiece;
        }
        bool more = true;
        while (more) {
            uint64_t km[kR];
            uint32_t pm[kR];
#pragma unroll
            for (uint32_t r = 0; r < kR; r++) {
                const uint32_t m = (lo[r] + hi[r]) >> 1;   // < n
                km[r] = lo[r] < hi[r] ? qk[m] : 0;
                pm[r] = lo[r] < hi[r] ? qp[m] : 0;
            }
            more = false;
#pragma unroll
            for (uint32_t r = 0; r < kR; r++) {
                if (lo[r] >= hi[r]) continue;
                const uint32_t m = (lo[r] + hi[r]) >> 1;
                if (am_less(km[r], pm[r], k[r], p[r])) lo[r] = m + 1u;
                else hi[r] = m;
                more |= lo[r] < hi[r];
            }
        }
#pragma unroll
        for (uint32_t r = 0; r < kR; r++) rank[r] += lo[r] - kRkPiece;
    }
    const uint32_t base = rk_start(a, qb);
#pragma unroll
    for (uint32_t r = 0; r < kR; r++)
        if (r * kRkT + t < cnt) rk_emit(a, grp, base, rank[r], k[r], p[r]);
}

__global__ __launch_bounds__(kRkT, 6) void k_am_rank(AmArgs a)
{
    __shared__ RkShared S;
    const uint32_t t = threadIdx.x, lane = (uint32_t)lane_id();
    // lane l: run l, its tile and how many of them; the block's run and tile
    // there (blocks are handed to the runs in order)
    const uint32_t start = rk_start(a, lane), len = wave_shl1(start, a.n) - start;
    uint32_t longest = len;   // (runs are lanes 0..15)
#pragma unroll
    for (int d = 8; d >= 1; d >>= 1) {
        const uint32_t o = (uint32_t)__shfl_xor((int)longest, d, 64);
        longest = o > longest ? o : longest;
    }
    longest = readlane32(longest, 0);
    const bool few = len <= a.n / kRkFew;
    const uint32_t tile = few ? kRkT : len >= longest / 8u ? kRkTile : len >= longest / 16u ? kRkTile / 2u : kRkTile / 4u;
    const uint32_t tiles = (len + tile - 1u) / tile, upto = wave_incl_scan_dpp(tiles);
    const uint64_t past = __ballot(blockIdx.x < upto);
    if (!past) return;   // the same for the whole block
    const uint32_t c = (uint32_t)__builtin_ctzll(past);
    const uint32_t mytile = readlane32(tile, (int)c), n = readlane32(len, (int)c), r0 = readlane32(start, (int)c);
    const uint32_t i0 = (blockIdx.x - readlane32(upto - tiles, (int)c)) * mytile;
    const uint32_t cnt = n - i0 < mytile ? n - i0 : mytile;
    // its group: runs [qb, qe)
    const uint32_t grp = c / a.per, qb = grp * a.per, qe = qb + a.per < a.K ? qb + a.per : a.K;
    if (readlane32(few ? 1u : 0u, (int)c)) {   // every entry searched in the whole of the other runs
        if (t >= cnt) return;
        const uint64_t x = a.rk[r0 + i0 + t];
        const uint32_t y = a.rp[r0 + i0 + t];
        uint32_t at = i0 + t;
        for (uint32_t q = qb; q < qe; q++) {
            if (q == c) continue;
            const uint32_t q0 = rk_start(a, q);
            at += lane_below(a.rk + q0, a.rp + q0, rk_start(a, q + 1u) - q0, x, y);
        }
        rk_emit(a, grp, rk_start(a, qb), at, x, y);
        return;
    }
    if (mytile == kRkTile) rank_tile<kRkPer>(a, S, c, i0, cnt, grp, qb, qe);
    else if (mytile == kRkTile / 2u) rank_tile<kRkPer / 2u>(a, S, c, i0, cnt, grp, qb, qe);
    else rank_tile<kRkPer / 4u>(a, S, c, i0, cnt, grp, qb, qe);
}

// A second set of run buffers: keys, FIFO positions, steps.
size_t runs_bytes(uint64_t n) { return align_up(n * 8, 256) + align_up(n * 4, 256) + am_steps_bytes(n); }

// scratch: runs_bytes(n).
void rank_launch(AmArgs a, void *scratch, hipStream_t s)
{
    auto launch = [&]() {
        // the tiles of all runs if they were of kRkTile, and what the smaller
        // ones make more: most of all, K - 1 runs of a sixteenth of the longest
        const uint32_t tiles = (uint32_t)cdiv(a.n, kRkTile) + a.K;
        const uint32_t more = (uint32_t)cdiv(3ull * (a.K - 1u) * a.n, (uint64_t)kRkTile * (15u + a.K));
        hipLaunchKernelGGL(k_am_rank, dim3(tiles + more), dim3(kRkT), 0, s, a);
    };
    a.stride = 1;
    a.per = a.K;
    a.ok = a.ohk = nullptr;
    a.op = a.ohp = nullptr;
    if (a.K >= kRkGroups) {
        uint8_t *q = static_cast<uint8_t *>(scratch);
        a.per = kRkGroup;
        a.ok = reinterpret_cast<uint64_t *>(q);
        q += align_up((uint64_t)a.n * 8, 256);
        a.op = reinterpret_cast<uint32_t *>(q);
        q += align_up((uint64_t)a.n * 4, 256);
        a.ohk = reinterpret_cast<uint64_t *>(q);
        a.ohp = am_steps_pos(a.ohk, a.n);
        launch();
        a.rk = a.ok;
        a.rp = a.op;
        a.hk = a.ohk;
        a.hp = a.ohp;
        a.ok = a.ohk = nullptr;
        a.op = a.ohp = nullptr;
        a.stride = a.per;
        a.K = (uint32_t)cdiv(a.K, a.per);
        a.per = a.K;
    }
    launch();
}

}  // namespace

size_t am_partition_ws_bytes(uint64_t n)
{
    const uint64_t tiles = cdiv(n ? n : 1, kAmTile);
    return align_up(tiles * kAmCls * 4, 256) + align_up(n * 8, 256) + align_up(n, 256);
}

hipError_t am_partition(const SortInput &in, uint32_t *run_pos, uint32_t *run_start, void *ws, hipStream_t s)
{
    const uint32_t n = in.n;
    if (n == 0) return hipSuccess;
    if (n > kAmMaxN || !in.fifo) return hipErrorInvalidValue;
    AmArgs a;
    memset(&a, 0, sizeof(a));
    a.in = in;
    a.n = n;
    a.tiles = (uint32_t)cdiv(n, kAmTile);
    a.K = kAmCls;
    uint8_t *p = static_cast<uint8_t *>(ws);
    a.cnt = reinterpret_cast<uint32_t *>(p);
    p += align_up((uint64_t)a.tiles * kAmCls * 4, 256);
    a.rk = reinterpret_cast<uint64_t *>(p);   // the scores are not used here
    p += align_up((uint64_t)n * 8, 256);
    a.tier = p;
    a.rp = run_pos;
    a.cstart = run_start;
    hipLaunchKernelGGL(k_am_count, dim3(a.tiles), dim3(kAmTPB), 0, s, a);
    hipLaunchKernelGGL(k_am_scan, dim3(1), dim3(1024), 0, s, a);
    hipLaunchKernelGGL(k_am_place, dim3(a.tiles), dim3(kAmTPB), 0, s, a);
    return hipGetLastError();
}

size_t am_ws_bytes(uint64_t n)
{
    const uint64_t tiles = cdiv(n ? n : 1, kAmTile);
    return align_up(tiles * kAmCls * 4, 256) + align_up((kAmCls + 1) * 4, 256) + align_up(n * 8, 256) +
           align_up(n * 4, 256) + align_up(n, 256) + am_steps_bytes(n) + runs_bytes(n);
}

hipError_t am_launch(const SortInput &in, uint32_t n_classes, uint32_t *perm, double *key_out, void *ws,
                     hipStream_t s, uint32_t *wait_status)
{
    const uint32_t n = in.n;
    if (n == 0) return hipSuccess;
    if (n > kAmMaxN || !in.fifo || n_classes < 1 || n_classes > kAmCls) return hipErrorInvalidValue;
    AmArgs a;
    a.in = in;
    a.n = n;
    a.tiles = (uint32_t)cdiv(n, kAmTile);
    a.K = n_classes;
    uint8_t *p = static_cast<uint8_t *>(ws);
    a.cnt = reinterpret_cast<uint32_t *>(p);
    p += align_up((uint64_t)a.tiles * kAmCls * 4, 256);
    a.cstart = reinterpret_cast<uint32_t *>(p);
    p += align_up((kAmCls + 1) * 4, 256);
    a.rk = reinterpret_cast<uint64_t *>(p);
    p += align_up((uint64_t)n * 8, 256);
    a.rp = reinterpret_cast<uint32_t *>(p);
    p += align_up((uint64_t)n * 4, 256);
    a.tier = p;
    p += align_up(n, 256);
    a.hk = reinterpret_cast<uint64_t *>(p);
    a.hp = am_steps_pos(a.hk, n);
    p += am_steps_bytes(n);
    a.perm = perm;
    a.key_out = key_out;
    a.wait_status = wait_status;
    hipLaunchKernelGGL(k_am_count, dim3(a.tiles), dim3(kAmTPB), 0, s, a);
    hipLaunchKernelGGL(k_am_scan, dim3(1), dim3(1024), 0, s, a);
    hipLaunchKernelGGL(k_am_place, dim3(a.tiles), dim3(kAmTPB), 0, s, a);
    rank_launch(a, p, s);
    return hipGetLastError();
}

hipError_t am_rank_launch(const SortInput &in, uint32_t n_classes, const LsRuns &runs, uint32_t *perm,
                          double *key_out, void *scratch, hipStream_t s)
{
    const uint32_t n = in.n;
    if (n == 0) return hipSuccess;
    if (n > kAmMaxN || !in.fifo || n_classes < 1 || n_classes > kAmCls) return hipErrorInvalidValue;
    AmArgs a;
    memset(&a, 0, sizeof(a));
    a.in = in;
    a.n = n;
    a.K = n_classes;
    a.cstart = runs.cstart;
    a.rk = runs.rk;
    a.rp = runs.rp;
    a.hk = runs.hk;
    a.hp = runs.hp;
    a.perm = perm;
    a.key_out = key_out;
    rank_launch(a, scratch, s);
    return hipGetLastError();
}

}  // namespace ds
