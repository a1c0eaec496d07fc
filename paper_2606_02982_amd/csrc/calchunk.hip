// Stage 2 for up to kCalGroupsChunked groups: Eq. (5) with the ratio of Eq. (6)
// (Sec. "Runtime Calibration and Feedback Adaptation") without a global
// partition of the events by group, so that every access is coalesced.
//
// The events, in completion order, are cut into C chunks of L events. With
// M(c, g) the composition of the affine maps x -> (1 - alpha) x + alpha r of
// group g's events in chunk c (in order):
//   small tables (at most kCalGroupsLds groups):
//   k_calc_agg    per chunk (one block): each sub-tile of 512 events is
//                 sorted by group in LDS (stable LSD passes, wave ballots),
//                 scanned as a segmented scan of maps, and each group's part
//                 is composed into that group's map in LDS; the chunk writes
//                 M(c, g) for every group (or "no usable event").
//   k_calc_apply  per chunk: the maps of the chunks before it applied to the
//                 initial factors (k_calc_agg keeps a copy of them), the same
//                 sub-tile sort and scan; every event then runs the exact
//                 update from its carried factor, in order, and the traces
//                 are staged in LDS and written in event order. The last
//                 chunk's block writes the final factors.
//   k_calc_one    when besides there are at most kOneChunks chunks of one
//                 sub-tile each: both in one pass over the events. Each block
//                 sorts and scans its sub-tile once, publishes its chunk's
//                 maps, reads those of the chunks before it (a bounded wait
//                 for words not yet written), and applies the updates; a
//                 small launch before it marks the words unwritten. Up to
//                 kOneBlock events a single chunk, and no such launch.
//   large tables:
//   k_calc_own    per chunk (one block, or one per range of 8192 groups): the
//                 waves own the groups between them, and each composes its
//                 groups' maps event by event in LDS. The chunk writes M(c, g)
//                 as a count k of usable events (its slope is (1 - alpha)^k)
//                 and an offset, and for traces each event's map from the
//                 chunk's start the same way (through the event when only the
//                 trace is wanted, else to just before it).
//   k_calc_scan   per 64 groups (one block, lane = group): the group's
//                 factor before chunk c is M(c-1, g) o ... o M(0, g) applied
//                 to its initial factor (sixteen stretches of chunks composed
//                 by sixteen waves, then chained in order); writes those
//                 carries over the maps' offsets, and the final factor.
//   k_calc_ev     per event: its chunk's carry through its map; without the
//                 event, followed by the exact update t1 = (1 - alpha) c,
//                 t2 = alpha r, c = t1 + t2.
// Results match the sequential recurrence up to the rounding of the
// composed maps (a few ulps; the contract is 1e-12 relative).
#include "common.h"
#include "kernels.h"
#include "lookback.h"

namespace ds {
namespace {

constexpr int kT = 512;                  // threads per block
// events per thread per sub-tile (kE) is a template parameter: 1, or 2 or 4 in
// one launch; kSub = kT * kE events per sub-tile
constexpr int kW = kT / 64;
constexpr uint32_t kG = kCalGroupsLds;   // groups held in LDS
constexpr uint32_t kMaxTable = 1u << 20; // C x G entries at most (C >= 1)
constexpr uint32_t kMaxTableR = 1u << 21;   // the same above kCalGroupsLds groups
constexpr uint32_t kMaxChunks = 512;
constexpr uint32_t kSmallTable = 16384;  // C x G at most of the one-launch path
// C x G at most of k_calc_agg and k_calc_apply with one sub-tile per chunk:
// every k_calc_apply block reads the maps of all chunks before it. Measured
// against k_calc_own and its two launches, with a trace: 131,073 events, 40
// groups 22.0 and 23.9 us, 50 groups 24.5 and 24.0; 150,000, 32 groups 23.8 and
// 25.0, 40 groups 26.2 and 24.3; 262,144, 4 groups 18.2 and 28, 20 groups 25.4
// and 25.4. Without one (k_calc_own then has one other launch): 131,073, 24
// groups 18.3 and 19.5, 32 groups 20.0 and 20.1.
constexpr uint32_t kSmallTraced = 10240, kSmallPair = 8192;
// The same with two sub-tiles per chunk and a trace: 262,145 events (a chunk per
// compute unit and one more), 1 group 20.3 and 26.8, 24 groups 23.7 and 25.5, 32
// groups 26.0 and 25.8; 300,000, 1 group 26.9 and 27.2, 4 groups 27.3 and 26.6;
// 524,288, 2 groups 27.6 and 29.8. (Three: 600,000, 1 group 37.8 and 31.0.)
constexpr uint32_t kPairTraced = 1024, kPairTraced256 = 6400;
// C x G at most of k_calc_agg and k_calc_apply with chunks of any length, which
// a workspace without room for k_calc_own's maps of every event gets.
constexpr uint32_t kFewTable = 16384;
constexpr uint32_t kCarryR = 4;          // chunk maps per thread held in registers for the carry

constexpr int kOT = 1024;                // k_calc_own: threads per block
constexpr uint32_t kOW = kOT / 64;       // its waves, the owners of the groups g = w (mod kOW)
constexpr uint32_t kOU = 4;              // events per thread per step
constexpr uint32_t kOStep = kOT * kOU;
constexpr uint32_t kOHeavy = 640;        // an owner's events of a step above which chunks combine theirs first
constexpr uint32_t kRangeGroups = 8192;  // groups per block above kCalGroupsLds groups

struct CalArgs {
    const uint32_t *group;
    const double *est;
    const uint32_t *obs;
    uint32_t E, G;
    double alpha, oma;       // alpha and 1 - alpha
    uint32_t C;              // chunks
    uint32_t L;              // events per chunk
    uint32_t passes;         // 8-bit LSD passes over the group key (key < 2^(8 passes))
    uint32_t keybits;        // bits of the largest key (G, for an event outside the groups)
    double *aggA, *aggB;     // [C][G]: M(c, g) = x -> A x + B; A < 0: no usable event
    uint32_t *aggK;          // large tables instead of aggA: A = (1 - alpha)^K; 0: no usable event
    uint32_t R;              // large tables: ranges of kRangeGroups groups (1: one block per chunk)
    double *carry;           // large tables: [C][G]: factor of g before chunk c, in the place of aggB
    double *s0;              // [G] the initial factors (small tables: no k_calc_scan)
    double *state;           // [G] in: before all events, out: after
    double *trace, *trace_before;
    uint32_t *status;        // the call's wait status word, or NULL: set by a wait that runs out
    uint32_t clear;          // the call's first kernel zeroes *status
    uint32_t no_wait;        // every wait gives up at once (a diagnostic of the error path)
    // large tables with traces: each event's map from its chunk's start to
    // just before it, x -> (1 - alpha)^xk x + xb, in event order; pw[j][d] =
    // (1 - alpha)^(d 256^j)
    // incl: the maps include the event itself (only the trace is wanted)
    double *xb;
    uint32_t *xk;
    double *pw;
    uint32_t incl;
};

// A composed affine map: x -> a x + b, f = a segment starts inside,
// u = some usable event inside, k = how many (a = (1 - alpha)^k).
struct Map {
    uint32_t f, u;
    double a, b;
    uint32_t k;
};

// x then y
__device__ __forceinline__ Map combine(const Map &x, const Map &y)
{
    if (y.f) return y;
    Map r;
    r.f = x.f;
    r.u = x.u | y.u;
    r.a = y.a * x.a;
    const double t = y.a * x.b;
    r.b = t + y.b;
    r.k = x.k + y.k;
    return r;
}

__device__ __forceinline__ double shfl_up_d(double x, int d)
{
    const long long v = __double_as_longlong(x);
    const int lo = __shfl_up((int)(uint32_t)v, d, 64), hi = __shfl_up((int)(uint32_t)(v >> 32), d, 64);
    return __longlong_as_double((long long)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
}

__device__ __forceinline__ double shfl_down_d(double x, int d)
{
    const long long v = __double_as_longlong(x);
    const int lo = __shfl_down((int)(uint32_t)v, d, 64), hi = __shfl_down((int)(uint32_t)(v >> 32), d, 64);
    return __longlong_as_double((long long)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo));
}

__device__ __forceinline__ Map shfl_up_map(const Map &m, int d)
{
    Map r;
    r.f = (uint32_t)__shfl_up((int)m.f, d, 64);
    r.u = (uint32_t)__shfl_up((int)m.u, d, 64);
    r.a = shfl_up_d(m.a, d);
    r.b = shfl_up_d(m.b, d);
    r.k = (uint32_t)__shfl_up((int)m.k, d, 64);
    return r;
}

// Inclusive scan of one map per lane over the wave (fixed order).
__device__ __forceinline__ Map wave_scan(Map v)
{
    const int lane = lane_id();
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const Map o = shfl_up_map(v, d);
        if (lane >= d) v = combine(o, v);
    }
    return v;
}

template <int kE>
struct SubShared {
    static constexpr uint32_t kSub = kT * kE;
    uint32_t wcnt[kW][256];
    uint32_t texcl[256];
    Map wagg[kW];
    uint16_t key[kSub];      // group (G for an event outside the groups)
    uint16_t slot[kSub];     // position in the sub-tile
    double b[kSub];          // alpha * r, or 0; reused for trace staging once read
    uint8_t ok[kSub];        // usable
};

// The raw events of a sub-tile (wave-major slots as in load_sort_scan).
template <int kE>
struct Raw {
    uint32_t g[kE], o[kE];
    double x[kE];
};

template <int kE>
__device__ __forceinline__ void load_raw(const CalArgs &a, uint32_t s0, uint32_t m, Raw<kE> &raw)
{
    const int w = (int)(threadIdx.x >> 6), lane = lane_id();
#pragma unroll
    for (int r = 0; r < kE; r++) {
        const uint32_t sl = (uint32_t)w * (64u * kE) + (uint32_t)r * 64u + (uint32_t)lane;
        raw.g[r] = 0;
        raw.o[r] = 0;
        raw.x[r] = 0.0;
        if (sl < m) {
            const uint32_t e = s0 + sl;
            raw.g[r] = a.group[e];
            raw.x[r] = a.est[e];
            raw.o[r] = a.obs[e];
        }
    }
}

// The sub-tile of m <= kSub events (m > 0) held in raw, sorted by group and
// scanned. On return (after a barrier that follows every thread's
// reads of sh.b, sh.slot and sh.ok), thread t holds sorted positions 4t ..
// 4t+3: key, slot, b, usable and the segment-start flags; and, when its first
// position continues a segment that starts at p < 4t, `excl`, the
// composition of the maps of positions p .. 4t-1. sh.key keeps the sorted
// keys.
template <int kE>
struct Sub {
    uint32_t key[kE], slot[kE], ok[kE], flag[kE];
    double b[kE];
    Map excl;
};

template <int kE>
__device__ void load_sort_scan(const CalArgs &a, const Raw<kE> &raw, uint32_t m, SubShared<kE> &sh, Sub<kE> &out)
{
    const uint32_t t = threadIdx.x;
    const int w = (int)(t >> 6), lane = lane_id();
    // wave-major slots: wave w holds slots [64 kE w, 64 kE (w + 1)), round r
    // the 64 slots from 64 kE w + 64 r; every load is coalesced
    uint32_t key[kE], slot[kE], ok[kE];
    double b[kE];
#pragma unroll
    for (int r = 0; r < kE; r++) {
        const uint32_t sl = (uint32_t)w * (64u * kE) + (uint32_t)r * 64u + (uint32_t)lane;
        slot[r] = sl;
        key[r] = 0;
        ok[r] = 0;
        b[r] = 0.0;
        if (sl < m) {
            const uint32_t g = raw.g[r];
            const double x = raw.x[r];
            const uint32_t o = raw.o[r];
            key[r] = g < a.G ? g : a.G;
            if (g < a.G && isfinite(x) && x > 0.0) {
                const double ratio = (double)o / x;
                b[r] = a.alpha * ratio;
                ok[r] = 1;
            }
        }
    }
    // stable LSD passes over the key (8 bits each); positions in LDS
    for (uint32_t p = 0; p < a.passes; p++) {
        for (uint32_t i = t; i < kW * 256u; i += kT) (&sh.wcnt[0][0])[i] = 0;
        lds_sync();
        uint32_t rk[kE];
#pragma unroll
        for (int r = 0; r < kE; r++) {
            const uint32_t sl = (uint32_t)w * (64u * kE) + (uint32_t)r * 64u + (uint32_t)lane;
            const bool v = sl < m;
            const uint32_t dg = (key[r] >> (8 * p)) & 255u;
            // (four bits at a time; bits no key has are left out)
            uint64_t peers = match_bits<4>(dg, __ballot(v));
            if (8 * p + 4 < a.keybits) peers = match_bits<4, 4>(dg, peers);
            const uint32_t below = (uint32_t)__popcll(peers & lanemask_lt());
            const uint32_t old = v ? sh.wcnt[w][dg] : 0u;
            rk[r] = old + below;
            if (v && below == 0) sh.wcnt[w][dg] = old + (uint32_t)__popcll(peers);
            __builtin_amdgcn_wave_barrier();
        }
        lds_sync();
        if (w == 0) {
            // digits 4 l .. 4 l + 3: per-wave exclusive offsets and digit starts
            uint32_t c[4][kW], tot[4];
#pragma unroll
            for (int e = 0; e < 4; e++)
#pragma unroll
                for (int q = 0; q < kW; q++) c[e][q] = sh.wcnt[q][4 * lane + e];
#pragma unroll
            for (int e = 0; e < 4; e++) {
                uint32_t acc = 0;
#pragma unroll
                for (int q = 0; q < kW; q++) {
                    sh.wcnt[q][4 * lane + e] = acc;
                    acc += c[e][q];
                }
                tot[e] = acc;
            }
            const uint32_t sum = tot[0] + tot[1] + tot[2] + tot[3];
            uint32_t ex = wave_incl_scan_dpp(sum) - sum;
#pragma unroll
            for (int e = 0; e < 4; e++) {
                sh.texcl[4 * lane + e] = ex;
                ex += tot[e];
            }
        }
        lds_sync();
#pragma unroll
        for (int r = 0; r < kE; r++) {
            const uint32_t sl = (uint32_t)w * (64u * kE) + (uint32_t)r * 64u + (uint32_t)lane;
            if (sl < m) {
                const uint32_t dg = (key[r] >> (8 * p)) & 255u;
                const uint32_t q = sh.texcl[dg] + sh.wcnt[w][dg] + rk[r];
                sh.key[q] = (uint16_t)key[r];
                sh.slot[q] = (uint16_t)slot[r];
                sh.b[q] = b[r];
                sh.ok[q] = (uint8_t)ok[r];
            }
        }
        lds_sync();
        if (p + 1 < a.passes) {
#pragma unroll
            for (int r = 0; r < kE; r++) {
                const uint32_t sl = (uint32_t)w * (64u * kE) + (uint32_t)r * 64u + (uint32_t)lane;
                if (sl < m) {
                    key[r] = sh.key[sl];
                    slot[r] = sh.slot[sl];
                    b[r] = sh.b[sl];
                    ok[r] = sh.ok[sl];
                }
            }
            lds_sync();
        }
    }
    // thread t takes sorted positions kE t .. kE t + kE - 1
    Map agg = {0u, 0u, 1.0, 0.0};
#pragma unroll
    for (int e = 0; e < kE; e++) {
        const uint32_t i = t * kE + (uint32_t)e;
        out.key[e] = kG;   // past the end: no group
        out.slot[e] = 0;
        out.ok[e] = 0;
        out.flag[e] = 0;
        out.b[e] = 0.0;
        if (i < m) {
            out.key[e] = sh.key[i];
            out.slot[e] = sh.slot[i];
            out.ok[e] = sh.ok[i];
            out.b[e] = sh.b[i];
            out.flag[e] = (i == 0 || sh.key[i - 1] != sh.key[i]) ? 1u : 0u;
            Map mp;
            mp.f = out.flag[e];
            mp.u = out.ok[e];
            mp.a = out.ok[e] ? a.oma : 1.0;
            mp.b = out.ok[e] ? out.b[e] : 0.0;
            mp.k = out.ok[e];
            agg = (e == 0) ? mp : combine(agg, mp);
        }
    }
    // exclusive scan of the threads' maps: wave scan, then the waves before
    const Map incl = wave_scan(agg);
    if (lane == 63) sh.wagg[w] = incl;
    lds_sync();
    Map before = {1u, 0u, 1.0, 0.0};   // nothing before
    for (int q = 0; q < w; q++) before = (q == 0) ? sh.wagg[0] : combine(before, sh.wagg[q]);
    Map ex = shfl_up_map(incl, 1);
    if (lane == 0) ex = before;
    else if (w > 0) ex = combine(before, ex);
    if (t == 0) ex = Map{1u, 0u, 1.0, 0.0};
    out.excl = ex;
}

template <int kE>
__global__ __launch_bounds__(kT) void k_calc_agg(CalArgs a)
{
    constexpr uint32_t kSub = kT * kE;
    __shared__ SubShared<kE> sh;
    __shared__ double sA[kG], sB[kG];   // the chunk's map per group so far (A < 0: none)
    const uint32_t t = threadIdx.x, c = blockIdx.x;
    if (a.clear && a.status && c == 0 && t == 0) *a.status = 0;
    for (uint32_t g = t; g < a.G; g += kT) {
        sA[g] = -1.0;
        sB[g] = 0.0;
        if (c == 0) a.s0[g] = a.state[g];
    }
    const uint64_t c0 = (uint64_t)c * a.L;
    const uint64_t c1 = c0 + a.L < a.E ? c0 + a.L : a.E;
    for (uint64_t s0 = c0; s0 < c1; s0 += kSub) {
        const uint32_t m = (uint32_t)(c1 - s0 < kSub ? c1 - s0 : kSub);
        Raw<kE> raw;
        load_raw<kE>(a, (uint32_t)s0, m, raw);
        Sub<kE> sub;
        load_sort_scan<kE>(a, raw, m, sh, sub);   // (its first barrier orders the sA/sB writes)
        // the segment of each group in this sub-tile, composed into the
        // group's map at the segment's last position (one thread per group)
        Map run = sub.excl;
#pragma unroll
        for (int e = 0; e < kE; e++) {
            const uint32_t i = t * kE + (uint32_t)e;
            if (i >= m) break;
            Map mp;
            mp.f = sub.flag[e];
            mp.u = sub.ok[e];
            mp.a = sub.ok[e] ? a.oma : 1.0;
            mp.b = sub.ok[e] ? sub.b[e] : 0.0;
            mp.k = sub.ok[e];
            run = mp.f ? mp : combine(run, mp);
            const bool last = (i + 1 == m) || (e + 1 < kE ? sub.flag[e + 1] != 0u : sh.key[i + 1] != sh.key[i]);
            const uint32_t g = sub.key[e];
            if (last && g < a.G && run.u) {
                const double pa = sA[g];
                if (pa < 0.0) {
                    sA[g] = run.a;
                    sB[g] = run.b;
                } else {
                    // the chunk so far, then this segment
                    sA[g] = run.a * pa;
                    const double tt = run.a * sB[g];
                    sB[g] = tt + run.b;
                }
            }
        }
        lds_sync();
    }
    for (uint32_t g = t; g < a.G; g += kT) {
        a.aggA[(uint64_t)c * a.G + g] = sA[g];
        a.aggB[(uint64_t)c * a.G + g] = sB[g];
    }
}

// ---- large tables ---------------------------------------------------------------

// One step's events in registers (event u * kOT + t of the step).
struct OwnStep {
    double x[kOU];
    uint32_t g[kOU], o[kOU];
};

__device__ __forceinline__ void own_load(const CalArgs &a, uint64_t s0, uint64_t c1, OwnStep &s)
{
#pragma unroll
    for (uint32_t u = 0; u < kOU; u++) {
        const uint64_t e = s0 + u * kOT + threadIdx.x;
        const bool in = e < c1;
        s.g[u] = in ? a.group[e] : 0xFFFFFFFFu;   // no group
        s.x[u] = in ? a.est[e] : 0.0;
        s.o[u] = in ? a.obs[e] : 0u;
    }
}

// Where a wave's share of the step lies: `at`: for lane l, the first place of
// owner l / 4's events of the wave's chunk l % 4; [lo, hi): the places of the
// wave's own events. heavy: some owner has more than kOHeavy.
struct OwnPlaces {
    uint32_t at, lo, hi;
    bool heavy;
};

// From the table of counts (every wave scans it for itself). bm: masks of the
// bytes of a 16-byte run that come before byte w.
__device__ __forceinline__ OwnPlaces own_places(const uint8_t *cnt, const uint32_t (&bm)[4], uint32_t w)
{
    // lane l holds owner l / 4, chunks 16 (l % 4) .. + 15 (of 64 events: u = l % 4)
    const uint4 v = *reinterpret_cast<const uint4 *>(&cnt[(uint32_t)lane_id() * 16]);
    uint32_t sum = 0, before = 0;
    sum = __builtin_amdgcn_sad_u8(v.x, 0u, sum);
    sum = __builtin_amdgcn_sad_u8(v.y, 0u, sum);
    sum = __builtin_amdgcn_sad_u8(v.z, 0u, sum);
    sum = __builtin_amdgcn_sad_u8(v.w, 0u, sum);
    before = __builtin_amdgcn_sad_u8(v.x & bm[0], 0u, before);
    before = __builtin_amdgcn_sad_u8(v.y & bm[1], 0u, before);
    before = __builtin_amdgcn_sad_u8(v.z & bm[2], 0u, before);
    before = __builtin_amdgcn_sad_u8(v.w & bm[3], 0u, before);
    const uint32_t incl = wave_incl_scan_dpp(sum);
    OwnPlaces o;
    o.at = incl - sum + before;
    o.lo = w ? readlane32(incl, (int)(4 * w - 1)) : 0u;
    o.hi = readlane32(incl, (int)(4 * w + 3));
    uint32_t own = sum + (uint32_t)__shfl_xor((int)sum, 1, 64);
    own += (uint32_t)__shfl_xor((int)own, 2, 64);
    o.heavy = __ballot(own > kOHeavy) != 0;
    return o;
}

// The lanes of one group (same: the live lanes with this lane's group) chained
// in lane order: on return A, B is the map of the group's lanes up to this
// one. rank: live lanes of the group before this one; prev0: the nearest.
__device__ __forceinline__ void own_chain(uint64_t same, double &A, double &B, uint32_t &rank, int &prev0)
{
    const uint64_t below = same & lanemask_lt();
    rank = (uint32_t)__popcll(below);
    prev0 = below ? 63 - __clzll((long long)below) : lane_id();
    int prev = prev0;
    for (uint32_t st = 1; __ballot(rank >= st); st <<= 1) {
        const double pA = __shfl(A, prev, 64), pB = __shfl(B, prev, 64);
        const int pp = __shfl(prev, prev, 64);
        if (rank >= st) {
            const double tt = A * pB;
            B = tt + B;
            A = A * pA;
            prev = pp;
        }
    }
}

// The chunk's maps and, with kEv, each event's map from the chunk's start.
// Wave w owns the groups g = w (mod 16) of the block's range. A step of 4096
// events is split by owner, stably, through LDS (four ballots per 64 events,
// one table of counts that every wave scans for itself), and each wave takes
// its own events 64 at a time, in event order: one ballot match finds the
// lanes of a group, log2 of the largest such set pointer jumps compose their
// maps (one jump for two lanes, six if one tenant holds all 64), the group's
// map so far is read and written once. The next step's loads are in flight
// meanwhile (the barriers wait on LDS alone). Where one owner would hold more
// than kOHeavy of a step's events (256 on average; a tenant with a large share
// of the traffic, or few groups), each wave first composes the lanes of a
// group in each of its 64 events, so that the owners chain one map per group
// and 64 events, and the events take their group's map from there.
//
// kGr = kCalGroupsLds: one block holds every group, and the events' maps are
// staged and written in event order; kGr = kRangeGroups: a.R blocks per
// chunk, each for a range of the groups, write their events' maps directly
// (the blocks of a chunk sit on one XCD, whose L2 they share).
//
// What bounds it: latency inside a CU (one block of 16 waves, 146 KB of LDS).
// 4,194,304 events over 4,096 groups: 57 us; the form before (sub-tiles of
// 4096 events sorted by two LSD passes and scanned by 8 waves) 83 us. With one
// group holding half or all of them: 75 and 57 us (without the heavy steps'
// combining 145 and 235).
// 1,048,575 events over 20,011 groups: 39 us; with a radix partition and
// gathers through it the whole call took 157 us, now 61 us.
template <uint32_t kGr, bool kEv>
__global__ __launch_bounds__(kOT) void k_calc_own(CalArgs a)
{
    constexpr bool kStage = kEv && kGr == kG;
    constexpr int kKeyBits = kGr == kG ? 8 : 9;
    static_assert(kGr <= kOW << kKeyBits, "a wave's groups fit the key");
    constexpr uint32_t kChunks = kOStep / 64;   // of 64 events per step: u * kOW + wave
    static_assert(kChunks * kOW == 64 * 16 && kOU == 4, "16 counts per lane");
    __shared__ double sB[kGr];            // the chunk's map per group so far: offset
    __shared__ uint32_t sK[kGr];          // and count of usable events
    __shared__ double stb[kOStep];        // staged events: alpha r (or 0),
    __shared__ uint32_t stm[kOStep];      // slot | key << 12 | usable << 31
    __shared__ double ob[kStage ? kOStep : 1];
    __shared__ uint32_t ok_[kStage ? kOStep : 1];
    __shared__ __align__(16) uint8_t cnt[kOW * kChunks];   // [owner][chunk]
    __shared__ double pw64[65];           // powers of 1 - alpha
    const uint32_t t = threadIdx.x, lane = (uint32_t)lane_id();
    const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(t >> 6));
    if (a.clear && a.status && blockIdx.x == 0 && t == 0) *a.status = 0;
    // block b: XCD b % 8, where it is the (b / 8)-th; the ranges of one chunk
    // follow each other there
    uint32_t c = blockIdx.x, r = 0;
    if (kGr != kG) {
        const uint32_t y = blockIdx.x / 8u;
        c = blockIdx.x % 8u + 8u * (y / a.R);
        r = y % a.R;
        if (c >= a.C) return;
    }
    const uint32_t g0 = r * kGr, gn = a.G - g0 < kGr ? a.G - g0 : kGr;
    for (uint32_t g = t; g < kGr; g += kOT) {
        sB[g] = 0.0;
        sK[g] = 0;
    }
    uint32_t bm[4];
#pragma unroll
    for (uint32_t q = 0; q < 4; q++)
        bm[q] = w >= 4 * q + 4 ? 0xFFFFFFFFu : w <= 4 * q ? 0u : (1u << (8 * (w - 4 * q))) - 1u;
    const uint64_t c0 = (uint64_t)c * a.L;
    const uint64_t c1 = c0 + a.L < a.E ? c0 + a.L : a.E;
    OwnStep cur;
    own_load(a, c0, c1, cur);
    // (while those loads are in flight) the powers of 1 - alpha: the block's,
    // and the tables that k_calc_scan and k_calc_ev read
    if (t <= 64) pw64[t] = pow(a.oma, (double)t);
    if (blockIdx.x == 0) a.pw[t] = pow(a.oma, (double)(t & 255u) * (double)(1u << (8 * (t >> 8))));
    lds_sync();
    for (uint64_t s0 = c0; s0 < c1; s0 += kOStep) {
        const OwnStep s = cur;
        if (s0 + kOStep < c1) own_load(a, s0 + kOStep, c1, cur);
        uint64_t peers[kOU];
        uint32_t lg[kOU];
        bool in[kOU];
#pragma unroll
        for (uint32_t u = 0; u < kOU; u++) {
            lg[u] = s.g[u] - g0;   // wraps below g0
            in[u] = s.g[u] >= g0 && lg[u] < gn;
            uint32_t mine;
            peers[u] = match_count<4>(lg[u], __ballot(in[u]), mine);
            if (lane < kOW) cnt[lane * kChunks + u * kOW + w] = (uint8_t)mine;   // owner = lane
        }
        lds_sync();
        const OwnPlaces pl = own_places(cnt, bm, w);
        if (pl.heavy) {
            // per event, its map from its lanes' first: offset B, and slope
            // (1 - alpha)^k; at: the place of its group's entry, k, the
            // group's last lane, the group's lane before this one
            double B[kOU];
            uint32_t at[kOU];
            lds_sync();   // (cnt has been read)
#pragma unroll
            for (uint32_t u = 0; u < kOU; u++) {
                const bool use = in[u] && isfinite(s.x[u]) && s.x[u] > 0.0;
                double A = 1.0;
                B[u] = 0.0;
                if (use) {
                    const double ratio = (double)s.o[u] / s.x[u];
                    A = a.oma;
                    B[u] = a.alpha * ratio;
                }
                uint64_t same = match_bits<kKeyBits + 4>(lg[u], __ballot(in[u]));
                if (!in[u]) same = 1ull << lane;
                uint32_t rank, mine;
                int prev0;
                own_chain(same, A, B[u], rank, prev0);
                const uint32_t k = (uint32_t)__popcll(__ballot(use) & same & lanemask_lt()) + (use ? 1u : 0u);
                const uint32_t l = 63u - (uint32_t)__clzll((long long)same);
                at[u] = (uint32_t)__popcll(match_count<4>(lg[u], __ballot(in[u] && l == lane), mine) & lanemask_lt()) |
                        k << 13 | l << 20 | (uint32_t)prev0 << 26;
                if (lane < kOW) cnt[lane * kChunks + u * kOW + w] = (uint8_t)mine;
            }
            lds_sync();
            const OwnPlaces ph = own_places(cnt, bm, w);
#pragma unroll
            for (uint32_t u = 0; u < kOU; u++) {
                at[u] += (uint32_t)__shfl((int)ph.at, (int)(4 * (lg[u] & (kOW - 1)) + u), 64);
                if (in[u] && ((at[u] >> 20) & 63u) == lane) {   // the group's last lane
                    stb[at[u] & 8191u] = B[u];
                    stm[at[u] & 8191u] = ((at[u] >> 13) & 127u) | (lg[u] / kOW) << 12;
                }
            }
            lds_sync();
            for (uint32_t i = ph.lo; i < ph.hi; i += 64) {
                const bool live = i + lane < ph.hi;
                // (no entry behind the last lane's: the places of earlier rounds hold maps by now)
                const uint32_t q = live ? i + lane : ph.lo;
                const uint32_t m = live ? stm[q] : 0u, key = m >> 12, g = key * kOW + w, k = m & 127u;
                double cA = pw64[k], cB = live ? stb[q] : 0.0;
                uint64_t cs = match_bits<kKeyBits>(key, __ballot(live));
                if (!live) cs = 0;
                uint32_t rank;
                int prev0;
                own_chain(cs, cA, cB, rank, prev0);
                const double gb = sB[g];
                const uint32_t gk = sK[g];
                const double tt = cA * gb;
                const double xb = tt + cB;
                uint32_t ks = live ? k : 0u;   // the lanes' counts up to this one
                int prev = prev0;
                for (uint32_t st = 1; __ballot(rank >= st); st <<= 1) {
                    const uint32_t pk = (uint32_t)__shfl((int)ks, prev, 64);
                    const int pp = __shfl(prev, prev, 64);
                    if (rank >= st) {
                        ks += pk;
                        prev = pp;
                    }
                }
                const uint32_t xk = gk + ks;
                const double qb = __shfl(xb, prev0, 64);
                const uint32_t qk = (uint32_t)__shfl((int)xk, prev0, 64);
                if (live) {   // the group's map before these lanes
                    stb[q] = rank ? qb : gb;
                    stm[q] = rank ? qk : gk;
                }
                if (live && (cs >> lane) >> 1 == 0) {
                    sB[g] = xb;
                    sK[g] = xk;
                }
            }
            if constexpr (kEv) {
                lds_sync();
#pragma unroll
                for (uint32_t u = 0; u < kOU; u++) {
                    const int l = (int)((at[u] >> 20) & 63u), pv = (int)(at[u] >> 26);
                    const bool last = in[u] && l == (int)lane;
                    const double hb = last ? stb[at[u] & 8191u] : 0.0;
                    const uint32_t hk = last ? stm[at[u] & 8191u] : 0u, k = (at[u] >> 13) & 127u;
                    const double gb = __shfl(hb, l, 64);
                    const uint32_t gk = (uint32_t)__shfl((int)hk, l, 64);
                    const double tt = pw64[k] * gb;
                    double eb = tt + B[u];
                    uint32_t ek = gk + k;
                    if (!a.incl) {
                        const double qb = __shfl(eb, pv, 64);
                        const uint32_t qk = (uint32_t)__shfl((int)ek, pv, 64);
                        eb = pv != (int)lane ? qb : gb;
                        ek = pv != (int)lane ? qk : gk;
                    }
                    if (in[u]) {
                        a.xb[s0 + u * kOT + t] = eb;
                        a.xk[s0 + u * kOT + t] = ek;
                    }
                }
            }
            continue;   // (the next step's first writes to LDS are to cnt, then a barrier)
        }
#pragma unroll
        for (uint32_t u = 0; u < kOU; u++) {
            const uint32_t p = (uint32_t)__shfl((int)pl.at, (int)(4 * (lg[u] & (kOW - 1)) + u), 64) +
                               (uint32_t)__popcll(peers[u] & lanemask_lt());
            if (in[u]) {
                const bool use = isfinite(s.x[u]) && s.x[u] > 0.0;
                double b = 0.0;
                if (use) {
                    const double ratio = (double)s.o[u] / s.x[u];
                    b = a.alpha * ratio;
                }
                stb[p] = b;
                stm[p] = (u * kOT + t) | (lg[u] / kOW) << 12 | (use ? 0x80000000u : 0u);
            }
        }
        lds_sync();
        for (uint32_t i = pl.lo; i < pl.hi; i += 64) {
            const bool live = i + lane < pl.hi;
            const uint32_t p = live ? i + lane : pl.lo;
            const uint32_t m = stm[p], key = (m >> 12) & ((1u << kKeyBits) - 1u), g = key * kOW + w;
            const bool use = live && (m >> 31);
            double A = use ? a.oma : 1.0, B = stb[p];
            uint64_t same = match_bits<kKeyBits>(key, __ballot(live));
            if (!live) same = 0;
            const uint64_t uses = __ballot(use) & same;
            uint32_t rank;
            int prev0;
            own_chain(same, A, B, rank, prev0);
            const double gb = sB[g];
            const uint32_t gk = sK[g];
            const double tt = A * gb;
            const double xb = tt + B;
            const uint32_t xk = gk + (uint32_t)__popcll(uses & lanemask_lt()) + (use ? 1u : 0u);
            if (live && (same >> lane) >> 1 == 0) {   // the group's last lane
                sB[g] = xb;
                sK[g] = xk;
            }
            if constexpr (kEv) {
                double eb = xb;
                uint32_t ek = xk;
                if (!a.incl) {   // up to the event before
                    const double qb = __shfl(xb, prev0, 64);
                    const uint32_t qk = (uint32_t)__shfl((int)xk, prev0, 64);
                    eb = rank ? qb : gb;
                    ek = rank ? qk : gk;
                }
                const uint32_t slot = m & (kOStep - 1u);
                if (live) {
                    if constexpr (kStage) {
                        ob[slot] = eb;
                        ok_[slot] = ek;
                    } else {
                        a.xb[s0 + slot] = eb;
                        a.xk[s0 + slot] = ek;
                    }
                }
            }
        }
        if constexpr (kStage) {
            lds_sync();
#pragma unroll
            for (uint32_t u = 0; u < kOU; u++)
                if (in[u]) {   // (an event of no group has no map)
                    a.xb[s0 + u * kOT + t] = ob[u * kOT + t];
                    a.xk[s0 + u * kOT + t] = ok_[u * kOT + t];
                }
        }
    }
    lds_sync();
    for (uint32_t g = t; g < gn; g += kOT) {
        a.aggK[(uint64_t)c * a.G + g0 + g] = sK[g];
        a.aggB[(uint64_t)c * a.G + g0 + g] = sB[g];
    }
}

// (1 - alpha)^k from the base-256 digits of k.
__device__ __forceinline__ double slope(const double *pw, uint32_t k)
{
    double p = pw[k & 255u];
    p *= pw[256u + ((k >> 8) & 255u)];
    if (k >> 16) {
        p *= pw[512u + ((k >> 16) & 255u)];
        p *= pw[768u + (k >> 24)];
    }
    return p;
}

// Carries before every chunk, and the final factors: one block per 64
// groups (lane = group, so every read of a chunk's row is 512 contiguous
// bytes), its sixteen waves over sixteen stretches of the chunks. Each wave
// composes its stretch's maps per group; each then takes the initial factor
// through the earlier stretches' maps in order and walks its own stretch,
// writing the factor before each chunk.
constexpr uint32_t kScanW = 16;
constexpr uint32_t kScanRegs = 16;   // a wave's stretch of chunk maps held in registers, at most
__global__ __launch_bounds__(64 * kScanW) void k_calc_scan(CalArgs a)
{
    __shared__ double sA[kScanW][64], sB[kScanW][64];
    __shared__ uint32_t sU[kScanW][64];
    __shared__ double pw[1024];
    pw[threadIdx.x] = a.pw[threadIdx.x];
    const uint32_t w = threadIdx.x >> 6;
    const int lane = lane_id();
    const uint32_t g = blockIdx.x * 64u + (uint32_t)lane;
    const bool in = g < a.G;
    const uint32_t per = (a.C + kScanW - 1) / kScanW;
    const uint32_t cb = w * per < a.C ? w * per : a.C, ce = cb + per < a.C ? cb + per : a.C;
    if (per <= kScanRegs) {
        // the stretch's maps in registers: one round of loads, walked twice
        double A[kScanRegs], B[kScanRegs];
        uint32_t K[kScanRegs];
        Map agg = {0u, 0u, 1.0, 0.0};
#pragma unroll
        for (uint32_t r = 0; r < kScanRegs; r++) {
            K[r] = 0;
            B[r] = 0.0;
            if (in && cb + r < ce) {
                K[r] = a.aggK[(uint64_t)(cb + r) * a.G + g];
                B[r] = a.aggB[(uint64_t)(cb + r) * a.G + g];
            }
        }
        __syncthreads();   // pw
#pragma unroll
        for (uint32_t r = 0; r < kScanRegs; r++) A[r] = K[r] ? slope(pw, K[r]) : -1.0;
#pragma unroll
        for (uint32_t r = 0; r < kScanRegs; r++)
            if (A[r] >= 0.0) agg = combine(agg, Map{0u, 1u, A[r], B[r]});
        sA[w][lane] = agg.a;
        sB[w][lane] = agg.b;
        sU[w][lane] = agg.u;
        double v = in ? a.state[g] : 0.0;   // (by every wave before the barrier, behind which one overwrites it)
        __syncthreads();
        if (!in) return;
        bool touched = false;
        for (uint32_t q = 0; q < kScanW; q++) {
            if (!sU[q][lane]) continue;
            touched = true;
            if (q < w) {
                const double tt = sA[q][lane] * v;
                v = tt + sB[q][lane];
            }
        }
#pragma unroll
        for (uint32_t r = 0; r < kScanRegs; r++) {
            if (cb + r >= ce) break;
            a.carry[(uint64_t)(cb + r) * a.G + g] = v;
            if (A[r] >= 0.0) {
                const double tt = A[r] * v;
                v = tt + B[r];
            }
        }
        // the wave holding the last chunk writes the factor after all events
        // (a group without usable events keeps its factor untouched)
        if (ce == a.C && cb < ce && touched) a.state[g] = v;
        return;
    }
    // four chunks' maps in flight at a time
    constexpr uint32_t kR = 4;
    Map agg = {0u, 0u, 1.0, 0.0};
    __syncthreads();   // pw
    if (in)
        for (uint32_t c0 = cb; c0 < ce; c0 += kR) {
            double A[kR], B[kR];
            uint32_t K[kR];
#pragma unroll
            for (uint32_t r = 0; r < kR; r++) {
                K[r] = 0;
                B[r] = 0.0;
                if (c0 + r < ce) {
                    K[r] = a.aggK[(uint64_t)(c0 + r) * a.G + g];
                    B[r] = a.aggB[(uint64_t)(c0 + r) * a.G + g];
                }
            }
#pragma unroll
            for (uint32_t r = 0; r < kR; r++) A[r] = K[r] ? slope(pw, K[r]) : -1.0;
#pragma unroll
            for (uint32_t r = 0; r < kR; r++)
                if (A[r] >= 0.0) agg = combine(agg, Map{0u, 1u, A[r], B[r]});
        }
    sA[w][lane] = agg.a;
    sB[w][lane] = agg.b;
    sU[w][lane] = agg.u;
    double v = in ? a.state[g] : 0.0;   // (before the barrier, as above)
    __syncthreads();
    if (!in) return;
    bool touched = false;
    for (uint32_t q = 0; q < kScanW; q++) {
        if (!sU[q][lane]) continue;
        touched = true;
        if (q < w) {
            const double tt = sA[q][lane] * v;
            v = tt + sB[q][lane];
        }
    }
    for (uint32_t c0 = cb; c0 < ce; c0 += kR) {
        double A[kR], B[kR];
        uint32_t K[kR];
#pragma unroll
        for (uint32_t r = 0; r < kR; r++) {
            K[r] = 0;
            B[r] = 0.0;
            if (c0 + r < ce) {
                K[r] = a.aggK[(uint64_t)(c0 + r) * a.G + g];
                B[r] = a.aggB[(uint64_t)(c0 + r) * a.G + g];
            }
        }
#pragma unroll
        for (uint32_t r = 0; r < kR; r++) A[r] = K[r] ? slope(pw, K[r]) : -1.0;
#pragma unroll
        for (uint32_t r = 0; r < kR; r++) {
            if (c0 + r >= ce) break;
            a.carry[(uint64_t)(c0 + r) * a.G + g] = v;
            if (A[r] >= 0.0) {
                const double tt = A[r] * v;
                v = tt + B[r];
            }
        }
    }
    // the wave holding the last chunk writes the factor after all events
    // (a group without usable events keeps its factor untouched)
    if (ce == a.C && cb < ce && touched) a.state[g] = v;
}

// Large tables: every event's factor from its chunk's carry and its map
// from the chunk's start. With incl (the trace alone) the map includes the
// event and gives its trace; otherwise it gives the factor before the
// event, followed by the exact update (Eq. 5 with the ratio of Eq. 6) for a
// usable event. Blocks of 1024 events, which lie in one chunk (chunks are a
// multiple of 2048 events). The dispatcher deals blocks to the 8 XCDs round
// robin; consecutive event ranges go to blocks on the same XCD, so that each
// chunk's row of carries is fetched into one XCD's L2 (not all eight).
constexpr uint32_t kEvR = 4;
constexpr uint32_t kXcds = 8;
static_assert(256 * kEvR == 1024, "");
__global__ __launch_bounds__(256) void k_calc_ev(CalArgs a)
{
    __shared__ double pw[1024];
    const uint32_t t = threadIdx.x;
    const uint32_t per = gridDim.x / kXcds, b = blockIdx.x;
    const uint32_t lb = b < per * kXcds ? (b % kXcds) * per + b / kXcds : b;
    const uint32_t e0 = lb * 1024u;
    const uint64_t row = (uint64_t)(e0 / a.L) * a.G;
    uint32_t g[kEvR], k[kEvR], o[kEvR];
    double xb[kEvR], x[kEvR];
#pragma unroll
    for (uint32_t r = 0; r < kEvR; r++) {
        const uint32_t i = e0 + r * 256u + t;
        g[r] = a.G;
        k[r] = 0;
        o[r] = 0;
        xb[r] = 0.0;
        x[r] = 0.0;
        if (i < a.E) {
            g[r] = a.group[i];
            k[r] = a.xk[i];
            xb[r] = a.xb[i];
            if (!a.incl) {
                x[r] = a.est[i];
                o[r] = a.obs[i];
            }
        }
    }
    double pv[4];
#pragma unroll
    for (uint32_t r = 0; r < 4; r++) pv[r] = a.pw[r * 256u + t];
    double cv[kEvR];
#pragma unroll
    for (uint32_t r = 0; r < kEvR; r++) cv[r] = g[r] < a.G ? a.carry[row + g[r]] : 0.0;
#pragma unroll
    for (uint32_t r = 0; r < 4; r++) pw[r * 256u + t] = pv[r];
    __syncthreads();
    const double nan = __builtin_nan("");
#pragma unroll
    for (uint32_t r = 0; r < kEvR; r++) {
        const uint32_t i = e0 + r * 256u + t;
        if (i >= a.E) break;
        double before = nan, after = nan;
        if (g[r] < a.G) {
            double v = cv[r];
            if (k[r]) {
                const double tt = slope(pw, k[r]) * v;
                v = tt + xb[r];
            }
            before = v;
            if (!a.incl && isfinite(x[r]) && x[r] > 0.0) {
                const double ratio = (double)o[r] / x[r];
                const double t1 = a.oma * v;
                v = t1 + a.alpha * ratio;
            }
            after = v;
        }
        if (a.trace) a.trace[i] = after;
        if (a.trace_before) a.trace_before[i] = before;
    }
}

template <int kE>
__global__ __launch_bounds__(kT) void k_calc_apply(CalArgs a)
{
    constexpr uint32_t kSub = kT * kE;
    __shared__ SubShared<kE> sh;
    __shared__ double trb[kSub];   // trace_before staging (the trace goes to sh.b)
    __shared__ double sv[kG];      // each group's factor at the current point of the chunk
    __shared__ uint8_t su[kG];     // the group has a usable event so far
    const uint32_t t = threadIdx.x, c = blockIdx.x;
    // the carry is the maps of the chunks before this one, composed in order (tpg threads per group, each over a contiguous range
    // of chunks, kCarryR maps loaded at a time, then an ordered tree of
    // shuffles), applied to the initial factor; a chunk without usable
    // events of the group leaves it untouched. The first kCarryR maps are
    // loaded before the first sub-tile's events and composed after them, so
    // that both loads are in flight together.
    uint32_t tpg = 1;
    while (tpg < 64 && tpg * 2 * a.G <= (uint32_t)kT) tpg *= 2;
    const bool quick = a.G <= (uint32_t)kT / tpg;
    double cA[kCarryR], cB[kCarryR];
    const uint32_t cjb = (t % tpg) * c / tpg, cje = (t % tpg + 1) * c / tpg;
    if (quick) {
        const uint32_t g = t / tpg, jb = cjb, je = cje;
#pragma unroll
        for (int r = 0; r < (int)kCarryR; r++) {
            const uint32_t j = jb + (uint32_t)r;
            cA[r] = -1.0;
            cB[r] = 0.0;
            if (g < a.G && j < je) {
                cA[r] = a.aggA[(uint64_t)j * a.G + g];
                cB[r] = a.aggB[(uint64_t)j * a.G + g];
            }
        }
    } else {
        for (uint32_t g = t; g < a.G; g += kT) {
            double v = a.s0[g];
            bool u = false;
            for (uint32_t j = 0; j < c; j++) {
                const double A = a.aggA[(uint64_t)j * a.G + g], B = a.aggB[(uint64_t)j * a.G + g];
                if (A >= 0.0) {
                    const double tt = A * v;
                    v = tt + B;
                    u = true;
                }
            }
            sv[g] = v;
            su[g] = (uint8_t)u;
        }
    }
    const uint64_t c0 = (uint64_t)c * a.L;
    const uint64_t c1 = c0 + a.L < a.E ? c0 + a.L : a.E;
    const double nan = __builtin_nan("");
    double *tr = sh.b;
    for (uint64_t s0 = c0; s0 < c1; s0 += kSub) {
        const uint32_t m = (uint32_t)(c1 - s0 < kSub ? c1 - s0 : kSub);
        Raw<kE> raw;
        load_raw<kE>(a, (uint32_t)s0, m, raw);
        Sub<kE> sub;
        load_sort_scan<kE>(a, raw, m, sh, sub);
        if (quick && s0 == c0) {
            const uint32_t g = t / tpg, p = t % tpg;
            Map mp = {0u, 0u, 1.0, 0.0};
#pragma unroll
            for (int r = 0; r < (int)kCarryR; r++)
                if (cA[r] >= 0.0) mp = combine(mp, Map{0u, 1u, cA[r], cB[r]});
            for (uint32_t j0 = cjb + kCarryR; j0 < cje; j0 += kCarryR) {
#pragma unroll
                for (int r = 0; r < (int)kCarryR; r++) {
                    const uint32_t j = j0 + (uint32_t)r;
                    cA[r] = -1.0;
                    cB[r] = 0.0;
                    if (g < a.G && j < cje) {
                        cA[r] = a.aggA[(uint64_t)j * a.G + g];
                        cB[r] = a.aggB[(uint64_t)j * a.G + g];
                    }
                }
#pragma unroll
                for (int r = 0; r < (int)kCarryR; r++)
                    if (cA[r] >= 0.0) mp = combine(mp, Map{0u, 1u, cA[r], cB[r]});
            }
            for (uint32_t d = 1; d < tpg; d <<= 1) {
                Map o;
                o.f = 0u;
                o.u = (uint32_t)__shfl_down((int)mp.u, (int)d, 64);
                o.a = shfl_down_d(mp.a, (int)d);
                o.b = shfl_down_d(mp.b, (int)d);
                if (p % (2 * d) == 0) mp = combine(mp, o);
            }
            if (g < a.G && p == 0) {
                double v = a.s0[g];
                if (mp.u) {
                    const double tt = mp.a * v;
                    v = tt + mp.b;
                }
                sv[g] = v;
                su[g] = (uint8_t)mp.u;
            }
            lds_sync();
        }
        // the factor before this thread's first position: the group's factor
        // at the sub-tile start, through the earlier positions of its
        // segment (their composed map, if any of them is usable)
        double cv;
        {
            const uint32_t g0 = sub.key[0];
            const double base = g0 < a.G ? sv[g0] : nan;
            cv = base;
            if (!sub.flag[0] && sub.excl.u) {
                const double tt = sub.excl.a * base;
                cv = tt + sub.excl.b;
            }
        }
        double after[kE];
#pragma unroll
        for (int e = 0; e < kE; e++) {
            const uint32_t i = t * kE + (uint32_t)e;
            after[e] = cv;
            if (i >= m) continue;
            const uint32_t g = sub.key[e];
            if (sub.flag[e]) cv = g < a.G ? sv[g] : nan;
            trb[sub.slot[e]] = cv;
            if (sub.ok[e]) su[g] = 1;
            if (sub.ok[e]) {
                // the exact sequential update
                const double t1 = a.oma * cv;
                cv = t1 + sub.b[e];
            }
            tr[sub.slot[e]] = cv;
            after[e] = cv;
        }
        lds_sync();   // every read of sv above precedes the updates below
#pragma unroll
        for (int e = 0; e < kE; e++) {
            const uint32_t i = t * kE + (uint32_t)e;
            if (i >= m) break;
            const bool last = (i + 1 == m) || (e + 1 < kE ? sub.flag[e + 1] != 0u : sh.key[i + 1] != sh.key[i]);
            const uint32_t g = sub.key[e];
            if (last && g < a.G) sv[g] = after[e];
        }
        // the traces in event order
        for (uint32_t i = t; i < m; i += kT) {
            if (a.trace) a.trace[s0 + i] = tr[i];
            if (a.trace_before) a.trace_before[s0 + i] = trb[i];
        }
        lds_sync();
    }
    if (c + 1 == a.C) {
        // the factors after all events: the groups with a usable event in
        // some chunk (the others keep theirs untouched)
        for (uint32_t g = t; g < a.G; g += kT)
            if (su[g]) a.state[g] = sv[g];
    }
}

// ---- one launch for small tables of one sub-tile per chunk -------------------
//
// Each block publishes its chunk's maps M(c, g) as two 64-bit words per group
// (A, then B) as soon as it has formed them, and only then reads the words
// of the chunks before it, so a block never waits before publishing. Every
// word was set to kUnset (a signalling NaN) by k_calc_unset just before: A
// is -1 or in [0, 1] and B an arithmetic result (never a signalling NaN), so
// each word shows by itself whether it has been written, and no ordering
// between the stores of a block is needed.
constexpr uint64_t kUnset = 0x7FF4DEADBEEF0001ull;
constexpr uint32_t kOneChunks = 64;   // chunks of the one-launch path at most
// Events that one block takes as a single chunk, without the unset words and
// their launch. Replays of a graph, chunks of 512 and one block: 500 events
// 7.8 and 6.2 us, 1,000 10.6 and 7.5, 2,048 11.7 and 9.3 (8 groups); 3,000 12.2
// and 12.3, 4,096 12.4 and 13.4 (1 group 9.9 and 14.4).
constexpr uint32_t kOneBlock = 4 * kT;
constexpr uint32_t kOneR = 16;   // chunk maps per thread loaded at once

__device__ __forceinline__ uint64_t ld_relaxed64(const uint64_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void st_relaxed64(uint64_t *p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__global__ __launch_bounds__(256) void k_calc_unset(uint64_t *w, uint32_t nw, uint32_t *wait_status)
{
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (wait_status && i == 0) *wait_status = 0;
    for (uint32_t k = i; k < nw; k += gridDim.x * 256u) w[k] = kUnset;
}

template <int kE>
__global__ __launch_bounds__(kT) void k_calc_one(CalArgs a)
{
    constexpr uint32_t kSub = kT * kE;
    static_assert(kSub <= kG, "the trace_before staging shares sA");
    __shared__ SubShared<kE> sh;
    __shared__ double sA[kG], sB[kG];   // this chunk's map per group; sA then stages trace_before
    __shared__ double sv[kG];           // each group's factor (initial, then at the current point)
    __shared__ uint8_t su[kG];          // the group has a usable event so far
    const uint32_t t = threadIdx.x, c = blockIdx.x;
    if (a.C == 1 && a.clear && a.status && t == 0) *a.status = 0;   // (else by k_calc_unset)
    // the initial factors are read before this block publishes anything: the
    // last block overwrites them only after every other block has published
    for (uint32_t g = t; g < a.G; g += kT) {
        sA[g] = -1.0;
        sB[g] = 0.0;
        sv[g] = a.state[g];
        su[g] = 0;
    }
    const uint64_t c0 = (uint64_t)c * kSub;
    const uint32_t m = (uint32_t)(a.E - c0 < kSub ? a.E - c0 : kSub);
    Raw<kE> raw;
    load_raw<kE>(a, (uint32_t)c0, m, raw);
    Sub<kE> sub;
    load_sort_scan<kE>(a, raw, m, sh, sub);   // (its first barrier orders the writes above)
    // which positions end their group's segment
    uint32_t lastm = 0;
#pragma unroll
    for (int e = 0; e < kE; e++) {
        const uint32_t i = t * kE + (uint32_t)e;
        if (i < m && ((i + 1 == m) || (e + 1 < kE ? sub.flag[e + 1] != 0u : sh.key[i + 1] != sh.key[i])))
            lastm |= 1u << e;
    }
    // this chunk's map of each group: its segment composed at its last position
    {
        Map run = sub.excl;
#pragma unroll
        for (int e = 0; e < kE; e++) {
            if (t * kE + (uint32_t)e >= m) break;
            Map mp;
            mp.f = sub.flag[e];
            mp.u = sub.ok[e];
            mp.a = sub.ok[e] ? a.oma : 1.0;
            mp.b = sub.ok[e] ? sub.b[e] : 0.0;
            mp.k = sub.ok[e];
            run = mp.f ? mp : combine(run, mp);
            const uint32_t g = sub.key[e];
            if (((lastm >> e) & 1u) && g < a.G && run.u) {
                sA[g] = run.a;
                sB[g] = run.b;
            }
        }
    }
    lds_sync();
    uint64_t *pubA = reinterpret_cast<uint64_t *>(a.aggA), *pubB = reinterpret_cast<uint64_t *>(a.aggB);
    if (c + 1 < a.C)   // the last chunk's maps are read by nobody
        for (uint32_t g = t; g < a.G; g += kT) {
            st_relaxed64(&pubA[(uint64_t)c * a.G + g], (uint64_t)__double_as_longlong(sA[g]));
            st_relaxed64(&pubB[(uint64_t)c * a.G + g], (uint64_t)__double_as_longlong(sB[g]));
        }
    // the carry of each group: the maps of chunks 0 .. c-1 composed in order
    // (tpg threads per group, each over a contiguous range of them, then an
    // ordered tree of shuffles), applied to the initial factor
    uint32_t tpg = 1;
    while (tpg < 64 && tpg * 2 * a.G <= (uint32_t)kT) tpg *= 2;
    const uint32_t p = t % tpg, jb = p * c / tpg, je = (p + 1) * c / tpg;
    bool gave_up = false;
    for (uint32_t g0 = 0; g0 < a.G; g0 += kT / tpg) {
        const uint32_t g = g0 + t / tpg;
        const bool gin = g < a.G;
        Map mp = {0u, 0u, 1.0, 0.0};
        if (c > 0 && a.no_wait) gave_up = true;
        for (uint32_t j0 = jb; gin && !gave_up && j0 < je; j0 += kOneR) {
            uint64_t A[kOneR], B[kOneR];
#pragma unroll
            for (uint32_t r = 0; r < kOneR; r++) {
                A[r] = 0;
                B[r] = 0;
                if (j0 + r < je) {
                    A[r] = ld_relaxed64(&pubA[(uint64_t)(j0 + r) * a.G + g]);
                    B[r] = ld_relaxed64(&pubB[(uint64_t)(j0 + r) * a.G + g]);
                }
            }
            // a word still unset is read again until it is written (bounded)
            uint32_t spins = 0;
            for (;;) {
                bool ready = true;
#pragma unroll
                for (uint32_t r = 0; r < kOneR; r++) ready = ready && A[r] != kUnset && B[r] != kUnset;
                if (ready) break;
                if (++spins > kSpinLimit) {
                    gave_up = true;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
#pragma unroll
                for (uint32_t r = 0; r < kOneR; r++) {
                    if (A[r] == kUnset) A[r] = ld_relaxed64(&pubA[(uint64_t)(j0 + r) * a.G + g]);
                    if (B[r] == kUnset) B[r] = ld_relaxed64(&pubB[(uint64_t)(j0 + r) * a.G + g]);
                }
            }
#pragma unroll
            for (uint32_t r = 0; r < kOneR; r++) {
                const double av = __longlong_as_double((long long)A[r]);
                if (j0 + r < je && av >= 0.0)
                    mp = combine(mp, Map{0u, 1u, av, __longlong_as_double((long long)B[r])});
            }
        }
        for (uint32_t d = 1; d < tpg; d <<= 1) {
            Map o;
            o.f = 0u;
            o.u = (uint32_t)__shfl_down((int)mp.u, (int)d, 64);
            o.a = shfl_down_d(mp.a, (int)d);
            o.b = shfl_down_d(mp.b, (int)d);
            if (p % (2 * d) == 0) mp = combine(mp, o);
        }
        if (gin && p == 0 && mp.u) {
            const double tt = mp.a * sv[g];
            sv[g] = tt + mp.b;
            su[g] = 1;
        }
    }
    if (gave_up && a.status) atomicOr(a.status, 1u);
    lds_sync();
    // every event's exact update from its factor before (as in k_calc_apply)
    const double nan = __builtin_nan("");
    double *tr = sh.b, *trb = sA;
    double cv;
    {
        const uint32_t g0 = sub.key[0];
        const double base = g0 < a.G ? sv[g0] : nan;
        cv = base;
        if (!sub.flag[0] && sub.excl.u) {
            const double tt = sub.excl.a * base;
            cv = tt + sub.excl.b;
        }
    }
    double after[kE];
#pragma unroll
    for (int e = 0; e < kE; e++) {
        const uint32_t i = t * kE + (uint32_t)e;
        after[e] = cv;
        if (i >= m) continue;
        const uint32_t g = sub.key[e];
        if (sub.flag[e]) cv = g < a.G ? sv[g] : nan;
        trb[sub.slot[e]] = cv;
        if (sub.ok[e]) {
            su[g] = 1;
            const double t1 = a.oma * cv;
            cv = t1 + sub.b[e];
        }
        tr[sub.slot[e]] = cv;
        after[e] = cv;
    }
    lds_sync();   // every read of sv above precedes the updates below
#pragma unroll
    for (int e = 0; e < kE; e++) {
        const uint32_t g = sub.key[e];
        if (((lastm >> e) & 1u) && g < a.G) sv[g] = after[e];
    }
    for (uint32_t i = t; i < m; i += kT) {
        if (a.trace) a.trace[c0 + i] = tr[i];
        if (a.trace_before) a.trace_before[c0 + i] = trb[i];
    }
    if (c + 1 == a.C) {
        lds_sync();
        for (uint32_t g = t; g < a.G; g += kT)
            if (su[g]) a.state[g] = sv[g];
    }
}

// Events per thread of the one-launch path for E events and G groups (a
// chunk is one sub-tile of kT times that many events), or 0 when the chunks
// would be too many or their table of maps too large for it.
uint32_t one_e(uint64_t E, uint32_t G)
{
    if (G > kG) return 0;
    for (uint32_t e = 1; e <= 4; e *= 2) {
        const uint64_t C = cdiv(E ? E : 1, (uint64_t)kT * e);
        if (C <= kOneChunks && C * G <= kSmallTable) return e;
    }
    return 0;
}

uint32_t sub_per_chunk(uint64_t E, uint32_t G, uint32_t kSub)
{
    uint64_t cmax = (G > kG ? kMaxTableR : kMaxTable) / (G ? G : 1);
    cmax = cmax < kMaxChunks ? cmax : kMaxChunks;
    cmax = cmax ? cmax : 1;
    const uint64_t subs = cdiv(E, kSub);
    return (uint32_t)(cdiv(subs, cmax) ? cdiv(subs, cmax) : 1);
}

}  // namespace

// Chunks of a multiple of sub events: events per chunk and chunks.
static void chunking(uint64_t n, uint32_t G, uint32_t sub, uint32_t &L, uint32_t &C)
{
    L = sub * sub_per_chunk(n, G, sub);
    C = (uint32_t)cdiv(n ? n : 1, L);
}

// The kernels that take n events of G groups.
enum class Route { One, Small, Own };

struct CalcPlan {
    Route route;
    uint32_t e;      // One: events per thread
    uint32_t L, C;   // events per chunk, chunks
};

// few: k_calc_agg and k_calc_apply wherever their table is at most kFewTable.
static CalcPlan calc_plan(uint64_t n, uint32_t G, bool few, bool traced)
{
    CalcPlan p;
    p.e = one_e(n, G);
    if (p.e) {
        p.route = Route::One;
        p.L = kT * p.e;
        p.C = (uint32_t)cdiv(n ? n : 1, p.L);
        return p;
    }
    p.route = Route::Small;
    chunking(n, G, kT, p.L, p.C);
    uint64_t most = 0;
    if (few) most = kFewTable;
    else if (p.L == (uint32_t)kT) most = traced ? kSmallTraced : kSmallPair;
    else if (p.L == 2u * kT && traced) most = p.C <= 257 ? kPairTraced256 : kPairTraced;
    if (G <= kG && (uint64_t)p.C * G <= most) return p;
    p.route = Route::Own;
    chunking(n, G, kOStep, p.L, p.C);
    return p;
}

// Bytes of a table of `entries` maps, and of the other arrays.
static size_t calc_bytes(Route route, uint64_t entries, uint64_t n, uint32_t G)
{
    if (route != Route::Own) return 2 * align_up(entries * 8, 256) + align_up((uint64_t)G * 8, 256);
    return align_up(entries * 4, 256) + align_up(entries * 8, 256) + align_up(1024 * 8, 256) + align_up(n * 8, 256) +
           align_up(n * 4, 256);
}

size_t calc_own_bytes(uint64_t n, uint32_t G)
{
    const CalcPlan p = calc_plan(n, G, false, false);
    return calc_bytes(p.route, (uint64_t)p.C * G, n, G);
}

size_t calc_need_bytes(uint64_t n, uint32_t G)
{
    const CalcPlan p = calc_plan(n, G, true, false);
    return calc_bytes(p.route, (uint64_t)p.C * G, n, G);
}

// Non-decreasing in n and in G: the tables of the most chunks that any call
// of at most n events and G groups makes.
size_t calc_ws_bytes(uint64_t n, uint32_t G)
{
    auto table = [n](uint64_t sub, uint64_t cap, uint64_t g) {
        const uint64_t chunks = cdiv(n ? n : 1, sub), most = (chunks < kMaxChunks ? chunks : kMaxChunks) * g;
        return most < cap ? most : cap;
    };
    const size_t small = calc_bytes(Route::Small, table(kT, kSmallTable, G < kG ? G : kG), n, G < kG ? G : kG);
    if (calc_plan(n, G, false, false).route != Route::Own) return small;
    const size_t own = calc_bytes(Route::Own, table(kOStep, G > kG ? kMaxTableR : kMaxTable, G), n, G);
    return own > small ? own : small;
}

hipError_t calc_launch(const uint32_t *group, const double *est, const uint32_t *obs, uint32_t n,
                       double alpha, uint32_t G, double *state, double *trace, double *trace_before,
                       void *ws, size_t ws_bytes, hipStream_t s, WaitCfg wait)
{
    if (n == 0) return hipSuccess;
    if (G == 0 || G > kCalGroupsChunked) return hipErrorInvalidValue;
    CalArgs a;
    a.group = group;
    a.est = est;
    a.obs = obs;
    a.E = n;
    a.G = G;
    a.alpha = alpha;
    a.oma = 1.0 - alpha;
    // few chunks of one sub-tile each: one launch (after the unset words);
    // else sub-tiles of 512 events when the table of chunk maps stays small
    // (the carries are then formed in k_calc_apply), else steps of 4096, which
    // keep 12 bytes of every event. In few groups the sub-tiles need none of
    // these, in any number of events, and serve a workspace without the room.
    CalcPlan plan = calc_plan(n, G, false, trace || trace_before);
    if (ws_bytes < calc_bytes(plan.route, (uint64_t)plan.C * G, n, G)) {
        plan = calc_plan(n, G, true, false);
        if (ws_bytes < calc_bytes(plan.route, (uint64_t)plan.C * G, n, G)) return hipErrorInvalidValue;
    }
    const uint32_t one = plan.e;
    a.L = plan.L;
    a.C = plan.C;
    a.R = G > kG ? (uint32_t)cdiv(G, kRangeGroups) : 1u;
    a.passes = G < 256 ? 1u : 2u;   // keys 0..G fit in 8 or 16 bits
    a.keybits = 1;
    while ((1u << a.keybits) <= G) a.keybits++;
    uint8_t *p = static_cast<uint8_t *>(ws);
    auto take = [&p](uint64_t bytes) {
        uint8_t *q = p;
        p += align_up(bytes, 256);
        return q;
    };
    const uint64_t entries = (uint64_t)a.C * G;
    a.aggA = nullptr;
    a.aggK = nullptr;
    a.carry = a.s0 = a.pw = a.xb = nullptr;
    a.xk = nullptr;
    if (plan.route == Route::Own) {
        a.aggK = reinterpret_cast<uint32_t *>(take(entries * 4));
        a.aggB = reinterpret_cast<double *>(take(entries * 8));
        a.carry = a.aggB;   // (each thread of k_calc_scan has read a map when it writes the carry there)
        a.pw = reinterpret_cast<double *>(take(1024 * 8));
        a.xb = reinterpret_cast<double *>(take((uint64_t)n * 8));
        a.xk = reinterpret_cast<uint32_t *>(take((uint64_t)n * 4));
    } else {
        a.aggA = reinterpret_cast<double *>(take(entries * 8));
        a.aggB = reinterpret_cast<double *>(take(entries * 8));
        a.s0 = reinterpret_cast<double *>(take((uint64_t)G * 8));
    }
    a.state = state;
    a.trace = trace;
    a.trace_before = trace_before;
    a.status = wait.status;
    a.clear = wait.clear ? 1u : 0u;
    a.no_wait = wait.no_wait ? 1u : 0u;
    a.incl = trace_before ? 0u : 1u;
    if (one) {
        // one sub-tile per chunk: the words the chunks publish are unset
        // first, then one launch does the rest
        // (up to kOneBlock events one chunk of them all: nothing is published,
        // so nothing to unset. DS_NO_WAIT exercises the waits between chunks.)
        if (n <= kOneBlock && !a.no_wait) {
            a.C = 1;
            if (n <= kT) hipLaunchKernelGGL(k_calc_one<1>, dim3(1), dim3(kT), 0, s, a);
            else if (n <= 2 * kT) hipLaunchKernelGGL(k_calc_one<2>, dim3(1), dim3(kT), 0, s, a);
            else hipLaunchKernelGGL(k_calc_one<4>, dim3(1), dim3(kT), 0, s, a);
            return hipGetLastError();
        }
        const uint32_t nw = (uint32_t)(align_up(entries * 8, 256) / 8 + entries);
        const uint32_t fb = (uint32_t)(cdiv(nw, 256) < 256 ? cdiv(nw, 256) : 256);
        hipLaunchKernelGGL(k_calc_unset, dim3(fb), dim3(256), 0, s, reinterpret_cast<uint64_t *>(a.aggA), nw,
                           a.clear ? a.status : nullptr);
        if (one == 1) hipLaunchKernelGGL(k_calc_one<1>, dim3(a.C), dim3(kT), 0, s, a);
        else if (one == 2) hipLaunchKernelGGL(k_calc_one<2>, dim3(a.C), dim3(kT), 0, s, a);
        else hipLaunchKernelGGL(k_calc_one<4>, dim3(a.C), dim3(kT), 0, s, a);
    } else if (plan.route == Route::Small) {
        hipLaunchKernelGGL(k_calc_agg<1>, dim3(a.C), dim3(kT), 0, s, a);
        hipLaunchKernelGGL(k_calc_apply<1>, dim3(a.C), dim3(kT), 0, s, a);
    } else {
        const bool ev = trace || trace_before;   // else the final factors alone
        const dim3 grid(G > kG ? (uint32_t)align_up(a.C, 8) * a.R : a.C);
        if (G > kG && ev)
            hipLaunchKernelGGL((k_calc_own<kRangeGroups, true>), grid, dim3(kOT), 0, s, a);
        else if (G > kG)
            hipLaunchKernelGGL((k_calc_own<kRangeGroups, false>), grid, dim3(kOT), 0, s, a);
        else if (ev)
            hipLaunchKernelGGL((k_calc_own<kG, true>), grid, dim3(kOT), 0, s, a);
        else
            hipLaunchKernelGGL((k_calc_own<kG, false>), grid, dim3(kOT), 0, s, a);
        hipLaunchKernelGGL(k_calc_scan, dim3((G + 63) / 64), dim3(64 * kScanW), 0, s, a);
        if (ev) hipLaunchKernelGGL(k_calc_ev, dim3((uint32_t)cdiv(n, 1024)), dim3(256), 0, s, a);
    }
    return hipGetLastError();
}

}  // namespace ds
