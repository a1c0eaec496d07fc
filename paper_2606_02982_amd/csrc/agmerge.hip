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
//               it in every other run; writes the permutation and the key
// Results are identical to sorting by (score, arrival, index): the scores
// are computed with the same operations as the other paths, and FIFO
// position order is (arrival, index) order.
#include <string.h>

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
// run, the entries below it there. A block takes 1024 entries of one run; one
// wave per other run and end of the tile finds where the tile's first and last
// entries fall (64-way probing), the stretch between is staged in LDS piece by
// piece (2048 entries) and each entry searched in it. Of a stretch of many
// pieces the first and the last are staged, and what falls between them is
// searched in memory (a run far shorter than another).
// What bounds it: latency (six blocks per CU, each a chain of about ten
// dependent reads and two staged pieces). In place of ceil(log2 K) rounds of
// pairwise merges, which wrote and read every entry each round: the whole
// Aging order of 2,097,152 requests, 3 classes 140 -> 99 us, 8 classes
// 165 -> 117, 16 classes 190 -> 134; of 4,194,304, 3 classes 279 -> 190 (of it the search
// itself 56 -> 34 us at 2,097,152). With 99% of 1,048,576 requests in one class
// the few tiles of the others set the time: 74 -> 86 us.
constexpr uint32_t kRkT = 256, kRkPer = 4, kRkTile = kRkT * kRkPer;
constexpr uint32_t kRkPiece = 2048, kRkPieces = 4;

// The entries of a run (k, p)[0, n) below (x, y), found by one wave: among
// the run's every kAmStep-th entries first (hk, hp: few pages, near each
// other), then among the 64 entries behind the last of those below.
static_assert(kAmStep == 64, "one probe of the wave");
__device__ inline uint32_t run_below(const uint64_t *k, const uint32_t *p, uint32_t n, const uint64_t *hk,
                                     const uint32_t *hp, uint64_t x, uint32_t y)
{
    uint32_t lo = 0, hi = (n + kAmStep - 1u) / kAmStep;
    const uint32_t lane = (uint32_t)lane_id();
    while (hi > lo) {
        const uint32_t span = hi - lo;
        const uint32_t m = lo + (uint32_t)(((uint64_t)span * lane) >> 6);   // lo <= m < hi
        const uint64_t km = hk[m];
        const bool b = km < x || (km == x && hp[m] < y);
        const uint32_t f = (uint32_t)__popcll(__ballot(b));   // probes 0..f-1 are below, f.. are not
        const uint32_t nlo = f ? lo + (uint32_t)(((uint64_t)span * (f - 1u)) >> 6) + 1u : lo;
        hi = f < 64u ? lo + (uint32_t)(((uint64_t)span * f) >> 6) : hi;
        lo = nlo;
    }
    if (lo == 0) return 0;
    const uint32_t base = (lo - 1u) * kAmStep, m = base + lane;
    const bool in = m < n;
    const uint64_t km = in ? k[m] : 0;
    const uint32_t pm = in ? p[m] : 0;
    return base + (uint32_t)__popcll(__ballot(in && (km < x || (km == x && pm < y))));
}

// The first n (at most kRkPiece) of the entries at (qk, qp), staged in LDS, and
// how many of them are below each of the thread's entries.
__device__ __forceinline__ void rk_piece(uint64_t *sk, uint32_t *sp, const uint64_t *qk, const uint32_t *qp,
                                         uint32_t n, const uint64_t (&k)[kRkPer], const uint32_t (&p)[kRkPer],
                                         uint32_t (&pos)[kRkPer])
{
    __syncthreads();
    for (uint32_t x = threadIdx.x; x < kRkPiece; x += kRkT) {
        const bool in = x < n;
        sk[x] = in ? qk[x] : ~0ull;   // (past the end: above every entry)
        sp[x] = in ? qp[x] : ~0u;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t r = 0; r < kRkPer; r++) pos[r] = 0;
    // steps of 1024 .. 1, the entries of a thread side by side, then the last
#pragma unroll
    for (uint32_t st = kRkPiece / 2; st > 0; st >>= 1) {
#pragma unroll
        for (uint32_t r = 0; r < kRkPer; r++) {
            const uint32_t y = pos[r] + st - 1u;
            if (am_less(sk[y], sp[y], k[r], p[r])) pos[r] += st;
        }
    }
#pragma unroll
    for (uint32_t r = 0; r < kRkPer; r++)
        if (am_less(sk[pos[r]], sp[pos[r]], k[r], p[r])) pos[r]++;   // (pos < kRkPiece before)
}

__global__ __launch_bounds__(kRkT) void k_am_rank(AmArgs a)
{
    __shared__ uint64_t sk[kRkPiece];
    __shared__ uint32_t sp[kRkPiece];
    __shared__ uint32_t from[kAmCls], to[kAmCls];
    const uint32_t t = threadIdx.x, w = t >> 6;
    // the block's run c and its tile there (blocks are handed to the runs in order)
    uint32_t b = blockIdx.x, c = 0, r0 = 0, len = 0;
    for (; c < a.K; c++) {
        r0 = a.cstart[c];
        len = a.cstart[c + 1u < a.K ? c + 1u : a.K] - r0;
        const uint32_t tiles = (len + kRkTile - 1u) / kRkTile;
        if (b < tiles) break;
        b -= tiles;
    }
    if (c >= a.K) return;   // the same for the whole block
    const uint32_t i0 = b * kRkTile, cnt = len - i0 < kRkTile ? len - i0 : kRkTile;
    const uint64_t *rk = a.rk;
    const uint32_t *rp = a.rp;
    uint64_t k[kRkPer];
    uint32_t p[kRkPer], rank[kRkPer];
#pragma unroll
    for (uint32_t r = 0; r < kRkPer; r++) {
        const uint32_t i = r * kRkT + t, g = r0 + i0 + (i < cnt ? i : 0u);
        k[r] = rk[g];
        p[r] = rp[g];
        rank[r] = i0 + i;
    }
    // wave w: the ends of searches w, w + 4, ... (run q, first or last entry)
    for (uint32_t x = w; x < 2u * a.K; x += kRkT / 64) {
        const uint32_t q = x >> 1, e = r0 + i0 + (x & 1u ? cnt - 1u : 0u);
        if (q == c) continue;
        const uint32_t q0 = a.cstart[q], qn = a.cstart[q + 1u < a.K ? q + 1u : a.K] - q0;
        const uint32_t h0 = am_step_at(q0, q);
        const uint32_t f = run_below(rk + q0, rp + q0, qn, a.hk + h0, a.hp + h0, rk[e], rp[e]);
        if (lane_id() == 0) (x & 1u ? to : from)[q] = f;
    }
    __syncthreads();
    for (uint32_t q = 0; q < a.K; q++) {
        if (q == c) continue;
        // the stretch (empty where the inputs break the contract and the run is not sorted)
        const uint32_t f = from[q], n = to[q] > f ? to[q] - f : 0u;
        const uint64_t *qk = rk + a.cstart[q] + f;
        const uint32_t *qp = rp + a.cstart[q] + f;
#pragma unroll
        for (uint32_t r = 0; r < kRkPer; r++) rank[r] += f;
        if (n <= kRkPiece * kRkPieces) {
            for (uint32_t x0 = 0; x0 < n; x0 += kRkPiece) {
                uint32_t pos[kRkPer];
                rk_piece(sk, sp, qk + x0, qp + x0, n - x0, k, p, pos);
#pragma unroll
                for (uint32_t r = 0; r < kRkPer; r++) rank[r] += pos[r];
            }
            continue;
        }
        // a long stretch: most entries fall into its first piece or its last
        // one (where the floor cuts the tile: the clamped entries tie with
        // their neighbours in time, the others follow every clamped one)
        uint32_t pos[kRkPer];
        bool open[kRkPer];
        rk_piece(sk, sp, qk, qp, kRkPiece, k, p, pos);
#pragma unroll
        for (uint32_t r = 0; r < kRkPer; r++) {
            open[r] = pos[r] == kRkPiece;
            rank[r] += pos[r];
        }
        rk_piece(sk, sp, qk + (n - kRkPiece), qp + (n - kRkPiece), kRkPiece, k, p, pos);
        // (the searches in memory side by side)
        uint32_t lo[kRkPer], hi[kRkPer];
#pragma unroll
        for (uint32_t r = 0; r < kRkPer; r++) {
            lo[r] = hi[r] = n - kRkPiece + pos[r];
            if (!open[r]) lo[r] = hi[r] = kRkPiece;
            else if (!pos[r]) lo[r] = kRkPiece;
        }
        bool more = true;
        while (more) {
            uint64_t km[kRkPer];
            uint32_t pm[kRkPer];
#pragma unroll
            for (uint32_t r = 0; r < kRkPer; r++) {
                const uint32_t m = (lo[r] + hi[r]) >> 1;   // < n
                km[r] = lo[r] < hi[r] ? qk[m] : 0;
                pm[r] = lo[r] < hi[r] ? qp[m] : 0;
            }
            more = false;
#pragma unroll
            for (uint32_t r = 0; r < kRkPer; r++) {
                if (lo[r] >= hi[r]) continue;
                const uint32_t m = (lo[r] + hi[r]) >> 1;
                if (am_less(km[r], pm[r], k[r], p[r])) lo[r] = m + 1u;
                else hi[r] = m;
                more |= lo[r] < hi[r];
            }
        }
#pragma unroll
        for (uint32_t r = 0; r < kRkPer; r++) rank[r] += lo[r] - kRkPiece;
    }
#pragma unroll
    for (uint32_t r = 0; r < kRkPer; r++) {
        if (r * kRkT + t >= cnt || rank[r] >= a.n) continue;
        uint32_t i = a.in.fifo[p[r]];
        i = i < a.n ? i : 0u;
        a.perm[rank[r]] = i;
        if (a.key_out) a.key_out[i] = am_aged(a.in, i, am_tier(a.in, i));
    }
}

void rank_launch(const AmArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(k_am_rank, dim3((uint32_t)cdiv(a.n, kRkTile) + a.K), dim3(kRkT), 0, s, a);
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
           align_up(n * 4, 256) + align_up(n, 256) + am_steps_bytes(n);
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
    a.perm = perm;
    a.key_out = key_out;
    a.wait_status = wait_status;
    hipLaunchKernelGGL(k_am_count, dim3(a.tiles), dim3(kAmTPB), 0, s, a);
    hipLaunchKernelGGL(k_am_scan, dim3(1), dim3(1024), 0, s, a);
    hipLaunchKernelGGL(k_am_place, dim3(a.tiles), dim3(kAmTPB), 0, s, a);
    rank_launch(a, s);
    return hipGetLastError();
}

hipError_t am_rank_launch(const SortInput &in, uint32_t n_classes, const LsRuns &runs, uint32_t *perm,
                          double *key_out, hipStream_t s)
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
    rank_launch(a, s);
    return hipGetLastError();
}

}  // namespace ds
