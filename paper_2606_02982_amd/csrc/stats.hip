// Estimation error of budget estimates against observed output lengths
// (Sec. "Impact of Workload Characterization and Runtime Calibration":
// tab:four_mode_token_error and tab:error_reduction) and runtime-class
// counts per semantic category (Eq. (4); tab:workload_mapping).
//
// Error: for every event with a usable estimate x = est[e] * factor[e]
// (finite and > 0; no factor = 1), d = x - obs[e]; per group and over all
// events: count, sum |d|, sum d^2 and sum obs / x. Each block takes a
// contiguous range of events and accumulates per-group sums in LDS (4096
// groups per pass over its range) and the all-events sums in registers; it
// stores its partial sums, and a last kernel adds the blocks' partials in a
// fixed order and forms MAE = sum|d| / count, RMSE = sqrt(sum d^2 / count),
// mean bias = sum(obs / x) / count. The sums in LDS are added to by LDS adds,
// each by one wave alone and in the order of its lanes, so that every order of
// addition is fixed by the data and the launch shape: results
// are the same from run to run and agree with any sequential sum within the
// rounding of an n-term sum.
#include "common.h"
#include "kernels.h"

namespace ds {
namespace {

constexpr uint32_t kT = 256;
constexpr uint32_t kMaxBlocks = 256;

constexpr uint32_t kEA = 1024;              // threads of an accumulating block
constexpr uint32_t kWaves = kEA / 64;
constexpr uint32_t kSlots = 4096;           // sums in LDS
constexpr uint32_t kWaveSlots = kSlots / kWaves;
constexpr uint32_t kU = 2;                  // events per thread per step
constexpr uint32_t kStep = kU * kEA;
constexpr uint32_t kChunks = kStep / 64;
constexpr uint32_t kNone = 0xFFFFFFFFu;

__device__ __forceinline__ bool usable(double x) { return isfinite(x) && x > 0.0; }

struct Sums {
    double a[kSlots], q[kSlots], r[kSlots];   // sum |d|, sum d^2, sum obs / x
    uint32_t n[kSlots];
};

// One step's events in registers.
struct Step {
    double x[kU], f[kU];
    uint32_t o[kU], g[kU];
};

__device__ __forceinline__ void load_step(const double *__restrict__ est,
                                          const double *__restrict__ factor,
                                          const uint32_t *__restrict__ obs,
                                          const uint32_t *__restrict__ group, uint64_t b0,
                                          uint64_t e1, Step &s)
{
#pragma unroll
    for (uint32_t u = 0; u < kU; u++) {
        const uint64_t e = b0 + u * kEA + threadIdx.x;
        const bool in = e < e1;
        s.x[u] = in ? est[e] : 0.0;           // 0: not usable
        s.f[u] = in && factor ? factor[e] : 1.0;
        s.o[u] = in ? obs[e] : 0u;
        s.g[u] = in && group ? group[e] : kNone;
    }
}

__device__ __forceinline__ double wave_sum_f64(double v)
{
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// s[slot] += v as one LDS instruction (no read back). Only one lane of a wave
// and one wave of the block ever adds to a slot at a time, and a wave's LDS
// instructions execute in order, so the order of additions is fixed.
template <typename T> __device__ __forceinline__ void lds_add(T *p, T v)
{
    __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Adds one event per lane (where ok) to the sum at `slot`. Lanes share a
// key (< 256) exactly when they share a slot, or with kCopies copies of a
// group's sums (copy = lane mod kCopies) a group; no other wave touches the
// slot, so a wave settles its collisions by itself: lanes of one slot add in
// lane order, one instruction after another; a key with many lanes (one tenant
// holding most of the events) is added up across the wave in a tree first.
template <uint32_t kCopies>
__device__ __forceinline__ void add_events(Sums &S, uint32_t slot, uint32_t key, bool ok, double a,
                                           double q, double r)
{
    constexpr uint32_t kHeavy = kCopies > 1 ? 2 * kCopies : 4;                 // more lanes take the tree
    constexpr uint32_t kLight = kCopies > 1 ? 64 / kCopies : kHeavy;           // lanes on one slot otherwise
    const uint32_t lane = (uint32_t)lane_id();
    uint64_t peers = match_bits<8>(key, __ballot(ok));
    if (!ok) peers = 0;
    for (;;) {
        const uint64_t heavy = __ballot((uint32_t)__popcll(peers) > kHeavy);
        if (!heavy) break;
        const int l = __builtin_ctzll(heavy);
        const uint64_t m = readlane64(peers, l);
        const bool in = (m >> lane) & 1u;
        const double ta = wave_sum_f64(in ? a : 0.0);
        const double tq = wave_sum_f64(in ? q : 0.0);
        const double tr = wave_sum_f64(in ? r : 0.0);
        if ((int)lane == l) {
            lds_add(&S.n[slot], (uint32_t)__popcll(m));
            lds_add(&S.a[slot], ta);
            lds_add(&S.q[slot], tq);
            lds_add(&S.r[slot], tr);
        }
        if (in) peers = 0;
    }
    if constexpr (kCopies > 1) {
        static_assert(kCopies == 8, "the lanes of a copy");
        peers &= 0x0101010101010101ull << (lane & (kCopies - 1));
    }
    const uint32_t rank = peers ? (uint32_t)__popcll(peers & lanemask_lt()) : kNone;
    if (rank == 0) lds_add(&S.n[slot], (uint32_t)__popcll(peers));
    for (uint32_t k = 0; k < kLight && __ballot(rank != kNone && rank >= k); k++) {
        if (rank == k) {
            lds_add(&S.a[slot], a);
            lds_add(&S.q[slot], q);
            lds_add(&S.r[slot], r);
        }
        // keeps the instructions of different ranks apart
        __builtin_amdgcn_wave_barrier();
    }
}

// partial layout: [block][4][G + 1] (count, sum |d|, sum d^2, sum obs/x);
// slot G holds the all-events sums.
//
// kOwn false (G <= 256): every wave has sums of its own, and
// where there is room rep = 256 / G (a power of two, at most 64) of them per
// group, one per lane mod rep, so that lanes of one wave seldom meet.
// kOwn true: wave w owns the groups g = w (mod 16), with kCopies sums of each
// (8 up to 512 groups, where a wave's 64 events else meet on 16 to 32 sums:
// 65,536 events of 257 groups 33.6 us with one, 17.4 with eight). A step's 2048 events are
// split by owner, stably, through LDS (4 ballots per 64 events, one table of
// counts that every wave scans for itself: two barriers a step), and each
// wave adds up its own events in event order. The next step's loads are in
// flight meanwhile (the barriers wait on LDS alone).
//
// What bounds it: LDS. At 4,194,304 events over 4,096 groups the block's sums
// take 112 KB, one block of 16 waves per CU, and the LDS pipe is busy 74% of
// the time (counters), mostly with the adds to random sums; every event is
// read and divided once. The form before (1,024 groups per pass, 4 waves that
// each walked every event of the block) took 634 us there, this one 79. The
// error statistics as a whole, before and after: 4,194,304 events, 4 groups
// 464 and 27 us, 256 groups 202 and 30, 4,096 groups 648 and 93, one group
// holding every event 1,740 and 205; 65,536 events, 1,000 groups 27 and 19.
template <bool kOwn, uint32_t kCopies = 1>
__global__ __launch_bounds__(kEA) void k_err_accum(uint64_t n, const double *__restrict__ est,
                                                   const double *__restrict__ factor,
                                                   const uint32_t *__restrict__ obs,
                                                   const uint32_t *__restrict__ group, uint32_t G,
                                                   uint32_t rep, double *__restrict__ partial)
{
    __shared__ Sums S;
    struct __align__(16) Staged {
        double x;
        uint32_t o, g;
    };
    __shared__ Staged st[kOwn ? kStep : 1];
    __shared__ __align__(16) uint16_t cnt[kOwn ? kWaves * kChunks : 8];   // [owner][chunk of 64]
    __shared__ double wsum[4][kWaves];
    const uint64_t slots = (uint64_t)G + 1;
    double *mine = partial + (uint64_t)blockIdx.x * 4 * slots;
    const uint64_t per = cdiv(n, gridDim.x);
    const uint64_t e0 = (uint64_t)blockIdx.x * per;
    const uint64_t e1 = e0 + per < n ? e0 + per : n;
    const uint32_t t = threadIdx.x, lane = (uint32_t)lane_id();
    const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(t >> 6));

    double c = 0.0, sa = 0.0, sq = 0.0, sr = 0.0;   // all events
    for (uint32_t c0 = 0; c0 == 0 || c0 < G; c0 += kSlots) {
        const uint32_t cn = G - c0 < kSlots ? G - c0 : kSlots;
        for (uint32_t i = t; i < kSlots; i += kEA) {
            S.n[i] = 0;
            S.a[i] = S.q[i] = S.r[i] = 0.0;
        }
        lds_sync();
        Step cur;
        load_step(est, factor, obs, group, e0, e1, cur);
        for (uint64_t b0 = e0; b0 < e1; b0 += kStep) {
            Step s = cur;
            if (b0 + kStep < e1) load_step(est, factor, obs, group, b0 + kStep, e1, cur);
#pragma unroll
            for (uint32_t u = 0; u < kU; u++) s.x[u] = s.x[u] * s.f[u];
            if constexpr (!kOwn) {
#pragma unroll
                for (uint32_t u = 0; u < kU; u++) {
                    const bool ok = usable(s.x[u]);
                    const double o = (double)s.o[u], d = s.x[u] - o;
                    const double a = fabs(d), q = d * d, r = o / s.x[u];
                    if (ok) {
                        c += 1.0;
                        sa += a;
                        sq += q;
                        sr += r;
                    }
                    const uint32_t key = (s.g[u] * rep + (lane & (rep - 1))) & (kWaveSlots - 1);
                    add_events<1>(S, w * kWaveSlots + key, key, ok && s.g[u] < G, a, q, r);
                }
            } else {
                // the wave's two chunks of 64 events by owner
                uint64_t peers[kU];
                bool ok[kU];
#pragma unroll
                for (uint32_t u = 0; u < kU; u++) {
                    s.g[u] -= c0;   // wraps below c0
                    // events of no group of this pass still count among all events (once)
                    ok[u] = usable(s.x[u]) && (c0 == 0 || s.g[u] < cn);
                    uint32_t mine;
                    peers[u] = match_count<4>(s.g[u], __ballot(ok[u]), mine);
                    if (lane < kWaves) cnt[lane * kChunks + u * kWaves + w] = (uint16_t)mine;   // owner = lane
                }
                lds_sync();
                // lane l holds owner l / 4, chunks 8 (l % 4) .. + 7
                const uint4 v = *reinterpret_cast<const uint4 *>(&cnt[lane * 8]);
                const uint32_t pk[4] = {v.x, v.y, v.z, v.w};
                uint32_t sum = 0, before = 0;   // before: the lane's chunks below w % 8
#pragma unroll
                for (uint32_t k = 0; k < 8; k++) {
                    if (k == (w & 7u)) before = sum;
                    sum += (pk[k >> 1] >> (16 * (k & 1u))) & 0xFFFFu;
                }
                const uint32_t incl = wave_incl_scan_dpp(sum);
                const uint32_t at = incl - sum + before;
                const uint32_t lo = w ? readlane32(incl, (int)(4 * w - 1)) : 0u;
                const uint32_t hi = readlane32(incl, (int)(4 * w + 3));
#pragma unroll
                for (uint32_t u = 0; u < kU; u++) {
                    const uint32_t ow = s.g[u] & (kWaves - 1);
                    const uint32_t p = (uint32_t)__shfl((int)at, (int)(4 * ow + 2 * u + (w >> 3)), 64) +
                                       (uint32_t)__popcll(peers[u] & lanemask_lt());
                    if (ok[u]) st[p] = {s.x[u], s.o[u], s.g[u]};
                }
                lds_sync();
                for (uint32_t i = lo; i < hi; i += 64) {
                    const bool in = i + lane < hi;
                    const Staged ev = st[in ? i + lane : lo];
                    const double x = ev.x, o = (double)ev.o;
                    const uint32_t g = ev.g;
                    const double d = x - o, a = fabs(d), q = d * d, r = o / x;
                    if (in && c0 == 0) {
                        c += 1.0;
                        sa += a;
                        sq += q;
                        sr += r;
                    }
                    const bool own = in && g < cn;
                    const uint32_t key = (g / kWaves) & (kWaveSlots - 1);   // (the wave's groups)
                    const uint32_t slot = kCopies > 1 ? (key * kCopies + lane % kCopies) * kWaves + w : g;
                    add_events<kCopies>(S, own ? slot : 0u, key, own, a, q, r);
                }
            }
        }
        __syncthreads();
        if constexpr (kOwn) {
            for (uint32_t i = t; i < cn; i += kEA) {
                double m[4] = {0.0, 0.0, 0.0, 0.0};
                for (uint32_t k = 0; k < kCopies; k++) {
                    const uint32_t j = ((i / kWaves) * kCopies + k) * kWaves + (i & (kWaves - 1));
                    m[0] += (double)S.n[j];
                    m[1] += S.a[j];
                    m[2] += S.q[j];
                    m[3] += S.r[j];
                }
                for (uint32_t k = 0; k < 4; k++) mine[k * slots + c0 + i] = m[k];
            }
            __syncthreads();
        } else if (t < kWaveSlots) {
            double m[4] = {0.0, 0.0, 0.0, 0.0};
            for (uint32_t k = 0; k < kWaves; k++) {
                const uint32_t i = k * kWaveSlots + t;
                m[0] += (double)S.n[i];
                m[1] += S.a[i];
                m[2] += S.q[i];
                m[3] += S.r[i];
            }
            for (uint32_t off = rep >> 1; off >= 1; off >>= 1)
                for (int k = 0; k < 4; k++) m[k] += __shfl_xor(m[k], (int)off, 64);
            if ((t & (rep - 1)) == 0 && t / rep < G)
                for (int k = 0; k < 4; k++) mine[k * slots + t / rep] = m[k];
        }
        if (!kOwn) break;
    }

    c = wave_sum_f64(c);
    sa = wave_sum_f64(sa);
    sq = wave_sum_f64(sq);
    sr = wave_sum_f64(sr);
    if (lane == 0) {
        wsum[0][w] = c;
        wsum[1][w] = sa;
        wsum[2][w] = sq;
        wsum[3][w] = sr;
    }
    __syncthreads();
    if (t < 4) {
        double v = 0.0;
        for (uint32_t k = 0; k < kWaves; k++) v += wsum[t][k];
        mine[t * slots + G] = v;
    }
}

// The all-events sums alone (no groups): 256 threads, and 1,024 above 2^20
// events, where 256 leave too few loads in flight. k_err_accum's cleared and
// folded LDS cost a small call a third: 2,000 events 8.4 us, 6.0 here; 1,048,576
// 11.6 and 9.4; 4,194,304 21.9 and 18.1.
template <uint32_t kTh>
__global__ __launch_bounds__(kTh) void k_err_all(uint64_t n, const double *__restrict__ est,
                                                 const double *__restrict__ factor,
                                                 const uint32_t *__restrict__ obs, double *__restrict__ partial)
{
    constexpr uint32_t kPer = kStep / kTh, kW = kTh / 64;
    __shared__ double wsum[4][kW];
    const uint64_t per = cdiv(n, gridDim.x);
    const uint64_t e0 = (uint64_t)blockIdx.x * per;
    const uint64_t e1 = e0 + per < n ? e0 + per : n;
    const uint32_t t = threadIdx.x;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    for (uint64_t b0 = e0; b0 < e1; b0 += kStep) {
        double x[kPer], f[kPer], o[kPer];
#pragma unroll
        for (uint32_t u = 0; u < kPer; u++) {
            const uint64_t e = b0 + u * kTh + t;
            const bool in = e < e1;
            x[u] = in ? est[e] : 0.0;   // 0: not usable
            f[u] = in && factor ? factor[e] : 1.0;
            o[u] = in ? (double)obs[e] : 0.0;
        }
#pragma unroll
        for (uint32_t u = 0; u < kPer; u++) {
            x[u] = x[u] * f[u];
            if (!usable(x[u])) continue;
            const double d = x[u] - o[u];
            v[0] += 1.0;
            v[1] += fabs(d);
            v[2] += d * d;
            v[3] += o[u] / x[u];
        }
    }
    for (uint32_t k = 0; k < 4; k++) {
        v[k] = wave_sum_f64(v[k]);
        if (lane_id() == 0) wsum[k][t >> 6] = v[k];
    }
    __syncthreads();
    if (t < 4) {
        double s = 0.0;
        for (uint32_t k = 0; k < kW; k++) s += wsum[t][k];
        partial[(uint64_t)blockIdx.x * 4 + t] = s;
    }
}

// stats[4 g ..]: a block per 16 group slots. Lane = (slot, which sum), wave =
// a sixteenth of the blocks' partials (64-byte and longer runs of a row,
// sixteen loads in flight), then the sixteen in order, then the means.
// (4,097 slots x 256 blocks: a wave per slot, lanes on blocks, took 26.6 us,
// this 11.2.)
constexpr uint32_t kFS = 16;

__global__ __launch_bounds__(kEA) void k_err_final(const double *__restrict__ partial,
                                                   uint32_t blocks, uint32_t G,
                                                   uint32_t with_groups, double *__restrict__ stats)
{
    __shared__ double part[kWaves][64];
    const uint64_t slots = (uint64_t)G + 1;
    const uint32_t lane = (uint32_t)lane_id(), w = threadIdx.x >> 6;
    const uint64_t g = (uint64_t)blockIdx.x * kFS + (lane & (kFS - 1));
    const uint32_t k = lane / kFS;
    double s = 0.0;
    if (g < slots && (g == G || with_groups)) {
        double v[kMaxBlocks / kWaves];
#pragma unroll
        for (uint32_t i = 0; i < kMaxBlocks / kWaves; i++) {
            const uint32_t b = i * kWaves + w;
            v[i] = b < blocks ? partial[((uint64_t)b * 4 + k) * slots + g] : 0.0;
        }
#pragma unroll
        for (uint32_t i = 0; i < kMaxBlocks / kWaves; i++) s += v[i];
    }
    part[w][lane] = s;
    __syncthreads();
    if (w) return;
    s = 0.0;
    for (uint32_t i = 0; i < kWaves; i++) s += part[i][lane];
    const double n = __shfl(s, (int)(lane & (kFS - 1)), 64);
    if (g >= slots) return;
    double *out = stats + 4 * g + k;
    if (k == 0)
        *out = s;
    else if (n > 0.0)
        *out = k == 2 ? sqrt(s / n) : s / n;
    else
        *out = __builtin_nan("");
}

// The one row of k_err_all's partials: a wave, lanes on blocks.
__global__ __launch_bounds__(64) void k_err_final_all(const double *__restrict__ partial, uint32_t blocks,
                                                      double *__restrict__ stats)
{
    const uint32_t lane = threadIdx.x;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    for (uint32_t b = lane; b < blocks; b += 64)
#pragma unroll
        for (uint32_t k = 0; k < 4; k++) v[k] += partial[(uint64_t)b * 4 + k];
#pragma unroll
    for (uint32_t k = 0; k < 4; k++) v[k] = wave_sum_f64(v[k]);
    if (lane != 0) return;
    const double n = v[0], nan = __builtin_nan("");
    stats[0] = n;
    stats[1] = n > 0.0 ? v[1] / n : nan;
    stats[2] = n > 0.0 ? sqrt(v[2] / n) : nan;
    stats[3] = n > 0.0 ? v[3] / n : nan;
}

__global__ void k_err_validate(uint64_t n, const uint32_t *__restrict__ group, uint32_t G,
                               uint32_t *__restrict__ flag)
{
    uint32_t bad = 0;
    for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (uint64_t)gridDim.x * blockDim.x)
        if (group[e] >= G) bad = 1;
    if (bad) atomicOr(flag, 1u);
}

__device__ __forceinline__ void hist_add(uint32_t *h, uint32_t c, uint32_t k, uint32_t n_cat)
{
    if (c < n_cat && k < 3) atomicAdd(&h[c * 3 + k], 1u);
}

// hist[c * 3 + k]: requests of category c in class k. kWide: both arrays are
// 16-byte aligned, 16 requests per load; otherwise byte loads. 4,194,304
// requests: 17.2 us with byte loads, 10.0 us with wide ones (128 blocks of
// 1,024 threads 12.2; copies of the cells per lane 9.7, not worth their code).
template <bool kWide>
__global__ __launch_bounds__(kT) void k_class_hist(uint32_t n, const uint8_t *__restrict__ category,
                                                    uint32_t n_cat, const uint8_t *__restrict__ cls,
                                                    uint32_t *__restrict__ hist)
{
    __shared__ uint32_t h[256 * 3];
    const uint32_t cells = n_cat * 3;
    for (uint32_t i = threadIdx.x; i < cells; i += kT) h[i] = 0;
    __syncthreads();
    const uint32_t id = blockIdx.x * kT + threadIdx.x, all = gridDim.x * kT;
    const uint32_t n16 = kWide ? n / 16 : 0;
    for (uint32_t i = id; i < n16; i += all) {
        const uint4 c = reinterpret_cast<const uint4 *>(category)[i];
        const uint4 k = reinterpret_cast<const uint4 *>(cls)[i];
        const uint32_t cw[4] = {c.x, c.y, c.z, c.w}, kw[4] = {k.x, k.y, k.z, k.w};
#pragma unroll
        for (int b = 0; b < 16; b++)
            hist_add(h, (cw[b >> 2] >> (8 * (b & 3))) & 0xFFu, (kw[b >> 2] >> (8 * (b & 3))) & 0xFFu, n_cat);
    }
    for (uint64_t i = (uint64_t)n16 * 16 + id; i < n; i += all) hist_add(h, category[i], cls[i], n_cat);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < cells; i += kT)
        if (h[i]) atomicAdd(&hist[i], h[i]);
}

__global__ void k_hist_validate(uint32_t n, const uint8_t *__restrict__ category, uint32_t n_cat,
                                const uint8_t *__restrict__ cls, uint32_t *__restrict__ flag)
{
    uint32_t bad = 0;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x)
        if (category[i] >= n_cat || cls[i] > 2) bad = 1;
    if (bad) atomicOr(flag, 1u);
}

uint32_t blocks_for(uint64_t n, uint32_t cap)
{
    uint64_t b = cdiv(n, kT);
    return (uint32_t)(b < 1 ? 1 : (b > cap ? cap : b));
}

}  // namespace

// Blocks of the error kernel: about 2048 events each, at most kMaxBlocks,
// and fewer when the partial sums of many groups would be large; at most 2^31
// events each.
static uint32_t err_blocks(uint64_t n, uint32_t G)
{
    uint64_t b = cdiv(n ? n : 1, 2048);
    const uint64_t cap = (1ull << 22) / ((uint64_t)G + 1);   // <= 128 MB of partials
    if (b > kMaxBlocks) b = kMaxBlocks;
    if (b > cap) b = cap;
    // (a block counts a group's events in 32 bits)
    const uint64_t least = cdiv(n ? n : 1, 1ull << 31);
    return (uint32_t)(b < least ? least : b);
}

size_t err_ws_bytes(uint64_t n, uint32_t n_groups)
{
    return align_up((uint64_t)err_blocks(n, n_groups) * 4 * ((uint64_t)n_groups + 1) * 8, 256);
}

hipError_t err_launch(uint64_t n, const double *est, const double *factor, const uint32_t *obs,
                      const uint32_t *group, uint32_t G, double *stats, void *ws, uint32_t *flag,
                      hipStream_t s)
{
    if (flag) {
        if (group && n)
            hipLaunchKernelGGL(k_err_validate, dim3(blocks_for(n, 1024)), dim3(kT), 0, s, n, group,
                               G, flag);
        return hipGetLastError();
    }
    double *partial = static_cast<double *>(ws);
    const uint32_t blocks = err_blocks(n, G);
    if (G == 0) {
        if (n <= 1u << 20)
            hipLaunchKernelGGL(k_err_all<256>, dim3(blocks), dim3(256), 0, s, n, est, factor, obs, partial);
        else
            hipLaunchKernelGGL(k_err_all<kEA>, dim3(blocks), dim3(kEA), 0, s, n, est, factor, obs, partial);
        hipLaunchKernelGGL(k_err_final_all, dim3(1), dim3(64), 0, s, (const double *)partial, blocks, stats);
        return hipGetLastError();
    }
    // up to 256 groups every wave's sums fit LDS beside the others'; up to 512
    // a wave owns at most 32 groups and keeps eight sums of each
    if (G <= kWaveSlots) {
        uint32_t rep = 64;
        while (rep > 1 && rep * G > kWaveSlots) rep >>= 1;
        hipLaunchKernelGGL(k_err_accum<false>, dim3(blocks), dim3(kEA), 0, s, n, est, factor, obs,
                           group, G, rep, partial);
    } else {
        const auto accum = G <= 2 * kWaveSlots ? k_err_accum<true, 8> : k_err_accum<true>;
        hipLaunchKernelGGL(accum, dim3(blocks), dim3(kEA), 0, s, n, est, factor, obs, group, G, 1u, partial);
    }
    hipLaunchKernelGGL(k_err_final, dim3((uint32_t)cdiv((uint64_t)G + 1, kFS)), dim3(kEA), 0, s,
                       (const double *)partial, blocks, G, group ? 1u : 0u, stats);
    return hipGetLastError();
}

hipError_t hist_launch(uint32_t n, const uint8_t *category, uint32_t n_cat, const uint8_t *cls,
                       uint32_t *hist, uint32_t *flag, hipStream_t s)
{
    if (flag) {
        if (n)
            hipLaunchKernelGGL(k_hist_validate, dim3(blocks_for(n, 1024)), dim3(kT), 0, s, n,
                               category, n_cat, cls, flag);
        return hipGetLastError();
    }
    hipError_t e = fill_u32(hist, 0u, (uint64_t)n_cat * 3, s);
    if (e != hipSuccess) return e;
    if (!n) return hipGetLastError();
    // below that the few blocks of wide loads lose to one request per thread:
    // 16,384 requests 4.1 and 3.9 us, 24,576 4.1 and 4.2, 65,536 4.1 and 6.0
    const bool wide = n >= 24576 && (((uintptr_t)category | (uintptr_t)cls) & 15u) == 0;
    const dim3 grid(wide ? blocks_for(cdiv(n, 16), 512) : blocks_for(n, 1024));
    if (wide)
        hipLaunchKernelGGL(k_class_hist<true>, grid, dim3(kT), 0, s, n, category, n_cat, cls, hist);
    else
        hipLaunchKernelGGL(k_class_hist<false>, grid, dim3(kT), 0, s, n, category, n_cat, cls, hist);
    return hipGetLastError();
}

}  // namespace ds
