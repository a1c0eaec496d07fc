// Orders of small batches by counting: a request's place under a policy is
// the number of requests before it. Up to kNoMaxN requests, comparing every
// pair in one launch takes less than the three dependent launches of the
// sample sorts (ssort.hip), whose time hardly depends on the batch there.
//
// A block takes cdiv(n, 256) rows (one block per compute unit) and every
// request of the batch once, one per lane: wave w the groups of 64 requests
// w, w + 16, ... For each row and pair of groups, the borrow of key - row's
// key - tie is the wave's mask of requests before the row:
//   F         by arrival, ties by index
//   SJF       by budget, ties by F
//   Aging     by score, ties by F
//   Priority  by class, ties by F
//   Weighted  F among the row's tier gives the rank in the tier, which the
//             closed form places
// The scalar unit counts the masks; the waves' counts are added in LDS.
//
// Bound by issue, n^2 / 64 row-group steps of some 10 vector and 12 scalar
// instructions over 1,024 SIMDs. Five orders, calls back to back: 1,024
// requests 49 us with the sample sorts and 11 here (bound by the host's
// launches), 4,096 39 and 18.0 (23.3 with two 64-bit comparisons per key),
// 6,144 37 and 32 (the waits behind the masks are 3% of it); 8,192 40 and
// about 50. FIFO alone: 4,096 23 and 9.2, 6,144 24 and 12.
#include "common.h"
#include "kernels.h"
#include "wrrplan.h"

namespace ds {
namespace {

constexpr uint32_t kNoTPB = 1024;
constexpr uint32_t kNoNW = kNoTPB / 64;
constexpr uint32_t kNoBlocks = 256;  // one per compute unit
constexpr uint32_t kNoRows = kNoMaxN / kNoBlocks;
constexpr uint32_t kNoQ = 16;
constexpr uint32_t kNoKey = 0xFFFFFFFFu;

struct NoBatch {
    SortInput in;
    uint32_t rows;
    uint32_t *perm[5];
    double *key[5];
};

struct NoKeys {
    uint64_t a, b, e;
    uint32_t cls, tier;
};

// The requests before a row (F, SJF, Aging, Priority), and its rank in its tier.
enum { kCntF = 0, kCntB = 1, kCntE = 2, kCntC = 3, kCntT = 4, kCnts = 5 };

// The aged score; each operation is rounded separately.
__device__ __forceinline__ double no_score(const SortInput &in, double a, double prio)
{
    double w = in.t_now - a;
    if (w < 0.0) w = 0.0;
    const double d = in.aging_rate * w;
    double e = prio - d;
    if (e < in.aging_floor) e = in.aging_floor;
    return e;
}

// The lanes of two groups whose key is below x, or equal to it where the
// lane's bit in t is set: the borrow of k - x - t, which the subtractions
// take and give as wave masks. (Written with comparisons, each key takes two
// of them, in 64 bits, and two scalar operations to combine them.) A vector
// instruction may read a mask two wait states after another one wrote it at the
// earliest. The compiler keeps that distance for its own instructions, but it
// does not see the writes in here: the waits at both ends are for a mask it
// wrote just before and for one it counts or spills just behind.
__device__ __forceinline__ void below2(uint64_t k0, uint64_t k1, uint64_t x, uint64_t t0, uint64_t t1, uint64_t &m0,
                                       uint64_t &m1)
{
    uint32_t d;
    uint64_t o0, o1;
    asm("s_nop 1\n\t"
        "v_subb_co_u32_e64 %[d], %[o0], %[l0], %[xl], %[t0]\n\t"
        "v_subb_co_u32_e64 %[d], %[o1], %[l1], %[xl], %[t1]\n\t"
        "s_nop 0\n\t"
        "v_subb_co_u32_e64 %[d], %[o0], %[h0], %[xh], %[o0]\n\t"
        "v_subb_co_u32_e64 %[d], %[o1], %[h1], %[xh], %[o1]\n\t"
        "s_nop 1"
        : [d] "=&v"(d), [o0] "=&s"(o0), [o1] "=&s"(o1)
        : [l0] "v"((uint32_t)k0), [h0] "v"((uint32_t)(k0 >> 32)), [l1] "v"((uint32_t)k1),
          [h1] "v"((uint32_t)(k1 >> 32)), [xl] "v"((uint32_t)x), [xh] "v"((uint32_t)(x >> 32)), [t0] "s"(t0),
          [t1] "s"(t1));
    m0 = o0;
    m1 = o1;
}

__device__ __forceinline__ void below2(uint32_t k0, uint32_t k1, uint32_t x, uint64_t t0, uint64_t t1, uint64_t &m0,
                                       uint64_t &m1)
{
    uint32_t d;
    uint64_t o0, o1;
    asm("s_nop 1\n\t"
        "v_subb_co_u32_e64 %[d], %[o0], %[k0], %[x], %[t0]\n\t"
        "v_subb_co_u32_e64 %[d], %[o1], %[k1], %[x], %[t1]\n\t"
        "s_nop 1"
        : [d] "=&v"(d), [o0] "=&s"(o0), [o1] "=&s"(o1)
        : [k0] "v"(k0), [k1] "v"(k1), [x] "v"(x), [t0] "s"(t0), [t1] "s"(t1));
    m0 = o0;
    m1 = o1;
}

// kG: groups per wave (an even number), at least n / (64 kNoNW); kB, kE, kP:
// SJF, Aging, and Priority or Weighted are wanted.
template <uint32_t kG, bool kB, bool kE, bool kP>
__global__ __launch_bounds__(kNoTPB) void k_no_rank(NoBatch b)
{
    __shared__ NoKeys s_row[kNoRows];
    __shared__ uint32_t s_cnt[kNoRows][kCnts];
    __shared__ uint32_t s_tot[kNoQ], s_weight[kNoQ], s_cls[kNoQ];
    __shared__ double s_prio[kNoQ];
    const uint32_t tid = threadIdx.x, lane = (uint32_t)lane_id();
    const uint32_t w = readlane32(tid >> 6, 0);
    const SortInput &in = b.in;
    const uint32_t n = in.n, rows = b.rows;
    const uint32_t i0 = blockIdx.x * rows, ig = i0 >> 6;
    const uint32_t nr = n - i0 < rows ? n - i0 : rows;   // i0 < n
    if (in.wait.clear && blockIdx.x == 0 && tid == 0 && in.wait.status) *in.wait.status = 0;
    if (tid < kNoQ) {
        s_tot[tid] = 0;
        s_weight[tid] = in.weight[tid];
        s_cls[tid] = in.cls[tid];
        s_prio[tid] = in.prio[tid];
    }
    if (tid < kNoRows * kCnts) (&s_cnt[0][0])[tid] = 0;

    // the keys of request j (beyond n: above every row's)
    auto load = [&](uint32_t j, double &a, double &bd, uint32_t &q) {
        a = 0.0;
        bd = 0.0;
        q = 0;
        if (j < n) {
            a = in.arrival[j];
            if constexpr (kB) bd = in.budget[j];
            if constexpr (kE || kP) q = in.tier[j];
        }
    };
    auto keys = [&](uint32_t j, double a, double bd, uint32_t q) {
        NoKeys k;
        const bool has = j < n;
        q = q < kNoQ ? q : kNoQ - 1u;
        k.a = has ? ordered_bits(a) : ~0ull;
        k.b = kB && has ? ordered_bits(bd) : ~0ull;
        k.e = ~0ull;
        if constexpr (kE)
            if (has) k.e = ordered_bits(no_score(in, a, s_prio[q]));
        k.cls = has ? s_cls[q] : kNoKey;
        k.tier = has ? q : kNoKey;
        return k;
    };
    double a[kG], bd[kG];
    uint32_t q[kG];
#pragma unroll
    for (uint32_t u = 0; u < kG; u++) load((w + u * kNoNW) * 64u + lane, a[u], bd[u], q[u]);
    double ra = 0.0, rb = 0.0;
    uint32_t rq = 0;
    if (tid < nr) load(i0 + tid, ra, rb, rq);
    lds_sync();
    if (tid < nr) s_row[tid] = keys(i0 + tid, ra, rb, rq);
    lds_sync();

    uint32_t tot = 0;   // lane q: requests of tier q
    NoKeys k[kG];
    uint64_t T[kG];     // requests whose index is below the row's
#pragma unroll
    for (uint32_t u = 0; u < kG; u++) {
        const uint32_t g = w + u * kNoNW;
        k[u] = keys(g * 64u + lane, a[u], bd[u], q[u]);
        T[u] = g < ig ? ~0ull : g > ig ? 0ull : (1ull << (i0 & 63u)) - 1ull;
        if constexpr (kP) {
            uint32_t mine;
            match_count<4>(k[u].tier, __ballot(k[u].tier < kNoQ), mine);
            tot += mine;
        }
    }
    for (uint32_t r = 0; r < nr; r++) {
        const NoKeys x = s_row[r];
        uint32_t cf = 0, cb = 0, ce = 0, cc = 0, ct = 0;
#pragma unroll
        for (uint32_t u = 0; u < kG; u += 2) {
            uint64_t f0, f1, m0, m1;
            below2(k[u].a, k[u + 1].a, x.a, T[u], T[u + 1], f0, f1);
            cf += (uint32_t)__popcll(f0) + (uint32_t)__popcll(f1);
            if constexpr (kB) {
                below2(k[u].b, k[u + 1].b, x.b, f0, f1, m0, m1);
                cb += (uint32_t)__popcll(m0) + (uint32_t)__popcll(m1);
            }
            if constexpr (kE) {
                below2(k[u].e, k[u + 1].e, x.e, f0, f1, m0, m1);
                ce += (uint32_t)__popcll(m0) + (uint32_t)__popcll(m1);
            }
            if constexpr (kP) {
                below2(k[u].cls, k[u + 1].cls, x.cls, f0, f1, m0, m1);
                cc += (uint32_t)__popcll(m0) + (uint32_t)__popcll(m1);
                ct += (uint32_t)__popcll(__ballot(k[u].tier == x.tier) & f0) +
                      (uint32_t)__popcll(__ballot(k[u + 1].tier == x.tier) & f1);
            }
        }
        // lane c adds count c
        const uint32_t v = lane == kCntF ? cf : lane == kCntB ? cb : lane == kCntE ? ce : lane == kCntC ? cc : ct;
        if (lane < kCnts) atomicAdd(&s_cnt[r][lane], v);
        // this row's index is below the next row's
#pragma unroll
        for (uint32_t u = 0; u < kG; u++)
            if (w + u * kNoNW == (i0 + r) >> 6) T[u] |= 1ull << ((i0 + r) & 63u);
    }
    if constexpr (kP)
        if (lane < kNoQ && tot) atomicAdd(&s_tot[lane], tot);
    lds_sync();
    if (tid >= nr) return;

    // one thread per row: its places and keys
    const uint32_t i = i0 + tid;
    auto place = [&](int p, uint32_t at, double key) {
        if (b.perm[p] && at < n) b.perm[p][at] = i;
        if (b.key[p]) b.key[p][i] = key;
    };
    rq = rq < kNoQ ? rq : kNoQ - 1u;
    place(0, s_cnt[tid][kCntF], ra);
    if constexpr (kB) place(3, s_cnt[tid][kCntB], rb);
    if constexpr (kE) place(4, s_cnt[tid][kCntE], no_score(in, ra, s_prio[rq]));
    if constexpr (kP) {
        place(1, s_cnt[tid][kCntC], s_prio[rq]);
        if (b.perm[2]) {
            const uint32_t kt = s_cnt[tid][kCntT];
            auto cnt = [&](uint32_t t) { return s_tot[t]; };
            uint64_t pos, rnd;
            if (in.wrr_mode == kWrrStride) {
                pos = wrr_stride_pos(rq, kt, s_weight, in.n_tiers, cnt);
                rnd = kt / (s_weight[rq] ? s_weight[rq] : 1u);
            } else {
                pos = wrr_blocked_pos(rq, kt, s_weight, in.n_tiers, cnt, rnd);
            }
            place(2, pos < n ? (uint32_t)pos : n, (double)rnd);
        }
    }
}

static_assert(kNoMaxN <= 6 * kNoTPB, "a wave holds all its groups");

template <uint32_t kG>
void no_start(uint32_t want, dim3 grid, dim3 block, hipStream_t s, const NoBatch &b)
{
    switch (want) {
    case 0: hipLaunchKernelGGL((k_no_rank<kG, false, false, false>), grid, block, 0, s, b); break;
    case 1: hipLaunchKernelGGL((k_no_rank<kG, true, false, false>), grid, block, 0, s, b); break;
    case 2: hipLaunchKernelGGL((k_no_rank<kG, false, true, false>), grid, block, 0, s, b); break;
    case 3: hipLaunchKernelGGL((k_no_rank<kG, true, true, false>), grid, block, 0, s, b); break;
    case 4: hipLaunchKernelGGL((k_no_rank<kG, false, false, true>), grid, block, 0, s, b); break;
    case 5: hipLaunchKernelGGL((k_no_rank<kG, true, false, true>), grid, block, 0, s, b); break;
    case 6: hipLaunchKernelGGL((k_no_rank<kG, false, true, true>), grid, block, 0, s, b); break;
    default: hipLaunchKernelGGL((k_no_rank<kG, true, true, true>), grid, block, 0, s, b); break;
    }
}

}  // namespace

hipError_t norder_launch(const SortInput &in, uint32_t *const perm[5], double *const key[5], hipStream_t s)
{
    if (in.n == 0) return hipSuccess;
    if (in.n > kNoMaxN) return hipErrorInvalidValue;
    NoBatch b;
    b.in = in;
    for (int p = 0; p < 5; p++) {
        b.perm[p] = perm[p];
        b.key[p] = perm[p] ? key[p] : nullptr;
    }
    b.rows = (uint32_t)cdiv(in.n, kNoBlocks);
    const dim3 grid((uint32_t)cdiv(in.n, b.rows)), block(kNoTPB);
    const uint32_t want = (perm[3] ? 1u : 0u) | (perm[4] ? 2u : 0u) | (perm[1] || perm[2] ? 4u : 0u);
    if (in.n <= 2 * kNoTPB) no_start<2>(want, grid, block, s, b);
    else if (in.n <= 4 * kNoTPB) no_start<4>(want, grid, block, s, b);
    else no_start<6>(want, grid, block, s, b);
    return hipGetLastError();
}

}  // namespace ds
