// Stage 4: dispatch orders (Sec. "Scheduling Engine").
//
// Every policy ends ties in FIFO order, so each one is a stable reordering
// of the FIFO sequence:
//   FIFO      order of (arrival, index)
//   Priority  stable partition of the FIFO sequence by priority class
//   Weighted  stable partition by tier, then each request goes straight to
//             its cyclic round-robin position (closed form of the round, or
//             of the smooth interleaving's period table)
//   SJF       stable sort of the FIFO sequence by budget
//   Aging     stable sort of the FIFO sequence by the aged score
// Up to kNoMaxN requests every place is counted in one launch. Up to kSsMaxN
// requests FIFO, SJF and Aging are sample sorts by the
// composite key (policy key, arrival, index), all in the same three
// launches, and the FIFO sort's last launch also places Priority and
// Weighted. Above that, the FIFO permutation is sorted first (unless the
// caller passes it in) and the other policies follow from the FIFO sequence
// in one set of launches: up to kLsMaxN SJF by a sample sort, Priority and
// Weighted by stable partitions, above by LSD radix sorts; Aging as the merge
// of the priority classes' runs.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace ds {
namespace {

__global__ void k_copy_fifo(const uint32_t *__restrict__ fifo, const double *__restrict__ arrival,
                            uint32_t n, uint32_t *__restrict__ perm, double *__restrict__ key,
                            uint32_t *__restrict__ wait_status)
{
    if (wait_status && blockIdx.x == 0 && threadIdx.x == 0) *wait_status = 0;
    for (uint32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < n; j += gridDim.x * blockDim.x) {
        perm[j] = fifo[j];
        if (key) key[j] = arrival[j];
    }
}

__global__ void k_order_validate(OrderArgs a, uint32_t *__restrict__ flag)
{
    uint32_t bad = 0;
    const bool need_budget = (a.mask >> 3) & 1u;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < a.n; i += gridDim.x * blockDim.x) {
        if (a.tier[i] >= a.n_tiers) bad = 1;
        if (isnan(a.arrival[i])) bad = 1;
        if (need_budget && isnan(a.budget[i])) bad = 1;
        if (a.fifo_in) {
            // strictly increasing in (arrival, index) and in range: a permutation
            uint32_t f = a.fifo_in[i];
            if (f >= a.n) {
                bad = 1;
            } else if (i + 1 < a.n) {
                uint32_t h = a.fifo_in[i + 1];
                if (h >= a.n) {
                    bad = 1;
                } else {
                    double x = a.arrival[f], y = a.arrival[h];
                    if (!(x < y || (x == y && f < h))) bad = 1;
                }
            }
        }
    }
    if (bad) atomicOr(flag, 1u);
}

}  // namespace

// Bytes of the batch over the FIFO sequence, behind the FIFO permutation: the
// FIFO-ordered copies of arrival, budget and tier, the Aging runs and the
// sorts (0 outside (kSsMaxN, kLsMaxN]).
static size_t batch_bytes(uint64_t n)
{
    const size_t lb = lsort_ws_bytes(n, 1, 2);
    return lb ? 2 * align_up(n * 8, 256) + align_up(n, 256) + align_up(n * 8, 256) + align_up(n * 4, 256) +
                    align_up(17 * 4, 256) + am_steps_bytes(n) + lsort_sample_bytes(n) + lb
              : 0;
}

// Above kSsMaxN requests: the FIFO permutation and the largest of `batch`,
// `runs` and the radix sorts, which share their workspace with the FIFO sort
// that runs before them on the stream; not less than the largest sample sorts.
static size_t large_bytes(uint64_t n, uint32_t npolicies, size_t batch, size_t runs)
{
    const uint32_t np = npolicies < 1 ? 1 : npolicies, nss = np + 1 > kSsMaxSorts ? kSsMaxSorts : np + 1;
    const size_t rs = sort_ws_bytes(n, np > kMaxSorts ? kMaxSorts : np);
    return std::max(ssort_ws_bytes(kSsMaxN, nss), align_up(n * 4, 256) + std::max(std::max(batch, rs), runs));
}

// The size does not fall with n.
size_t order_ws_bytes(uint64_t n, uint32_t npolicies)
{
    if (n <= kSsMaxN) return ssort_ws_bytes(n, npolicies + 1 > kSsMaxSorts ? kSsMaxSorts : npolicies + 1);
    // (the Aging runs take the radix sorts' place after them)
    const size_t bytes = large_bytes(n, npolicies, batch_bytes(n), n <= kAmMaxN ? am_ws_bytes(n) : 0);
    return n > kLsMaxN ? std::max(bytes, order_ws_bytes(kLsMaxN, npolicies)) : bytes;
}

size_t order_need_bytes(uint64_t n, uint32_t npolicies)
{
    return n <= kLsNeedN ? order_ws_bytes(n, npolicies) : large_bytes(n, npolicies, 0, 0);
}

hipError_t order_launch(const OrderArgs &a, void *ws, size_t ws_bytes, uint32_t *flag, hipStream_t s, WaitCfg wait)
{
    const uint32_t n = a.n;
    if (flag) {
        uint64_t nb = cdiv(n, 256);
        uint32_t vb = (uint32_t)(nb < 1024 ? nb : 1024);
        if (vb) hipLaunchKernelGGL(k_order_validate, dim3(vb), dim3(256), 0, s, a, flag);
        return hipGetLastError();
    }
    if (n == 0 || a.mask == 0) return hipSuccess;

    SortInput in = {};
    in.n = n;
    in.arrival = a.arrival;
    in.budget = a.budget;
    in.tier = a.tier;
    in.n_tiers = a.n_tiers;
    for (int q = 0; q < 16; q++) {
        in.prio[q] = a.prio[q];
        in.weight[q] = a.weight[q];
    }
    in.wrr_mode = a.wrr_mode;
    in.aging_rate = a.aging_rate;
    in.t_now = a.t_now;
    in.aging_floor = a.aging_floor;
    in.wait = wait;
    uint32_t n_classes = 1;
    if (a.mask & ((1u << 1) | (1u << 4))) {
        // priority classes: rank of each tier's priority among the distinct values
        double vals[16];
        for (uint32_t q = 0; q < a.n_tiers; q++) vals[q] = a.prio[q];
        std::sort(vals, vals + a.n_tiers);
        uint32_t nd = (uint32_t)(std::unique(vals, vals + a.n_tiers) - vals);
        n_classes = nd;
        for (uint32_t q = 0; q < 16; q++) {
            uint32_t c = 0;
            if (q < a.n_tiers)
                while (c + 1 < nd && vals[c] < a.prio[q]) c++;
            in.cls[q] = c;
        }
    }
    const bool want_fifo = a.mask & 1u;
    if (want_fifo && a.fifo_in) {
        uint64_t nb = cdiv(n, 256);
        uint32_t blocks = (uint32_t)(nb < 4096 ? nb : 4096);
        hipLaunchKernelGGL(k_copy_fifo, dim3(blocks), dim3(256), 0, s, a.fifo_in, a.arrival, n, a.perm[0],
                           a.key[0], wait.clear ? wait.status : nullptr);
        in.wait.clear = false;
    }
    // Counting up to 6,144 requests, one limit for every set of policies: the
    // five orders of 6,144 take 32 us against 37, of 8,192 about 50 against 40
    // (fewer policies cost less, and their line lies higher: FIFO alone takes
    // 12 us against 24 at 6,144); not with the smooth mode, whose period table the sample
    // sorts' launches build. A given fifo_in is the order that is counted.
    // (DS_SERIAL_SORT and DS_NO_WAIT exercise the sorts.)
    if (n <= kNoMaxN && !a.serial_sort && !wait.no_wait &&
        !((a.mask & (1u << 2)) && a.wrr_mode == kWrrSmooth)) {
        uint32_t *perm[5];
        for (int p = 0; p < 5; p++) perm[p] = a.perm[p];
        if (a.fifo_in) perm[0] = nullptr;   // copied above
        if ((a.mask & ~1u) == 0 && !perm[0]) return hipGetLastError();
        return norder_launch(in, perm, a.key, s);
    }
    if (n <= kSsMaxN) {
        // one batch of sample sorts: FIFO (carrying Priority and Weighted),
        // SJF, Aging; a given fifo_in only saves the FIFO sort when neither
        // partition is wanted
        const bool parts = a.mask & 6u;
        SsPartitions pw = {{nullptr, nullptr}, {nullptr, nullptr}};
        for (int e = 0; e < 2; e++)
            if (a.mask & (2u << e)) {
                pw.perm[e] = a.perm[1 + e];
                pw.key[e] = a.key[1 + e];
            }
        SortJob all[kSsMaxSorts];
        uint32_t na = 0;
        const bool fifo_out = want_fifo && !a.fifo_in;
        if (fifo_out || parts)
            all[na++] = {SortKind::Fifo, 64, fifo_out ? a.key[0] : nullptr, fifo_out ? a.perm[0] : nullptr};
        if (a.mask & (1u << 3)) all[na++] = {SortKind::Budget, 64, a.key[3], a.perm[3]};
        if (a.mask & (1u << 4)) all[na++] = {SortKind::Aging, 64, a.key[4], a.perm[4]};
        if (na == 0) return hipGetLastError();
        return ssort_launch(in, all, na, a.serial_sort, ws, s, parts ? &pw : nullptr);
    }

    uint8_t *p = static_cast<uint8_t *>(ws);
    uint32_t *fifo_ws = reinterpret_cast<uint32_t *>(p);
    void *sort_ws = p + align_up((uint64_t)n * 4, 256);
    const size_t sort_bytes = ws_bytes - align_up((uint64_t)n * 4, 256);
    // Aging alone over a given FIFO order (a dispatch tick's re-sort): its runs
    // and places straight from it. Measured against the batch below with the
    // class partition alone: 400,000 requests 31 and 41 us, 1,048,576 55 and 67.
    const bool runs_fit = n <= kAmMaxN && am_ws_bytes(n) <= sort_bytes;
    if (a.fifo_in && (a.mask & 0x1Eu) == (1u << 4) && runs_fit) {
        in.fifo = a.fifo_in;
        return am_launch(in, n_classes, a.perm[4], a.key[4], sort_ws, s,
                         in.wait.clear ? in.wait.status : nullptr);
    }
    // Sample sorts where the workspace holds them (above kLsNeedN requests the
    // radix sorts need less than half: SJF of 4,194,304 requests 413 us against
    // 773). (DS_NO_WAIT above kLsNeedN exercises the radix passes'
    // waits: the sample sorts wait for nothing)
    if (n <= (wait.no_wait ? kLsNeedN : kLsMaxN) && batch_bytes(n) <= sort_bytes) {
        // the FIFO sort, then every other policy over the FIFO sequence in
        // one batch of sample sorts and partitions (lsort.hip)
        uint8_t *q = static_cast<uint8_t *>(sort_ws);
        LsCopies cp;
        cp.arr = reinterpret_cast<double *>(q);
        q += align_up((uint64_t)n * 8, 256);
        cp.bud = (a.mask & (1u << 3)) ? reinterpret_cast<double *>(q) : nullptr;
        q += align_up((uint64_t)n * 8, 256);
        cp.tier = q;
        q += align_up(n, 256);
        LsRuns runs;
        runs.rk = reinterpret_cast<uint64_t *>(q);
        q += align_up((uint64_t)n * 8, 256);
        runs.rp = reinterpret_cast<uint32_t *>(q);
        q += align_up((uint64_t)n * 4, 256);
        runs.cstart = reinterpret_cast<uint32_t *>(q);
        q += align_up(17 * 4, 256);
        runs.hk = reinterpret_cast<uint64_t *>(q);
        runs.hp = am_steps_pos(runs.hk, n);
        q += am_steps_bytes(n);
        LsSample sjf = lsort_sample_at(n, q);
        q += lsort_sample_bytes(n);
        void *batch_ws = q;
        const bool more = a.mask & ~1u;   // policies over the FIFO sequence
        const uint32_t *fifo = a.fifo_in;
        bool sjf_drawn = false;
        if (!fifo) {
            // (SJF's splitters are drawn in the same launches)
            sjf_drawn = (a.mask & (1u << 3)) != 0;
            SortJob job = {SortKind::Fifo, 64, want_fifo ? a.key[0] : nullptr, want_fifo ? a.perm[0] : fifo_ws};
            hipError_t err = lsort_launch(in, &job, 1, batch_ws, s, nullptr, more ? &cp : nullptr, nullptr,
                                          sjf_drawn ? &sjf : nullptr);
            if (err != hipSuccess) return err;
            fifo = job.out;
            in.wait.clear = false;
        }
        sjf.draw = false;
        in.fifo = fifo;
        // SJF sorts; Priority partitions (and lays out the priority classes'
        // runs, from which each request's Aging place follows); Weighted partitions
        const bool prio = a.mask & (1u << 1), aging = a.mask & (1u << 4);
        SortJob jobs[3];
        uint32_t nj = 0;
        if (a.mask & (1u << 3)) jobs[nj++] = {SortKind::Budget, 64, a.key[3], a.perm[3]};
        if (prio || aging)
            jobs[nj++] = {SortKind::Class, 8, prio ? a.key[1] : nullptr, prio ? a.perm[1] : nullptr};
        if (a.mask & (1u << 2)) jobs[nj++] = {SortKind::Tier, 8, a.key[2], a.perm[2]};
        if (nj == 0) return hipGetLastError();
        hipError_t err = lsort_launch(in, jobs, nj, batch_ws, s, a.fifo_in ? nullptr : &cp, nullptr,
                                      aging ? &runs : nullptr, sjf_drawn ? &sjf : nullptr);
        if (err != hipSuccess || !aging) return err;
        return am_rank_launch(in, n_classes, runs, a.perm[4], a.key[4], batch_ws, s);   // (the batch is done with it)
    }

    // the policy sorts over the FIFO sequence; Aging as the merge of the
    // priority classes' runs of that sequence (agmerge.hip), in the sort
    // workspace, or where they do not fit, and above kAmMaxN, as one more radix
    // sort
    const bool aging_merge = (a.mask & (1u << 4)) && runs_fit;
    SortJob jobs[kMaxSorts];
    uint32_t nj = 0;
    if (a.mask & (1u << 1)) jobs[nj++] = {SortKind::Class, 8, a.key[1], a.perm[1]};
    if (a.mask & (1u << 2)) jobs[nj++] = {SortKind::Tier, 8, a.key[2], a.perm[2]};
    if (a.mask & (1u << 3)) jobs[nj++] = {SortKind::Budget, 64, a.key[3], a.perm[3]};
    if ((a.mask & (1u << 4)) && !aging_merge) jobs[nj++] = {SortKind::Aging, 64, a.key[4], a.perm[4]};

    // radix sorts: the FIFO permutation first, then the policies over it
    const uint32_t *fifo = a.fifo_in;
    if (!fifo) {
        SortJob job = {SortKind::Fifo, 64, want_fifo ? a.key[0] : nullptr, want_fifo ? a.perm[0] : fifo_ws};
        hipError_t err = sort_launch(in, &job, 1, sort_ws, s);
        if (err != hipSuccess) return err;
        fifo = job.out;
        in.wait.clear = false;
    }
    in.fifo = fifo;
    if (nj > 0) {
        hipError_t err = sort_launch(in, jobs, nj, sort_ws, s);
        if (err != hipSuccess) return err;
        in.wait.clear = false;
    }
    // (after the sorts on the stream: the runs reuse their workspace)
    if (aging_merge)
        return am_launch(in, n_classes, a.perm[4], a.key[4], sort_ws, s,
                         in.wait.clear ? in.wait.status : nullptr);
    return hipGetLastError();
}

__global__ void k_fill_u32(uint32_t *__restrict__ p, uint32_t v, uint64_t n)
{
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

hipError_t fill_u32(uint32_t *p, uint32_t v, uint64_t n, hipStream_t s)
{
    uint64_t nb = cdiv(n, 256);
    uint32_t blocks = (uint32_t)(nb < 1024 ? nb : 1024);
    if (blocks) hipLaunchKernelGGL(k_fill_u32, dim3(blocks), dim3(256), 0, s, p, v, n);
    return hipGetLastError();
}

}  // namespace ds
