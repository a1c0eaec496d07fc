// The large-table calibration kernels on the CPU (cpu/hip/hip_runtime.h): every
// index into shared memory checked, and the results against the event-by-event
// recurrence whichever wave goes on first behind a barrier.
#include "../../paper_2606_02982_amd/csrc/calchunk.hip"

#include <random>

namespace {

int failures = 0;

bool close(double a, double b) { return a == b || fabs(a - b) <= 1e-12 * fabs(b) || (std::isnan(a) && std::isnan(b)); }

// n events over G groups; share: part of them in the groups 0, 16, 32, .. below
// 16 * spread, which one wave owns.
void calibrate(const char *name, uint32_t n, uint32_t G, double share, uint32_t spread, bool before)
{
    std::mt19937_64 rng(n + G);
    auto u = [&] { return (double)(rng() >> 11) * 0x1p-53; };
    std::vector<uint32_t> group(n), obs(n);
    std::vector<double> est(n), state(G), trace(n), tb(n), want(G), wt(n), wb(n);
    const double alpha = 0.1;
    for (uint32_t g = 0; g < G; g++) state[g] = want[g] = 0.5 + u();
    for (uint32_t e = 0; e < n; e++) {
        group[e] = u() < share ? 16u * (uint32_t)(u() * spread) : (uint32_t)(u() * G);
        est[e] = u() < 0.05 ? 0.0 : 1.0 + 500.0 * u();
        obs[e] = (uint32_t)(u() * 1000.0);
        double &c = want[group[e]];
        wb[e] = c;
        if (est[e] > 0.0) {
            const double t1 = (1.0 - alpha) * c;
            c = t1 + alpha * ((double)obs[e] / est[e]);
        }
        wt[e] = c;
    }
    std::vector<char> ws(ds::calc_ws_bytes(n, G) + 256);
    void *w = (void *)(((uintptr_t)ws.data() + 255) & ~(uintptr_t)255);
    if (ds::calc_launch(group.data(), est.data(), obs.data(), n, alpha, G, state.data(), trace.data(),
                        before ? tb.data() : nullptr, w, ds::calc_ws_bytes(n, G), nullptr, {}) != hipSuccess)
        failures++;
    uint32_t bad = 0;
    for (uint32_t g = 0; g < G; g++) bad += !close(state[g], want[g]);
    for (uint32_t e = 0; e < n; e++) bad += !close(trace[e], wt[e]) + (before && !close(tb[e], wb[e]));
    printf("%s: n %u G %u, last wave %s: %u wrong\n", name, n, G, emu::last_wave_first ? "first" : "last", bad);
    fflush(stdout);
    failures += bad != 0;
}

// One chunk of several steps: its maps, and each event's (to just before it).
void chunk(uint32_t n, uint32_t G, uint32_t spread)
{
    std::mt19937_64 rng(n);
    auto u = [&] { return (double)(rng() >> 11) * 0x1p-53; };
    std::vector<uint32_t> group(n), obs(n), K(G), xk(n), wk(n), wantK(G);
    std::vector<double> est(n), B(G), xb(n), pw(1024), wx(n), wantB(G);
    for (uint32_t e = 0; e < n; e++) {
        group[e] = 16u * (uint32_t)(u() * spread);
        est[e] = 1.0 + 500.0 * u();
        obs[e] = (uint32_t)(u() * 1000.0);
    }
    ds::CalArgs a;
    memset(&a, 0, sizeof a);
    a.group = group.data();
    a.est = est.data();
    a.obs = obs.data();
    a.E = a.L = n;
    a.G = G;
    a.C = a.R = 1;
    a.alpha = 0.1;
    a.oma = 1.0 - a.alpha;
    a.aggK = K.data();
    a.aggB = B.data();
    a.xb = xb.data();
    a.xk = xk.data();
    a.pw = pw.data();
    hipLaunchKernelGGL((ds::k_calc_own<ds::kG, true>), dim3(1), dim3(ds::kOT), 0, nullptr, a);
    uint32_t bad = 0;
    for (uint32_t e = 0; e < n; e++) {
        const uint32_t g = group[e];
        bad += xk[e] != wantK[g] || !close(xb[e], wantB[g]);
        wantB[g] = a.oma * wantB[g] + a.alpha * ((double)obs[e] / est[e]);
        wantK[g]++;
    }
    for (uint32_t g = 0; g < G; g++) bad += K[g] != wantK[g] || !close(B[g], wantB[g]);
    printf("chunk: n %u, %u groups of one owner, last wave %s: %u wrong\n", n, spread,
           emu::last_wave_first ? "first" : "last", bad);
    fflush(stdout);
    failures += bad != 0;
}

// The carries of C chunks alone, from given maps of every chunk.
void scan(uint32_t C, uint32_t G)
{
    std::vector<uint32_t> K((size_t)C * G);
    std::vector<double> B((size_t)C * G), carry((size_t)C * G), state(G), pw(1024), want(G);
    ds::CalArgs a;
    memset(&a, 0, sizeof a);
    a.C = C;
    a.G = G;
    a.oma = 0.9;
    a.aggK = K.data();
    a.aggB = B.data();
    a.carry = carry.data();
    a.state = state.data();
    a.pw = pw.data();
    for (uint32_t t = 0; t < 1024; t++) pw[t] = pow(a.oma, (double)(t & 255u) * (double)(1u << (8 * (t >> 8))));
    for (uint32_t i = 0; i < C * G; i++) {
        K[i] = (i * 7u) % 5u;
        B[i] = K[i] ? 0.1 * (double)(i % 13u + 1u) : 0.0;
    }
    uint32_t bad = 0;
    for (uint32_t g = 0; g < G; g++) state[g] = want[g] = 1.0 + g;
    std::vector<double> wc((size_t)C * G);
    for (uint32_t c = 0; c < C; c++)
        for (uint32_t g = 0; g < G; g++) {
            wc[(size_t)c * G + g] = want[g];
            if (K[(size_t)c * G + g]) want[g] = pow(a.oma, K[(size_t)c * G + g]) * want[g] + B[(size_t)c * G + g];
        }
    hipLaunchKernelGGL(ds::k_calc_scan, dim3((G + 63) / 64), dim3(64 * ds::kScanW), 0, nullptr, a);
    for (uint32_t i = 0; i < C * G; i++) bad += !close(carry[i], wc[i]);
    for (uint32_t g = 0; g < G; g++) bad += !close(state[g], want[g]);
    printf("scan: C %u G %u, last wave %s: %u wrong\n", C, G, emu::last_wave_first ? "first" : "last", bad);
    fflush(stdout);
    failures += bad != 0;
}

}  // namespace

int main()
{
    for (int order = 0; order < 2; order++) {
        emu::last_wave_first = order != 0;
        scan(3, 70);
        scan(200, 64);   // a wave's stretch in registers
        scan(400, 64);   // and read twice
        chunk(3 * 4096 + 77, 4096, 40);
        chunk(2 * 4096, 4096, 250);
        calibrate("uniform", 9001, 4096, 0.0, 1, true);
        calibrate("one owner, 40 groups", 9001, 4096, 0.9, 40, order == 0);
        calibrate("one group", 9001, 4096, 1.0, 1, true);
        calibrate("one owner, ranges", 8193, 8200, 0.9, 300, order != 0);
    }
    printf(failures ? "FAILED\n" : "ok\n");
    return failures != 0;
}
