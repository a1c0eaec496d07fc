// Stage 1: whitespace-proxy word counts over a packed UTF-8 prompt buffer.
//
// counts[i] = number of maximal runs of non-whitespace characters in prompt
// i, whitespace being the 29 code points str.split() separates on
// (Sec. "Workload Characterization and Token Budget Estimation").
//
// Byte formulation used here: byte p of prompt i is a word start when p is
// not whitespace and either p is the prompt's first byte or byte p-1 is
// whitespace. A byte is whitespace when it is one of the ASCII separators
// 09-0D, 1C-20, or belongs to one of the multi-byte separators
// C2 85, C2 A0, E1 9A 80, E2 80 80..8A, E2 80 A8, E2 80 A9, E2 80 AF,
// E2 81 9F, E3 80 80 lying entirely inside the prompt. Because none of these
// sequences starts with a continuation byte, this equals decoding each prompt
// on its own (undecodable bytes as ordinary characters) and splitting.
//
// Layout of the work: the text is cut into equal byte ranges, one per
// resident wave; each wave streams its range in super-rounds of 4 KiB (four
// 1 KiB rounds of 64 lanes x 16 bytes, all loads issued together) and works
// on them as two sets of 2 KiB, 32 bytes per lane. A set's bytes are
// transposed into eight bit planes (plane b holds bit b of the lane's 32
// bytes), and everything after that is a Boolean function of planes, 32 bytes
// per instruction: the ASCII separators, the pieces of the multi-byte ones,
// the word starts. Neighbouring bytes meet through byte and lane shifts of a
// plane. Per 2 KiB set (counters) ASCII text takes 107 vector instructions, a
// set with leads of multi-byte separators about 70 more, one with prompt
// boundaries about 60 more; the form before this, 8 bits per byte and 4 bytes
// per instruction, took 141 for ASCII, listed lead bytes through LDS and went
// round by round where they were dense or met a boundary.
// What bounds it: HBM (6.9 TB/s is this card's read rate) on ASCII and on
// long prompts, the vector units on text of 2- and 3-byte letters. Measured
// with the final kernel and the scores, before and after: 16,384 long prompts,
// 5% of the bytes not ASCII, 2.94 GB: 531 and 457 us (6.4 TB/s); 1,048,576
// chat prompts, 1.2 GB: 238 and 213 us; 65,536 prompts of 2- and 3-byte
// letters with multi-byte spaces, 310 MB: 286 and 80 us.
// Word starts are attributed to prompts through prefix sums: each prompt
// boundary receives the number of word starts in its wave's range before it,
// each wave its total; a second kernel forms counts[i] from the two
// boundaries' local prefixes and the totals of the waves between them. No
// atomics; results are exact integers independent of scheduling.
#include "common.h"
#include "kernels.h"
#include "scoremath.h"

namespace ds {
namespace {

constexpr uint32_t kRound = 1024;        // bytes per wave per round
constexpr uint32_t kLoadRounds = 4;      // rounds loaded together
constexpr uint32_t kSet = 2 * kRound;    // bytes turned into one set of planes
constexpr uint32_t kBlock = 256;         // 4 independent waves per block
// Each wave takes one contiguous range of the buffer. Four ranges per
// resident wave slot: waves that start late (their slot held by an earlier
// wave or by another stream's kernel) leave a short tail, not a long one.
constexpr uint32_t kRangesPerSlot = 4;
constexpr uint32_t kMaxWaves = 32768;

typedef unsigned int v4u __attribute__((ext_vector_type(4)));

// 16 bytes at c (bytes >= B read as 0). The text is streamed once: the
// full-chunk load is marked nontemporal.
__device__ __forceinline__ uint4 load16(const uint8_t *t, uint64_t B, uint64_t c)
{
    if (c + 16 <= B) {
        v4u v = __builtin_nontemporal_load(reinterpret_cast<const v4u *>(t + c));
        return make_uint4(v.x, v.y, v.z, v.w);
    }
    uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int k = 0; k < 16; k++)
        if (c + k < B) w[k >> 2] |= (uint32_t)t[c + k] << (8 * (k & 3));
    return make_uint4(w[0], w[1], w[2], w[3]);
}

__device__ __forceinline__ uint32_t load4(const uint8_t *t, uint64_t B, uint64_t c)
{
    if (c + 4 <= B) return *reinterpret_cast<const uint32_t *>(t + c);
    uint32_t w = 0;
#pragma unroll
    for (int k = 0; k < 4; k++)
        if (c + k < B) w |= (uint32_t)t[c + k] << (8 * k);
    return w;
}

// First index i in [0, count) with off[i] >= x, or count (wave-cooperative
// 64-ary search; every step is one round of loads).
__device__ uint32_t lower_bound_wave(const uint64_t *off, uint64_t count, uint64_t x, int lane)
{
    uint64_t lo = 0, hi = count;
    while (hi - lo > 64) {
        uint64_t step = (hi - lo + 63) / 64;
        uint64_t idx = lo + (uint64_t)lane * step;
        bool lt = idx < hi && off[idx] < x;
        uint32_t k = (uint32_t)__popcll(__ballot(lt));
        if (k == 0) { hi = lo; break; }
        uint64_t nlo = lo + (uint64_t)(k - 1) * step + 1;
        uint64_t nhi = lo + (uint64_t)k * step;
        lo = nlo;
        hi = nhi < hi ? nhi : hi;
    }
    bool lt = (lo + (uint64_t)lane < hi) && off[lo + lane] < x;
    return (uint32_t)(lo + (uint64_t)__popcll(__ballot(lt)));
}

// A value that is the same in every lane, known so to the compiler.
__device__ __forceinline__ uint32_t uniform(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}

// Positions inside a wave's range are 32-bit distances from its start (a
// range is a small part of the buffer; kFar stands for anything beyond).
constexpr uint32_t kFar = 0xFFFFFFFFu;

struct WaveState {
    uint32_t s_ptr;     // first boundary index not yet consumed
    uint32_t wb;        // boundary index held by lane 0 of win
    uint32_t win;       // offsets[wb + lane] - ws_start (kFar past the range or the end)
    uint32_t next;      // win of s_ptr
    uint64_t running;   // word starts in [ws_start, current set), less acc
    uint32_t acc;       // per-lane starts not yet in running
    uint32_t ws_prev;   // whitespace bit of the byte before the set
    uint32_t spill;     // separator bits spilling into the set's first two bytes
};

struct RangeCtx {
    const uint64_t *off;
    uint32_t N;
    uint64_t ws_start;
    uint32_t len;       // bytes of the range
    uint32_t *ploc;
};

__device__ __forceinline__ void load_window(WaveState &st, const RangeCtx &rc, uint32_t s, int lane)
{
    const uint64_t i = (uint64_t)s + (uint64_t)lane;
    st.wb = uniform(s);
    st.win = kFar;
    if (i <= (uint64_t)rc.N) {
        const uint64_t d = rc.off[i] - rc.ws_start;   // wraps far beyond if before the range
        if (d < rc.len) st.win = (uint32_t)d;
    }
}

__device__ __forceinline__ void ensure_window(WaveState &st, const RangeCtx &rc, uint32_t s, int lane)
{
    if (s < st.wb || s - st.wb >= 64) load_window(st, rc, s, lane);
}

// Does a prompt start at byte x? (rare: only beside a separator that crosses
// a set's end)
__device__ __noinline__ bool boundary_at(const uint64_t *off, uint32_t N, uint64_t x, int lane)
{
    const uint32_t i = lower_bound_wave(off, (uint64_t)N + 1, x, lane);
    return i <= N && off[i] == x;
}

// Length (2 or 3) of the multi-byte separator starting at the low byte of v
// (bytes little-endian), or 0; branch-free.
__device__ __forceinline__ uint32_t mb_space_len_nb(uint32_t v)
{
    const uint32_t v2 = v & 0xFFFFu, v3 = v & 0xFFFFFFu, b2 = (v >> 16) & 0xFFu;
    const bool two = (v2 == 0x85C2u) | (v2 == 0xA0C2u);
    const bool e2 = (v2 == 0x80E2u) & ((b2 - 0x80u <= 0x0Au) | (b2 == 0xA8u) | (b2 == 0xA9u) | (b2 == 0xAFu));
    const bool three = (v3 == 0x809AE1u) | (v3 == 0x9F81E2u) | (v3 == 0x8080E3u) | e2;
    return two ? 2u : (three ? 3u : 0u);
}

// Coverage by the separator of len bytes (0: none) that starts at byte p - k
// (k = 1..3; p counts from the range's start), unless a prompt boundary cuts
// it: bits 0, 1 = bytes p - 2, p - 1, bits 2, 3 = bytes p, p + 1.
__device__ __forceinline__ uint32_t coverage(const RangeCtx &rc, uint32_t p, uint32_t k, uint32_t len, int lane)
{
    for (uint32_t i = 1; i < len; i++)
        if (boundary_at(rc.off, rc.N, rc.ws_start + p - k + i, lane)) return 0;
    return (((1u << len) - 1u) << (3u - k)) >> 1;
}

// The bytes from p - k on, k = 1..3, of the dwords before and at p.
__device__ __forceinline__ uint32_t bytes_from(uint32_t before, uint32_t at, uint32_t k)
{
    return (uint32_t)((((uint64_t)at << 32) | before) >> (32u - 8u * k));
}

// Coverage of the two bytes before p and the two from p on by a separator that
// starts before p and ends at or behind it (dwords before and at p: the same
// values in every lane).
__device__ __forceinline__ uint32_t crossing(const RangeCtx &rc, uint32_t before, uint32_t at, uint32_t p, int lane)
{
    const uint32_t l1 = mb_space_len_nb(bytes_from(before, at, 1));
    const uint32_t l2 = mb_space_len_nb(bytes_from(before, at, 2));
    if (!(l1 || l2 == 3)) return 0;
    return coverage(rc, p, l1 ? 1u : 2u, l1 ? l1 : l2, lane);
}

// (x & m) | (y & ~m) as one instruction (from the expression the compiler
// makes several where it sees parts shared)
__device__ __forceinline__ uint32_t bfi(uint32_t m, uint32_t x, uint32_t y)
{
    uint32_t r;
    asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(r) : "s"(m), "v"(x), "v"(y));
    return r;
}

// The eight bit planes of a lane's 32 bytes: a is its chunk of the set's first
// round, b of the second. Bit 8c + i of plane j is bit j of byte c of dword i
// (i < 4 in a, else b): an 8 x 8 bit transposition in each byte column, three
// stages of pairwise exchanges.
__device__ __forceinline__ void planes(const uint4 &a, const uint4 &b, uint32_t (&w)[8])
{
    w[0] = a.x; w[1] = a.y; w[2] = a.z; w[3] = a.w;
    w[4] = b.x; w[5] = b.y; w[6] = b.z; w[7] = b.w;
    constexpr uint32_t mask[3] = {0x55555555u, 0x33333333u, 0x0F0F0F0Fu};
#pragma unroll
    for (int e = 2; e >= 0; e--) {
        const int sft = 1 << e;
#pragma unroll
        for (int i = 0; i < 8; i++) {
            if (i & sft) continue;
            const uint32_t x = w[i], y = w[i + sft];
            w[i] = bfi(mask[e], x, y << sft);
            w[i + sft] = bfi(mask[e], x >> sft, y);
        }
    }
}

// ASCII separators 09-0D, 1C-20.
__device__ __forceinline__ uint32_t ascii_space(const uint32_t (&b)[8])
{
    const uint32_t f = (b[2] & ~b[1]) | (~b[2] & (b[1] | b[0]));            // low three bits 1..5
    const uint32_t g = (b[4] & b[2]) | (~b[4] & f);                         // 1C-1F or 09-0D, given bit 3
    const uint32_t n = ~(b[2] | b[1] | b[0]) & ~b[3] & ~b[4];               // 20, given bit 5
    const uint32_t m = (b[5] & n) | (~b[5] & (b[3] & g));
    return m & ~b[7] & ~b[6];
}

// Planes move by whole bytes of the text: inside a lane bytes of one dword are
// 8 bits apart and dwords one bit; a round's lanes follow each other. Across
// the rounds' ends only `edge` enters (0 for the pieces of separators, whose
// crossings of a round's end are looked up apart).
// prev1: each byte's predecessor; bits 27 and 31 of edge: those of lane 0's
// first byte in the two rounds.
__device__ __forceinline__ uint32_t prev1(uint32_t x, uint32_t edge)
{
    const uint32_t z = bfi(0x11111111u, wave_shr1(x, edge) >> 3, x << 1);
    return __builtin_amdgcn_alignbyte(x, z, 3);
}

__device__ __forceinline__ uint32_t prev1(uint32_t x)
{
    // (zero into lane 0)
    const uint32_t p = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x138, 0xF, 0xF, true);
    return __builtin_amdgcn_alignbyte(x, bfi(0x11111111u, p >> 3, x << 1), 3);
}

// next1: each byte's successor in its round.
__device__ __forceinline__ uint32_t next1(uint32_t x)
{
    const uint32_t n = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x130, 0xF, 0xF, true);
    return __builtin_amdgcn_alignbyte(bfi(0x88888888u, n << 3, x >> 1), x, 1);
}

// The bytes covered by multi-byte separators that lie inside one round and
// inside one prompt (bd: bytes that prompts start at; none continues a
// separator). Leads that can start one: C2, E1, E2, E3; z: 11x000xx.
__device__ __forceinline__ uint32_t wide_space(const uint32_t (&b)[8], uint32_t z, uint32_t bd)
{
    // lead codes: k3 = C2; (k1, k2) = E1: (1, 0), E2: (0, 1), E3: (1, 1)
    const uint32_t k1 = z & b[5] & b[0], k2 = z & b[5] & b[1], k3 = z & ~b[5] & b[1] & ~b[0];
    const uint32_t q1 = prev1(k1), q2 = prev1(k2), q3 = prev1(k3);
    // second bytes
    const uint32_t c = b[7] & ~b[6] & ~bd, lo5 = c & ~b[5];
    const uint32_t n0 = ~(b[2] | b[1] | b[0]), n1 = n0 & ~b[3] & ~b[4];
    const uint32_t is80 = lo5 & n1;
    const uint32_t top = lo5 & ~b[4] & ~b[3] & ~b[1] & b[0];                // 81 or 85
    const uint32_t is1a = lo5 & b[4] & b[3] & b[1];                         // 9A, 9B, 9E, 9F
    const uint32_t t2 = q3 & ((top & b[2]) | (c & b[5] & n1));              // C2 85, C2 A0
    const uint32_t pa = (q2 & is80) | (q1 & ~q2 & is1a & ~b[2] & ~b[0]);    // E2 80, E3 80, E1 9A
    const uint32_t pb = q2 & ~q1 & (is80 | (top & ~b[2]));                  // E2 80, E2 81
    if (__ballot((t2 | pa | pb) != 0) == 0) return 0;
    // third bytes: E2 80 takes 80-8A, A8, A9, AF; E1 9A and E3 80 take 80;
    // E2 81 takes 9F
    const uint32_t u5 = b[3] & ((b[2] & b[1] & b[0]) | ~(b[2] | b[1]));
    const uint32_t u4 = ~b[3] | (~b[2] & ~(b[1] & b[0]));
    const uint32_t wide = c & ~b[4] & ((b[5] & u5) | (~b[5] & u4));
    const uint32_t pa1 = prev1(pa), pb1 = prev1(pb);
    const uint32_t t3 = (pa1 & ((pb1 & wide) | (~pb1 & is80))) | (~pa1 & pb1 & is1a & b[2] & b[0]);
    const uint32_t v = t2 | t3;
    return v | next1(v | next1(t3));
}

// The prompt boundaries before `end`, from s_ptr on: body(m) runs for each
// window of 64 offsets, m the lanes that hold such boundaries. Returns the
// first index past them.
template <typename F>
__device__ __forceinline__ uint32_t for_boundaries(WaveState &st, const RangeCtx &rc, uint32_t end, int lane,
                                                   F body)
{
    uint32_t s = st.s_ptr;
    for (;;) {
        ensure_window(st, rc, s, lane);
        const uint32_t kk = s - st.wb;
        const uint64_t m = __ballot((uint32_t)lane >= kk && st.win < end);
        body(m);
        if (!((m >> 63) & 1ull)) return uniform(st.wb + kk + (uint32_t)__popcll(m));
        s = uniform(st.wb + 64);
        if (s > rc.N) return s;
    }
}

// May a separator begin in the last two bytes of this dword and end behind it?
__device__ __forceinline__ bool may_cross(uint32_t last)
{
    const uint32_t c1 = last >> 24, c2 = (last >> 16) & 0xFFu;
    return c1 == 0xC2u || c1 - 0xE1u <= 2u || c2 - 0xE1u <= 2u;
}

// One 2 KiB set, pos bytes into the range: word starts counted, boundaries
// given their prefixes. next: the dword behind the set.
__device__ __forceinline__ void process_set(WaveState &st, const RangeCtx &rc, const uint4 &d0, const uint4 &d1,
                                            uint32_t next, uint32_t pos, int lane)
{
    uint32_t b[8];
    planes(d0, d1, b);
    const bool bnd = st.next < pos + kSet;
    uint32_t bd = 0;
    if (bnd)
        for_boundaries(st, rc, pos + kSet, lane, [&](uint64_t m) {
            const uint32_t wrel = st.win - pos;
            // empty prompts start where the next one does: in a window full of
            // starts each place once (65,536 empty prompts in a row: 4.6 ms
            // offset by offset, 0.67 so)
            if (m == ~0ull) m = __ballot(wave_shr1(st.win, kFar) != st.win);
            for (; m; m &= m - 1) {
                const uint32_t rel = readlane32(wrel, __builtin_ctzll(m));
                const uint32_t bit = 1u << (8u * (rel & 3u) + 4u * ((rel >> 10) & 1u) + ((rel >> 2) & 3u));
                bd |= (uint32_t)lane == ((rel >> 4) & 63u) ? bit : 0u;
            }
        });
    uint32_t ws = ascii_space(b);
    const uint32_t z = b[7] & b[6] & ~b[4] & ~b[3] & ~b[2];
    if (__ballot(z != 0)) ws |= wide_space(b, z, bd);
    // separators across the rounds' ends
    const uint32_t last0 = readlane32(d0.w, 63), last1 = readlane32(d1.w, 63);
    uint32_t cross0 = 0, cross1 = 0;
    if (may_cross(last0) || may_cross(last1)) {
        // lanes 0..3: the first and the second round's end, from its last
        // byte and from the one before
        const bool second = lane & 1, two = lane & 2;
        const uint32_t before = second ? last1 : last0, at = second ? next : readlane32(d1.x, 0);
        const uint32_t len = mb_space_len_nb(two ? __builtin_amdgcn_alignbyte(at, before, 2)
                                                 : __builtin_amdgcn_alignbyte(at, before, 3));
        uint64_t hits = __ballot(lane < 4 && (two ? len == 3 : len != 0));
        for (; hits; hits &= hits - 1) {
            const int l = __builtin_ctzll(hits);
            const uint32_t c = coverage(rc, pos + (1u + (l & 1)) * kRound, 1u + (uint32_t)(l >> 1), readlane32(len, l), lane);
            if (l & 1) cross1 |= c;
            else cross0 |= c;
        }
    }
    if (st.spill | cross0 | cross1) {
        // lane 0: bytes 0, 1 of dwords 0 and 4; lane 63: bytes 2, 3 of dwords 3 and 7
        const uint32_t s0 = cross0 >> 2;
        if (lane == 0) ws |= (st.spill & 1u) | ((st.spill & 2u) << 7) | ((s0 & 1u) << 4) | ((s0 & 2u) << 11);
        if (lane == 63)
            ws |= ((cross0 & 1u) << 19) | ((cross0 & 2u) << 26) | ((cross1 & 1u) << 23) | ((cross1 & 2u) << 30);
    }
    st.spill = cross1 >> 2;
    const uint32_t top = readlane32(ws, 63);
    const uint32_t before = prev1(ws, (st.ws_prev << 27) | ((top << 4) & 0x80000000u));
    st.ws_prev = top >> 31;
    uint32_t start = ~ws & (before | bd);
    if (pos + kSet > rc.len) {   // the text's end: bytes past it do not count
        for (uint32_t i = 0; i < 8; i++)
            for (uint32_t c = 0; c < 4; c++)
                if (pos + (i >> 2) * kRound + 16u * (uint32_t)lane + 4u * (i & 3u) + c >= rc.len)
                    start &= ~(1u << (8u * c + i));
    }
    if (!bnd) {
        st.acc += (uint32_t)__popc(start);
        return;
    }
    // starts of the two rounds before each lane, as packed 16-bit sums
    st.running += readlane32(wave_incl_scan_dpp(st.acc), 63);
    st.acc = 0;
    const uint32_t cnt = (uint32_t)__popc(start & 0x0F0F0F0Fu) | ((uint32_t)__popc(start & 0xF0F0F0F0u) << 16);
    const uint32_t incl = wave_incl_scan_dpp(cnt), excl = incl - cnt, tot = readlane32(incl, 63);
    st.s_ptr = for_boundaries(st, rc, pos + kSet, lane, [&](uint64_t m) {
        const uint32_t rel = st.win - pos;
        const int src = (int)((rel >> 4) & 63u);
        const uint32_t ex = (uint32_t)__shfl((int)excl, src, 64), sw = (uint32_t)__shfl((int)start, src, 64);
        const uint32_t r4 = 4u * ((rel >> 10) & 1u), i = r4 + ((rel >> 2) & 3u);
        // the round's dwords before i, and dword i's bytes before the boundary
        const uint32_t rows = ((1u << i) - (1u << r4)) * 0x01010101u;
        const uint32_t cols = (0x01010101u & ((1u << (8u * (rel & 3u))) - 1u)) << i;
        const uint32_t val = (uint32_t)st.running + (r4 ? (tot & 0xFFFFu) + (ex >> 16) : ex & 0xFFFFu) +
                             (uint32_t)__popc(sw & (rows | cols));
        if ((m >> lane) & 1ull) rc.ploc[st.wb + (uint32_t)lane] = val;
    });
    st.running += (tot & 0xFFFFu) + (tot >> 16);
    ensure_window(st, rc, st.s_ptr, lane);
    st.next = readlane32(st.win, (int)(st.s_ptr - st.wb));
}

// 8 waves per SIMD (64 registers): 7 cost 1% more, 6 4%; a second super-round
// in flight per wave (5 or 4 waves) 20%.
__global__ __launch_bounds__(kBlock, 8) void k_char_main(const uint8_t *__restrict__ text, uint64_t B,
                                                      const uint64_t *__restrict__ off, uint32_t N,
                                                      uint64_t Rw, uint32_t nwaves,
                                                      uint32_t *__restrict__ ploc,
                                                      uint64_t *__restrict__ wavetot)
{
    const int lane = lane_id();
    // the wave index, known to the compiler to be uniform across the wave
    const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)));
    if (w >= nwaves) return;
    RangeCtx rc;
    rc.off = off;
    rc.N = N;
    rc.ws_start = (uint64_t)w * Rw;
    rc.ploc = ploc;
    if (rc.ws_start >= B) {
        if (lane == 0) wavetot[w] = 0;
        return;
    }
    const uint64_t left = B - rc.ws_start;
    rc.len = (uint32_t)(left < Rw ? left : Rw);
    // super-rounds that end at or before `whole` bytes into the range have
    // every chunk and the dword behind them inside the buffer
    const uint32_t whole = left < 4 ? 0u : (uint32_t)(left - 4 < Rw ? left - 4 : Rw);
    WaveState st;
    st.s_ptr = uniform(lower_bound_wave(off, (uint64_t)N + 1, rc.ws_start, lane));
    load_window(st, rc, st.s_ptr, lane);
    st.next = readlane32(st.win, 0);
    st.running = 0;
    st.acc = 0;
    st.ws_prev = 1;
    st.spill = 0;
    if (rc.ws_start > 0) {   // then ws_start >= Rw >= 4 KiB
        // whether the byte before the range is whitespace, and what a
        // separator begun there covers of the range
        const uint32_t before = uniform(load4(text, B, rc.ws_start - 4)), at = uniform(load4(text, B, rc.ws_start));
        const uint32_t c = crossing(rc, before, at, 0u, lane), p = before >> 24;
        st.spill = c >> 2;
        st.ws_prev = (c >> 1) & 1u;
        if (p - 0x09u <= 4u || p - 0x1Cu <= 4u) st.ws_prev = 1;
        // or one that ends there
        if (mb_space_len_nb(bytes_from(before, at, 2)) == 2) st.ws_prev |= coverage(rc, 0u, 2, 2, lane) >> 1;
        if (mb_space_len_nb(bytes_from(before, at, 3)) == 3) st.ws_prev |= coverage(rc, 0u, 3, 3, lane) >> 1;
    }
    constexpr uint32_t sr_bytes = kRound * kLoadRounds;
    for (uint32_t pos = 0; pos < rc.len; pos += sr_bytes) {
        const uint8_t *src = text + rc.ws_start + pos;
        uint4 d[kLoadRounds];
        uint32_t tail = 0;
        if (pos + sr_bytes <= whole) {
#pragma unroll
            for (uint32_t u = 0; u < kLoadRounds; u++) {
                v4u v = __builtin_nontemporal_load(reinterpret_cast<const v4u *>(src + u * kRound + 16u * (uint32_t)lane));
                d[u] = make_uint4(v.x, v.y, v.z, v.w);
            }
            tail = *reinterpret_cast<const uint32_t *>(src + sr_bytes);
        } else {
            const uint64_t sb = rc.ws_start + pos;
#pragma unroll
            for (uint32_t u = 0; u < kLoadRounds; u++) {
                uint64_t c = sb + (uint64_t)u * kRound + 16u * (uint32_t)lane;
                d[u] = c < B ? load16(text, B, c) : make_uint4(0u, 0u, 0u, 0u);
            }
            tail = uniform(load4(text, B, sb + sr_bytes));
        }
#pragma unroll
        for (uint32_t u = 0; u < kLoadRounds; u += 2) {
            if (pos + u * kRound >= rc.len) break;
            const uint32_t next = u + 2 < kLoadRounds ? readlane32(d[u + 2 < kLoadRounds ? u + 2 : u].x, 0) : tail;
            process_set(st, rc, d[u], d[u + 1], next, pos + u * kRound, lane);
        }
    }
    uint64_t total = st.running + readlane32(wave_incl_scan_dpp(st.acc), 63);
    if (lane == 0) wavetot[w] = total;
}

// counts[i] from the per-boundary local prefixes and the per-wave totals:
// the word starts of [a, b) are the starts after a in a's wave, those of the
// whole waves in between, and the starts before b in b's wave.
// Per prompt: the word count from the waves' totals and the boundary
// positions; with sc.n != 0 the request is also scored (stage 3) from that
// count.
__global__ __launch_bounds__(256) void k_char_fin(const uint64_t *__restrict__ off, uint32_t N,
                                                  uint64_t B, uint32_t rw_kib, uint32_t nwaves,
                                                  const uint64_t *__restrict__ wavetot,
                                                  const uint32_t *__restrict__ ploc,
                                                  uint32_t *__restrict__ counts, ScoreArgs sc)
{
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N;
         i += (uint64_t)gridDim.x * blockDim.x) {
        uint64_t a = off[i], b = off[i + 1];
        if (b <= a || a >= B) {
            counts[i] = 0;
            if (sc.n) score_one(sc, (uint32_t)i, 0u);
            continue;
        }
        uint32_t wa = (uint32_t)(a >> 10) / rw_kib;
        uint32_t wb;
        uint64_t tail;
        if (b >= B) {
            wb = nwaves;
            tail = 0;
        } else {
            wb = (uint32_t)(b >> 10) / rw_kib;
            tail = ploc[i + 1];
        }
        uint64_t sum = tail;
        for (uint32_t w = wa; w < wb && w < nwaves; w++) sum += wavetot[w];
        const uint32_t cnt = (uint32_t)(sum - ploc[i]);
        counts[i] = cnt;
        if (sc.n) score_one(sc, (uint32_t)i, cnt);
    }
}

// DS_VALIDATE: offsets nondecreasing and offsets[N] <= B.
__global__ void k_char_validate(const uint64_t *__restrict__ off, uint32_t N, uint64_t B,
                                uint32_t *__restrict__ flag)
{
    uint32_t bad = 0;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N;
         i += (uint64_t)gridDim.x * blockDim.x)
        if (off[i] > off[i + 1]) bad = 1;
    if (blockIdx.x == 0 && threadIdx.x == 0 && off[N] > B) bad = 1;
    if (bad) atomicOr(flag, 1u);
}

// The read side of k_char_main alone: the same wave ranges and 16-byte
// nontemporal loads, four rounds in flight per wave, and no classification;
// each wave's XOR of its words goes to sink[w], so that no load is dropped.
// B is a multiple of 16.
__global__ __launch_bounds__(kBlock) void k_read_stream(const uint8_t *__restrict__ p, uint64_t B, uint64_t Rw,
                                                      uint32_t nwaves, uint32_t *__restrict__ sink)
{
    const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)));
    if (w >= nwaves) return;
    const int lane = lane_id();
    const uint64_t b = (uint64_t)w * Rw, e = b + Rw < B ? b + Rw : B;
    uint32_t acc = 0;
    for (uint64_t sb = b; sb < e; sb += (uint64_t)kRound * kLoadRounds) {
        v4u d[kLoadRounds];
#pragma unroll
        for (uint32_t u = 0; u < kLoadRounds; u++) {
            const uint64_t c = sb + (uint64_t)u * kRound + 16u * (uint32_t)lane;   // c < e: c + 16 <= e
            d[u] = c < e ? __builtin_nontemporal_load(reinterpret_cast<const v4u *>(p + c)) : v4u{0u, 0u, 0u, 0u};
        }
#pragma unroll
        for (uint32_t u = 0; u < kLoadRounds; u++) acc ^= d[u].x ^ d[u].y ^ d[u].z ^ d[u].w;
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) acc ^= (uint32_t)__shfl_xor((int)acc, m, 64);
    if (lane == 0) sink[w] = acc;
}

// Wave ranges of k_char_main for B bytes: one per resident wave slot (CUs x
// resident waves of k_char_main per CU) times kRangesPerSlot, whole 4 KiB
// super-rounds.
hipError_t char_waves(uint64_t B, uint64_t &Rw, uint32_t &nwaves)
{
    static int resident_cache[64];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    int resident = dev >= 0 && dev < 64 ? resident_cache[dev] : 0;
    if (resident == 0) {
        int n_cu = 0, per_cu = 0;
        e = hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return e;
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_char_main, kBlock, 0);
        if (e != hipSuccess) return e;
        resident = (n_cu > 0 ? n_cu : 1) * (per_cu > 0 ? per_cu : 1) * (int)(kBlock / 64);
        if (dev >= 0 && dev < 64) resident_cache[dev] = resident;
    }
    uint64_t target = (uint64_t)resident * kRangesPerSlot;
    if (target > kMaxWaves) target = kMaxWaves;
    Rw = align_up(cdiv(B ? B : 1, target), (uint64_t)kRound * kLoadRounds);
    nwaves = (uint32_t)cdiv(B, Rw);
    return hipSuccess;
}

}  // namespace

size_t char_ws_bytes(uint64_t n)
{
    return align_up((n + 1) * 4, 256) + align_up((uint64_t)kMaxWaves * 8, 256);
}

hipError_t char_launch(const uint8_t *text, uint64_t B, const uint64_t *offsets, uint32_t n,
                       uint32_t *counts, void *ws, uint32_t *flag, hipStream_t s, const ScoreArgs *score)
{
    uint8_t *p = static_cast<uint8_t *>(ws);
    uint32_t *ploc = reinterpret_cast<uint32_t *>(p);
    p += align_up(((uint64_t)n + 1) * 4, 256);
    uint64_t *wavetot = reinterpret_cast<uint64_t *>(p);

    if (flag) {
        uint32_t blocks = (uint32_t)(cdiv(n, 256) < 1024 ? cdiv(n, 256) : 1024);
        if (blocks == 0) blocks = 1;
        hipLaunchKernelGGL(k_char_validate, dim3(blocks), dim3(256), 0, s, offsets, n, B, flag);
        return hipGetLastError();
    }
    uint64_t Rw = 0;
    uint32_t nwaves = 0;
    hipError_t e = char_waves(B, Rw, nwaves);
    if (e != hipSuccess) return e;
    if (nwaves > 0) {
        uint32_t blocks = (uint32_t)cdiv(nwaves, kBlock / 64);
        hipLaunchKernelGGL(k_char_main, dim3(blocks), dim3(kBlock), 0, s, text, B, offsets, n, Rw,
                           nwaves, ploc, wavetot);
    }
    uint64_t fb = cdiv(n, 256);
    uint32_t fblocks = (uint32_t)(fb < 4096 ? fb : 4096);
    if (fblocks)
        hipLaunchKernelGGL(k_char_fin, dim3(fblocks), dim3(256), 0, s, offsets, n, B,
                           (uint32_t)(Rw >> 10), nwaves, wavetot, ploc, counts,
                           score ? *score : ScoreArgs{});
    return hipGetLastError();
}

hipError_t readbw_launch(const void *buf, uint64_t bytes, uint32_t *xor_out, hipStream_t s)
{
    hipError_t e = fill_u32(xor_out, 0u, kReadBwWords, s);   // a fill kernel, not a memset
    if (e != hipSuccess || bytes == 0) return e;
    uint64_t Rw = 0;
    uint32_t nwaves = 0;
    e = char_waves(bytes, Rw, nwaves);
    if (e != hipSuccess) return e;
    static_assert(kMaxWaves <= kReadBwWords, "a word per wave");
    const uint32_t blocks = (uint32_t)cdiv(nwaves, kBlock / 64);
    hipLaunchKernelGGL(k_read_stream, dim3(blocks), dim3(kBlock), 0, s, static_cast<const uint8_t *>(buf), bytes, Rw,
                       nwaves, xor_out);
    return hipGetLastError();
}

}  // namespace ds
