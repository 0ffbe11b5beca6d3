// Helicity-summed |M|^2 of u(p1) ubar(p2) -> n photons with the helicities of
// a point spread over the lanes of a wave, so that every subset current is
// formed once per point for exactly the helicities it depends on.
//
// The algebra is that of meet_sets in me2_tree.hpp: with K = (n + 1) / 2,
//     sum over all orderings = sum over |A| = K of W(B) . J(A),  B = the rest,
//     J(Q) = d(q_Q) P(q_Q) sum_{j in Q} V_j J(Q \ j),  q_Q = -p2 + sum_Q k,
//     R(C) = [sum_{c in C} R(C \ c) V_c] d(p1 - sum_C k) P(p1 - sum_C k),
//     W(B) = sum_{b in B} R(B \ b) V_b.
// J(Q) depends on the helicities of the photons in Q only, R and W likewise:
// a set of m photons has 2^m values, the contraction of a set A 2^n.  One
// lane per point can share them only among the helicities it holds in
// registers at once (two at n = 8, where the held currents of two already
// spill), so its walks form most values many times over: 5.1e6 operations per
// point at n = 8 instead of 6.0e5.  Here S = 2^(n-2) lanes hold one point (P =
// 64 / S points per wave): lane s owns the four configurations whose photons
// 2 .. n-1 have the bits of s (photons 0 and 1 run over the lane's four FP64
// accumulators), and the currents pass between lanes through the wave's LDS.
//
// Phases, each reading what the phase before wrote (two waves share a point's
// LDS, take the rounds of a phase in turn and meet at a barrier per phase):
//   1. lane s < n: photon s (scaled light-cone momentum, both vertex blocks);
//   2. propagators of all sets of up to K - 1 (v-bar end), n - K - 1 (u end);
//   3. J level by level up to K - 1, then R up to n - K - 1: a task is one set
//      with the helicities of all its photons but the last, whose two a lane
//      forms together (they share the children and blocks that they read);
//   4. propagators of the sets of K photons;
//   5. per chunk of four sets A, the waves taking every other chunk through an
//      LDS buffer of their own: the 2^K values of every J(A) and the 2^(n-K) of
//      every W(B) go to the buffer, and the lanes contract them, each for its
//      four configurations.  Within a wave LDS operations execute in order, so
//      no barrier is met; the waves add their accumulators at the end.
// Sets A are walked grouped by which of photons 0 and 1 they hold, so that the
// pattern of a lane's four contractions is known at compile time.  Where the J
// (or the W) of a chunk would leave lanes idle (n = 8) one round forms both:
// a row's step is a column's with the halves of the vertex block swapped, so the
// u end's lanes read swapped copies of the blocks and a propagator of unity.
// All LDS addresses of a lane come from tables made at compile time.
//
// What bounds it: in FP32 VALU issue (n = 8: 7 000 instructions per point; at
// four waves per SIMD the counters show the issue slots full, LDS busy half of
// the clocks), in FP64 the LDS reads, 16 bytes each and two per value, of two
// waves per SIMD (40 KiB of LDS per workgroup; more waves through a shared
// buffer and barriers ran 5% slower).
// Measured (us; helicities by one lane per point -> one task per value and one
// to two waves -> this form; 131 101, 65 537 and 20 001 points): FP32 n = 6
// 397 -> 191 -> 154, n = 7 1 530 -> 284 -> 243, n = 8 3 100 -> 249 -> 220; FP64
// n = 6 1 350 -> 281 -> 272, n = 7 7 400 -> 447 -> 428, n = 8 16 700 -> 395 ->
// 387.  At 2053 points FP32: n = 6 11.0 -> 8.4, n = 7 19.4 -> 14.6, n = 8 32.0 ->
// 28.7.  Every FP32 value is formed by the same operations in the same order in
// all of these, so FP32 results have the same bits (up to the order in which the
// waves add the sets).
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "kernels.hpp"
#include "me2_item.hpp"
#include "me2_tree.hpp"
#include "reduce.hpp"

namespace heget {
namespace lanes {

// Fixed numbers of the split for n photons with W = 2 waves on a workgroup's points
// (one wave, two chunk buffers in turn, was slower at every size: FP32 n = 7, 65 537
// points 276 us instead of 243, 2053 points 18.2 instead of 14.6).
template <int N, int WAVES>
struct Split {
    static constexpr int W = WAVES;
    static constexpr int K = (N + 1) / 2, U = N - K;
    static constexpr int S = 1 << (N - 2), P = 64 / S;
    static constexpr int kSets = binomial(N, K);
    // first walked set that holds photon 0 only, 1 only, neither of the two
    static constexpr int kFrom1 = binomial(N - 2, K - 2), kFrom2 = kFrom1 + binomial(N - 2, K - 1),
                         kFrom0 = kFrom2 + binomial(N - 2, K - 1);
    // of photons 0 and 1, those in the set of walking slot `slot`
    static constexpr uint32_t held(int slot) { return slot < kFrom1 ? 3u : slot < kFrom2 ? 1u : slot < kFrom0 ? 2u : 0u; }
    // sets per chunk: the values of J and W of a chunk fill whole rounds of S lanes
    static constexpr int C = 4;
    static constexpr int kChunks = (kSets + C - 1) / C;
    static constexpr int kSlots = kChunks * C;
    // a lane forms a set's values for both helicities of its last photon where
    // that fills the rounds; J and W share a round where each alone would not
    static constexpr bool kMixed = (C << (K - 1)) % S != 0;
    static constexpr int kOutJ = 2, kOutW = kMixed || (C << (U - 1)) % S == 0 ? 2 : 1;
    static constexpr int kTasksJ = (C << K) / kOutJ, kTasksW = (C << U) / kOutW;
    static constexpr int kRounds = (kTasksJ + kTasksW) / S;  // of a chunk
    static_assert((kTasksJ + kTasksW) % S == 0 && (kMixed ? K == U && kRounds == 1 : kTasksJ % S == 0));
    static constexpr int props_j()
    {
        int r = 0;
        for (int l = 1; l < K; ++l) r += binomial(N, l);
        return r;
    }
    static constexpr int props_r()
    {
        int r = 0;
        for (int l = 1; l < U; ++l) r += binomial(N, l);
        return r;
    }
    static constexpr int level_size(int l) { return binomial(N, l) << l; }
    static constexpr int max2(int a, int b) { return a > b ? a : b; }
    // LDS regions of one point, in entries of four values (16 bytes per plane)
    static constexpr int kChunkJ = C << K, kChunk = kChunkJ + (C << U);
    // level 2 where it does not stay (of the v-bar end, then of the u end)
    static constexpr int lower() { return K - 1 > 2 ? level_size(2) : 0; }
    static constexpr int kJ = 0;                               // J of level K - 1
    static constexpr int kR = kJ + level_size(K - 1);          // R of level n - K - 1
    static constexpr int kT = kR + level_size(U - 1);          // a zero momentum, level 2; then a chunk per wave
    static constexpr int kT2 = kT + max2(lower(), 1);          // u-end propagators, level 1
    static constexpr int kProp = max2(kT2 + props_r() + level_size(1), kT + W * kChunk);  // v-bar-end propagators
    static constexpr int kSwap = kProp + kSlots;               // then those of level K, and where J and W share a
    static constexpr int kOne = kSwap + 2 * N;                 // round the blocks as a row takes them, and unity
    static constexpr int kRec = kProp + max2(props_j(), kMixed ? kSlots + 2 * N + 1 : kSlots);
    static constexpr int kRecSize = 3;                         // photon: block of helicity -, +, momentum
    // LDS of a point: with four or more points per wave an odd multiple of eight
    // entries, half the 256 bytes that the banks span, so that two points' reads
    // of the same entries fall into different banks (n = 6: a third of the LDS
    // clocks were conflicts with 287 entries; FP64 4.23e8 -> 4.82e8 points/s,
    // FP32 7.4e8 -> 7.6e8; strides of 0, 1, 2, 4 or 12 beyond a multiple of
    // sixteen lie between)
    static constexpr int kUsed = kRec + kRecSize * N;
    static constexpr int kEntries = P >= 4 ? (kUsed + 7) / 16 * 16 + 8 : kUsed;
    static_assert(kEntries * P * 16 <= 65536, "byte offsets of a plane are 16 bits");
    // entry of level l of the v-bar end or (row) the u end
    static constexpr int level_at(bool row, int l)
    {
        return l == (row ? U : K) - 1 ? (row ? kR : kJ) : l == 1 ? kT2 + props_r() : kT;
    }
    // propagators of the levels below l of one end
    static constexpr int props_below(int l)
    {
        int a = 0;
        for (int i = 1; i < l; ++i) a += binomial(N, i);
        return a;
    }
    // rounds of level l (2 or more), two helicity configurations per lane
    static constexpr int level_rounds(int l) { return (level_size(l) / 2 + S - 1) / S; }
};

// Byte offsets into a plane of the workgroup's LDS, worked out for each of the
// 64 lanes at compile time (lane l of a wave: point l / S, lane l % S of it).
struct alignas(16) LaneRow {
    uint32_t w[4];  // per photon of the lane's set: the child's value | the vertex block's << 16
};

template <int N, int W>
struct alignas(16) Tables {
    using L = Split<N, W>;
    LaneRow build[L::kChunks][L::kRounds][64];  // rounds of a chunk: its J, then its W
    LaneRow lev[2][5][64];                      // rounds of levels 2 and 3 (index l - 2; both ends)
    LaneRow con[L::kChunks][64];                // per set of a chunk: the lane's J | W << 16 in the chunk buffer
    uint16_t prop[256][4];                      // photon momenta of each propagator task (from the point's LDS)
    uint16_t set_of[L::kSlots];                 // the sets A in walking order (padded with the last one)
};

// Bits of h at the positions of `set`, packed to the bottom.
constexpr uint32_t pack_bits(uint32_t h, uint32_t set)
{
    uint32_t r = 0;
    int at = 0;
    for (int j = 0; j < 8; ++j)
        if (set >> j & 1u) r |= (h >> j & 1u) << at++;
    return r;
}

// h without bit p.
constexpr uint32_t without_bit(uint32_t h, int p)
{
    return (h & ((1u << p) - 1u)) | ((h >> (p + 1)) << p);
}

// Row of the lane of point `pt` that forms the values of `set` for the helicities
// f of its photons but (out = 2) the last, from the level below at entry `from`.
template <int N, int W>
constexpr LaneRow lane_row(const uint8_t (&rank)[256], uint32_t set, uint32_t f, int out, int from, int pt,
                           bool swapped = false)
{
    using L = Split<N, W>;
    LaneRow r{};
    const int l = __builtin_popcount(set);
    int p = 0;
    for (int j = 0; j < N; ++j) {
        if (!(set >> j & 1u)) continue;
        const int child = from + (rank[set & ~(1u << j)] << (l - 1)) + static_cast<int>(without_bit(f, p));
        const int e = out == 2 && p == l - 1 ? 0 : static_cast<int>(f >> p & 1u);
        const int block = swapped ? L::kSwap + 2 * j + e : L::kRec + L::kRecSize * j + e;
        r.w[p] = static_cast<uint32_t>((pt * L::kEntries + child) * 16) |
                 static_cast<uint32_t>((pt * L::kEntries + block) * 16) << 16;
        ++p;
    }
    return r;
}

template <int N, int W>
constexpr void momentum_entries(uint32_t set, uint16_t (&out)[4])
{
    using L = Split<N, W>;
    for (int p = 0; p < 4; ++p)
        out[p] = static_cast<uint16_t>(
            (p < __builtin_popcount(set) ? L::kRec + L::kRecSize * nth_bit(set, p) + 2 : L::kT) * 16);
}

template <int N, int W>
constexpr Tables<N, W> make_tables()
{
    using L = Split<N, W>;
    Tables<N, W> t{};
    uint8_t rank[256] = {}, of_rank[N + 1][70] = {};
    int seen[N + 1] = {};
    for (uint32_t m = 1; m < (1u << N); ++m) {  // as subset_rank
        const int l = __builtin_popcount(m);
        of_rank[l][seen[l]] = static_cast<uint8_t>(m);
        rank[m] = static_cast<uint8_t>(seen[l]++);
    }
    // sets A of K photons: those holding photons 0 and 1, 0 only, 1 only, neither
    int at = 0;
    while (at < L::kSets) {
        const uint32_t held = L::held(at);
        for (uint32_t m = 1; m < (1u << N); ++m)
            if (__builtin_popcount(m) == L::K && (m & 3u) == held) t.set_of[at++] = static_cast<uint16_t>(m);
    }
    for (; at < L::kSlots; ++at) t.set_of[at] = t.set_of[L::kSets - 1];
    constexpr uint32_t kAll = (1u << N) - 1u;
    for (int lane = 0; lane < 64; ++lane) {
        const int s = lane % L::S, pt = lane / L::S;
        for (int c = 0; c < L::kChunks; ++c)
            for (int r = 0; r < L::kRounds; ++r) {
                const bool row = r * L::S + s >= L::kTasksJ;
                const int lv = row ? L::U : L::K, out = row ? L::kOutW : L::kOutJ, h = (1 << lv) / out;
                const int task = r * L::S + s - (row ? L::kTasksJ : 0);
                const uint32_t A = t.set_of[c * L::C + task / h];
                t.build[c][r][lane] = lane_row<N, W>(rank, row ? kAll & ~A : A, static_cast<uint32_t>(task % h), out,
                                                     row ? L::kR : L::kJ, pt, row && L::kMixed);
            }
        for (int i = 0; i < L::kSlots; ++i) {
            const uint32_t A = t.set_of[i], h = static_cast<uint32_t>(s) << 2;
            const int base = pt * L::kEntries + L::kT + i / L::C % W * L::kChunk, in = i % L::C;
            t.con[i / L::C][lane].w[in] = (base + (in << L::K) + pack_bits(h, A)) * 16u |
                             ((base + L::kChunkJ + (in << L::U) + pack_bits(h, kAll & ~A)) * 16u) << 16;
        }
        for (int l = 2; l <= 3; ++l)
            if (l <= L::K - 1)
                for (int r = 0; r < L::level_rounds(l); ++r) {
                    // lanes past the last task repeat the last set
                    const int h = 1 << (l - 1), task = r * L::S + s, last = binomial(N, l) - 1;
                    t.lev[l - 2][r][lane] = lane_row<N, W>(rank, of_rank[l][task / h < last ? task / h : last],
                                                           static_cast<uint32_t>(task % h), 2, L::level_at(false, l - 1), pt);
                }
    }
    // propagator tasks: v-bar end levels 1 .. K - 1, u end 1 .. U - 1, level K
    at = 0;
    for (int end = 0; end < 2; ++end)
        for (int l = 1; l < (end == 0 ? L::K : L::U); ++l)
            for (uint32_t m = 1; m < (1u << N); ++m)
                if (__builtin_popcount(m) == l) momentum_entries<N, W>(m, t.prop[at++]);
    for (int i = 0; i < L::kSets; ++i) momentum_entries<N, W>(t.set_of[i], t.prop[at++]);
    return t;
}

template <int N, int W>
__constant__ constexpr Tables<N, W> kTables = make_tables<N, W>();

// The tables are read through an address the compiler cannot see through
// (fresh_tables, once per phase or chunk): it would otherwise take every
// table load, the same for every item, out of the loop over items and spill.
#define HEGET_CONST_AS __attribute__((address_space(4)))
template <int N, int W>
using TabPtr = const HEGET_CONST_AS Tables<N, W> *;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

template <int N, int W>
__device__ __forceinline__ TabPtr<N, W> fresh_tables()
{
    TabPtr<N, W> t = (TabPtr<N, W>)&kTables<N, W>;
    asm volatile("" : "+s"(t));
    return t;
}

// Lane `lane`'s row of a table row of the wave: from a scalar address.
__device__ __forceinline__ u32x4 row4(const HEGET_CONST_AS LaneRow *wave_row, int lane)
{
    asm volatile("" : "+s"(wave_row));
    return *(const HEGET_CONST_AS u32x4 *)(wave_row + static_cast<uint32_t>(lane));
}

// Four values of one LDS entry.  FP64 entries lie in two planes of 16 bytes
// per entry (so that consecutive entries are consecutive 16-byte words, as in
// FP32, and offsets are the same), `PLANE` bytes apart.
template <typename R>
struct Quad {
    R a, b, c, d;
};

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

template <int PLANE>
__device__ __forceinline__ Quad<float> get(const char *p, float)
{
    const f32x4 v = *reinterpret_cast<const f32x4 *>(p);
    return {v.x, v.y, v.z, v.w};
}

template <int PLANE>
__device__ __forceinline__ Quad<double> get(const char *p, double)
{
    const f64x2 u = *reinterpret_cast<const f64x2 *>(p), v = *reinterpret_cast<const f64x2 *>(p + PLANE);
    return {u.x, u.y, v.x, v.y};
}

template <int PLANE>
__device__ __forceinline__ void put(char *p, const Quad<float> &q)
{
    *reinterpret_cast<f32x4 *>(p) = f32x4{q.a, q.b, q.c, q.d};
}

template <int PLANE>
__device__ __forceinline__ void put(char *p, const Quad<double> &q)
{
    *reinterpret_cast<f64x2 *>(p) = f64x2{q.a, q.b};
    *reinterpret_cast<f64x2 *>(p + PLANE) = f64x2{q.c, q.d};
}

// What a lane of this wave wrote to LDS is read by others of the wave after it:
// the LDS unit executes one wave's operations in order, so only the compiler
// has to keep that order.
__device__ __forceinline__ void wave_phase_end()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

// Sum (or product) of v over the S lanes of a point, left in every lane.
template <int S>
__device__ __forceinline__ double group_sum(double v)
{
    v += dpp_f64<0xB1>(v);
    v += dpp_f64<0x4E>(v);
    v += dpp_f64<0x141>(v);
    if constexpr (S >= 16) v += dpp_f64<0x140>(v);
    if constexpr (S >= 32) {
        double lo, hi;
        swap_f64<16>(v, lo, hi);
        v = lo + hi;
    }
    if constexpr (S >= 64) {
        double lo, hi;
        swap_f64<32>(v, lo, hi);
        v = lo + hi;
    }
    return v;
}

__device__ __forceinline__ double octet_product(double v)
{
    v *= dpp_f64<0xB1>(v);
    v *= dpp_f64<0x4E>(v);
    v *= dpp_f64<0x141>(v);
    return v;
}

// Sum of v, |v| <= 1, over each eight lanes less `target`, which lies close to it, to
// well below a rounding of v: the multiples of 2^-40 in v add exactly, and the rest
// of it is that small.
__device__ __forceinline__ double octet_excess(double v, double target)
{
    constexpr double kGrid = 0x1.8p+12;
    double hi = (v + kGrid) - kGrid, lo = v - hi;
    hi += dpp_f64<0xB1>(hi), lo += dpp_f64<0xB1>(lo);
    hi += dpp_f64<0x4E>(hi), lo += dpp_f64<0x4E>(lo);
    hi += dpp_f64<0x141>(hi), lo += dpp_f64<0x141>(lo);
    return (hi - target) + lo;
}

// s (+)= V c for a current c = (g2, g3) (or c V for a row, ROW) with one
// lane's vertex block v = (beta, gamma).
template <bool ROW, bool FIRST, typename R>
__device__ __forceinline__ void vertex(const Quad<R> &v, const Quad<R> &c, Quad<R> &s)
{
    // a column takes beta into its first component and gamma into its second,
    // a row the other way round
    const R b1r = ROW ? v.c : v.a, b1i = ROW ? v.d : v.b, b2r = ROW ? v.a : v.c, b2i = ROW ? v.b : v.d;
    const R x = FIRST ? c.a : s.a + c.a, y = FIRST ? c.b : s.b + c.b;
    const R z = FIRST ? -c.c : s.c - c.c, w = FIRST ? -c.d : s.d - c.d;
    s.a = fma(b1r, c.c, fma(-b1i, c.d, x));
    s.b = fma(b1r, c.d, fma(b1i, c.c, y));
    s.c = fma(b2r, c.a, fma(-b2i, c.b, z));
    s.d = fma(b2r, c.b, fma(b2i, c.a, w));
}

// d P(q) s (a column) or s d P(q) (a row), with P = d (q-, q+, qx, qy).
template <bool ROW, typename R>
__device__ __forceinline__ Quad<R> propagated(const Quad<R> &P, const Quad<R> &s)
{
    const R m = P.a, p = P.b, x = P.c, y = ROW ? -P.d : P.d;
    Quad<R> o;
    o.a = m * s.a - x * s.c + y * s.d;
    o.b = m * s.b - x * s.d - y * s.c;
    o.c = p * s.c - x * s.a - y * s.b;
    o.d = p * s.d - x * s.b + y * s.a;
    return o;
}

// sum_p V_p c(set \ p) of a set of LV photons for OUT helicity configurations
// (rows: c V): those of the lane's table row, and (OUT = 2) of the last photon
// both.  The pair shares all vertex blocks but the last photon's, which are the
// same four values in another order, and that photon's child: 2 LV + (2 LV - 1)
// reads from LDS instead of 4 LV.
template <typename R, int LV, bool ROW, int OUT, int PLANE>
__device__ __forceinline__ void vertices(const char *lds_all, const u32x4 &row, Quad<R> (&sum)[OUT])
{
    static_for<0, LV>([&](auto pi) {
        constexpr int p = decltype(pi)::value;
        const char *child = lds_all + (row[p] & 0xffffu);
        const Quad<R> v = get<PLANE>(lds_all + (row[p] >> 16), R());
        if constexpr (OUT == 2 && p == LV - 1) {
            const Quad<R> c = get<PLANE>(child, R());
            vertex<ROW, p == 0>(v, c, sum[0]);
            vertex<ROW, p == 0>(Quad<R>{v.c, -v.d, v.a, -v.b}, c, sum[1]);
        } else {
#pragma unroll
            for (int o = 0; o < OUT; ++o)
                vertex<ROW, p == 0>(v, get<PLANE>(child + o * (16 << (LV - 2)), R()), sum[o]);
        }
    });
}

// Propagators of the COUNT tasks from FIRST in the table on, to entry `AT`
// (rest: where REST is set):
// d (q-, q+, qx, qy) with q = base + sign * (sum of the task's photons) + rest.
template <typename R, int N, int W, int FIRST, int COUNT, int AT, int PLANE, bool REST = false>
__device__ __forceinline__ void propagators(char *lds, int s, int first, R base_p, R base_m, R sign,
                                            const Quad<R> &rest = {})
{
    using L = Split<N, W>;
    constexpr int S = L::S;
    const TabPtr<N, W> tab = fresh_tables<N, W>();
    constexpr int kRounds = (COUNT + S - 1) / S;
#pragma unroll
    for (int i = 0; i < (kRounds + W - 1) / W; ++i) {
        const int r = i * W + first;
        if (kRounds % W != 0 && r >= kRounds) break;
        const int t = r * S + s < COUNT ? r * S + s : COUNT - 1;
        const u32x2 w = *(const HEGET_CONST_AS u32x2 *)tab->prop[FIRST + t];
        const uint32_t off[4] = {w.x & 0xffffu, w.x >> 16, w.y & 0xffffu, w.y >> 16};
        R p = base_p, m = base_m, x = R(0), y = R(0);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (j >= L::K) continue;
            const Quad<R> k = get<PLANE>(lds + off[j], R());
            p = fma(sign, k.a, p);
            m = fma(sign, k.b, m);
            x = fma(sign, k.c, x);
            y = fma(sign, k.d, y);
        }
        if constexpr (REST) p += rest.a, m += rest.b, x += rest.c, y += rest.d;
        const R q2 = p * m - x * x - y * y;
        const R d = neg_recip(q2);
        put<PLANE>(lds + (AT + t) * 16, Quad<R>{d * m, d * p, d * x, d * y});
    }
}

// Level 1 of one end (ROW: the u end).
template <typename R, int N, int W, bool ROW, int PLANE>
__device__ __forceinline__ void build_first(char *lds, int s, int first)
{
    using L = Split<N, W>;
    constexpr int S = L::S, TO = L::level_at(ROW, 1), PR = ROW ? L::kT2 : L::kProp;
    static_assert(2 * N <= S, "one round");
    if (first != 0) return;
    // lanes past the last task repeat the last photon (same values, same place)
    const int photon = s / 2 < N ? s / 2 : N - 1, e = s & 1;
    const Quad<R> P = get<PLANE>(lds + (PR + photon) * 16, R());
    const Quad<R> v = get<PLANE>(lds + (L::kRec + L::kRecSize * photon + e) * 16, R());
    Quad<R> o;
    if constexpr (!ROW)  // V (1, 0) = (1, gamma)
        o = {fma(-P.c, v.c, fma(P.d, v.d, P.a)), -fma(P.c, v.d, P.d * v.c), fma(P.b, v.c, -P.c),
             fma(P.b, v.d, P.d)};
    else  // (gamma, -1)
        o = {fma(v.c, P.a, P.c), fma(v.d, P.a, -P.d), -fma(v.c, P.c, fma(-v.d, P.d, P.b)),
             -fma(v.c, P.d, v.d * P.c)};
    put<PLANE>(lds + (TO + 2 * photon + e) * 16, o);
}

// Level LV (2 or more) of one end (ROW: the u end) from the level below.
template <typename R, int N, int W, int LV, bool ROW, int PLANE>
__device__ __forceinline__ void build_level(char *lds_all, char *lds, int lane, int first)
{
    using L = Split<N, W>;
    constexpr int S = L::S, H = 1 << (LV - 1), kTasks = L::level_size(LV) / 2, kRounds = L::level_rounds(LV);
    constexpr int TO = L::level_at(ROW, LV), PR = (ROW ? L::kT2 : L::kProp) + L::props_below(LV);
    static_assert(!ROW || L::level_at(true, LV - 1) == L::level_at(false, LV - 1), "the ends share their table");
    const TabPtr<N, W> tabs = fresh_tables<N, W>();
    const int s = lane % S;
#pragma unroll
    for (int i = 0; i < (kRounds + W - 1) / W; ++i) {
        const int r = i * W + first;
        if (kRounds % W != 0 && r >= kRounds) break;
        // lanes past the last task repeat the last set (same values, same place)
        int set = (r * S + s) / H;
        if (kTasks % S != 0) set = set < binomial(N, LV) ? set : binomial(N, LV) - 1;
        const Quad<R> P = get<PLANE>(lds + (PR + set) * 16, R());
        Quad<R> sum[2];
        vertices<R, LV, ROW, 2, PLANE>(lds_all, row4(tabs->lev[LV - 2][r], lane), sum);
        char *to = lds + (TO + (set << LV) + s % H) * 16;
#pragma unroll
        for (int o = 0; o < 2; ++o) put<PLANE>(to + o * H * 16, propagated<ROW>(P, sum[o]));
    }
}

// Table words of a chunk, loaded a chunk before their use.
template <int N, int W>
struct ChunkRows {
    u32x4 build[Split<N, W>::kRounds], con;
};

template <int N, int W>
__device__ __forceinline__ ChunkRows<N, W> load_chunk(int lane, int chunk)
{
    using L = Split<N, W>;
    const TabPtr<N, W> t = fresh_tables<N, W>();
    ChunkRows<N, W> c;
#pragma unroll
    for (int r = 0; r < L::kRounds; ++r) c.build[r] = row4(t->build[chunk][r], lane);
    c.con = row4(t->con[chunk], lane);
    return c;
}

// The values of J and W of chunk CH to its wave's buffer.  In a mixed round every
// lane forms a column: a row's vertex blocks come with their halves swapped, and
// its propagator is unity.
template <typename R, int N, int W, int CH, int PLANE>
__device__ __forceinline__ void build_chunk(char *lds_all, char *lds, int s, const ChunkRows<N, W> &rows)
{
    using L = Split<N, W>;
    char *buf = lds + (L::kT + CH % W * L::kChunk) * 16;
    static_for<0, L::kRounds>([&](auto ri) {
        constexpr int r = decltype(ri)::value;
        constexpr bool kRow = !L::kMixed && r * L::S >= L::kTasksJ;
        constexpr int LV = kRow ? L::U : L::K, OUT = kRow ? L::kOutW : L::kOutJ, H = (1 << LV) / OUT;
        Quad<R> sum[OUT];
        vertices<R, LV, kRow, OUT, PLANE>(lds_all, rows.build[r], sum);
        constexpr int kFirst = kRow ? r * L::S - L::kTasksJ : r * L::S;
        const int in = (kFirst + s) / H;
        if constexpr (!kRow) {
            int at = (L::kProp + CH * L::C) + in;
            if constexpr (L::kMixed) at = s < L::kTasksJ ? at : L::kOne;
            const Quad<R> P = get<PLANE>(lds + at * 16, R());
#pragma unroll
            for (int o = 0; o < OUT; ++o) sum[o] = propagated<false>(P, sum[o]);
        }
        // W follows J in the buffer: a mixed round's sets are numbered on
        static_assert(L::kChunkJ == L::C << L::K);
        char *to = buf + ((kRow ? L::kChunkJ : 0) + (in << LV) + s % H) * 16;
#pragma unroll
        for (int o = 0; o < OUT; ++o) put<PLANE>(to + o * H * 16, sum[o]);
    });
}

// Add w . g, in the working precision, to an FP64 sum.
template <typename R>
__device__ __forceinline__ void add_product(const Quad<R> &w, const Quad<R> &g, double &re, double &im)
{
    R ar = w.a * g.a;
    ar = fma(-w.b, g.b, ar);
    ar = fma(w.c, g.c, ar);
    ar = fma(-w.d, g.d, ar);
    R ai = w.a * g.b;
    ai = fma(w.b, g.a, ai);
    ai = fma(w.c, g.d, ai);
    ai = fma(w.d, g.c, ai);
    re += static_cast<double>(ar);
    im += static_cast<double>(ai);
}

// Add the contraction W(B) . J(A) of one set for the lane's four
// configurations: configuration bit 0 is photon 0, bit 1 photon 1, and a set
// that holds a photon sees its bit lowest.  kHeld: of photons 0 and 1, those in
// A; `con`: the lane's places in the chunk buffer.
template <typename R, uint32_t kHeld, int PLANE>
__device__ __forceinline__ void contract(const char *lds_all, uint32_t con, double (&re)[4], double (&im)[4])
{
    const char *jb = lds_all + (con & 0xffffu), *wb = lds_all + (con >> 16);
    constexpr int nj = kHeld == 3u ? 4 : kHeld == 0u ? 1 : 2, nw = 4 / nj;
    Quad<R> jv[nj], wv[nw];
#pragma unroll
    for (int i = 0; i < nj; ++i) jv[i] = get<PLANE>(jb + 16 * i, R());
#pragma unroll
    for (int i = 0; i < nw; ++i) wv[i] = get<PLANE>(wb + 16 * i, R());
#pragma unroll
    for (int h = 0; h < 4; ++h) {
        const Quad<R> &g = jv[kHeld == 3u ? h : kHeld == 0u ? 0 : kHeld == 1u ? (h & 1) : (h >> 1)];
        const Quad<R> &w = wv[kHeld == 3u ? 0 : kHeld == 0u ? h : kHeld == 1u ? (h >> 1) : (h & 1)];
        add_product(w, g, re[h], im[h]);
    }
}

// What one lane loads of a point: the beams and photon min(s, n - 1).
struct LaneLoad {
    double e1, x1, y1, z1, e2, x2, y2, z2, e, x, y, z;
};

template <bool BEAM>
__device__ __forceinline__ LaneLoad load_lane(const double *__restrict__ mom, int64_t ld, uint32_t src,
                                              int photon)
{
    const double *k = mom + (kBeamRows<BEAM> + 4 * photon) * ld + src;
    const double *b = mom + src;
    if constexpr (BEAM)
        return {b[0], 0.0, 0.0, b[0], b[0], 0.0, 0.0, -b[0], k[0], k[ld], k[2 * ld], k[3 * ld]};
    else
        return {b[0], b[ld], b[2 * ld], b[3 * ld], b[4 * ld], b[5 * ld], b[6 * ld], b[7 * ld],
                k[0], k[ld], k[2 * ld], k[3 * ld]};
}

// Work item: P consecutive points of the list.  Resident waves, each walking
// its items in turn and loading the next item's inputs ahead; |M|^2 of point
// i at out[i].  Arguments as me2_kernel's (one chunk, no weighted epilogue).
template <typename R, int N, int W, int WPE, bool BEAM>
__global__ void __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(WPE)))
me2_lanes_kernel(const double *__restrict__ mom, int64_t ld, const int32_t *__restrict__ index,
                 const uint16_t *__restrict__, const int64_t *__restrict__ d_count, int64_t count, int,
                 double coef, double *__restrict__ out, int64_t, const double *__restrict__,
                 double *__restrict__, double *__restrict__, unsigned *__restrict__ flags)
{
    using L = Split<N, W>;
    constexpr int S = L::S, P = L::P;
    constexpr bool kF32 = std::is_same<R, float>::value;
    constexpr int PLANE = L::kEntries * P * 16;
    __shared__ __align__(16) char lds_all[(kF32 ? 1 : 2) * PLANE];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int s = lane % S, pt = lane / S;
    char *lds = lds_all + pt * (L::kEntries * 16);
    const int64_t npts = d_count ? *d_count : count;
    const int64_t nitems = (npts + P - 1) / P;
    int64_t stride = gridDim.x, item = blockIdx.x, end = nitems;
    // one contiguous range of items per XCD (blocks go round-robin to the
    // eight), so that points sharing cache lines are read through one L2
    constexpr unsigned kXcds = 8;
    if (gridDim.x % kXcds == 0) {
        const int64_t x = blockIdx.x % kXcds, per = (nitems + kXcds - 1) / kXcds;
        stride = gridDim.x / kXcds;
        item = x * per + blockIdx.x / kXcds;
        end = (x + 1) * per < nitems ? (x + 1) * per : nitems;
    }
    if (item >= end) return;
    // The photons' momenta add up to p1 + p2 only to a rounding, and the u end
    // starts from p1: at a soft set its momenta are then another event's than the
    // v-bar end's by more than their own rounding.  Where one lane per point walked
    // from the v-bar end alone (FP64 n = 8) the u end takes what is left over,
    // rest = sum of the photons - p1 - p2, with every momentum.  Against the oracle's
    // 1024 stored points, that walk -> p1 as it is -> with the rest: median 9.8e-15
    // -> 1.15e-14 -> 7.8e-15, 99th percentile 1.36e-13 -> 1.54e-13 -> 9.1e-14, maximum
    // 2.5e-13 -> 2.9e-13 -> 2.1e-13; 20 001 points 384.6 -> 386.6 us.  n = 6 and 7
    // met in the middle before too, with the same errors as now.
    constexpr bool kBalance = !kF32 && N == 8;
    // (every eight lanes hold all photons where their sum is formed)
    const int own = kBalance ? s & 7 : s;
    const int photon = own < N ? own : N - 1;
    // loads past the last point repeat it (never stored)
    auto column = [&](int64_t it) -> uint32_t {
        const int64_t i = it * P + pt;
        const int64_t ic = i < npts ? i : npts - 1;
        return index ? static_cast<uint32_t>(index[ic]) : static_cast<uint32_t>(ic);
    };
    // A point's inputs are loaded an item ahead (their columns two) at two waves
    // per SIMD, and at its start (the column one ahead) at four, where the
    // registers are short and the other waves cover the latency.
    constexpr bool kAhead = WPE < 4;
    LaneLoad q;
    uint32_t src_next = column(item);
    if constexpr (kAhead) {
        q = load_lane<BEAM>(mom, ld, src_next, photon);
        src_next = column(item + stride);
    }
    for (;;) {
        if constexpr (!kAhead) {
            q = load_lane<BEAM>(mom, ld, src_next, photon);
            src_next = column(item + stride);
        }
        // ---- phase 1: FP64 set-up (as me2_compute's), one photon per lane
        bool ok = q.x1 == 0.0 && q.y1 == 0.0 && q.z1 > 0.0 && q.x2 == 0.0 && q.y2 == 0.0 && q.z2 < 0.0;
        int m = 0;
        frexp(q.e1 + q.e2, &m);
        const double sc = ldexp(1.0, -m);
        const double norm = ((q.e1 + q.z1) * sc) * (2.0 * q.e2 * sc);
        const R q0p = static_cast<R>(-(q.e2 + q.z2) * sc), q0m = static_cast<R>(-(q.e2 - q.z2) * sc);
        const R p1p = static_cast<R>((q.e1 + q.z1) * sc), p1m = static_cast<R>((q.e1 - q.z1) * sc);
        const double E = q.e * sc, kx = q.x * sc, ky = q.y * sc, kz = q.z * sc;
        const double pt2 = kx * kx + ky * ky;
        ok = ok && E > 0.0 && pt2 > 0.0;
        const double big = E + fabs(kz);
        R small;
        if constexpr (kF32)
            small = static_cast<float>(pt2) * __builtin_amdgcn_rcpf(static_cast<float>(big));
        else
            small = pt2 / big;
        const R kp = kz >= 0.0 ? static_cast<R>(big) : small;
        const R km = kz >= 0.0 ? small : static_cast<R>(big);
        R ip, im_;
        if constexpr (kF32) {
            ip = __builtin_amdgcn_rcpf(kp);
            im_ = __builtin_amdgcn_rcpf(km);
        } else {
            ip = 1.0 / kp;
            im_ = 1.0 / km;
        }
        const double norm_den = octet_product(s < N ? 2.0 * E * E / pt2 : 1.0);
        Quad<R> rest{};
        if constexpr (kBalance) {
            const bool in = own < N;
            rest = {octet_excess(in ? kp : 0.0, p1p - q0p), octet_excess(in ? km : 0.0, p1m - q0m),
                    octet_excess(in ? kx : 0.0, 0.0), octet_excess(in ? ky : 0.0, 0.0)};
        }
        if (wave == 0 && s < N) {
            const R fx = static_cast<R>(kx), fy = static_cast<R>(ky);
            const R xp = fx * ip, yp = fy * ip, xm = fx * im_, ym = fy * im_;
            char *rec = lds + (L::kRec + L::kRecSize * s) * 16;
            put<PLANE>(rec, Quad<R>{xp, yp, -xm, ym});
            put<PLANE>(rec + 16, Quad<R>{-xm, -ym, xp, -yp});
            put<PLANE>(rec + 32, Quad<R>{kp, km, fx, fy});
        }
        if (wave == 0 && s == 0) put<PLANE>(lds + L::kT * 16, Quad<R>{R(0), R(0), R(0), R(0)});
        const uint64_t votes = __ballot(ok);
        const uint64_t group = (S == 64 ? ~0ull : ((1ull << (S & 63)) - 1ull)) << (pt * S & 63);
        const bool all_ok = (votes & group) == group;
        // the next item's inputs, loaded behind the walk (past the last item:
        // the last point again, never used)
        LaneLoad nxt;
        uint32_t src_after = 0;
        if constexpr (kAhead) {
            nxt = load_lane<BEAM>(mom, ld, src_next, photon);
            src_after = column(item + 2 * stride);
        }
        __syncthreads();

        // ---- phase 2 (two waves take the rounds of each end in turn)
        constexpr int kPj = L::props_j(), kPr = L::props_r();
        const int first = wave, other = W - 1 - wave;
        propagators<R, N, W, 0, kPj, L::kProp, PLANE>(lds, s, first, q0p, q0m, R(1));
        propagators<R, N, W, kPj, kPr, L::kT2, PLANE, kBalance>(lds, s, other, p1p, p1m, R(-1), rest);
        __syncthreads();

        // ---- phase 3
        build_first<R, N, W, false, PLANE>(lds, s, first);
        __syncthreads();
        static_for<2, L::K>([&](auto li) {
            build_level<R, N, W, decltype(li)::value, false, PLANE>(lds_all, lds, lane, first);
            __syncthreads();
        });
        build_first<R, N, W, true, PLANE>(lds, s, other);
        __syncthreads();
        static_for<2, L::U>([&](auto li) {
            build_level<R, N, W, decltype(li)::value, true, PLANE>(lds_all, lds, lane, other);
            __syncthreads();
        });

        // ---- phase 4
        propagators<R, N, W, kPj + kPr, L::kSets, L::kProp, PLANE>(lds, s, first, q0p, q0m, R(1));
        if constexpr (L::kMixed)
            if (wave == W - 1 && s <= 2 * N) {
                Quad<R> v = {R(1), R(1), R(0), R(0)};
                if (s < 2 * N) {
                    const Quad<R> u = get<PLANE>(lds + (L::kRec + L::kRecSize * (s >> 1) + (s & 1)) * 16, R());
                    v = {u.c, u.d, u.a, u.b};
                }
                put<PLANE>(lds + (L::kSwap + s) * 16, v);
            }
        __syncthreads();

        // ---- phase 5: each wave takes every W-th chunk, through a buffer of its own
        double re[4] = {0.0, 0.0, 0.0, 0.0}, im[4] = {0.0, 0.0, 0.0, 0.0};
        auto walk = [&](auto wi) {
            constexpr int w = decltype(wi)::value;
            ChunkRows<N, W> rows = load_chunk<N, W>(lane, w);
            static_for<0, (L::kChunks - w + W - 1) / W>([&](auto ci) {
                constexpr int c = w + W * decltype(ci)::value;
                ChunkRows<N, W> next = rows;
                if constexpr (c + W < L::kChunks) next = load_chunk<N, W>(lane, c + W);
                build_chunk<R, N, W, c, PLANE>(lds_all, lds, s, rows);
                wave_phase_end();
                static_for<0, L::C>([&](auto ii) {
                    constexpr int slot = c * L::C + decltype(ii)::value;
                    if constexpr (slot < L::kSets)
                        contract<R, L::held(slot), PLANE>(lds_all, rows.con[decltype(ii)::value], re, im);
                });
                rows = next;
                wave_phase_end();
            });
        };
        static_assert(W == 2);
        if (wave == 0)
            walk(std::integral_constant<int, 0>{});
        else
            walk(std::integral_constant<int, 1>{});
        __syncthreads();
        static_assert((W - 1) * 8 * 64 * sizeof(double) <= sizeof(lds_all));
        double *share = reinterpret_cast<double *>(lds_all) + lane;
        if (wave > 0) {
#pragma unroll
            for (int h = 0; h < 4; ++h) {
                share[(wave - 1) * 512 + (2 * h) * 64] = re[h];
                share[(wave - 1) * 512 + (2 * h + 1) * 64] = im[h];
            }
        }
        __syncthreads();
        if (wave == 0) {
#pragma unroll
            for (int w = 0; w < W - 1; ++w)
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    re[h] += share[w * 512 + (2 * h) * 64];
                    im[h] += share[w * 512 + (2 * h + 1) * 64];
                }
        }
        double total = 0.0;
#pragma unroll
        for (int h = 0; h < 4; ++h) total += re[h] * re[h] + im[h] * im[h];
        total = group_sum<S>(total);
        const int64_t i = item * P + pt;
        if (wave == 0 && s == 0 && i < npts) {
            double me2 = ldexp(coef * (norm / norm_den) * total, 2 * m * (2 - N));
            if (!all_ok) me2 = __builtin_nan("");
            if (!isfinite(me2)) atomicOr(flags, 1u);
            out[i] = me2;
        }
        item += stride;
        if (item >= end) break;
        if constexpr (kAhead) {
            q = nxt;
            src_next = src_after;
        }
        __syncthreads();
    }
}

}  // namespace lanes
}  // namespace heget
