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
// Phases, each reading what the phase before wrote:
//   1. lane s < n: photon s (scaled light-cone momentum, both vertex blocks);
//   2. propagators of all sets of up to K - 1 (v-bar end), n - K - 1 (u end);
//   3. J level by level up to K - 1, then R up to n - K - 1: a task is one
//      (set, helicities of the set), 2^m consecutive lanes share a set;
//   4. propagators of the sets of K photons;
//   5. per chunk of sets A: the 2^K values of every J(A) and the 2^(n-K) of
//      every W(B) go to an LDS buffer, and the lanes contract them, each for
//      its four configurations.
// Sets A are walked grouped by which of photons 0 and 1 they hold, so that
// the pattern of a lane's four contractions is known at compile time.
//
// With W = 1 a workgroup is one wave: the LDS operations of a wave execute in
// order, so a phase ends with a compiler fence and no barrier, and phase 5
// fills one of two buffers while it contracts the other.  With W = 2 two waves
// share the same points (and LDS): they take the rounds of a phase and the
// chunks in turn, each through a buffer of its own, meet at a barrier per
// phase and add their accumulators at the end.
//
// What bounds it: VALU issue, 7 000 (FP32) and 6 600 (FP64) instructions per
// point and wave at n = 8 (counters: 0.23 per clock and SIMD in FP32, where
// 0.25 is the rate of one wave; LDS busy 48% of the clocks).  LDS (20 KiB per
// wave in FP32, 40 in FP64) allows two waves per SIMD in FP32 but one in FP64,
// which stood still 41% of the time: hence W = 2 there (points/s, W = 1 -> 2:
// n = 8 3.95e7 -> 5.09e7, n = 7 1.14e8 -> 1.48e8, n = 6 3.66e8 -> 4.23e8).  In
// FP32 a third wave per SIMD gains at n = 8 only (8.08e7 -> 8.37e7; at 2053
// points 46.8 -> 34.6 us); at n = 7 it spills, at n = 6 both forms run alike.
// Measured (points/s, one-lane-per-point kernel before -> this one; 524 288,
// 200 003 and 111 040 points at 1.5 TeV): FP32 n = 6 3.3e8 -> 7.6e8, n = 7
// 4.3e7 -> 2.3e8, n = 8 6.4e6 -> 8.4e7; FP64 n = 6 9.7e7 -> 4.8e8, n = 7
// 8.9e6 -> 1.5e8, n = 8 1.2e6 -> 5.1e7.  Every FP32 value is formed by the
// same operations in the same order, so FP32 results have the same bits (up to
// the order in which W = 2 adds the sets).
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "kernels.hpp"
#include "me2_tree.hpp"
#include "reduce.hpp"

namespace heget {
namespace lanes {

// Fixed numbers of the split for n photons with W waves on a wave's points.
template <int N, int WAVES>
struct Split {
    static constexpr int W = WAVES;
    static constexpr int K = (N + 1) / 2, U = N - K;
    static constexpr int S = 1 << (N - 2), P = 64 / S;
    static constexpr int kSets = binomial(N, K);
    // sets per chunk: the values of J of a chunk fill whole rounds of S lanes
    static constexpr int C = N <= 6 && W == 2 ? 2 : 4;
    static constexpr int kChunks = (kSets + C - 1) / C;
    static constexpr int kSlots = kChunks * C;
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
    static constexpr int kChunkJ = C << K, kChunkW = C << U, kChunk = kChunkJ + kChunkW;
    // level 2 where it does not stay (of the v-bar end, then of the u end)
    static constexpr int lower() { return K - 1 > 2 ? level_size(2) : 0; }
    static constexpr int kJ = 0;                               // J of level K - 1
    static constexpr int kR = kJ + level_size(K - 1);          // R of level n - K - 1
    static constexpr int kT = kR + level_size(U - 1);          // a zero momentum, level 2, chunk buffer 0
    static constexpr int kT2 = kT + max2(lower(), kChunk);     // u-end propagators, level 1, chunk buffer 1
    static constexpr int kProp = kT2 + max2(props_r() + level_size(1), kChunk);  // v-bar-end propagators
    static constexpr int kRec = kProp + max2(props_j(), kSets);  // then those of level K
    static constexpr int kRecSize = 3;                         // photon: block of helicity -, +, momentum
    // LDS of a point: with four or more points per wave an odd multiple of eight
    // entries, half the 256 bytes that the banks span, so that two points' reads
    // of the same entries fall into different banks (n = 6: a third of the LDS
    // clocks were conflicts with 287 entries; FP64 4.23e8 -> 4.82e8 points/s,
    // FP32 7.4e8 -> 7.6e8; strides of 0, 1, 2, 4 or 12 beyond a multiple of
    // sixteen lie between)
    static constexpr int kUsed = kRec + kRecSize * N;
    static constexpr int kEntries = P >= 4 ? (kUsed + 7) / 16 * 16 + 8 : kUsed;
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
};

// Index tables (byte offsets within a region, at 16 bytes per entry), built
// at compile time.
template <int N, int W>
struct alignas(16) Tables {
    using L = Split<N, W>;
    uint32_t con[L::kSlots][L::S];  // lane s: J entry | W entry << 16 within the chunk's set
    uint32_t mj[L::kSlots][4];      // per photon of A: J(A \ j) at level K - 1 | record << 16
    uint32_t mw[L::kSlots][4];      // per photon of B: R(B \ b) at level U - 1 | record << 16
    uint32_t lev[3][56][4];         // levels 2, 3 (index l - 1): as mj, for sets in increasing order
    uint16_t prop[256][4];          // photon momenta of each propagator task (offsets from the point's LDS)
    uint16_t set_of[L::kSlots];     // the sets A in walking order (padded with the last one)
};

// Sets A of K photons: those holding photons 0 and 1, 0 only, 1 only, neither.
template <int N>
constexpr uint32_t walk_set(int i)
{
    constexpr int K = (N + 1) / 2;
    constexpr uint32_t kPattern[4] = {3u, 1u, 2u, 0u};
    int at = 0;
    for (int t = 0; t < 4; ++t)
        for (uint32_t m = 1; m < (1u << N); ++m)
            if (__builtin_popcount(m) == K && (m & 3u) == kPattern[t]) {
                if (at == i) return m;
                ++at;
            }
    return 0u;
}

// Bits of h at the positions of `set`, packed to the bottom.
constexpr uint32_t pack_bits(uint32_t h, uint32_t set)
{
    uint32_t r = 0;
    int at = 0;
    for (int j = 0; j < 8; ++j)
        if (set >> j & 1u) r |= (h >> j & 1u) << at++;
    return r;
}

// Per photon of `set`: entry of set \ photon on the level below | record << 16.
template <int N, int W>
constexpr void child_entries(uint32_t set, uint32_t (&out)[4])
{
    using L = Split<N, W>;
    const int l = __builtin_popcount(set);
    for (int p = 0; p < 4; ++p) out[p] = 0;
    for (int p = 0; p < l; ++p) {
        const int j = nth_bit(set, p);
        const uint32_t e = static_cast<uint32_t>(subset_rank<N>(set & ~(1u << j))) << (l - 1);
        out[p] = e * 16u | static_cast<uint32_t>(L::kRecSize * j * 16) << 16;
    }
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
    for (int i = 0; i < L::kSlots; ++i) {
        const uint32_t A = walk_set<N>(i < L::kSets ? i : L::kSets - 1);
        const uint32_t B = ((1u << N) - 1u) & ~A;
        t.set_of[i] = static_cast<uint16_t>(A);
        child_entries<N, W>(A, t.mj[i]);
        child_entries<N, W>(B, t.mw[i]);
        for (int s = 0; s < L::S; ++s) {
            const uint32_t h = static_cast<uint32_t>(s) << 2;
            t.con[i][s] = pack_bits(h, A) * 16u | (pack_bits(h, B) * 16u) << 16;
        }
    }
    for (int l = 2; l <= 3; ++l)
        if (l <= L::K - 1) {
            int r = 0;
            for (uint32_t m = 1; m < (1u << N); ++m)
                if (__builtin_popcount(m) == l) child_entries<N, W>(m, t.lev[l - 1][r++]);
        }
    // propagator tasks: v-bar end levels 1 .. K - 1, u end 1 .. U - 1, level K
    int at = 0;
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

__device__ __forceinline__ u32x4 row4(const HEGET_CONST_AS uint32_t *p)
{
    return *(const HEGET_CONST_AS u32x4 *)p;
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

// End of a phase: what the point's lanes wrote to LDS is read by other lanes
// after it.  The LDS unit executes one wave's operations in order, so within a
// wave only the compiler has to keep that order; two waves meet at a barrier.
__device__ __forceinline__ void wave_phase_end()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

template <int W>
__device__ __forceinline__ void phase_end()
{
    if constexpr (W == 1)
        wave_phase_end();
    else
        __syncthreads();
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

// Entry offset of helicity bits e without bit p.
__device__ __forceinline__ uint32_t drop_bit(uint32_t e, int p)
{
    return (e & ((1u << p) - 1u)) | ((e >> (p + 1)) << p);
}

// Propagators of the COUNT tasks from FIRST in the table on, to entry `AT`:
// d (q-, q+, qx, qy) with q = base + sign * (sum of the task's photons).
template <typename R, int N, int W, int FIRST, int COUNT, int AT, int PLANE>
__device__ __forceinline__ void propagators(char *lds, int s, int first, R base_p, R base_m, R sign)
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
        const R q2 = p * m - x * x - y * y;
        const R d = neg_recip(q2);
        put<PLANE>(lds + (AT + t) * 16, Quad<R>{d * m, d * p, d * x, d * y});
    }
}

// Level LV of one end (ROW: the u end) from the level below.
template <typename R, int N, int W, int LV, bool ROW, int PLANE>
__device__ __forceinline__ void build_level(char *lds, int s, int first)
{
    using L = Split<N, W>;
    constexpr int S = L::S, H = 1 << LV, kTasks = L::level_size(LV);
    constexpr int FROM = L::level_at(ROW, LV - 1), TO = L::level_at(ROW, LV);
    constexpr int PR = (ROW ? L::kT2 : L::kProp) + L::props_below(LV);
    const TabPtr<N, W> tabs = fresh_tables<N, W>();
    const uint32_t e = static_cast<uint32_t>(s) & (H - 1);
    uint32_t child[LV], block[LV];
#pragma unroll
    for (int p = 0; p < LV; ++p) {
        child[p] = drop_bit(e, p) * 16u;
        block[p] = (e >> p & 1u) * 16u;
    }
    constexpr int kRounds = (kTasks + S - 1) / S;
#pragma unroll
    for (int i = 0; i < (kRounds + W - 1) / W; ++i) {
        const int r = i * W + first;
        if (kRounds % W != 0 && r >= kRounds) break;
        // lanes past the last task repeat the last set (same values, same place)
        const int t = r * S + s;
        int set = t >> LV;
        if (kTasks % S != 0) set = set < binomial(N, LV) ? set : binomial(N, LV) - 1;
        const Quad<R> P = get<PLANE>(lds + (PR + set) * 16, R());
        Quad<R> o;
        if constexpr (LV == 1) {
            const Quad<R> v = get<PLANE>(lds + L::kRec * 16 + set * (L::kRecSize * 16) + block[0], R());
            if constexpr (!ROW)  // V (1, 0) = (1, gamma)
                o = {fma(-P.c, v.c, fma(P.d, v.d, P.a)), -fma(P.c, v.d, P.d * v.c), fma(P.b, v.c, -P.c),
                     fma(P.b, v.d, P.d)};
            else  // (gamma, -1)
                o = {fma(v.c, P.a, P.c), fma(v.d, P.a, -P.d), -fma(v.c, P.c, fma(-v.d, P.d, P.b)),
                     -fma(v.c, P.d, v.d * P.c)};
        } else {
            const u32x4 tab = row4(tabs->lev[LV - 1][set]);
            Quad<R> sum;
            static_for<0, LV>([&](auto pi) {
                constexpr int p = decltype(pi)::value;
                const Quad<R> c = get<PLANE>(lds + FROM * 16 + ((tab[p] & 0xffffu) + child[p]), R());
                const Quad<R> v = get<PLANE>(lds + L::kRec * 16 + ((tab[p] >> 16) + block[p]), R());
                vertex<ROW, p == 0>(v, c, sum);
            });
            o = propagated<ROW>(P, sum);
        }
        put<PLANE>(lds + (TO + (set << LV)) * 16 + e * 16u, o);
    }
}

// Table entries of one chunk, loaded a chunk before their use.
template <int N, int W>
struct ChunkTab {
    using L = Split<N, W>;
    u32x4 j[L::kChunkJ / L::S], w[L::kChunkW / L::S];
    uint32_t con[L::C];
};

template <int N, int W>
__device__ __forceinline__ ChunkTab<N, W> load_chunk_tab(int s, int chunk)
{
    using L = Split<N, W>;
    static_assert(L::kChunkJ % L::S == 0 && L::kChunkW % L::S == 0, "a chunk fills whole rounds");
    const TabPtr<N, W> t = fresh_tables<N, W>();
    ChunkTab<N, W> c;
#pragma unroll
    for (int r = 0; r < L::kChunkJ / L::S; ++r) c.j[r] = row4(t->mj[chunk * L::C + ((r * L::S + s) >> L::K)]);
#pragma unroll
    for (int r = 0; r < L::kChunkW / L::S; ++r) c.w[r] = row4(t->mw[chunk * L::C + ((r * L::S + s) >> L::U)]);
#pragma unroll
    for (int i = 0; i < L::C; ++i) c.con[i] = t->con[chunk * L::C + i][s];
    return c;
}

// The values of J (or W, ROW) of one chunk of sets to `to`.
template <typename R, int N, int W, bool ROW, int PLANE>
__device__ __forceinline__ void build_chunk(char *lds, int s, int chunk, const ChunkTab<N, W> &ct, char *to)
{
    using L = Split<N, W>;
    constexpr int S = L::S, LV = ROW ? L::U : L::K, H = 1 << LV;
    constexpr int FROM = ROW ? L::kR : L::kJ;
    const uint32_t e = static_cast<uint32_t>(s) & (H - 1);
#pragma unroll
    for (int r = 0; r < (L::C << LV) / S; ++r) {
        const u32x4 tab = ROW ? ct.w[r] : ct.j[r];
        Quad<R> sum;
        static_for<0, LV>([&](auto pi) {
            constexpr int p = decltype(pi)::value;
            const Quad<R> c = get<PLANE>(lds + FROM * 16 + ((tab[p] & 0xffffu) + drop_bit(e, p) * 16u), R());
            const Quad<R> v = get<PLANE>(lds + L::kRec * 16 + ((tab[p] >> 16) + (e >> p & 1u) * 16u), R());
            vertex<ROW, p == 0>(v, c, sum);
        });
        if constexpr (!ROW) {
            const int slot = chunk * L::C + ((r * S + s) >> LV);
            // padding slots repeat the last set
            const int at = L::kSlots > L::kSets ? (slot < L::kSets ? slot : L::kSets - 1) : slot;
            sum = propagated<false>(get<PLANE>(lds + (L::kProp + at) * 16, R()), sum);
        }
        put<PLANE>(to + (r * S + s) * 16, sum);
    }
}

// Add the contraction W(B) . J(A) of walking slot SLOT (place I of the chunk
// in `buf`) for the lane's four configurations: configuration bit 0 is photon
// 0, bit 1 photon 1, and a set that holds a photon sees its bit lowest.
template <typename R, int N, int W, int SLOT, int PLANE>
__device__ __forceinline__ void contract(const char *buf, uint32_t con, double (&re)[4], double (&im)[4])
{
    using L = Split<N, W>;
    constexpr int I = SLOT % L::C;
    constexpr uint32_t kHeld = walk_set<N>(SLOT) & 3u;  // of photons 0 and 1, those in A
    const char *jb = buf + I * (16 << L::K) + (con & 0xffffu);
    const char *wb = buf + L::kChunkJ * 16 + I * (16 << L::U) + (con >> 16);
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
        R ar = w.a * g.a;
        ar = fma(-w.b, g.b, ar);
        ar = fma(w.c, g.c, ar);
        ar = fma(-w.d, g.d, ar);
        R ai = w.a * g.b;
        ai = fma(w.b, g.a, ai);
        ai = fma(w.c, g.d, ai);
        ai = fma(w.d, g.c, ai);
        re[h] += static_cast<double>(ar);
        im[h] += static_cast<double>(ai);
    }
}

// What one lane loads of a point: the beams and photon min(s, n - 1).
struct LaneLoad {
    double e1, x1, y1, z1, e2, x2, y2, z2, e, x, y, z;
};

__device__ __forceinline__ LaneLoad load_lane(const double *__restrict__ mom, int64_t ld, uint32_t src,
                                              int photon)
{
    const double *k = mom + (8 + 4 * photon) * ld + src;
    const double *b = mom + src;
    return {b[0], b[ld], b[2 * ld], b[3 * ld], b[4 * ld], b[5 * ld], b[6 * ld], b[7 * ld],
            k[0], k[ld], k[2 * ld], k[3 * ld]};
}

// Work item: P consecutive points of the list.  Resident waves, each walking
// its items in turn and loading the next item's inputs ahead; |M|^2 of point
// i at out[i].  Arguments as me2_kernel's (one chunk, no weighted epilogue).
template <typename R, int N, int W, int WPE>
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
    const int wave = W == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
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
    const int photon = s < N ? s : N - 1;
    // loads past the last point repeat it (never stored)
    auto column = [&](int64_t it) -> uint32_t {
        const int64_t i = it * P + pt;
        const int64_t ic = i < npts ? i : npts - 1;
        return index ? static_cast<uint32_t>(index[ic]) : static_cast<uint32_t>(ic);
    };
    LaneLoad q = load_lane(mom, ld, column(item), photon);
    uint32_t src_next = column(item + stride);
    for (;;) {
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
        const LaneLoad nxt = load_lane(mom, ld, src_next, photon);
        const uint32_t src_after = column(item + 2 * stride);
        phase_end<W>();

        // ---- phase 2 (two waves take the rounds of each end in turn)
        constexpr int kPj = L::props_j(), kPr = L::props_r();
        const int first = wave, other = W - 1 - wave;
        propagators<R, N, W, 0, kPj, L::kProp, PLANE>(lds, s, first, q0p, q0m, R(1));
        propagators<R, N, W, kPj, kPr, L::kT2, PLANE>(lds, s, other, p1p, p1m, R(-1));
        phase_end<W>();

        // ---- phase 3
        static_for<1, L::K>([&](auto li) {
            build_level<R, N, W, decltype(li)::value, false, PLANE>(lds, s, first);
            phase_end<W>();
        });
        static_for<1, L::U>([&](auto li) {
            build_level<R, N, W, decltype(li)::value, true, PLANE>(lds, s, other);
            phase_end<W>();
        });

        // ---- phase 4
        propagators<R, N, W, kPj + kPr, L::kSets, L::kProp, PLANE>(lds, s, first, q0p, q0m, R(1));
        phase_end<W>();

        // ---- phase 5
        double re[4] = {0.0, 0.0, 0.0, 0.0}, im[4] = {0.0, 0.0, 0.0, 0.0};
        if constexpr (W == 1) {
            ChunkTab<N, W> ct = load_chunk_tab<N, W>(s, 0), ct_next = load_chunk_tab<N, W>(s, 1);
            build_chunk<R, N, W, false, PLANE>(lds, s, 0, ct, lds + L::kT * 16);
            build_chunk<R, N, W, true, PLANE>(lds, s, 0, ct, lds + (L::kT + L::kChunkJ) * 16);
            wave_phase_end();
            static_for<0, L::kChunks>([&](auto ci) {
                constexpr int c = decltype(ci)::value;
                ChunkTab<N, W> ct_after = ct_next;
                if constexpr (c + 2 < L::kChunks) ct_after = load_chunk_tab<N, W>(s, c + 2);
                if constexpr (c + 1 < L::kChunks) {
                    char *to = lds + (c % 2 == 0 ? L::kT2 : L::kT) * 16;
                    build_chunk<R, N, W, false, PLANE>(lds, s, c + 1, ct_next, to);
                    build_chunk<R, N, W, true, PLANE>(lds, s, c + 1, ct_next, to + L::kChunkJ * 16);
                }
                const char *buf = lds + (c % 2 == 0 ? L::kT : L::kT2) * 16;
                static_for<0, L::C>([&](auto ii) {
                    constexpr int slot = c * L::C + decltype(ii)::value;
                    if constexpr (slot < L::kSets) contract<R, N, W, slot, PLANE>(buf, ct.con[decltype(ii)::value], re, im);
                });
                ct = ct_next;
                ct_next = ct_after;
                wave_phase_end();
            });
        } else {
            // each wave takes every other chunk, through a buffer of its own
            auto walk = [&](auto wi) {
                constexpr int w = decltype(wi)::value;
                constexpr int kMine = (L::kChunks - w + W - 1) / W;
                char *buf = lds + (w == 0 ? L::kT : L::kT2) * 16;
                ChunkTab<N, W> ct = load_chunk_tab<N, W>(s, w);
                static_for<0, kMine>([&](auto ci) {
                    constexpr int c = w + W * decltype(ci)::value;
                    ChunkTab<N, W> next = ct;
                    if constexpr (c + W < L::kChunks) next = load_chunk_tab<N, W>(s, c + W);
                    build_chunk<R, N, W, false, PLANE>(lds, s, c, ct, buf);
                    build_chunk<R, N, W, true, PLANE>(lds, s, c, ct, buf + L::kChunkJ * 16);
                    wave_phase_end();
                    static_for<0, L::C>([&](auto ii) {
                        constexpr int slot = c * L::C + decltype(ii)::value;
                        if constexpr (slot < L::kSets) contract<R, N, W, slot, PLANE>(buf, ct.con[decltype(ii)::value], re, im);
                    });
                    ct = next;
                    wave_phase_end();
                });
            };
            if (wave == 0)
                walk(std::integral_constant<int, 0>{});
            else
                walk(std::integral_constant<int, 1>{});
            __syncthreads();
            double *share = reinterpret_cast<double *>(lds_all) + lane;
            if (wave == 1) {
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    share[(2 * h) * 64] = re[h];
                    share[(2 * h + 1) * 64] = im[h];
                }
            }
            __syncthreads();
            if (wave == 0) {
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    re[h] += share[(2 * h) * 64];
                    im[h] += share[(2 * h + 1) * 64];
                }
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
        q = nxt;
        src_next = src_after;
        phase_end<W>();
    }
}

}  // namespace lanes
}  // namespace heget
