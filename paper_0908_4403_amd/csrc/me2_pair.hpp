// Helicity-summed |M|^2 of u(p1) ubar(p2) -> n photons with a point's helicities
// over two lanes, for n = 5, where one lane per point has too many values for its
// registers and the lanes of me2_lanes.hpp too little work for what they pass on.
//
// The algebra is that of meet_sets in me2_tree.hpp (W(B) . J(A) over the sets A of
// K photons), each value formed once per point.  The last photon's helicity is
// the lane's: - in the even, + in the odd one.  A lane labels the other photons'
// helicities by whether they are its own (label 0) or not, so that both lanes
// run the same code with the vertex blocks of all photons exchanged in the odd
// one.  A set with the last photon has its values for the lane's own helicity;
// the values of a set without it are the same in both lanes, label l of the one
// being label ~l of the other: each lane forms those with the first photon's label
// 0 and takes the others from its partner by a DPP move.  So a lane does half of
// a point's work, with 16 instead of 32 FP64 accumulators and two thirds of the
// values, and a wave holds 32 points: it walks a tile of 64 in two halves.
//
// What bounds it: in FP32 VALU issue at two waves per SIMD, 2 x 5760 instructions
// per tile (the walk of all 32 configurations in a lane had 12 070, an eighth of
// them moves to and from the upper half of its 512 registers, 96 KB of code, and
// one wave per SIMD that waited a tenth of its time); in FP64 registers (one wave,
// 90 spills).  Measured, us, before -> this: FP32 (that walk) 100 000 points 51 ->
// 49, 300 000 124 -> 107, 1e6 368 -> 312, 2.4e6 858 -> 734; FP64 (eight per walk)
// 65 536 points 68 -> 46, 1e6 923 -> 634, 2.4e6 2203 -> 1540.  Loading the next
// half tile ahead, by registers or through LDS, costs more instructions than it
// hides waits (FP32 1e6 points 348 and 362 us); n = 4 (FP64) loses: its set-up and
// propagators, which both lanes need, are a third of it (1e6 points 116 -> 149).
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>

#include <type_traits>

#include "kernels.hpp"
#include "me2_item.hpp"
#include "me2_lanes.hpp"
#include "me2_tree.hpp"
#include "reduce.hpp"

namespace heget {
namespace pairs {

using lanes::Quad;

__device__ __forceinline__ float from_partner(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, true));
}

__device__ __forceinline__ double from_partner(double v) { return dpp_f64<0xB1>(v); }

template <typename R>
__device__ __forceinline__ Quad<R> from_partner(const Quad<R> &v)
{
    return {from_partner(v.a), from_partner(v.b), from_partner(v.c), from_partner(v.d)};
}

constexpr uint32_t without_bit(uint32_t h, int p) { return (h & ((1u << p) - 1u)) | ((h >> (p + 1)) << p); }

// Labels of the photons in `set` (all but the last photon), from those of all of them.
constexpr uint32_t labels_of(uint32_t h, uint32_t set)
{
    uint32_t r = 0;
    int at = 0;
    for (int j = 0; j < 8; ++j)
        if (set >> j & 1u) r |= (h >> j & 1u) << at++;
    return r;
}

// Per-point values that all sets share.
template <typename R, int N>
struct Point {
    LMom<R> k[N], q0, p1;
    Quad<R> v[N];  // vertex block (beta, gamma) of label 0; of the last photon the lane's
};

// Block of photon j for label b.
template <typename R, int N>
__device__ __forceinline__ Quad<R> block(const Point<R, N> &s, int j, uint32_t b)
{
    const Quad<R> &v = s.v[j];
    return b ? Quad<R>{v.c, -v.d, v.a, -v.b} : v;
}

// d (q-, q+, qx, qy) of q = base + SIGN * (sum of the photons of SET).
template <int SIGN, uint32_t SET, typename R, int N>
__device__ __forceinline__ Quad<R> propagator(const LMom<R> &base, const Point<R, N> &s)
{
    R p = base.p, m = base.m, x = base.x, y = base.y;
    for_each_bit<SET>([&](auto bit) {
        constexpr int b = decltype(bit)::value;
        if constexpr (SIGN > 0) {
            p += s.k[b].p, m += s.k[b].m, x += s.k[b].x, y += s.k[b].y;
        } else {
            p -= s.k[b].p, m -= s.k[b].m, x -= s.k[b].x, y -= s.k[b].y;
        }
    });
    const R d = neg_recip(p * m - x * x - y * y);
    return {d * m, d * p, d * x, d * y};
}

// Value of SET for label L of the lane: without the last photon only even labels
// (the first photon's label 0) are held, label L of this lane is label ~L of the
// partner.
template <uint32_t SET, uint32_t L, typename R, int N, int M>
__device__ __forceinline__ Quad<R> value_of(const Quad<R> (&v)[M])
{
    constexpr uint32_t kAll = (1u << __builtin_popcount(SET)) - 1u;
    if constexpr ((SET >> (N - 1) & 1u) == 0u && (L & 1u) != 0u)
        return from_partner(v[~L & kAll]);
    else
        return v[L];
}

// The values of SET for its labels, from those of its subsets; without the last
// photon only for even labels (the first photon's label 0).
template <uint32_t SET, bool ROW, typename R, int N, int M>
__device__ __forceinline__ void vertices(const Point<R, N> &s, const Quad<R> (&from)[1 << N][M], Quad<R> (&to)[M])
{
    constexpr uint32_t kLast = 1u << (N - 1), kOthers = SET & ~kLast;
    constexpr int kBits = __builtin_popcount(kOthers);
    static_for<0, (1 << kBits)>([&](auto li) {
        constexpr uint32_t l = decltype(li)::value;
        if constexpr ((SET & kLast) != 0u || (l & 1u) == 0u) {
            constexpr int kFirst = __builtin_ctz(SET);
            for_each_bit<SET>([&](auto bit) {
                constexpr int j = decltype(bit)::value;
                constexpr int p = __builtin_popcount(kOthers & ((1u << j) - 1u));
                constexpr uint32_t child = j == N - 1 ? l : without_bit(l, p);
                constexpr uint32_t b = j == N - 1 ? 0u : l >> p & 1u;
                constexpr uint32_t kChild = SET & ~(1u << j);
                lanes::vertex<ROW, j == kFirst>(block(s, j, b), value_of<kChild, child, R, N, M>(from[kChild]), to[l]);
            });
        }
    });
}

// The other half of a set without the last photon: label l of this lane is label
// ~l of the partner.
template <uint32_t SET, typename R, int N, int M>
__device__ __forceinline__ void complete(Quad<R> (&v)[M])
{
    if constexpr ((SET >> (N - 1) & 1u) == 0u) {
        constexpr int kBits = __builtin_popcount(SET);
        constexpr uint32_t kAll = (1u << kBits) - 1u;
        static_for<0, (1 << (kBits - 1))>([&](auto li) {
            constexpr uint32_t l = 2u * decltype(li)::value + 1u;
            v[l] = from_partner(v[~l & kAll]);
        });
    }
}

// Values of all sets of up to LEVELS photons of one end (ROW: the u end).
template <int LEVELS, bool ROW, typename R, int N, int M>
__device__ __forceinline__ void build(const Point<R, N> &s, Quad<R> (&J)[1 << N][M])
{
    static_for<1, LEVELS + 1>([&](auto li) {
        constexpr int L = decltype(li)::value;
        for_each_subset<N, L>([&](auto mi) {
            constexpr uint32_t set = decltype(mi)::value;
            const Quad<R> P = propagator<ROW ? -1 : 1, set>(ROW ? s.p1 : s.q0, s);
            if constexpr (L == 1) {
                const Quad<R> v = s.v[__builtin_ctz(set)];
                if constexpr (!ROW)  // V (1, 0) = (1, gamma)
                    J[set][0] = {fma(-P.c, v.c, fma(P.d, v.d, P.a)), -fma(P.c, v.d, P.d * v.c), fma(P.b, v.c, -P.c),
                                 fma(P.b, v.d, P.d)};
                else  // (gamma, -1)
                    J[set][0] = {fma(v.c, P.a, P.c), fma(v.d, P.a, -P.d), -fma(v.c, P.c, fma(-v.d, P.d, P.b)),
                                 -fma(v.c, P.d, v.d * P.c)};
            } else {
                vertices<set, ROW, R, N, M>(s, J, J[set]);
                constexpr bool kWhole = (set >> (N - 1) & 1u) != 0u;
                constexpr int kLabels = 1 << __builtin_popcount(set & ~(1u << (N - 1)));
#pragma unroll
                for (int l = 0; l < kLabels; l += kWhole ? 1 : 2) J[set][l] = lanes::propagated<ROW>(P, J[set][l]);
            }
        });
    });
}

// |ordering sum|^2 over the lane's 2^(n-1) configurations.
template <typename R, int N>
__device__ __forceinline__ double pair_sum(const Point<R, N> &s)
{
    constexpr int K = (N + 1) / 2, U = N - K, C = 1 << (N - 1);
    constexpr int MJ = 1 << K, MW = 1 << U;
    constexpr uint32_t kAll = (1u << N) - 1u, kLast = 1u << (N - 1);
    Quad<R> J[1 << N][MJ], W[1 << N][MW];
    build<K - 1, false>(s, J);
    build<U - 1, true>(s, W);
    double re[C], im[C];
#pragma unroll
    for (int h = 0; h < C; ++h) re[h] = im[h] = 0.0;
    // From the highest set down: the sets with the last photon come first, so that the
    // currents only they read are dead for the rest and fewer registers spill (FP32 53
    // -> 35, FP64 110 -> 94 at n = 5; from the lowest up FP32 1e6 points 345 us, 312 so).
    constexpr int kSets = binomial(N, K);
    static_for<0, kSets>([&](auto si) {
        constexpr uint32_t A = nth_subset(K, kSets - 1 - decltype(si)::value), B = kAll & ~A;
        Quad<R> j[MJ], w[MW];
        vertices<A, false, R, N, MJ>(s, J, j);
        const Quad<R> P = propagator<1, A>(s.q0, s);
        constexpr int kStep = (A & kLast) != 0u ? 1 : 2;
#pragma unroll
        for (int l = 0; l < 1 << __builtin_popcount(A & ~kLast); l += kStep) j[l] = lanes::propagated<false>(P, j[l]);
        complete<A, R, N, MJ>(j);
        vertices<B, true, R, N, MW>(s, W, w);
        complete<B, R, N, MW>(w);
        static_for<0, C>([&](auto hi) {
            constexpr int h = decltype(hi)::value;
            lanes::add_product(w[labels_of(h, B & ~kLast)], j[labels_of(h, A & ~kLast)], re[h], im[h]);
        });
    });
    double total = 0.0;
#pragma unroll
    for (int h = 0; h < C; ++h) total += re[h] * re[h] + im[h] * im[h];
    return total;
}

// |M|^2 of one point per pair of lanes, in both of them.
template <typename R, int N, bool BEAM>
__device__ __forceinline__ double pair_value(const PointLoad<N, BEAM> &q, double coef, bool odd)
{
    double E1 = q.x[0], p1x = 0.0, p1y = 0.0, p1z = E1, E2 = E1, p2x = 0.0, p2y = 0.0, p2z = -E1;
    if constexpr (!BEAM) {
        p1x = q.x[1], p1y = q.x[2], p1z = q.x[3];
        E2 = q.x[4], p2x = q.x[5], p2y = q.x[6], p2z = q.x[7];
    }
    bool ok = p1x == 0.0 && p1y == 0.0 && p1z > 0.0 && p2x == 0.0 && p2y == 0.0 && p2z < 0.0;
    int m = 0;
    frexp(E1 + E2, &m);
    const double sc = ldexp(1.0, -m);
    const double norm = ((E1 + p1z) * sc) * (2.0 * E2 * sc);
    Point<R, N> s;
    s.q0 = {static_cast<R>(-(E2 + p2z) * sc), static_cast<R>(-(E2 - p2z) * sc), R(0), R(0), R(0), R(0)};
    s.p1 = {static_cast<R>((E1 + p1z) * sc), static_cast<R>((E1 - p1z) * sc), R(0), R(0), R(0), R(0)};
    double norm_den = 1.0;
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const int r = kBeamRows<BEAM> + 4 * j;
        const double E = q.x[r] * sc, kx = q.x[r + 1] * sc, ky = q.x[r + 2] * sc, kz = q.x[r + 3] * sc;
        const double pt2 = kx * kx + ky * ky;
        ok = ok && E > 0.0 && pt2 > 0.0;
        const double big = E + fabs(kz);
        R small, ip, im;
        if constexpr (std::is_same<R, float>::value)
            small = static_cast<float>(pt2) * __builtin_amdgcn_rcpf(static_cast<float>(big));
        else
            small = pt2 / big;
        const R kp = kz >= 0.0 ? static_cast<R>(big) : small;
        const R km = kz >= 0.0 ? small : static_cast<R>(big);
        if constexpr (std::is_same<R, float>::value) {
            ip = __builtin_amdgcn_rcpf(kp);
            im = __builtin_amdgcn_rcpf(km);
        } else {
            ip = 1.0 / kp;
            im = 1.0 / km;
        }
        norm_den *= 2.0 * E * E / pt2;
        const R fx = static_cast<R>(kx), fy = static_cast<R>(ky);
        s.k[j] = {kp, km, fx, fy, ip, im};
        // block of helicity -, or + in the odd lane
        const R xp = fx * ip, yp = fy * ip, xm = fx * im, ym = fy * im;
        s.v[j] = {odd ? -xm : xp, odd ? -ym : yp, odd ? xp : -xm, odd ? -yp : ym};
    }
    double sum = pair_sum<R, N>(s);
    sum += from_partner(sum);
    const double me2 = ldexp(coef * (norm / norm_den) * sum, 2 * m * (2 - N));
    return ok ? me2 : __builtin_nan("");
}

// One tile of 64 points per wave; arguments as me2_kernel's (one chunk).
template <typename R, int N, int WPE, bool BEAM>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(WPE)))
me2_pair_kernel(const double *__restrict__ mom, int64_t ld, const int32_t *__restrict__ index,
                const uint16_t *__restrict__, const int64_t *__restrict__ d_count, int64_t count, int,
                double coef, double *__restrict__ out, int64_t, const double *__restrict__ wfac,
                double *__restrict__ partials, double *__restrict__ wout, unsigned *__restrict__ flags)
{
    const int lane = threadIdx.x;
    const int64_t npts = d_count ? *d_count : count;
    const int64_t ntiles = (npts + 63) >> 6;
    int64_t tile = blockIdx.x;
    // one contiguous range of tiles per XCD, as me2_kernel
    constexpr unsigned kXcds = 8;
    if (gridDim.x % kXcds == 0) {
        const int64_t per = (ntiles + kXcds - 1) / kXcds;
        if (blockIdx.x / kXcds >= per) return;
        tile = blockIdx.x % kXcds * per + blockIdx.x / kXcds;
    }
    if (tile >= ntiles) return;
    const double *wf = partials ? wfac : nullptr;
    // column of this pair's point of a half tile (past the last point: that again)
    auto column = [&](int half) -> uint32_t {
        const int64_t i = tile * 64 + half * 32 + (lane >> 1), ic = i < npts ? i : npts - 1;
        return index ? static_cast<uint32_t>(index[ic]) : static_cast<uint32_t>(ic);
    };
    uint32_t src = column(0);
    double value = 0.0, weight = 0.0;  // of point `lane` of the tile
#pragma unroll 1
    for (int half = 0; half < 2; ++half) {
        // row addresses formed here, not held across the halves
        int64_t rows = ld;
        asm volatile("" : "+s"(rows));
        const PointLoad<N, BEAM> q = load_point<N, BEAM>(mom, rows, src, wf, nullptr);
        src = column(1);
        const double me2 = pair_value<R, N, BEAM>(q, coef, lane & 1);
        const double mine = __shfl(me2, 2 * (lane & 31), 64), factor = __shfl(q.wf, 2 * (lane & 31), 64);
        if (lane >> 5 == half) {
            value = mine;
            weight = mine * factor;
        }
    }
    const int64_t i = tile * 64 + lane;
    const bool valid = i < npts;
    if (partials) {
        const double w = valid ? weight : 0.0;
        if (!isfinite(w)) atomicOr(flags, 1u);
        if (wout && valid) wout[i] = w;
        tile_partial(w, lane, partials, tile);
    } else if (valid) {
        if (!isfinite(value)) atomicOr(flags, 1u);
        out[i] = value;
    }
}

}  // namespace pairs
}  // namespace heget
