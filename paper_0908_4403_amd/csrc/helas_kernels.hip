// Batch kernels over the HELAS device library (helas.hpp):
//  * helas_eval_kernel: one library function on independent records, one
//    lane per record (FP64 records in and out; the arithmetic in FP32 or FP64);
//  * me2_frame_kernel: helicity-summed |M|^2 of u(p1) ubar(p2) -> n photons for
//    momenta in any frame, one lane per point.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>

#include "helas.hpp"
#include "kernels.hpp"
#include "me2_tree.hpp"

namespace heget {
namespace {

using helas::Cx;
using helas::Wave;

// record layouts: a wavefunction is 12 doubles (re, im of four components,
// then the momentum along the flow)
template <typename R>
__device__ inline Wave<R> load_wave(const double *x)
{
    Wave<R> w;
#pragma unroll
    for (int m = 0; m < 4; ++m) w.c[m] = helas::cx(R(x[2 * m]), R(x[2 * m + 1]));
#pragma unroll
    for (int m = 0; m < 4; ++m) w.p[m] = R(x[8 + m]);
    return w;
}

template <typename R>
__device__ inline void store_wave(const Wave<R> &w, double *y)
{
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        y[2 * m] = double(w.c[m].re);
        y[2 * m + 1] = double(w.c[m].im);
    }
#pragma unroll
    for (int m = 0; m < 4; ++m) y[8 + m] = double(w.p[m]);
}

template <typename R>
__global__ __launch_bounds__(256) void helas_eval_kernel(int func, int64_t count,
                                                         const double *__restrict__ in,
                                                         double *__restrict__ out)
{
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= count) return;
    const double *x = in + i * helas_in_size(func);
    double *y = out + i * helas_out_size(func);
    if (func <= kHelasVxxxx2) {
        const R p[4] = {R(x[0]), R(x[1]), R(x[2]), R(x[3])};
        const int nhel = int(x[4]), nsf = int(x[5]);
        Wave<R> w;
        switch (func) {
        case kHelasIxxxx0: w = helas::ixxxx0(p, nhel, nsf); break;
        case kHelasIxxxx1: w = helas::ixxxx1(p, nhel, nsf); break;
        case kHelasIxxxx2: w = helas::ixxxx2(p, nhel, nsf); break;
        case kHelasOxxxx0: w = helas::oxxxx0(p, nhel, nsf); break;
        case kHelasOxxxx1: w = helas::oxxxx1(p, nhel, nsf); break;
        case kHelasOxxxx2: w = helas::oxxxx2(p, nhel, nsf); break;
        case kHelasVxxxx0: w = helas::vxxxx0(p, nhel, nsf); break;
        case kHelasVxxxx1: w = helas::vxxxx1(p, nhel); break;
        default: w = helas::vxxxx2(p, nhel); break;
        }
        store_wave(w, y);
        return;
    }
    if (func == kHelasIovxxx) {
        const Cx<R> v = helas::iovxxx(load_wave<R>(x), load_wave<R>(x + 12), load_wave<R>(x + 24),
                                      R(x[36]), R(x[37]));
        y[0] = double(v.re);
        y[1] = double(v.im);
        return;
    }
    const Wave<R> a = load_wave<R>(x), b = load_wave<R>(x + 12);
    const R g0 = R(x[24]), g1 = R(x[25]);
    Wave<R> w;
    if (func == kHelasFvixx0) w = helas::fvixx0(a, b, g0, g1);
    else if (func == kHelasFvoxx0) w = helas::fvoxx0(a, b, g0, g1);
    else w = helas::jioxx0(a, b, g0, g1);
    store_wave(w, y);
}

// ---- |M|^2 for momenta in any frame
//
// The helicity sum is a Lorentz invariant, so a point is evaluated in the
// frame where u moves along +z and ubar along -z with the same energy, by the
// subset currents of the amplitude kernels (me2_tree.hpp).  That frame's
// light-cone momenta are spinor products of the given ones: with the Weyl
// spinor lam(p) = (sqrt(p+), (px + i py) / sqrt(p+)) of ixxxx0, <pq> = lam_0(p)
// lam_1(q) - lam_1(p) lam_0(q), |<pq>|^2 = 2 p.q,
//     sqrt(s) = |<12>|,  k- = |<1k>|^2 / sqrt(s),  k+ = |<2k>|^2 / sqrt(s),
//     kx + i ky = <1k> conj(<2k>) / sqrt(s)
// up to a rotation about z common to all photons and a reflection, which the
// sum does not see.  A spinor product loses accuracy only where its two
// momenta are nearly collinear, where the amplitude itself does; a photon
// along an axis of the given frame is nothing special.  Formed in FP64 for
// both precisions.
struct Spinor {
    double a, re, im;  // lam_0 (real) and lam_1
};

__device__ inline Spinor spinor(const double p[4])
{
    const double pp = helas::light_cone_plus(p);
    if (!(pp > 0.0)) return {0.0, sqrt(2.0 * p[0]), 0.0};  // along -z
    const double s = sqrt(pp), r = 1.0 / s;
    return {s, p[1] * r, p[2] * r};
}

__device__ inline Cx<double> product(const Spinor &p, const Spinor &q)
{
    return helas::cx(p.a * q.re - q.a * p.re, p.a * q.im - q.a * p.im);
}

// W waves per workgroup share a tile of 64 points (one per lane), each taking
// its part of the helicity walks of H configurations; their sums meet in LDS
// in wave order.  W = 1 does not repeat the set-up, W = 4 fills the chip and
// shortens the walk of a wave where tiles are few.
// Bound by VALU issue from some 1e5 points on, below that by one wave's
// latency.  Time, with the chains over all orderings of 4-spinors for both
// quark helicities that this replaces -> now: 20 011 points n = 4 FP64 564 ->
// 9.9 us, n = 5 FP64 5600 -> 37 us, n = 5 FP32 5160 -> 25 us; 200 003 points
// n = 3 FP64 159 -> 18 us, n = 4 FP32 997 -> 31 us, n = 5 FP64 22.5 -> 0.21
// ms; n = 2 is bound by the launch on both.  Errors against 64-bit values are
// no larger (median at n = 4 2.2e-15 -> 2.0e-15 in FP64, 7.9e-7 -> 1.1e-7 in
// FP32; at a boost of gamma = 20 1.5e-12 -> 9e-15 and 8e-4 -> 1.1e-7).
template <typename R, int N, int H, int CL, int PS, int W>
__global__ __launch_bounds__(64 * W) void me2_frame_kernel(const double *__restrict__ mom, int64_t ld,
                                                           int64_t np, double coef,
                                                           double *__restrict__ out,
                                                           unsigned *__restrict__ flags)
{
    constexpr int kPasses = (1 << N) / H;
    static_assert(kPasses % W == 0, "every wave takes the same number of walks");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t i = int64_t(blockIdx.x) * 64 + lane;
    const int64_t c = i < np ? i : np - 1;  // lanes past the last point repeat it and store nothing
    int ex = 0;
    frexp(mom[c] + mom[4 * ld + c], &ex);
    // scaled by ldexp: 2^-ex itself overflows for energies below 2^-1024
    auto load = [&](int particle) {
        double p[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) p[m] = ldexp(mom[(4 * particle + m) * ld + c], -ex);
        return spinor(p);
    };
    const Spinor l1 = load(0), l2 = load(1);
    const Cx<double> p12 = product(l1, l2);
    const double s = p12.re * p12.re + p12.im * p12.im, rs = sqrt(s), inv = 1.0 / rs;
    PointIn<R, N> in;
    in.q0 = {R(0), R(-rs), R(0), R(0), R(0), R(0)};
    in.p1 = {R(rs), R(0), R(0), R(0), R(0), R(0)};
    double den = 1.0;  // product of the photons' 2 E^2 / pT^2
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const Spinor k = load(j + 2);
        const Cx<double> u = product(l1, k), v = product(l2, k);
        const double km = (u.re * u.re + u.im * u.im) * inv, kp = (v.re * v.re + v.im * v.im) * inv;
        const Cx<double> t = u * helas::conj(v);
        in.k[j] = {R(kp), R(km), R(t.re * inv), R(t.im * inv), R(1.0 / kp), R(1.0 / km)};
        den *= 0.5 * (kp + km) * (kp + km) / (kp * km);
    }
    constexpr int ppw = kPasses / W;
    double sum = tree_sum<R, N, N, H, CL, PS>(in, static_cast<R *>(nullptr), lane, wave * ppw, (wave + 1) * ppw);
    if constexpr (W > 1) {
        __shared__ double part[W][64];
        part[wave][lane] = sum;
        __syncthreads();
        if (wave != 0) return;
#pragma unroll
        for (int w = 1; w < W; ++w) sum += part[w][lane];
    }
    if (i >= np) return;
    // |u|^2 |vbar|^2 = s; 2: the other quark pair is the mirror image
    const double r = ldexp(2.0 * coef * (s / den) * sum, 2 * ex * (2 - N));
    out[i] = r;
    if (!isfinite(r)) atomicOr(flags, 1u);
}

// Tiles up to which the walks of a point are split over four waves.  Four waves a
// tile fill the 1024 SIMDs of 256 CUs at 256 tiles, and at one wave per SIMD (278 to
// 498 registers in FP64, 372 in FP32 at n = 5) any more wait for a second round: at
// n = 4 that is longer than the undivided walk, at n = 5 two rounds are still shorter.
// us, four waves and one: n = 4 FP64 16 384 points 8.2 and 9.7, 20 011 12.8 and 9.9,
// 131 072 45 and 19; FP32 16 384 8.8 and 9.4, 20 011 10.7 and 9.6; n = 5 FP64 16 384 21
// and 47, 32 768 40 and 52, 65 536 75 and 61; FP32 32 768 26 and 30, 65 536 49 and 32.
template <int N>
constexpr int64_t kFrameSplitTiles = N >= 5 ? 512 : 256;

template <typename R, int N, int H, int CL, int PS, int HS>
hipError_t launch_frame_n(int64_t np, const double *mom, int64_t ld, double coef, double *out,
                          unsigned *flags, hipStream_t s)
{
    const int64_t tiles = (np + 63) / 64;
    constexpr int W = (1 << N) / HS >= 4 ? 4 : 1;  // n = 2, 3 have too few walks to split
    if constexpr (W > 1) {
        if (tiles <= kFrameSplitTiles<N>) {
            hipLaunchKernelGGL((me2_frame_kernel<R, N, HS, CL, PS, W>), dim3(unsigned(tiles)), dim3(64 * W), 0, s,
                               mom, ld, np, coef, out, flags);
            return hipGetLastError();
        }
    }
    hipLaunchKernelGGL((me2_frame_kernel<R, N, H, CL, PS, 1>), dim3(unsigned(tiles)), dim3(64), 0, s, mom, ld, np,
                       coef, out, flags);
    return hipGetLastError();
}

// The walk shapes (helicities per walk, closing, prefix sets; helicities per
// walk where four waves share a point) follow the amplitude kernel's defaults,
// but for n = 5 FP32, where all 32 helicities per walk spill here (200 003
// points 154 us, eight per walk 132).
template <typename R>
hipError_t launch_frame(int n, int64_t np, const double *mom, int64_t ld, double coef, double *out,
                        unsigned *flags, hipStream_t s)
{
    constexpr bool f32 = std::is_same<R, float>::value;
    switch (n) {
    case 2: return launch_frame_n<R, 2, 2, 2, 0, 2>(np, mom, ld, coef, out, flags, s);
    case 3: return launch_frame_n<R, 3, f32 ? 8 : 4, 2, 0, 4>(np, mom, ld, coef, out, flags, s);
    case 4: return launch_frame_n<R, 4, 16, 3, 0, 4>(np, mom, ld, coef, out, flags, s);
    case 5: return launch_frame_n<R, 5, 8, 2, f32 ? 2 : 3, f32 ? 8 : 4>(np, mom, ld, coef, out, flags, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_helas(int func, int prec, int64_t count, const double *in, double *out,
                        hipStream_t s)
{
    if (count <= 0) return hipSuccess;
    const unsigned blocks = unsigned((count + 255) / 256);
    if (prec == 0)
        hipLaunchKernelGGL(helas_eval_kernel<double>, dim3(blocks), dim3(256), 0, s, func, count, in, out);
    else
        hipLaunchKernelGGL(helas_eval_kernel<float>, dim3(blocks), dim3(256), 0, s, func, count, in, out);
    return hipGetLastError();
}

hipError_t launch_me2_frame(int n, int prec, int64_t np, const double *mom, int64_t ld, double coef,
                            double *out, unsigned *flags, hipStream_t s)
{
    if (np <= 0) return hipSuccess;
    return prec == 0 ? launch_frame<double>(n, np, mom, ld, coef, out, flags, s)
                     : launch_frame<float>(n, np, mom, ld, coef, out, flags, s);
}

}  // namespace heget
