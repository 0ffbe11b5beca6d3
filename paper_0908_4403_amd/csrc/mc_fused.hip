// Cross section of small n in one pass over the points: generation, cuts,
// |M|^2, weight and the block's partial sums in one kernel, one lane per
// generated point.  Helicity sums up to n = 4, sampled helicities up to n = 5.
//
// For these the amplitude is no longer than the generation by much (300, 1220
// and 4388 operations for n = 2, 3, 4), and apart from it it was bound by
// writing and gathering the momenta (32 (n + 2) + 13 bytes a point) and by the
// launches, which become two.  Lanes of rejected points compute |M|^2 for
// nothing (1 to 40% of them).  Time of the whole path, FP32, before -> fused: n
// = 2, 16 384 points 17.6 -> 11.6 us, 4 194 304 points 285 -> 115 us; n = 3 18
// -> 12.5 and 352 -> 200; n = 4 23 -> 17 and 519 -> 488 (1 048 576 points at
// sqrt(shat) = 700 GeV 137 -> 130; pp, where a third is cut, 135 -> 138);
// sampled n = 4 424 -> 246, n = 5 1 048 576 points 130 -> 120 (FP64 152 -> 141).
// With the generation's tables since: n = 2, 4 194 304 points 108, n = 4, 1 048 576
// points 125; sampled n = 5 111 (FP64 135).
// Bound by VALU issue of FP64 and integer instructions, as gen_kernel.
#include <hip/hip_runtime.h>
#include <math.h>

#include <type_traits>

#include "kernels.hpp"
#include "me2_item.hpp"

namespace heget {

// Points up to which the FP64 n = 4 sum runs fused: its walk of sixteen
// configurations leaves one wave per SIMD, which the generation in the same
// kernel then has too (300 007 points 81 apart, 73 fused, 399 999 96 and 90,
// 500 003 106 and 104, 600 003 115 and 121, 1e6 160 and 185).
constexpr int64_t kFusedWide = 400000;

// partials[3 b ..]: (sum, compensation, sum of squares) of block b's 256
// weights; block_acc[b]: its accepted points, kBlockNonfinite added if one of
// their weights is not finite.  H = 0: the drawn helicity configuration.  The
// walk (unrolled n, closing, meeting in the middle) is that of the amplitude
// kernel's default, but for n = 2 and FP64 n = 3 of all helicities at once, not half
// of them.  FP32 and sampled points have the same bits in both; in FP64 sums the
// compiler contracts products differently (up to 2e-14 of a point).
// FP64 n = 5 is held to two waves per SIMD: a few spills cost less than the
// generation at one (300 007 points 62 -> 52 us, 49 with its tables); n = 4 with
// sixteen walks is not (62 -> 80 us).
template <typename R, int N, int MODE, int H>
__global__ void __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(N == 5 && std::is_same<R, double>::value ? 2 : 1)))
fused_kernel(GenParams g, double coef, double *__restrict__ partials, int32_t *__restrict__ block_acc,
             double *__restrict__ wout, double *__restrict__ xout, int observable)
{
    constexpr int CL = N == 2 && H > 0 && std::is_same<R, float>::value ? 1 : N == 4 ? 3 : 2;
    constexpr int PS = N >= 5 ? 2 : 0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    __shared__ fm::PhotonTables tab;
    load_photon_tables(tab);
    clear_bins(g);
    __syncthreads();
    bool acc = false;
    double w = 0.0;
    if (i < g.npoints) {
        const uint64_t point = static_cast<uint64_t>(g.first + i);
        Vec4 k[N];
        double e, wf, y;
        int s = point_setup_screened<N, MODE>(g, point, tab, k, e, wf, y);
        if (s < 0) s = pass_cuts_fp64<N>(k, y, g.pt_min, g.eta_max, g.dr_min) ? 1 : 0;
        acc = s == 1;
        PointLoad<N> q;
        const double beams[8] = {e, 0.0, 0.0, e, e, 0.0, 0.0, -e};
#pragma unroll
        for (int r = 0; r < 8; ++r) q.x[r] = beams[r];
#pragma unroll
        for (int j = 0; j < N; ++j) {
            q.x[8 + 4 * j] = k[j].e;
            q.x[9 + 4 * j] = k[j].x;
            q.x[10 + 4 * j] = k[j].y;
            q.x[11 + 4 * j] = k[j].z;
        }
        q.wf = wf;
        q.hel = H == 0 ? static_cast<uint32_t>(draw_helicity<N>(g.seed, point)) : 0u;
        const double me2 = me2_value<R, N, N, H, CL, PS>(q, 0, 1, coef, static_cast<R *>(nullptr), lane);
        w = acc ? me2 * wf : 0.0;
        if (wout) wout[i] = w;
        if (xout)
            xout[i] = observable == 0 ? event_observable<N, 0>(k) : event_observable<N, 1>(k);
    }
    CSum cs{w, 0.0};
    double sq = w * w;
    wave_reduce(cs, sq);
    __shared__ double part[3][4];
    if (lane == 0) {
        part[0][wave] = cs.s;
        part[1][wave] = cs.c;
        part[2][wave] = sq;
    }
    const int count = __syncthreads_count(acc ? 1 : 0);
    const int bad = __syncthreads_or(acc && !isfinite(w) ? 1 : 0);
    if (threadIdx.x != 0) return;
    for (int v = 1; v < 4; ++v) {
        cs = csum_add(cs, CSum{part[0][v], part[1][v]});
        sq += part[2][v];
    }
    const int64_t b = blockIdx.x;
    partials[3 * b + 0] = cs.s;
    partials[3 * b + 1] = cs.c;
    partials[3 * b + 2] = sq;
    block_acc[b] = count + (bad ? kBlockNonfinite : 0);
}

struct FusedOut {
    double coef, *partials;
    int32_t *block_acc;
    double *wout, *xout;
    int observable;
};

template <typename R, int N, int H>
static hipError_t fused_n(const GenParams &g, const FusedOut &o, hipStream_t s)
{
    const int64_t blocks = (g.npoints + 255) / 256;
    if (blocks == 0) return hipSuccess;
    const auto kern = g.mode == 1 ? fused_kernel<R, N, 1, H> : g.mode == 2 ? fused_kernel<R, N, 2, H>
                                                                           : fused_kernel<R, N, 0, H>;
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, g, o.coef, o.partials,
                       o.block_acc, o.wout, o.xout, o.observable);
    return hipGetLastError();
}

template <typename R>
static hipError_t fused(int n, bool sampled, const GenParams &g, const FusedOut &o, hipStream_t s)
{
    switch (n) {
    case 2: return sampled ? fused_n<R, 2, 0>(g, o, s) : fused_n<R, 2, 4>(g, o, s);
    case 3: return sampled ? fused_n<R, 3, 0>(g, o, s) : fused_n<R, 3, 8>(g, o, s);
    case 4: return sampled ? fused_n<R, 4, 0>(g, o, s) : fused_n<R, 4, 16>(g, o, s);
    case 5: return sampled ? fused_n<R, 5, 0>(g, o, s) : hipErrorInvalidValue;
    default: return hipErrorInvalidValue;
    }
}

bool has_fused(int n, int prec, bool sampled, int64_t points)
{
    if (n > (sampled ? 5 : 4)) return false;
    return prec == 1 || n != 4 || sampled || points <= kFusedWide;
}

hipError_t launch_fused(int n, int prec, bool sampled, const GenParams &g, double coef, double *partials,
                        int32_t *block_acc, double *wout, double *xout, int observable, hipStream_t stream)
{
    const FusedOut o{coef, partials, block_acc, wout, xout, observable};
    return prec == 1 ? fused<float>(n, sampled, g, o, stream) : fused<double>(n, sampled, g, o, stream);
}

}  // namespace heget
