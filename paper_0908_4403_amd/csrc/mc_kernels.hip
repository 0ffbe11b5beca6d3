// Monte-Carlo side of the path: phase-space generation with cuts, stream
// compaction of the surviving points into an index list; per-point weights of
// eq. (1)-(2) are applied in the amplitude pass; a deterministic compensated
// reduction gives sigma and its error.  All FP64.
//
// Determinism: compaction keeps point order (block counts -> each block's
// offset, the sum of its predecessors' counts -> in-block ballot ranks), and
// every sum is a fixed tree (64-point tiles by a fixed tree of cross-lane
// moves, tiles in index order), so a configuration gives bitwise the same
// sigma on every run.
#include <hip/hip_runtime.h>
#include <math.h>

#include "kernels.hpp"
#include "reduce.hpp"

namespace heget {

// SoA rows of one point: quark momenta (E, 0, 0, +-E), then the photons; with
// `beam` only E for the quarks: 21 rows instead of 28 at n = 5, for this kernel
// and for the gathering reads of the next (hadronic n = 5 of 4.2e6 points 217 ->
// 209 us here and 913 -> 885 in the amplitude kernel, which also needs fewer
// registers; FP64 n = 4 of 1e6 points 45 -> 43 and 108 -> 106).  The row of the workgroup's first point is uniform (scalar
// address arithmetic), a lane adds its place in the workgroup.
template <int N>
__device__ __forceinline__ void store_point(double *__restrict__ mom, int64_t ld, bool beam, double e,
                                            const Vec4 (&k)[N])
{
    double *block = mom + static_cast<int64_t>(blockIdx.x) * 256;
    const uint32_t t = threadIdx.x;
    block[t] = e;
    if (!beam) {
        const double rest[7] = {0.0, 0.0, e, e, 0.0, 0.0, -e};
#pragma unroll
        for (int r = 0; r < 7; ++r) {
            block += ld;
            block[t] = rest[r];
        }
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const double v[4] = {k[j].e, k[j].x, k[j].y, k[j].z};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            block += ld;
            block[t] = v[c];
        }
    }
}

// Every point, in point order; rejected points keep their momenta, weight 0.
// Optionally the accept flag per point and the accept count per block of 256.
template <int N, int MODE>
__global__ void __launch_bounds__(256)
gen_kernel(GenParams g, double *__restrict__ mom, int64_t ld, double *__restrict__ wout,
           uint8_t *__restrict__ flag, int32_t *__restrict__ block_count)
{
    __shared__ fm::PhotonTables tab;
    load_photon_tables(tab);
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (g.clear_word && i == 0) *g.clear_word = 0u;
    clear_bins(g);
    __syncthreads();
    bool acc = false;
    if (i < g.npoints) {
        double w, y;
        int s;
        {
            Vec4 k[N];
            double e;
            s = point_setup_screened<N, MODE>(g, static_cast<uint64_t>(g.first + i), tab, k, e, w, y);
            store_point<N>(mom, ld, g.beam, e, k);
        }
        if (s < 0) {
            // Rare: decide in FP64 from the momenta just stored.  The row
            // pointer is passed through an empty asm statement so that the
            // compiler reloads them instead of keeping every momentum live
            // through the whole kernel (which costs two waves per SIMD).
            __threadfence_block();  // this thread's stores above are visible to its loads
            const double *m = mom + (g.beam ? 1 : 8) * ld + i;
            asm volatile("" : "+v"(m));
            Vec4 k[N];
#pragma unroll
            for (int j = 0; j < N; ++j)
                k[j] = {m[4 * j * ld], m[(4 * j + 1) * ld], m[(4 * j + 2) * ld], m[(4 * j + 3) * ld]};
            s = pass_cuts_fp64<N>(k, y, g.pt_min, g.eta_max, g.dr_min) ? 1 : 0;
        }
        acc = s == 1;
        wout[i] = acc ? w : 0.0;
        if (flag) flag[i] = acc ? 1 : 0;
        if (g.hel_out) g.hel_out[i] = draw_helicity<N>(g.seed, static_cast<uint64_t>(g.first + i));
    }
    if (block_count) {
        const int c = __syncthreads_count(acc ? 1 : 0);
        if (threadIdx.x == 0) block_count[blockIdx.x] = c;
    }
}

// Exclusive prefix sums of the nb per-block counts, in place, and their total
// into *d_count: one workgroup of 1024 threads walks the counts in chunks of
// 4096 (four consecutive counts per thread), carrying the running total.
// Used for large point counts, where the blocks of compact_kernel would
// otherwise each sum all their predecessors' counts (work growing as nb^2).
constexpr int kScanThreads = 1024;

__global__ void __launch_bounds__(kScanThreads)
block_scan_kernel(int32_t *__restrict__ counts, int nb, int64_t *__restrict__ d_count)
{
    __shared__ int wave_tot[kScanThreads / 64];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    int64_t carry = 0;
    for (int base = 0; base < nb; base += 4 * kScanThreads) {
        int v[4], own = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int idx = base + 4 * t + j;
            v[j] = idx < nb ? counts[idx] : 0;
            own += v[j];
        }
        // inclusive scan of `own` over the wave, then over the waves
        int inc = own;
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) {
            const int up = __shfl_up(inc, m, 64);
            if (lane >= m) inc += up;
        }
        if (lane == 63) wave_tot[w] = inc;
        __syncthreads();
        int before = 0, chunk = 0;
        for (int k = 0; k < kScanThreads / 64; ++k) {
            if (k < w) before += wave_tot[k];
            chunk += wave_tot[k];
        }
        int run = static_cast<int>(carry) + before + inc - own;  // offsets stay below 2^31
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int idx = base + 4 * t + j;
            if (idx < nb) counts[idx] = run;
            run += v[j];
        }
        carry += chunk;
        __syncthreads();  // wave_tot is rewritten by the next chunk
    }
    if (t == 0) *d_count = carry;
}

// Survivor list: index[offset_b + rank] = point, in point order, where block b
// (256 points) takes offset_b, the survivors of blocks 0..b-1, from `counts`
// already scanned into offsets (scanned = 1, block_scan_kernel wrote
// *d_count), or sums its predecessors' counts itself (a few KiB of
// L2-resident reads per block at the sizes this is used for, so no separate
// scan pass; the last block writes the total to *d_count).
__global__ void __launch_bounds__(256)
compact_kernel(const uint8_t *__restrict__ flag, int64_t np, const int32_t *__restrict__ counts,
               int nb, int scanned, int32_t *__restrict__ index, int64_t *__restrict__ d_count)
{
    __shared__ int part[4];
    __shared__ int wave_count[4];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int b = static_cast<int>(blockIdx.x);
    int s = 0;
    if (scanned) {
        s = t == 0 ? counts[b] : 0;
    } else {
        // the counts of blocks 0..b-1, four per 16-byte load (the count
        // buffer is 256-byte aligned), loads batched so their latencies overlap
        const int4 *c4 = reinterpret_cast<const int4 *>(counts);
        const int nfull = b >> 2;
#pragma unroll 4
        for (int j = t; j < nfull; j += 256) {
            const int4 v = c4[j];
            s += (v.x + v.y) + (v.z + v.w);
        }
        if (t < b - (nfull << 2)) s += counts[(nfull << 2) + t];
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) s += __shfl_xor(s, m, 64);
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + t;
    const bool f = i < np && flag[i] != 0;
    const uint64_t bal = __ballot(f);
    const int rank = __popcll(bal & ((1ull << lane) - 1ull));
    if (lane == 0) {
        part[w] = s;
        wave_count[w] = __popcll(bal);
    }
    __syncthreads();
    const int offset = part[0] + part[1] + part[2] + part[3];
    int base = offset;
    for (int k = 0; k < w; ++k) base += wave_count[k];
    if (f) index[base + rank] = static_cast<int32_t>(i);
    if (!scanned && t == 0 && b == nb - 1)
        *d_count = offset + wave_count[0] + wave_count[1] + wave_count[2] + wave_count[3];
}

// ---------------------------------------------------------------- event records

// Per generated point of an events call: weight 0 (the survivors' weights
// are scattered in afterwards), the rapidity of the partonic frame in the lab,
// the helicity configuration drawn in sampling mode (bit layout of
// draw_helicity_raw).
template <int MODE>
__global__ void __launch_bounds__(256)
event_fill_kernel(GenParams g, int n, double *__restrict__ w_all, double *__restrict__ y_out,
                  uint16_t *__restrict__ hel_out)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i >= g.npoints) return;
    const uint64_t point = static_cast<uint64_t>(g.first + i);
    w_all[i] = 0.0;
    if (y_out) y_out[i] = point_kinematics<MODE>(g, point).y;
    if (hel_out) hel_out[i] = static_cast<uint16_t>(draw_helicity_raw(g.seed, point, n));
}

// Survivor weights back to point order: w_all[index[k]] = w[k], k < *d_count.
__global__ void __launch_bounds__(256)
event_scatter_kernel(const int32_t *__restrict__ index, const double *__restrict__ w,
                     const int64_t *__restrict__ d_count, int64_t max_count,
                     double *__restrict__ w_all)
{
    const int64_t k = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int64_t count = *d_count;
    if (k >= count || k >= max_count) return;
    w_all[index[k]] = w[k];
}

// ---------------------------------------------------------------- sums

__global__ void __launch_bounds__(256)
sum_chunks_kernel(const double *__restrict__ part, int nchunks, int64_t ld,
                  const int64_t *__restrict__ d_count, int64_t count, double *__restrict__ out,
                  const int32_t *__restrict__ index, const double *__restrict__ wfac,
                  double *__restrict__ partials, double *__restrict__ wout,
                  unsigned *__restrict__ flags)
{
    const int64_t k = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int64_t n = d_count ? *d_count : count;
    if (partials) {
        // whole waves stay for the tile reduction
        if ((k & ~int64_t(63)) >= n) return;
        double w = 0.0;
        if (k < n) {
            double s = 0.0;
            for (int c = 0; c < nchunks; ++c) s += part[c * ld + k];
            w = s * wfac[index ? static_cast<int64_t>(index[k]) : k];
            if (!isfinite(w)) atomicOr(flags, 1u);
            if (wout) wout[k] = w;
        }
        tile_partial(w, threadIdx.x & 63, partials, k >> 6);
        return;
    }
    if (k >= n) return;
    double s = 0.0;
    for (int c = 0; c < nchunks; ++c) s += part[c * ld + k];
    if (!isfinite(s)) atomicOr(flags, 1u);
    out[k] = s;
}

constexpr int kFinalThreads = 1024;
constexpr int kFinalBatch = 8;

// Block reduction of (sum, compensation, sum of squares) into thread 0.
__device__ __forceinline__ void block_reduce(CSum &cs, double &sq)
{
    constexpr int kWaves = kFinalThreads / 64;
    __shared__ double sh[3][kWaves];
    wave_reduce(cs, sq);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) {
        sh[0][w] = cs.s;
        sh[1][w] = cs.c;
        sh[2][w] = sq;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        cs = {sh[0][0], sh[1][0]};
        sq = sh[2][0];
        for (int q = 1; q < kWaves; ++q) {
            cs = csum_add(cs, CSum{sh[0][q], sh[1][q]});
            sq += sh[2][q];
        }
    }
}

// One block: thread t folds triples t, t + T, t + 2T, ... in that order (loads
// issued kFinalBatch at a time), then a fixed tree.  The record is {sigma,
// err, sum, comp, sum2 (double), n_gen, n_acc (int64)}, sigma = sum / n_gen
// and err^2 = (sum2/N - sigma^2)/(N - 1).  `host` (pinned host memory) receives
// res and the call's status flags: the host needs no copy after the kernel.
__global__ void __launch_bounds__(kFinalThreads)
final_kernel(const double *__restrict__ partials, const int64_t *__restrict__ d_count,
             const int32_t *__restrict__ block_acc, int64_t n_gen, double *__restrict__ res, void *record,
             const unsigned *__restrict__ flags, double *__restrict__ host)
{
    const int t = threadIdx.x;
    int64_t nacc, nt;
    unsigned status;
    if (block_acc) {
        // the blocks' accepted points and non-finite marks
        nt = (n_gen + 255) / 256;
        __shared__ int64_t wave_acc[kFinalThreads / 64];
        int64_t own = 0;
        int mark = 0;
        for (int64_t b = t; b < nt; b += kFinalThreads) {
            const int32_t v = block_acc[b];
            own += v & (kBlockNonfinite - 1);
            mark |= v & kBlockNonfinite;
        }
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) own += __shfl_xor(own, m, 64);
        if ((t & 63) == 0) wave_acc[t >> 6] = own;
        status = __syncthreads_or(mark) ? 1u : 0u;
        nacc = 0;
        for (int q = 0; q < kFinalThreads / 64; ++q) nacc += wave_acc[q];
    } else {
        nacc = *d_count;
        nt = (nacc + 63) / 64;
        status = flags ? *flags : 0u;
    }
    CSum cs{0.0, 0.0};
    double sq = 0.0;
    for (int64_t j0 = t; j0 < nt; j0 += int64_t(kFinalThreads) * kFinalBatch) {
        double v[kFinalBatch][3];
#pragma unroll
        for (int u = 0; u < kFinalBatch; ++u) {
            const int64_t j = j0 + int64_t(u) * kFinalThreads;
            const bool in = j < nt;
            v[u][0] = in ? partials[3 * j + 0] : 0.0;
            v[u][1] = in ? partials[3 * j + 1] : 0.0;
            v[u][2] = in ? partials[3 * j + 2] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < kFinalBatch; ++u) {
            cs = csum_add(cs, CSum{v[u][0], v[u][1]});
            sq += v[u][2];
        }
    }
    block_reduce(cs, sq);
    if (t != 0) return;
    const double sum = cs.s + cs.c;
    res[0] = sum;
    res[1] = cs.c;
    res[2] = sq;
    res[3] = static_cast<double>(nacc);
    if (host) {
        host[0] = sum;
        host[1] = cs.c;
        host[2] = sq;
        host[3] = static_cast<double>(nacc);
        host[4] = static_cast<double>(status);
    }
    if (record) {
        double *d = static_cast<double *>(record);
        int64_t *q = static_cast<int64_t *>(record);
        const double N = static_cast<double>(n_gen);
        const double sigma = n_gen > 0 ? sum / N : 0.0;
        const double var = n_gen > 1 ? (sq / N - sigma * sigma) / (N - 1.0) : 0.0;
        d[0] = sigma;
        d[1] = sqrt(var > 0.0 ? var : 0.0);
        d[2] = sum;
        d[3] = cs.c;
        d[4] = sq;
        q[5] = n_gen;
        q[6] = nacc;
    }
}

// ---------------------------------------------------------------- histograms

// Fixed-point exponent: every weight and every partial sum stays below 2^62.
__device__ __forceinline__ int hist_shift(const double *res)
{
    int e = 0;
    frexp(res[0], &e);  // sum of weights < 2^e
    return 62 - e;
}

// Bins of one workgroup, summed in LDS: four copies where the bins are few, so
// that fewer waves wait for each other at a bin.
constexpr int kHistSlots = kHistMaxBins + 2;

__device__ __forceinline__ void hist_add(unsigned long long *lb, double x, double wk, int shift, int nbins,
                                         double lo, double hi, double scale)
{
    if (!(wk > 0.0) || !isfinite(wk)) return;
    int b;
    if (x < lo) {
        b = 0;
    } else if (!(x < hi)) {
        b = nbins + 1;
    } else {
        b = 1 + static_cast<int>((x - lo) * scale);
        b = b > nbins ? nbins : b;
    }
    atomicAdd(&lb[b], static_cast<unsigned long long>(llrint(ldexp(wk, shift))));
}

// The histogram of the survivors' observable (N photons from mom through
// index, or N = 0: x and w per generated point, as the fused pass writes them).
// At most 128 workgroups (kHistBlocks): every one adds each of its bins to the same
// words in memory, one after the other (some 20 ns each).  The last one to
// finish (bins[nbins + 2] counts them) converts the sums to sum(w) / n_gen per
// bin into `hist`.  300 007 sampled n = 5 points, of which the fused pass left
// weight and observable: 7 us; 23 us when a workgroup of 256 took every 256
// survivors from their momenta, and 10 more for the conversion and the zeroing
// of the bins in kernels of their own.
//
// Delta R of gathered survivors is work (n logarithms, arctangents, n (n - 1) / 2
// roots): a workgroup for each CU, and from n = 6 half as many threads, which 128
// registers are too few for.  us, one kernel per 256 survivors -> 128 workgroups of
// 1024 -> this: pp n = 5 of 4.2e6 points 138 -> 217 -> 138, n = 5 of 1e6 57 -> 69 ->
// 44, FP64 n = 4 of 1e6 54 -> 59 -> 42, sampled n = 6, 7, 8 of 1e6 58 -> 75 -> 49, 59 -> 89
// -> 54, 59 -> 103 -> 58; n = 8 of 65 536 17 -> 31 -> 16.  The largest pT gains nothing by
// either (n = 5 of 1e6 22 and 22, FP64 n = 4 18 and 21).
template <int N, int WHICH>
constexpr bool kHistWork = N > 0 && WHICH == 1;
template <int N, int WHICH>
constexpr int kHistBlocks = kHistWork<N, WHICH> ? 256 : 128;
template <int N, int WHICH>
constexpr int kHistThreads = kHistWork<N, WHICH> && N >= 6 ? 512 : 1024;

template <int N, int WHICH>
__global__ void __launch_bounds__((kHistThreads<N, WHICH>))
hist_kernel(const double *__restrict__ mom, int64_t ld, const int32_t *__restrict__ index,
            const double *__restrict__ w, const int64_t *__restrict__ d_count, int64_t points,
            const double *__restrict__ res, int nbins, double lo, double hi, unsigned long long *bins,
            int64_t n_gen, double *__restrict__ hist)
{
    constexpr int kThreads = kHistThreads<N, WHICH>;
    __shared__ unsigned long long lb[kHistSlots];
    __shared__ int last;
    const int slots = nbins + 2;
    const int copies = slots * 4 <= kHistSlots ? 4 : 1;
    for (int b = threadIdx.x; b < slots * copies; b += kThreads) lb[b] = 0ull;
    __syncthreads();
    unsigned long long *mine = lb + (copies == 4 ? (threadIdx.x >> 6 & 3) * slots : 0);
    const int64_t count = N == 0 ? points : *d_count;
    const int shift = hist_shift(res);
    const double scale = static_cast<double>(nbins) / (hi - lo);
    for (int64_t k = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; k < count;
         k += static_cast<int64_t>(gridDim.x) * kThreads) {
        double x;
        if constexpr (N == 0) {
            x = mom[k];
        } else {
            const int64_t col = index[k];
            Vec4 p[N];
#pragma unroll
            for (int j = 0; j < N; ++j)
                p[j] = {0.0, mom[(9 + 4 * j) * ld + col], mom[(10 + 4 * j) * ld + col],
                        WHICH == 0 ? 0.0 : mom[(11 + 4 * j) * ld + col]};
            x = event_observable<N, WHICH>(p);
        }
        hist_add(mine, x, w[k], shift, nbins, lo, hi, scale);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < slots; b += kThreads) {
        unsigned long long v = lb[b];
        for (int c = 1; c < copies; ++c) v += lb[c * slots + b];
        if (v) __hip_atomic_fetch_add(&bins[b], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // Every wave waits until its own additions are done, then the barrier, then
    // thread 0 counts the workgroup in.  Neither of the two waits for them: the
    // barrier waits for no memory operation and thread 0's release for those of
    // its own wave.  (A fence by every thread took 20 us: each one writes back
    // the L2; the additions are done at memory and leave nothing in it.)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0)
        last = __hip_atomic_fetch_add(&bins[slots], 1ull, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) ==
               gridDim.x - 1u;
    __syncthreads();
    if (!last) return;
    for (int b = threadIdx.x; b < slots; b += kThreads) {
        const unsigned long long v = __hip_atomic_load(&bins[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        hist[b] = n_gen > 0 ? ldexp(static_cast<double>(v), -shift) / static_cast<double>(n_gen) : 0.0;
    }
}

__global__ void zero_u32_kernel(unsigned *p, int count)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0u;
}

// ---------------------------------------------------------------- launchers

template <int N>
static hipError_t gen_n(const GenParams &g, double *mom, int64_t ld, double *w, uint8_t *flag,
                        int32_t *block_count, hipStream_t stream)
{
    const int64_t blocks = (g.npoints + 255) / 256;
    if (blocks == 0) return hipSuccess;
    // one kernel per partonic mode: the fixed-energy one needs far fewer registers
    const auto kern = g.mode == 1 ? gen_kernel<N, 1> : g.mode == 2 ? gen_kernel<N, 2> : gen_kernel<N, 0>;
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, stream, g, mom, ld,
                       w, flag, block_count);
    return hipGetLastError();
}

hipError_t launch_gen(int n, const GenParams &g, double *mom, int64_t ld, double *w,
                      uint8_t *flag, int32_t *block_count, hipStream_t stream)
{
    switch (n) {
    case 2: return gen_n<2>(g, mom, ld, w, flag, block_count, stream);
    case 3: return gen_n<3>(g, mom, ld, w, flag, block_count, stream);
    case 4: return gen_n<4>(g, mom, ld, w, flag, block_count, stream);
    case 5: return gen_n<5>(g, mom, ld, w, flag, block_count, stream);
    case 6: return gen_n<6>(g, mom, ld, w, flag, block_count, stream);
    case 7: return gen_n<7>(g, mom, ld, w, flag, block_count, stream);
    case 8: return gen_n<8>(g, mom, ld, w, flag, block_count, stream);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_events(int n, const GenParams &g, double *w_all, double *y, uint16_t *hel,
                         hipStream_t stream)
{
    const int64_t blocks = (g.npoints + 255) / 256;
    if (blocks == 0) return hipSuccess;
    const auto kern = g.mode == 1 ? event_fill_kernel<1> : g.mode == 2 ? event_fill_kernel<2>
                                                                         : event_fill_kernel<0>;
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, stream, g, n, w_all,
                       y, hel);
    return hipGetLastError();
}

hipError_t launch_event_scatter(const int32_t *index, const double *w, const int64_t *d_count,
                                int64_t max_count, double *w_all, hipStream_t stream)
{
    const int64_t blocks = (max_count + 255) / 256;
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(event_scatter_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0,
                       stream, index, w, d_count, max_count, w_all);
    return hipGetLastError();
}

// Above this many 256-point blocks (2^20 points) the block counts are scanned
// by one workgroup first instead of each block summing its predecessors'.
constexpr int64_t kScanAboveBlocks = 4096;

hipError_t launch_compact(int32_t *counts, const uint8_t *flag, int64_t np, int32_t *index,
                          int64_t *d_count, hipStream_t stream)
{
    const int64_t blocks = (np + 255) / 256;
    // no points (an empty configuration of a batch): what follows reads the count all the same
    if (blocks == 0) return launch_zero_u32(reinterpret_cast<unsigned *>(d_count), 2, stream);
    const int scanned = blocks > kScanAboveBlocks ? 1 : 0;
    if (scanned)
        hipLaunchKernelGGL(block_scan_kernel, dim3(1), dim3(kScanThreads), 0, stream, counts,
                           static_cast<int>(blocks), d_count);
    hipLaunchKernelGGL(compact_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, stream,
                       flag, np, counts, static_cast<int>(blocks), scanned, index, d_count);
    return hipGetLastError();
}

hipError_t launch_sum_chunks(const double *part, int nchunks, int64_t ld, const int64_t *d_count,
                             int64_t count, double *out, const int32_t *index, const double *wfac,
                             double *partials, double *wout, unsigned *flags, hipStream_t stream)
{
    const int64_t blocks = (count + 255) / 256;
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(sum_chunks_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, stream,
                       part, nchunks, ld, d_count, count, out, index, wfac, partials, wout, flags);
    return hipGetLastError();
}

hipError_t launch_final(const double *partials, const int64_t *d_count, const int32_t *block_acc, int64_t n_gen,
                        double *res, void *record, const unsigned *flags, double *host, hipStream_t stream)
{
    hipLaunchKernelGGL(final_kernel, dim3(1), dim3(kFinalThreads), 0, stream, partials, d_count, block_acc,
                       n_gen, res, record, flags, host);
    return hipGetLastError();
}

template <int N, int WHICH>
static hipError_t hist_nw(const HistArgs &a, hipStream_t stream)
{
    constexpr int kThreads = kHistThreads<N, WHICH>;
    int64_t blocks = (a.points + kThreads - 1) / kThreads;
    blocks = blocks < 1 ? 1 : (blocks > kHistBlocks<N, WHICH> ? kHistBlocks<N, WHICH> : blocks);
    hipLaunchKernelGGL((hist_kernel<N, WHICH>), dim3(static_cast<unsigned>(blocks)), dim3(kThreads), 0, stream,
                       a.mom, a.ld, a.index, a.w, a.d_count, a.points, a.res, a.nbins, a.lo, a.hi, a.bins, a.n_gen,
                       a.hist);
    return hipGetLastError();
}

template <int N>
static hipError_t hist_n(const HistArgs &a, hipStream_t stream)
{
    return a.observable == 0 ? hist_nw<N, 0>(a, stream) : hist_nw<N, 1>(a, stream);
}

hipError_t launch_hist(int n, const HistArgs &a, hipStream_t stream)
{
    switch (n) {
    case 0: return hist_nw<0, 0>(a, stream);
    case 2: return hist_n<2>(a, stream);
    case 3: return hist_n<3>(a, stream);
    case 4: return hist_n<4>(a, stream);
    case 5: return hist_n<5>(a, stream);
    case 6: return hist_n<6>(a, stream);
    case 7: return hist_n<7>(a, stream);
    case 8: return hist_n<8>(a, stream);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_zero_u32(unsigned *p, int count, hipStream_t stream)
{
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(zero_u32_kernel, dim3((count + 255) / 256), dim3(256), 0, stream, p, count);
    return hipGetLastError();
}

}  // namespace heget
