// Registry of the compiled amplitude-kernel shapes and their launcher.
#include <hip/hip_runtime.h>

#include <map>
#include <mutex>
#include <vector>

#include "kernels.hpp"

namespace heget {

// Tables defined in the me2_shapes_*.hip translation units.
extern const Me2Variant kShapesF32Lo[], kShapesF32Mid[], kShapesF32Meet7[], kShapesF32Meet8[],
    kShapesF32Hi[];
extern const Me2Variant kShapesF64Lo[], kShapesF64Mid[], kShapesF64Hi[];
extern const int kShapesF32LoCount, kShapesF32MidCount, kShapesF32Meet7Count, kShapesF32Meet8Count,
    kShapesF32HiCount;
extern const int kShapesF64LoCount, kShapesF64MidCount, kShapesF64HiCount;
extern const Me2Variant kShapesSampled[], kShapesSampledMeet8[];
extern const int kShapesSampledCount, kShapesSampledMeet8Count;
extern const Me2Variant kShapesLanes[];
extern const int kShapesLanesCount;
extern const Me2Variant kShapesPair[];
extern const int kShapesPairCount;
extern const Me2Variant kShapesWhole[];
extern const int kShapesWholeCount;

static const std::vector<Me2Variant> &all_variants()
{
    static const std::vector<Me2Variant> v = [] {
        std::vector<Me2Variant> r;
        // the meeting-in-the-middle tables come before the other n = 7, 8
        // shapes: their first entries are the defaults
        const Me2Variant *tabs[] = {kShapesF32Lo, kShapesF32Mid, kShapesF32Meet7, kShapesF32Meet8,
                                    kShapesF32Hi, kShapesF64Lo, kShapesF64Mid, kShapesF64Hi};
        const int counts[] = {kShapesF32LoCount, kShapesF32MidCount, kShapesF32Meet7Count,
                              kShapesF32Meet8Count, kShapesF32HiCount, kShapesF64LoCount,
                              kShapesF64MidCount, kShapesF64HiCount};
        for (int t = 0; t < 8; ++t)
            for (int i = 0; i < counts[t]; ++i) r.push_back(tabs[t][i]);
        return r;
    }();
    return v;
}

const Me2Variant *me2_variants(int *count)
{
    *count = static_cast<int>(all_variants().size());
    return all_variants().data();
}

const Me2Variant *me2_default(int prec, int n)
{
    for (const Me2Variant &v : all_variants())
        if (v.prec == prec && v.n == n) return &v;
    return nullptr;
}

const Me2Variant *me2_shared(int prec, int n, int i)
{
    const Me2Variant *tabs[] = {kShapesLanes, kShapesPair, kShapesWhole};
    const int counts[] = {kShapesLanesCount, kShapesPairCount, kShapesWholeCount};
    for (int t = 0; t < 3; ++t)
        for (int k = 0; k < counts[t]; ++k)
            if (tabs[t][k].prec == prec && tabs[t][k].n == n && i-- == 0) return &tabs[t][k];
    return nullptr;
}

const Me2Variant *me2_sampled(int prec, int n)
{
    for (int i = 0; i < kShapesSampledCount; ++i)
        if (kShapesSampled[i].prec == prec && kShapesSampled[i].n == n) return &kShapesSampled[i];
    for (int i = 0; i < kShapesSampledMeet8Count; ++i)
        if (kShapesSampledMeet8[i].prec == prec && kShapesSampledMeet8[i].n == n) return &kShapesSampledMeet8[i];
    return nullptr;
}

// Blocks of a kernel that fit on the device at once (resident), per kernel.
static int64_t resident_blocks(const void *func, int wpb)
{
    static std::mutex mu;
    static std::map<const void *, int64_t> cache;
    std::lock_guard<std::mutex> lk(mu);
    auto it = cache.find(func);
    if (it != cache.end()) return it->second;
    int dev = 0, per_cu = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, func, wpb * 64, 0) != hipSuccess ||
        per_cu <= 0 || cus <= 0)
        return 0;  // unknown: one wave per item
    const int64_t r = static_cast<int64_t>(per_cu) * cus;
    cache[func] = r;
    return r;
}

hipError_t launch_me2(const Me2Variant &v, const Me2Args &a, hipStream_t stream)
{
    const void *func = a.beam ? v.beam_func : v.func;
    if (!func) return hipErrorInvalidValue;
    const int64_t ntiles = (a.count + 63) / 64;
    int64_t items = (ntiles + v.ppl - 1) / v.ppl * a.nchunks;
    if (v.ps == kLanesPs) {  // a workgroup's wave(s) share 2^(8 - n) points, |M|^2 of each to out
        const int64_t per = int64_t(1) << (8 - v.n);
        if (a.nchunks != 1 || a.partials || !a.out) return hipErrorInvalidValue;
        items = (a.count + per - 1) / per;
    }
    if (items == 0) return hipSuccess;
    int64_t blocks = v.ps == kLanesPs ? items : (items + v.wpb - 1) / v.wpb;
    if (v.pf) {
        const int64_t r = resident_blocks(func, v.wpb);
        if (r > 0 && r < blocks) blocks = r;
    }
    void *args[] = {const_cast<double **>(&a.mom), const_cast<int64_t *>(&a.ld),
                    const_cast<int32_t **>(&a.index), const_cast<uint16_t **>(&a.hel),
                    const_cast<int64_t **>(&a.d_count), const_cast<int64_t *>(&a.count),
                    const_cast<int *>(&a.nchunks), const_cast<double *>(&a.coef),
                    const_cast<double **>(&a.out), const_cast<int64_t *>(&a.ld_out),
                    const_cast<double **>(&a.wfac), const_cast<double **>(&a.partials),
                    const_cast<double **>(&a.wout), const_cast<unsigned **>(&a.flags)};
    return hipLaunchKernel(func, dim3(static_cast<unsigned>(blocks)), dim3(v.wpb * 64), args, 0,
                           stream);
}

}  // namespace heget
