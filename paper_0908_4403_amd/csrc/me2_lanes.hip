// Amplitude kernels with the helicities of a point over the lanes of a wave
// (me2_lanes.hpp), float and double.
#include "me2_lanes.hpp"

namespace heget {

template <typename R, int N, int W, int WPE>
constexpr Me2Variant lanes_variant()
{
    return Me2Variant{std::is_same<R, float>::value ? 1 : 0, N, N, 1 << N, 2, W, 1, WPE, 1, kLanesPs,
                      reinterpret_cast<const void *>(&lanes::me2_lanes_kernel<R, N, W, WPE, false>),
                      reinterpret_cast<const void *>(&lanes::me2_lanes_kernel<R, N, W, WPE, true>)};
}

// (waves on a wave's points, waves per SIMD): see me2_lanes.hpp
extern const Me2Variant kShapesLanes[] = {
    lanes_variant<float, 6, 2, 4>(),  lanes_variant<float, 7, 2, 4>(),  lanes_variant<float, 8, 2, 4>(),
    lanes_variant<double, 6, 2, 2>(), lanes_variant<double, 7, 2, 2>(), lanes_variant<double, 8, 2, 2>(),
};
extern const int kShapesLanesCount = sizeof(kShapesLanes) / sizeof(Me2Variant);

}  // namespace heget
