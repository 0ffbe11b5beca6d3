// Amplitude kernels with the helicities of a point over the lanes of a wave
// (me2_lanes.hpp), float and double.
#include "me2_lanes.hpp"

namespace heget {

template <typename R, int N>
constexpr Me2Variant lanes_variant()
{
    return Me2Variant{std::is_same<R, float>::value ? 1 : 0, N, N, 1 << N, 2, 1, 1, 0, 1, kLanesPs,
                      reinterpret_cast<const void *>(&lanes::me2_lanes_kernel<R, N>)};
}

extern const Me2Variant kShapesLanes[] = {
    lanes_variant<float, 6>(),  lanes_variant<float, 7>(),  lanes_variant<float, 8>(),
    lanes_variant<double, 6>(), lanes_variant<double, 7>(), lanes_variant<double, 8>(),
};
extern const int kShapesLanesCount = sizeof(kShapesLanes) / sizeof(Me2Variant);

}  // namespace heget
