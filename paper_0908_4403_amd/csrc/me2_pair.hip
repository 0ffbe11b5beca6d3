// Amplitude kernels with two lanes per point (me2_pair.hpp), float and double,
// n = 5.
#include "me2_pair.hpp"

namespace heget {

template <typename R, int N, int WPE>
constexpr Me2Variant pair_variant()
{
    return Me2Variant{std::is_same<R, float>::value ? 1 : 0, N, N, 1 << N, 2, 1, 0, WPE, 1, kPairPs,
                      reinterpret_cast<const void *>(&pairs::me2_pair_kernel<R, N, WPE, false>),
                      reinterpret_cast<const void *>(&pairs::me2_pair_kernel<R, N, WPE, true>)};
}

extern const Me2Variant kShapesPair[] = {pair_variant<float, 5, 2>(), pair_variant<double, 5, 1>()};
extern const int kShapesPairCount = sizeof(kShapesPair) / sizeof(Me2Variant);

}  // namespace heget
