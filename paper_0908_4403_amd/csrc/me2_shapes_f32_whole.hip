// The float n = 5 walk of all 32 helicity configurations at once (fields as in
// me2_shapes_f32_lo.hip), in its own translation unit and table: it is the
// default for n = 5 where the tiles give every SIMD up to one wave, and no shape
// of the list that the autotuner's callers see, because every value it shares is
// formed once (helicities_per_walk = 2^n, as the kernels of me2_lanes.hpp).
// It needs all 512 registers of a lane (40 held currents of two photons, 32
// FP64 accumulators), 13% of its instructions move values to and from the
// upper half, and still it is ahead of eight configurations per walk: 12 100
// instructions per point instead of 20 300, 1e6 points in 371 instead of 442
// us; sixteen per walk 415 us.  Bound by one wave's issue rate (0.23
// instructions per clock and SIMD); beyond 65 536 points two lanes per point are
// ahead (me2_pair.hpp).
#include "me2_item.hpp"

namespace heget {

extern const Me2Variant kShapesWhole[] = {
    mc_variant<float, 5, 5, 32, 2, 1, 0, 0, 1, 2>(),
};
extern const int kShapesWholeCount = sizeof(kShapesWhole) / sizeof(Me2Variant);

}  // namespace heget
