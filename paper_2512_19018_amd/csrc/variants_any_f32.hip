// fp32, any alignment and size, all four layouts.
#include "variant_any.h"

namespace peak {

static const Variant rows_any_f32[] = {
    // four waves of 64x64, two workgroups per CU
    TILED_LOOSE_LAYOUTS("f32_r128x128", DT_F32, 128, 128, 2, 2, 1, 128, 2, 2),
    // four waves of 32x32, and of 32x32 on half of the rounds each: fp32 MFMAs are slow enough that small tiles cost
    // little, and they fill the chip evenly where the tiles are few
    TILED_LOOSE_LAYOUTS("f32_r64x64", DT_F32, 64, 64, 2, 2, 1, 128, 3, 4),
    // (three stages and four workgroups per CU; five and two: 1728x1184x547 TT 26.7 us against 24.3, 2575x2944x4496 TN 572 and 525)
    TILED_LOOSE_LAYOUTS("f32_r64x32", DT_F32, 64, 32, 2, 1, 2, 128, 3, 4),
    // one 32x32 tile by four waves that share K: latency-bound sizes
    TILED_LOOSE_LAYOUTS("f32_r32x32", DT_F32, 32, 32, 1, 1, 4, 256, 3, 4),
};

PEAK_VARIANT_GROUP(variants_any_f32, rows_any_f32)

}  // namespace peak
