// fp32, any alignment and size, all four layouts.
#include "variant_any.h"

namespace peak {

static const Variant rows_any_f32[] = {
    // four waves of 64x64, two workgroups per CU
    TILED_ANY_LAYOUTS("f32_r128x128", DT_F32, 128, 128, 2, 2, 1, 128, 1, 2),
    // four waves of 32x32, and of 32x32 on half of the rounds each: fp32 MFMAs are slow enough that small tiles cost
    // little, and they fill the chip evenly where the tiles are few
    TILED_ANY_LAYOUTS("f32_r64x64", DT_F32, 64, 64, 2, 2, 1, 128, 2, 4),
    // (one tile on its way in registers, as in 16 bits: 777x1234x1555 TT 42.2 us against 45.3 with two, 43.4 against 47.8
    // for the 32x32 tile; the 64x64 tile is level)
    TILED_ANY_LAYOUTS("f32_r64x32", DT_F32, 64, 32, 2, 1, 2, 128, 1, 4),
    // one 32x32 tile by four waves that share K: latency-bound sizes
    TILED_ANY_LAYOUTS("f32_r32x32", DT_F32, 32, 32, 1, 1, 4, 256, 1, 4),
};

PEAK_VARIANT_GROUP(variants_any_f32, rows_any_f32)

}  // namespace peak
