// fp32, aligned operands, small tiles with a ring of K tiles.
#include "variant_any.h"

namespace peak {

static const Variant rows_ring_f32[] = {
    // four waves of 32x32, three stages of 16 KB, three workgroups per CU (five stages: 1024^3 NT 23.5 us against 22.2)
    TILED_RING_LAYOUTS("f32_m64x64q3", DT_F32, 64, 64, 2, 2, 1, 128, 3, 4),
    // ... of 32x32 on half of the rounds each, 64x32 in all
    TILED_RING_LAYOUTS("f32_m64x32q5", DT_F32, 64, 32, 2, 1, 2, 128, 5, 4),
    // one 32x32 tile by four waves that share K, 64 k per stage
    TILED_RING_LAYOUTS("f32_m32x32q3", DT_F32, 32, 32, 1, 1, 4, 256, 3, 4),
};

PEAK_VARIANT_GROUP(variants_ring_f32, rows_ring_f32)

}  // namespace peak
