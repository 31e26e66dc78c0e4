// 16-bit storage, A stored K x M: 256 x 256 tile kernels built on the 16x16x32 MFMA.
#include "variant16.h"

namespace peak {

static const Variant rows_mf16t[] = {
    // as those for A along K (variants_mf16.hip)
    TILED_MF16("bf16_m256x256w4a3_tt", DT_BF16, 1, 0, 256, 2),
    TILED_MF16("f16_m256x256w4a3_tt", DT_F16, 1, 0, 256, 2),
    TILED_MF16("bf16_m256x256w4a3_tn", DT_BF16, 1, 1, 256, 2),
    TILED_MF16("f16_m256x256w4a3_tn", DT_F16, 1, 1, 256, 2),
};

PEAK_VARIANT_GROUP(variants_mf16t, rows_mf16t)

}  // namespace peak
