#define V16_DT DT_F16
#define V16_PRE "f16"
#define V16_FN variants_ring_f16
#include "variants_ring16.inc"
