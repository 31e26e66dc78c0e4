#define V16_DT DT_BF16
#define V16_PRE "bf16"
#define V16_FN variants_ring_bf16
#include "variants_ring16.inc"
