// Launch of the ring kernels and the macros for their rows of the variant table.
#pragma once

#include "variant.h"
#include "gemm_any_device.h"

namespace peak {

template <class C>
static int launch_gemm_any(const GemmArgs &a, unsigned grid, void *stream)
{
    hipLaunchKernelGGL((gemm_any_kernel<C>), dim3(grid), dim3(C::NT), C::OWN_LDS ? 0 : C::lds_of(a.ktiles_per_slice), (hipStream_t)stream, a);
    return hipGetLastError() == hipSuccess ? 0 : 1;
}

// operands of any alignment straight to LDS, STAGES K tiles in a ring
#define TILED_LOOSE(NAME, DT, AKM, BKN, BM, BN, WMW, WNW, WKW, RB, STAGES, EU)                         \
    {NAME, KIND_TILED, DT, AKM, BKN, 0, BM, BN, PEAK_BK(DT, RB), WMW * WNW * WKW * 64, STAGES,         \
     CfgAny<DT, AKM != 0, BKN != 0, BM, BN, WMW, WNW, WKW, RB, EU, STAGES, true>::LDS_BYTES, 0,     \
     &launch_gemm_any<CfgAny<DT, AKM != 0, BKN != 0, BM, BN, WMW, WNW, WKW, RB, EU, STAGES, true>>, 0, 0, 0, 0, 0, 0, \
     CfgAny<DT, AKM != 0, BKN != 0, BM, BN, WMW, WNW, WKW, RB, EU, STAGES, true>::LDS_LEAST, EU}

#define TILED_LOOSE_LAYOUTS(NAME, DT, BM, BN, WMW, WNW, WKW, RB, STAGES, EU)                           \
    TILED_LOOSE(NAME "_nt", DT, 0, 0, BM, BN, WMW, WNW, WKW, RB, STAGES, EU),                          \
    TILED_LOOSE(NAME "_nn", DT, 0, 1, BM, BN, WMW, WNW, WKW, RB, STAGES, EU),                          \
    TILED_LOOSE(NAME "_tt", DT, 1, 0, BM, BN, WMW, WNW, WKW, RB, STAGES, EU),                          \
    TILED_LOOSE(NAME "_tn", DT, 1, 1, BM, BN, WMW, WNW, WKW, RB, STAGES, EU)

// aligned operands straight to LDS, STAGES K tiles in a ring (the registers of all of them, 118 at most, leave room for four waves per SIMD)
#define TILED_RING(NAME, DT, AKM, BKN, BM, BN, WMW, WNW, WKW, RB, STAGES, EU)                          \
    {NAME, KIND_TILED, DT, AKM, BKN, 1, BM, BN, PEAK_BK(DT, RB), WMW * WNW * WKW * 64, STAGES,         \
     CfgAny<DT, AKM != 0, BKN != 0, BM, BN, WMW, WNW, WKW, RB, EU, STAGES, false>::LDS_BYTES, 0,           \
     &launch_gemm_any<CfgAny<DT, AKM != 0, BKN != 0, BM, BN, WMW, WNW, WKW, RB, EU, STAGES, false>>,       \
     BKN, AKM, 0, 0, 0, 1, CfgAny<DT, AKM != 0, BKN != 0, BM, BN, WMW, WNW, WKW, RB, EU, STAGES, false>::LDS_SHORTEST, 4}

#define TILED_RING_LAYOUTS(NAME, DT, BM, BN, WMW, WNW, WKW, RB, STAGES, EU)                            \
    TILED_RING(NAME "_nt", DT, 0, 0, BM, BN, WMW, WNW, WKW, RB, STAGES, EU),                           \
    TILED_RING(NAME "_nn", DT, 0, 1, BM, BN, WMW, WNW, WKW, RB, STAGES, EU),                           \
    TILED_RING(NAME "_tt", DT, 1, 0, BM, BN, WMW, WNW, WKW, RB, STAGES, EU),                           \
    TILED_RING(NAME "_tn", DT, 1, 1, BM, BN, WMW, WNW, WKW, RB, STAGES, EU)

}  // namespace peak
