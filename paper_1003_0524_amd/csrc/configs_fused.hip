// Instances of the fused kernel (see configs.hpp).
#include "configs.hpp"

namespace exc {

#define FCFG(MODE, RTW, NCT, NB8M, KC, ID)                                                       \
  FusedKCfg{MODE, RTW, NCT, NB8M, KC, 16, 1, fused_kernel<MODE, RTW, NCT, NB8M, KC, 16, 1>,        \
            FusedCfg<MODE, RTW, NCT, NB8M, KC, 16, 1>::LDS_B, ID, false, 256, false,                \
            FusedCfg<MODE, RTW, NCT, NB8M, KC, 16, 1>::GCHAIN, FusedCfg<MODE, RTW, NCT, NB8M, KC, 16, 1>::GR, \
            FusedCfg<MODE, RTW, NCT, NB8M, KC, 16, 1>::GR}
// two workgroups per CU: at most 256 registers per lane and half the LDS each
#define FCFG2(MODE, RTW, NCT, NB8M, ID)                                                          \
  FusedKCfg{MODE, RTW, NCT, NB8M, 32, 16, 2, fused_kernel<MODE, RTW, NCT, NB8M, 32, 16, 2>,       \
            FusedCfg<MODE, RTW, NCT, NB8M, 32, 16, 2>::LDS_B, ID, false, 256, false,               \
            FusedCfg<MODE, RTW, NCT, NB8M, 32, 16, 2>::GCHAIN, FusedCfg<MODE, RTW, NCT, NB8M, 32, 16, 2>::GR, \
            FusedCfg<MODE, RTW, NCT, NB8M, 32, 16, 2>::GR}

// real-factor instances (inversion symmetry): the same kernels without the
// products with the factor's zero imaginary parts
#define FCFG2R(MODE, RTW, NCT, NB8M, ID)                                                         \
  FusedKCfg{MODE, RTW, NCT, NB8M, 32, 16, 2, fused_kernel<MODE, RTW, NCT, NB8M, 32, 16, 2, true>, \
            FusedCfg<MODE, RTW, NCT, NB8M, 32, 16, 2>::LDS_B, ID, true, 256, false,                \
            FusedCfg<MODE, RTW, NCT, NB8M, 32, 16, 2>::GCHAIN, FusedCfg<MODE, RTW, NCT, NB8M, 32, 16, 2>::GR, \
            FusedCfg<MODE, RTW, NCT, NB8M, 32, 16, 2>::GR}

// Listed in order of preference among equal band-tile capacity (the two-per-CU
// instances first: they hide more memory latency).
const FusedKCfg kFusedCfgs[kNumFused] = {
    FCFG2(M_F32, 2, 6, 3, 150),        FCFG2(M_F32, 3, 6, 3, 151),
    FCFG2(M_BF16X3, 3, 6, 3, 161),     FCFG2(M_BF16X3, 2, 6, 3, 160),   // 161 first: 3-5 % ahead
    FCFG2(M_BF16X6, 2, 6, 3, 170),     FCFG2(M_BF16X6, 3, 6, 3, 171),
    FCFG2(M_BF16X3, 2, 8, 8, 162),
    FCFG(M_F32, 3, 12, 3, 32, 120),    FCFG(M_F32, 5, 6, 3, 32, 124),
    FCFG(M_F32, 4, 8, 8, 32, 121),     FCFG(M_F32, 2, 13, 13, 32, 123),
    FCFG(M_F32, 2, 16, 16, 32, 122),
    FCFG(M_BF16X3, 3, 12, 3, 32, 130), FCFG(M_BF16X3, 5, 6, 3, 32, 134),
    FCFG(M_BF16X3, 4, 8, 8, 32, 131),  FCFG(M_BF16X3, 2, 13, 13, 32, 133),
    FCFG(M_BF16X3, 2, 16, 16, 32, 132),
    FCFG(M_BF16X6, 3, 12, 3, 32, 140), FCFG(M_BF16X6, 5, 6, 3, 32, 144),
    FCFG(M_BF16X6, 4, 8, 8, 32, 141),  FCFG(M_BF16X6, 2, 13, 13, 32, 143),
    FCFG(M_BF16X6, 2, 16, 16, 32, 142),
    FCFG2R(M_F32, 2, 6, 3, 250),       FCFG2R(M_F32, 3, 6, 3, 251),
    FCFG2R(M_BF16X3, 3, 6, 3, 261),    FCFG2R(M_BF16X3, 2, 6, 3, 260),
    FCFG2R(M_BF16X6, 2, 6, 3, 270),    FCFG2R(M_BF16X6, 3, 6, 3, 271),
};

}  // namespace exc
