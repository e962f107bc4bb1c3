// Instances of the wide kernel (see configs.hpp).
#include "configs.hpp"
#include "wide.hpp"

namespace exc {

// wide kernel (large pairs, complex64 M): 8 wavefronts, 256-row dense blocks, NB8M band tiles
#define WCFG(MODE, NB8M, RT, ID)                                                                  \
  FusedKCfg{MODE, RT, NB8M, NB8M, 32, 32, 1, wide_kernel<MODE, NB8M, RT>, WideCfg<MODE, NB8M, RT>::LDS_B, \
            ID, false, 512, true, WideCfg<MODE, NB8M, RT>::GCHAIN, WideCfg<MODE, NB8M, RT>::GCH_RS,        \
            WideCfg<MODE, NB8M, RT>::GCH_RD}

const FusedKCfg kWideCfgs[kNumWide] = {
    WCFG(M_F32, 13, 2, 180),           WCFG(M_BF16X3, 13, 2, 181),        WCFG(M_BF16X6, 13, 2, 182),
    WCFG(M_F32, 16, 2, 183),           WCFG(M_BF16X3, 16, 2, 184),
    WCFG(M_F32, 13, 1, 186),           WCFG(M_BF16X3, 13, 1, 187),        WCFG(M_BF16X6, 13, 1, 188),
    WCFG(M_F32, 8, 2, 189),            WCFG(M_BF16X3, 8, 2, 190),         WCFG(M_BF16X6, 8, 2, 191),
};

}  // namespace exc
