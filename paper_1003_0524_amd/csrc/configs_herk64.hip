// Instances of the FP64 Cholesky/HERK kernel (see configs.hpp).
#include "configs.hpp"

namespace exc {

#define HCFG(NBT, NG)                                                                              \
  Herk64K{{NBT, NG, Herk64Cfg<NBT, NG, false>::NW, Herk64Cfg<NBT, NG, false>::NPW,                  \
           Herk64Cfg<NBT, NG, false>::CTW}, herk64_kernel<NBT, NG, false>, herk64_kernel<NBT, NG, true>}
const Herk64K kHerk64[kNumHerk64] = {
    HCFG(1, 1), HCFG(1, 2), HCFG(1, 4), HCFG(1, 8), HCFG(1, 12),
    HCFG(2, 1), HCFG(2, 2), HCFG(2, 3), HCFG(2, 4), HCFG(2, 6),
    HCFG(3, 1), HCFG(3, 2), HCFG(3, 3), HCFG(3, 4),
    HCFG(4, 1), HCFG(4, 2), HCFG(5, 1), HCFG(6, 1), HCFG(7, 1), HCFG(8, 1),
    HCFG(9, 1), HCFG(10, 1), HCFG(11, 1), HCFG(12, 1), HCFG(13, 1), HCFG(14, 1), HCFG(15, 1), HCFG(16, 1),
};

}  // namespace exc
