// Tables of the main kernels' instances. Each table lives in a translation unit of its own
// (configs_fused.hip, configs_wide.hip, configs_herk64.hip) so that they compile side by side.
#pragma once
#include "fused.hpp"
#include "herk64.hpp"
#include "plan64.hpp"

namespace exc {

// coefficients per multipole-free row staged by the fused kernel (its MAXT)
constexpr int kRunPad = FusedCfg<M_BF16X3, 1, 1, 1, 32>::MAXT;
// chunks of multipole-free rows: rows (one per lane), multipole rows, chunks (at most)
constexpr int kChunkRows = FusedCfg<M_BF16X3, 1, 1, 1, 32>::GR;
constexpr int kChunkMP = FusedCfg<M_BF16X3, 1, 1, 1, 32>::MPC;
constexpr int kMaxChunks = FusedCfg<M_BF16X3, 1, 1, 1, 32>::MAXCK;

// Fused reduced-precision HERK kernels: RTW row tiles per wavefront (row
// blocks of 64 RTW rows), NCT band tiles per pass, NB8M the largest band-tile
// count per n'' value, KC complex k per K-loop panel.
struct FusedKCfg {
  int mode, RTW, NCT, NB8M, KC, CB, OCC;
  void (*fn)(FusedArgs);
  size_t lds;
  int id;
  bool realf = false;               // real factor only (inversion-symmetric contexts)
  int nt = 256;                     // threads per workgroup
  bool c64only = false;             // reads complex64 M only (the wide kernel)
  int gchain = 0, grs = 64, grd = 64;   // binary32 Gram chains: kind, rows per chunk (sparse, dense)
};

// Listed in order of preference among equal band-tile capacity.
constexpr int kNumFused = 28, kNumWide = 11, kNumHerk64 = 28;
extern const FusedKCfg kFusedCfgs[kNumFused];
extern const FusedKCfg kWideCfgs[kNumWide];

// FP64 Cholesky/HERK kernels (herk64.hpp): nbt band tiles, ng n'' values per pass. The planner picks
// the smallest nbt that holds the context's bands and the ng of the cheapest plan (build_plan64).
struct Herk64K {
  Shape64 shape;
  void (*fn)(Herk64Args);           // complex128 M
  void (*fn64)(Herk64Args);         // complex64 M
  int id() const { return 2000 + 16 * shape.nbt + shape.ng; }
};
extern const Herk64K kHerk64[kNumHerk64];

}  // namespace exc
