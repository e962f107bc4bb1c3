// Block-sparse rows on the FP64 matrix cores, for some of the reduced-precision kernels (the FP64 kernel has its own form):
// a wavefront forms 16 rows of a chunk, Y_s = W A with the 16 x K matrix W of the channel factors,
//   W[r][k] = conj(L_c[k][r]) for the rows k >= r of r's channel, l_c[r] for its multipole row,
// in units of up to eight consecutive rows of M (two steps of the 16x16x4 product, one for up to four). K runs from the rows' first one to the
// end of their last channel, then over their channels' multipole rows. W is laid out once per context in operand
// order (pack_units_kernel).
//
// M goes from memory straight into operand registers, a unit ahead, and needs no LDS and no barrier; formed on the
// vector cores (a lane per row, the rows of a run brought by DPP shifts, or a lane per column with the rows in LDS)
// there are a sixth of the multiplications, but shifts and LDS reads beside them. Bound by the 64 cycles of a product:
// the instances that gain by it say so.
#pragma once
#include "common.hpp"
#include "tile.hpp"

namespace exc {

// rows [row, row + rows) of M: five to eight in two steps, up to four in one, none: padding
struct RowUnit { int32_t row, rows; };
constexpr int kUnitRing = 4;                           // a group's units come in fours

struct RowUnits {
  const RowUnit* units;           // those of the first 16 rows of every chunk, of the second ones, ...
  const int32_t* count;           // [4][n_chunk] units of each chunk's 16 rows
  int32_t n_chunk, n_units;
  const d2_t* w;                  // [n_units][2 steps][64 lanes]
  int64_t w_qs;                   // elements between the copies of q and q + 1 (0: one copy)
  int32_t begin[4];               // first unit of each group of 16 rows
};

// The row of its 16 that lane l16 supplies: the four accumulator elements of a lane group are then consecutive rows.
__device__ __forceinline__ constexpr int unit_row(int l16) { return 4 * (l16 & 3) + (l16 >> 2); }

// One wavefront's rows of every chunk: group t (rows 16 t .. 16 t + 15 of a chunk) and NJ tiles of eight columns whose
// byte offsets from the resource's base are co[j] (lanes 2 c and 2 c + 1: column c; out of range: zeros), the first
// `nj` of them used. done(ck, y) takes each chunk's rows: lane (l16, lq) holds Re (even lanes) or Im of column
// l16 / 2 of each tile, rows 4 lq .. 4 lq + 3 of the group.
// ONLY64: M is complex64 (else c64 says); RING (2 or 4): units in flight.
template <int NJ, bool REALF, bool ONLY64, int RING, class F>
__device__ __forceinline__ void sparse_units(const RowUnits& R, int q, __amdgpu_buffer_rsrc_t mrs, const uint32_t (&co)[NJ],
                                             int nj, bool c64, int t, int lane, F&& done) {
  static_assert(kUnitRing % RING == 0, "whole rounds of the ring");
  using raw_t = std::conditional_t<ONLY64, u2_t, u4_t>;
  const int lq = lane >> 4, part = lane & 1;
  const uint32_t sgn = part == 0 ? 0x80000000u : 0u;
  const auto* units = (const __attribute__((address_space(4))) RowUnit*)R.units;        // (scalar loads)
  const auto* count = (const __attribute__((address_space(4))) int32_t*)R.count + t * R.n_chunk;
  const d2_t* W = R.w + q * R.w_qs + lane;
  int u = R.begin[t];
  struct Unit { raw_t x[NJ]; d2_t w[2]; int rows; };
  // two steps: a lane loads row 2 lq + part, step e contracts rows 2 lq + e, the other one of the pair comes from the
  // neighbouring lane; one step: both lanes load row lq
  auto load = [&](Unit& n, int i) {
    i = min(i, R.n_units - 1);
    const int row = units[i].row;
    n.rows = units[i].rows;
    const int k = n.rows > 4 ? 2 * lq + part : lq;
    if constexpr (ONLY64) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) n.x[j] = buf_load<u2_t>(mrs, k < n.rows ? co[j] + k * 8 : 0x80000000u, (uint32_t)(row * 8));
    } else if (c64) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const u2_t v = buf_load<u2_t>(mrs, k < n.rows ? co[j] + k * 8 : 0x80000000u, (uint32_t)(row * 8));
        n.x[j].x = v.x;
        n.x[j].y = v.y;
      }
    } else {
#pragma unroll
      for (int j = 0; j < NJ; ++j) n.x[j] = buf_load<u4_t>(mrs, k < n.rows ? co[j] + k * 16 : 0x80000000u, (uint32_t)(row * 16));
    }
    n.w[0] = W[(long)i * 128];
    n.w[1] = W[(long)i * 128 + 64];
  };
  auto dpp = [](uint32_t x) -> uint32_t { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, true); };
  auto swap = [&](raw_t v) -> raw_t {
#pragma unroll
    for (int i = 0; i < (int)(sizeof(raw_t) / 4); ++i) v[i] = dpp(v[i]);
    return v;
  };
  auto re = [](raw_t v) -> double {
    if constexpr (ONLY64) return (double)__uint_as_float(v[0]);
    else return __hiloint2double((int)v[1], (int)v[0]);
  };
  auto im = [](raw_t v) -> double {
    if constexpr (ONLY64) return (double)__uint_as_float(v[1]);
    else return __hiloint2double((int)v[3], (int)v[2]);
  };
  auto neg = [&](double x) -> double { return __hiloint2double(__double2hiint(x) ^ (int)sgn, __double2loint(x)); };
  Unit c[RING];
  static_for<0, RING>([&](auto rc) { load(c[decltype(rc)::value], u + decltype(rc)::value); });
  for (int ck = 0; ck < R.n_chunk; ++ck) {
    const int m = count[ck];
    d4_t y[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) y[j] = d4_t{0, 0, 0, 0};
    for (int i = 0; i < m; i += RING) {
      static_for<0, RING>([&](auto rc) {
        Unit& n = c[decltype(rc)::value];
        if constexpr (!ONLY64)
          if (c64) {
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
              const double vr = (double)__uint_as_float(n.x[j][0]), vi = (double)__uint_as_float(n.x[j][1]);
              n.x[j] = u4_t{(uint32_t)__double2loint(vr), (uint32_t)__double2hiint(vr), (uint32_t)__double2loint(vi),
                            (uint32_t)__double2hiint(vi)};
            }
          }
        if (n.rows > 4) {
#pragma unroll
          for (int j = 0; j < NJ; ++j)
            if (j < nj) {                              // uniform
              const raw_t v = n.x[j], o = swap(v);
              y[j] = mfma(n.w[0].x, part ? im(o) : re(v), y[j]);
              if constexpr (!REALF) y[j] = mfma(n.w[0].y, neg(part ? re(o) : im(v)), y[j]);
              y[j] = mfma(n.w[1].x, part ? im(v) : re(o), y[j]);
              if constexpr (!REALF) y[j] = mfma(n.w[1].y, neg(part ? re(v) : im(o)), y[j]);
            }
        }
        if (n.rows <= 4 && n.rows > 0) {
#pragma unroll
          for (int j = 0; j < NJ; ++j)
            if (j < nj) {
              const raw_t v = n.x[j];
              y[j] = mfma(n.w[0].x, part ? im(v) : re(v), y[j]);
              if constexpr (!REALF) y[j] = mfma(n.w[0].y, neg(part ? re(v) : im(v)), y[j]);
            }
        }
        load(n, u + RING + decltype(rc)::value);
      });
      u += RING;
    }
    done(ck, y);
  }
}

// W of every unit in operand order: lane (l16, lq) of step e, row unit_row(l16) of the 16 and row 2 lq + e (one
// step: lq) of the unit. blockIdx.x: unit, blockIdx.y: copy of the channel blocks. owner[unit]: the first of the 16 rows, how many.
__global__ __launch_bounds__(128) inline void pack_units_kernel(RowUnits R, const int2* owner, const double2* coef,
                                                                const double2* cvec, const int4* rowinfo, int n_s,
                                                                int64_t coef_qs, int64_t cvec_qs, d2_t* out) {
  const int u = blockIdx.x, lane = threadIdx.x & 63, e = threadIdx.x >> 6, l16 = lane & 15, lq = lane >> 4;
  const int i = unit_row(l16);
  int kk = 2 * lq + e;
  const int2 own = owner[u];
  const RowUnit un = R.units[u];
  const bool one = un.rows <= 4;                       // (one step)
  if (one) kk = e == 0 ? lq : 8;
  d2_t v{0.0, 0.0};
  if (i < own.y && kk < un.rows) {
    const int r = own.x + i, k = un.row + kk;
    const int4 ri = rowinfo[r];                        // {run start, run length, multipole row}
    if (k < n_s) {
      if (k >= r && k - r < ri.y) {
        const double2 l = coef[blockIdx.y * coef_qs + ri.x + (k - r)];
        v = d2_t{l.x, -l.y};
      }
    } else if (k == ri.z) {
      const double2 l = cvec[blockIdx.y * cvec_qs + r];
      v = d2_t{l.x, l.y};
    }
  }
  out[blockIdx.y * R.w_qs + ((long)u * 2 + e) * 64 + lane] = v;
}

}  // namespace exc
