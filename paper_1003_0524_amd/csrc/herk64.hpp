// FP64 kernel of the Cholesky/HERK form: one work item is a pair (k,q), a range of
// n'' values processed ngc at a time, and a range of row parts (part 0 the block-sparse
// rows, part 1 + j the dense rows [64 j, 64 j + 64)); it adds
//
//   G = sum_{n''} Y^H Y,   Y = rows of [ Y_s ; L22^H A_d ]
//
// into its own partial slot (Sec. III.C, eq. "vec-mat-vec" with v = L L^H). Bound by the
// FP64 matrix cores: a 16x16x4 instruction takes 64 cycles of its SIMD, so what counts is
// that every SIMD always has one ready and that few of them multiply zeros.
//
//  * Four wavefronts side by side over the 64 rows of a block (16 rows each, every column
//    tile of the pass, so each wavefront reads its own rows of the factor from L2 straight
//    into registers, one panel ahead), two workgroups per CU: while one waits at a barrier
//    or runs the short panels of its diagonal, the other keeps the SIMDs busy. More than
//    8 band tiles: eight wavefronts, the column tiles split over two, one workgroup per CU.
//  * K panels of A_d (16 k of every column) go global -> LDS by direct buffer loads, three
//    buffers, two panels ahead, one barrier a panel. A 1 KB load covers 16 columns x 64
//    contiguous bytes; the 16-byte units of a column are permuted within those 64 bytes so
//    that the operand reads of a half-wave meet distinct LDS banks.
//  * Tile columns interleave re and im (column 2 c + part), the order in which M holds them,
//    so [Ar|Ai] and [-Ai|Ar] are plain 8-byte reads of the raw panel: no conversion pass.
//  * A panel that ends above a wavefront's first row meets only zeros of the triangular
//    factor and is skipped by that wavefront.
//  * Gram tiles stay in registers for the whole item. The accumulator layout of the
//    16x16x4 instruction (lane group lq, element i: row lq + 4 i) is its operand layout for
//    k = rows 4 i .. 4 i + 3, so with at most three band tiles a wavefront contracts its 16
//    rows straight from its accumulators into its own copy of all Gram tiles (summed over
//    the wavefronts once per item); with more, the 64 rows pass through LDS and each
//    wavefront holds its share of the tiles.
//
// Measured against the kernel it replaces (tile_kernel's FP64 instances: one item per pair, operands through
// registers, Gram tiles of more than three band tiles added in global memory once per 64 rows): one outer
// iteration of the Si-like workload 844 -> 655 us; one k of the ZnO-like one (144 pairs, which left 112 of the
// 256 CUs without work) 30.8 -> 7.9 ms; one k of eight small pairs (N_MB 300, 16 bands) 299 -> 73 us.
//
// Partial slots: [tile pair][element i][lane], rows and columns of a tile interleaved as above.
#pragma once
#include "common.hpp"
#include "tile.hpp"
#include "wide.hpp"

namespace exc {

struct Herk64Args {
  const PairInfo* pairs;
  const WorkItem* items;
  int32_t n_items;
  const void* const* mtab;       // [n_k] device pointers to M_k
  int32_t n_s, n_occ;
  const double* U;               // factor planes (re, im) of L22^H
  const double2* ws;             // block-sparse rows Y_s
  double* gpart;                 // Gram partials
  int32_t gstride;
  const uint64_t* tmask;         // [n_k][3] band-tile pairs to compute
};

template <int NBT_, int NG_, bool C64>
struct Herk64Cfg {
  static constexpr int NBT = NBT_, NG = NG_;           // band tiles, n'' values of a pass
  static constexpr int NWC = NBT * NG > 12 || (NBT > 8) ? 2 : 1;
  static constexpr int NWR = 4, NW = NWR * NWC, NT = 64 * NW, BM = 16 * NWR, KC = 16;
  static constexpr int NCT = (NBT * NG + NWC - 1) / NWC * NWC, CTW = NCT / NWC;   // column tiles: pass, wavefront
  static constexpr int NCB = (NCT + 1) / 2, NCC = 16 * NCB;      // load blocks of 16 columns, columns
  static constexpr bool REGG = NBT <= 3;               // Gram straight from the accumulators
  static_assert(NWC == 1 || NG == 1, "column tiles split over two wavefronts: one n'' value a pass");
  static constexpr int NPT = NBT * (NBT + 1) / 2;
  static constexpr int NPW = REGG ? NPT : (NPT + NW - 1) / NW;   // Gram tiles a wavefront holds
  // a panel: blocks of 16 columns x 64 bytes (4 k of complex128, 8 of complex64)
  static constexpr int UK = C64 ? 2 : 1, BK = 4 * UK, NBLK = (KC / BK) * NCB;
  static constexpr int DL = (NBLK + NW - 1) / NW;      // direct loads per wavefront and panel
  static constexpr int PANEL_B = NBLK * 1024;
  static constexpr bool TRASH = NBLK % NW != 0;        // the loads past the panel land in a spare KB
  static constexpr int P2_B = 4 * NCB * 1024, DL2 = (4 * NCB + NW - 1) / NW;   // panels of Y_s (complex128)
  static constexpr int MAXP = PANEL_B > P2_B ? PANEL_B : P2_B;
  static constexpr size_t KLOOP_B = 3 * (size_t)MAXP + 1024;     // (the last KB: trash)
  static constexpr int YP = 2 * NCC + 16;              // row pitch of the Gram stage (doubles)
  static constexpr size_t STAGE_B = REGG ? (size_t)NW * NPT * 256 * 8 : (size_t)BM * YP * 8;
  static constexpr size_t LDS_B = KLOOP_B > STAGE_B ? KLOOP_B : STAGE_B;
  static_assert(LDS_B * (NWC == 1 ? 2 : 1) <= 163840, "the workgroups of a CU share 160 KB of LDS");
};

template <int NBT, int NG, bool C64>
__global__ __launch_bounds__((256 * Herk64Cfg<NBT, NG, C64>::NWC), 2) void herk64_kernel(Herk64Args a) {
  using C = Herk64Cfg<NBT, NG, C64>;
  constexpr int NWC = C::NWC, NCT = C::NCT, NW = C::NW, CTW = C::CTW, BM = C::BM, KC = C::KC, DL = C::DL, DL2 = C::DL2;
  constexpr int NCB = C::NCB, NPW = C::NPW, NPT = C::NPT, YP = C::YP;
  constexpr int ESZ = C64 ? 8 : 16;
  constexpr uint32_t OOB = 0xFFFFFFF0u;                // past every resource: reads zero
  __shared__ __align__(1024) unsigned char smem[C::LDS_B];

  const WorkItem wi0 = a.items[blockIdx.x];
  const int pair = uni(wi0.pair);
  if (pair < 0) return;                                // padding of the launch order
  const int g0 = uni(wi0.g0), g1 = uni(wi0.g1), rb0 = uni(wi0.rb0), rb1 = uni(wi0.rb1);
  const PairInfo pi = a.pairs[pair];
  const int nb = uni(pi.nb), nmb = uni(pi.nmb), nd = uni(pi.nd), ldu = uni(pi.ldu);
  const int kk = uni(pi.k);
  const char* mbase = uni((const char*)a.mtab[kk]) + uni(pi.m_off) * ESZ;
  const double* Ug = a.U + uni(pi.u_off);
  const long plane = (long)ldu * ldu;

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = uni(tid >> 6), wr = w & 3, wc = w >> 2;
  const int l16 = lane & 15, lq = lane >> 4, c8 = l16 >> 1, part = l16 & 1;

  // direct loads of a panel of 4 UPB units: block b = w + NW t holds 16 columns x 64 bytes; lane l brings
  // the unit at slot l % 4 of column l / 4 (units permuted within the 64 bytes)
  auto unit_k = [&](int t, bool c64) -> int {          // first k (within the panel) of this lane's unit
    const int qd = (w + NW * t) / NCB, col16 = lane >> 2, slot = lane & 3;
    const int sw = c64 ? ((col16 >> 2) & 1) : (((col16 >> 2) & 1) + 2 * (qd & 1));
    return c64 ? qd * 8 + (slot ^ sw) * 2 : qd * 4 + (slot ^ sw);
  };
  // byte offset of this lane's unit of load t from the pass's first column (OOB: none)
  auto unit_off = [&](int t, int ng, int pitch, int row0, bool c64) -> uint32_t {
    const int b = w + NW * t, qd = b / NCB, col = (b - qd * NCB) * 16 + (lane >> 2);
    const int g = col / (8 * NBT), n = col - g * 8 * NBT;
    const bool ok = qd < (c64 ? 2 : 4) && g < ng && n < nb;
    return ok ? (uint32_t)(((g * nb + n) * pitch + row0 + unit_k(t, c64)) * (c64 ? 8 : 16)) : OOB;
  };
  auto rd = [&](const unsigned char* p) -> double {
    if constexpr (C64) return (double)*(const float*)p;
    else return *(const double*)p;
  };

  d4_t gacc[NPW];
#pragma unroll
  for (int s = 0; s < NPW; ++s) gacc[s] = d4_t{0, 0, 0, 0};
  // REGG: the products of one k step's operands (one per column tile) into the Gram tiles
  auto gram_step = [&](auto&& op) {
    static_for<0, NG>([&](auto gc) {
      constexpr int g = decltype(gc)::value;
      static_for<0, NBT>([&](auto jc) {
        constexpr int J = decltype(jc)::value;
        static_for<0, J + 1>([&](auto ic) {
          constexpr int I = decltype(ic)::value, tp = J * (J + 1) / 2 + I;
          gacc[tp] = mfma(op(g * NBT + I), op(g * NBT + J), gacc[tp]);
        });
      });
    });
  };
  // LDS form: this wavefront's Gram tiles (w + NW s; past the last one, that one again, not written) over NS
  // steps of 4 rows read through addr(column tile, step)
  auto gram_lds = [&](int ng, auto ns_c, auto&& addr) {
    constexpr int NS = decltype(ns_c)::value;
#pragma unroll
    for (int s = 0; s < NPW; ++s) {
      int I, J;
      tp_to_ij(min(w + NW * s, NPT - 1), I, J);
      for (int g = 0; g < ng; ++g) {
#pragma unroll 1
        for (int k0 = 0; k0 < NS; k0 += 4) {
          double x[4], y[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            x[u] = addr(g * NBT + I, k0 + u);
            y[u] = addr(g * NBT + J, k0 + u);
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) gacc[s] = mfma(x[u], y[u], gacc[s]);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  for (int gbase = g0; gbase < g1; gbase += NG) {
    const int ng = min(NG, g1 - gbase);

    // ================= block-sparse rows =================
    if (rb0 == 0 && a.n_s > 0) {
      const int ldw = uni(pi.ldw), np = (a.n_s + KC - 1) / KC;
      const auto rs = make_rsrc((const char*)(a.ws + uni(pi.ws_off) + (long)gbase * nb * ldw), (uint32_t)((long)ng * nb * ldw * 16));
      uint32_t vo[DL2];
#pragma unroll
      for (int t = 0; t < DL2; ++t) vo[t] = unit_off(t, ng, ldw, 0, false);
      uint32_t adr[4];
#pragma unroll
      for (int s = 0; s < 4; ++s)
        adr[s] = lq * NCB * 1024 + c8 * 64 + ((s ^ (((c8 >> 2) & 1) + 2 * (lq & 1))) * 16) + part * 8;
      auto issue2 = [&](int p) {
#pragma unroll
        for (int t = 0; t < DL2; ++t) {
          const int b = w + NW * t;
          unsigned char* dst = smem + (b < 4 * NCB ? (p % 3) * C::P2_B + b * 1024 : 3 * C::MAXP);
          lds_load16(rs, dst, p * KC + unit_k(t, false) < a.n_s ? vo[t] : OOB, (uint32_t)(p * KC * 16));
        }
      };
      __syncthreads();
      issue2(0);
      if (np > 1) issue2(1);
      for (int p = 0; p < np; ++p) {
        if (p + 1 < np) wait_vm<DL2>();                // panel p landed, p + 1 may fly
        else wait_vm<0>();
        __syncthreads();                               // (every wavefront is past panel p - 1, whose
        if (p + 2 < np) issue2(p + 2);                 //  buffer takes panel p + 2)
        const unsigned char* pb = smem + (p % 3) * C::P2_B;
        if constexpr (C::REGG) {
          const unsigned char* pl = pb + (w == 0 ? adr[0] : (w == 1 ? adr[1] : (w == 2 ? adr[2] : adr[3])));
          double op[NCT];
#pragma unroll
          for (int j = 0; j < NCT; ++j) op[j] = *(const double*)(pl + j * 512);
          gram_step([&](int j) { return op[j]; });
        } else {
          gram_lds(ng, std::integral_constant<int, 4>{}, [&](int ct, int ks) { return *(const double*)(pb + adr[ks] + ct * 512); });
        }
      }
    }

    // ================= dense rows: blocks of 64 =================
    const int r_lo = max(rb0 - 1, 0) * BM, r_hi = min(nd, (rb1 - 1) * BM);
    const auto mrs = make_rsrc(mbase + (long)gbase * nb * nmb * ESZ, (uint32_t)((long)ng * nb * nmb * ESZ));
    uint32_t voff[DL];
#pragma unroll
    for (int t = 0; t < DL; ++t) voff[t] = unit_off(t, ng, nmb, a.n_s, C64);
    // LDS byte offset (within a panel) of this lane's operand of its first column tile, step s: k = 4 lq + s
    uint32_t adr[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      if constexpr (C64)
        adr[s] = wc * CTW * 512 + (lq >> 1) * NCB * 1024 + c8 * 64 +
                 ((((lq & 1) * 2 + (s >> 1)) ^ ((c8 >> 2) & 1)) * 16) + (s & 1) * 8 + part * 4;
      else
        adr[s] = wc * CTW * 512 + lq * NCB * 1024 + c8 * 64 + ((s ^ (((c8 >> 2) & 1) + 2 * (lq & 1))) * 16) + part * 8;
    }
    constexpr uint32_t PFLIP = C64 ? 4 : 8;            // the other part of the same value
    const uint32_t sgn = part == 0 ? 0x80000000u : 0u; // -Im in the real columns of the second product
    for (int r0 = r_lo; r0 < r_hi; r0 += BM) {
      const int rw = r0 + 16 * wr;                     // this wavefront's first row
      const int np = (nd - r0 + KC - 1) / KC;          // K panels (r0 is a multiple of KC)
      // panels before this one meet only zeros of the triangular factor in this wavefront's rows
      const int pact = rw < nd ? wr : np;
      // the panel of k [r0 + p KC, + KC) into its buffer; k at or past N_d read zero
      auto issue = [&](int p) {
        const int kc = r0 + p * KC;
#pragma unroll
        for (int t = 0; t < DL; ++t) {
          const int b = w + NW * t;
          unsigned char* dst = smem + (!C::TRASH || b < C::NBLK ? (p % 3) * C::PANEL_B + b * 1024 : 3 * C::MAXP);
          uint32_t vo = voff[t];
          if (kc + KC > nd && kc + unit_k(t, C64) >= nd) vo = OOB;
          lds_load16(mrs, dst, vo, (uint32_t)(kc * ESZ));
        }
      };
      // the factor of panel p: lane (l16, lq) takes k = 4 lq .. 4 lq + 3 of row l16
      const double* fp = Ug + (long)(rw + l16) * ldu + r0 + 4 * lq;
      struct Fac { double2 r0, r1, i0, i1; };
      auto load_f = [&](int p) -> Fac {
        const double2 *q = (const double2*)(fp + p * KC), *qi = (const double2*)(fp + plane + p * KC);
        return Fac{q[0], q[1], qi[0], qi[1]};
      };
      d4_t yacc[CTW];
#pragma unroll
      for (int j = 0; j < CTW; ++j) yacc[j] = d4_t{0, 0, 0, 0};
      __syncthreads();                                 // LDS of the previous phase is free
      issue(0);
      Fac f = load_f(0), fn = f;
      if (np > 1) {
        issue(1);
        wait_vm<DL>();
      } else {
        wait_vm<0>();
      }
      __syncthreads();
      // requests of iteration p: the next panel's factor, then the raw panel two ahead (so that waiting for the
      // former leaves the latter in flight); at its end panel p + 1 has landed for every wavefront
      auto request = [&](int p) {
        if (p + 1 < np) fn = load_f(p + 1);
        if (p + 2 < np) issue(p + 2);
      };
      auto finish = [&](int p) {
        if (p + 2 < np) wait_vm<DL>();
        else wait_vm<0>();
        __syncthreads();
        f = fn;
      };
      int p = 0;
      for (; p < min(pact, np); ++p) {
        request(p);
        finish(p);
      }
      for (; p < np; ++p) {
        request(p);
        const unsigned char* pb = smem + (p % 3) * C::PANEL_B;
        const int klim = nd - (r0 + p * KC) - 4 * lq;  // (complex64: a unit may straddle N_d)
        const double fr[4] = {f.r0.x, f.r0.y, f.r1.x, f.r1.y}, fi[4] = {f.i0.x, f.i0.y, f.i1.x, f.i1.y};
        // operands two column tiles ahead of their products
        auto bload = [&](int s, int hj) -> double {
          const int h = hj >= CTW, j = h ? hj - CTW : hj;
          double x = rd(pb + (h ? adr[s] ^ PFLIP : adr[s]) + j * 512);
          if (C64 && s >= klim) x = 0.0;
          return x;
        };
        constexpr int N = 8 * CTW;                     // products of a panel: (step, Re / Im of the factor, tile)
        double b[3];
        b[0] = bload(0, 0);
        b[1] = bload(N > 2 * CTW ? 1 / (2 * CTW) : 0, 1 % (2 * CTW));
        static_for<0, N>([&](auto ic) {
          constexpr int i = decltype(ic)::value, s = i / (2 * CTW), hj = i % (2 * CTW);
          constexpr int i2 = i + 2;
          if constexpr (i2 < N) b[i2 % 3] = bload(i2 / (2 * CTW), i2 % (2 * CTW));
          if constexpr (hj >= CTW) {
            const double x = __hiloint2double(__double2hiint(b[i % 3]) ^ (int)sgn, __double2loint(b[i % 3]));
            yacc[hj - CTW] = mfma(fi[s], x, yacc[hj - CTW]);
          } else {
            yacc[hj] = mfma(fr[s], b[i % 3], yacc[hj]);
          }
          __builtin_amdgcn_sched_barrier(0);
        });
        finish(p);
      }
      // ---- contraction of the block's rows ----
      if constexpr (C::REGG) {
#pragma unroll
        for (int i = 0; i < 4; ++i) gram_step([&](int j) { return yacc[j][i]; });
      } else {
        double* Ys = (double*)smem;                    // [64 rows][YP]
#pragma unroll
        for (int j = 0; j < CTW; ++j)
#pragma unroll
          for (int i = 0; i < 4; ++i) Ys[(16 * wr + lq + 4 * i) * YP + (wc * CTW + j) * 16 + l16] = yacc[j][i];
        __syncthreads();
        const double* yl = Ys + lq * YP + l16;
        gram_lds(ng, std::integral_constant<int, 16>{}, [&](int ct, int ks) { return yl[4 * ks * YP + ct * 16]; });
      }
    }
  }

  // ---- the item's Gram tiles to its slot (tiles left out by the band mask: zeros) ----
  double* gp = a.gpart + (long)uni(wi0.slot) * a.gstride;
  const int nbt = (nb + 7) >> 3, npt = nbt * (nbt + 1) / 2;
  auto kept = [&](int tp) -> bool { return !a.tmask || ((a.tmask[3 * kk + (tp >> 6)] >> (tp & 63)) & 1); };
  if constexpr (C::REGG) {
    double* red = (double*)smem;                       // [NW][NPT][4][64]
    __syncthreads();
#pragma unroll
    for (int s = 0; s < NPW; ++s)
#pragma unroll
      for (int i = 0; i < 4; ++i) red[((w * NPT + s) * 4 + i) * 64 + lane] = gacc[s][i];
    __syncthreads();
    for (int e = tid; e < npt * 256; e += C::NT) {
      double x = red[e];
#pragma unroll
      for (int v = 1; v < NW; ++v) x += red[v * NPT * 256 + e];
      gp[e] = kept(e >> 8) ? x : 0.0;
    }
  } else {
#pragma unroll
    for (int s = 0; s < NPW; ++s) {
      const int tp = w + NW * s;
      if (tp < npt) {
        const bool k1 = kept(tp);
#pragma unroll
        for (int i = 0; i < 4; ++i) gp[(tp * 4 + i) * 64 + lane] = k1 ? gacc[s][i] : 0.0;
      }
    }
  }
}

}  // namespace exc
