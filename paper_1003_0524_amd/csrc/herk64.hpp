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
//  * Requests run ahead of everything: panels two ahead, the factor one, operands four column tiles ahead of their
//    products, the next block's first panel and factor while this one is contracted; row tiles rotate over the
//    wavefronts from block to block, so that the short ones (a triangular factor) meet every SIMD.
//  * Block-sparse rows: a chunk of whole channels (at most 16 rows, four multipole rows) per wavefront, formed as
//    W A on the matrix cores with W's 16 x 20 entries gathered from the channel factors and M's rows read straight
//    into operand registers, a tile or more ahead: no LDS, no barrier (forming them on the vector cores from rows in
//    LDS takes a fifth of the multiplications, but is bound by LDS reads and took 630 us where this takes 530 for
//    one outer iteration of the Si-like workload; a kernel of its own before this one, 680 us: it writes and this
//    one reads 240 MB). Where a channel is longer than a chunk sparse_kernel writes Y_s and its panels are read here.
//  * Gram tiles stay in registers for the whole item. The accumulator layout of the
//    16x16x4 instruction (lane group lq, element i: row lq + 4 i) is its operand layout for
//    k = rows 4 i .. 4 i + 3, so with at most three band tiles a wavefront contracts its 16
//    rows straight from its accumulators into its own copy of all Gram tiles (summed over
//    the wavefronts once per item); with more, the 64 rows pass through LDS and each
//    wavefront holds its share of the tiles.
//
// Measured against the kernel it replaces (tile_kernel's FP64 instances: one item per pair, operands through
// registers, Gram tiles of more than three band tiles added in global memory once per 64 rows): one outer
// iteration of the Si-like workload 844 -> 530 us; one k of the ZnO-like one (144 pairs, which left 112 of the
// 256 CUs without work) 30.8 -> 6.9 ms, 50 TFLOP/s of its real work where a large matrix product reaches 70; one k
// of eight small pairs (N_MB 300, 16 bands) 299 -> 28 us.
//
// Partial slots: [tile pair][element i][lane], rows and columns of a tile interleaved as above.
#pragma once
#include "common.hpp"
#include "tile.hpp"
#include "wide.hpp"

namespace exc {

// A chunk of block-sparse rows: rows [row, row + rows) of whole channels, their first multipole row.
struct Chunk64 { int32_t row, rows, mp, pad; };

struct Herk64Args {
  const PairInfo* pairs;
  const WorkItem* items;
  int32_t n_items;
  const void* const* mtab;       // [n_k] device pointers to M_k
  int32_t n_s, n_occ;
  const double* U;               // factor planes (re, im) of L22^H
  const double2* ws;             // block-sparse rows Y_s (sparse_kernel), when n_chunk is 0
  const Chunk64* chunks;         // [n_chunk] of whole channels
  int32_t n_chunk;               // 0: Y_s comes from ws
  const int4* rowinfo;           // [n_s] {run start in coef, run length, multipole row}
  const double2* coef;           // channel factors L_c
  const double2* cvec;           // [n_s] l_c
  int64_t coef_qs, cvec_qs;      // elements between the copies of q and q + 1 (0: one copy)
  double* gpart;                 // Gram partials
  int32_t gstride;
  const uint64_t* tmask;         // [n_k][3] band-tile pairs to compute
};

// chunks of the block-sparse rows: whole channels, one panel of rows and four (consecutive) multipole rows at most
constexpr int kH64Rows = 16, kH64MP = 4;

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
  // LDS of the dense rows: two panel buffers where the Gram stage goes at the end of a block, and a third one for
  // every third panel, the first of a block among them (requested before the block ahead of it is contracted)
  static constexpr int SROW = (NCT + 1) / 2 * 256;     // bytes of a stage row
  static constexpr size_t STAGE_B = REGG ? 0 : (size_t)BM * SROW;
  static constexpr size_t EOFF = STAGE_B > 2 * (size_t)PANEL_B ? STAGE_B : 2 * (size_t)PANEL_B;
  static constexpr size_t DENSE_B = EOFF + PANEL_B + (TRASH ? 1024 : 0);
  static constexpr size_t WS_B = 3 * (size_t)P2_B + 1024;   // three panels of Y_s
  static constexpr size_t RED_B = REGG ? (size_t)NW * NPT * 256 * 8 : 0;
  static constexpr size_t max2(size_t x, size_t y) { return x > y ? x : y; }
  static constexpr size_t LDS_B = max2(DENSE_B, max2(WS_B, RED_B));
  static_assert(LDS_B * (NWC == 1 ? 2 : 1) <= 163840, "the workgroups of a CU share 160 KB of LDS");
};

template <int NBT, int NG, bool C64>
__global__ __launch_bounds__((256 * Herk64Cfg<NBT, NG, C64>::NWC), 2) void herk64_kernel(Herk64Args a) {
  using C = Herk64Cfg<NBT, NG, C64>;
  constexpr int NWC = C::NWC, NCT = C::NCT, NW = C::NW, CTW = C::CTW, BM = C::BM, KC = C::KC, DL = C::DL, DL2 = C::DL2;
  constexpr int NCB = C::NCB, NPW = C::NPW, NPT = C::NPT;
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

  const int tid = threadIdx.x;
  const int w = uni(tid >> 6), wc = w >> 2;
  // the lane index, opaque per use: each phase forms its addresses afresh instead of keeping those of every
  // phase live (or spilled) through the others
  auto lane_id = [&]() -> int {
    int l = tid & 63;
    asm volatile("" : "+v"(l));
    return l;
  };

  // direct loads of a panel of 4 UPB units: block b = w + NW t holds 16 columns x 64 bytes; lane l brings
  // the unit at slot l % 4 of column l / 4 (units permuted within the 64 bytes)
  auto unit_k = [&](int lane, int t, bool c64) -> int {   // first k (within the panel) of this lane's unit
    const int qd = (w + NW * t) / NCB, col16 = lane >> 2, slot = lane & 3;
    const int sw = c64 ? ((col16 >> 2) & 1) : (((col16 >> 2) & 1) + 2 * (qd & 1));
    return c64 ? qd * 8 + (slot ^ sw) * 2 : qd * 4 + (slot ^ sw);
  };
  // byte offset of this lane's unit of load t from the pass's first column (OOB: none)
  auto unit_off = [&](int lane, int t, int ng, int pitch, int row0, bool c64) -> uint32_t {
    const int b = w + NW * t, qd = b / NCB, col = (b - qd * NCB) * 16 + (lane >> 2);
    const int g = col / (8 * NBT), n = col - g * 8 * NBT;
    const bool ok = qd < (c64 ? 2 : 4) && g < ng && n < nb;
    return ok ? (uint32_t)(((g * nb + n) * pitch + row0 + unit_k(lane, t, c64)) * (c64 ? 8 : 16)) : OOB;
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

  // contraction of 64 rows, 16 of them (row tile wr) in this wavefront's accumulators
  auto contract = [&](const d4_t (&yacc)[CTW], int wr, int ng) {
    if constexpr (C::REGG) {
#pragma unroll
      for (int i = 0; i < 4; ++i) gram_step([&](int j) { return yacc[j][i]; });
    } else {
      // stage [64 rows][column tile][16]: odd rows swap neighbouring tiles, so that the rows of a half-wave's
      // operand read meet distinct banks
      const int lane = lane_id(), l16 = lane & 15, lq = lane >> 4;
#pragma unroll
      for (int j = 0; j < CTW; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int ct = wc * CTW + j;
          *(double*)(smem + (16 * wr + lq + 4 * i) * C::SROW + ((ct ^ (lq & 1)) * 128) + l16 * 8) = yacc[j][i];
        }
      lds_barrier();
      gram_lds(ng, std::integral_constant<int, 16>{}, [&](int ct, int ks) {
        return *(const double*)(smem + (4 * ks + lq) * C::SROW + ((ct ^ (lq & 1)) * 128) + l16 * 8);
      });
      lds_barrier();                                 // the stage is free
    }
  };

  // ================= block-sparse rows of a pass =================
  // 64 rows at a time, a chunk of 16 per wavefront: Y_s = W A with W[r][k] = conj(L_c[k - r]) for the chunk's own rows
  // k and l_c for its multipole rows, five steps of four k
  auto sparse_rows = [&](int gbase, int ng) {
    if (a.n_chunk > 0) {
      const int lane = lane_id(), l16 = lane & 15, lq = lane >> 4, c8 = l16 >> 1, part = l16 & 1, wr = w & 3;
      constexpr int R = CTW % 2 == 0 ? 2 : (CTW % 3 == 0 ? 3 : 1);   // tiles in flight
      using raw_t = std::conditional_t<C64, u2_t, u4_t>;
      const int q = uni(pi.q);
      const double2 *coef = a.coef + q * a.coef_qs, *cvec = a.cvec + q * a.cvec_qs;
      const auto rs = make_rsrc(mbase + (long)gbase * nb * nmb * ESZ, (uint32_t)((long)ng * nb * nmb * ESZ));
      // this lane's column of each tile, no column: past every resource also with a row's offset added (0xFFFFFFF0
      // would wrap around to the first columns)
      constexpr uint32_t NOCOL = 0xFFFFFF00u;
      static_assert((kH64Rows - 1) * 16 <= 0xF0, "NOCOL with a row's offset");
      uint32_t co[CTW];
#pragma unroll
      for (int j = 0; j < CTW; ++j) {
        const int ct = wc * CTW + j, g = ct / NBT, n = (ct - g * NBT) * 8 + c8;
        co[j] = g < ng && n < nb ? (uint32_t)((g * nb + n) * nmb * ESZ) : NOCOL;
      }
      // A load brings rows 8 i + 2 lq + part of the chunk (i = 0, 1): a lane holds one of the two rows that the
      // lanes of its column contract in steps 2 i and 2 i + 1 and gets the other one from its neighbour
      struct Tile { raw_t a[2], m; };
      struct Desc { int row, rows, mp; };
      const auto* chunks = (const __attribute__((address_space(4))) Chunk64*)a.chunks;   // (scalar loads)
      auto desc = [&](int ck) -> Desc {
        const auto* p = chunks + min(ck, a.n_chunk - 1);
        return Desc{p->row, ck < a.n_chunk ? p->rows : 0, p->mp};
      };
      auto load = [&](const Desc& d, int j) -> Tile {
        Tile t;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const int k = 8 * i + 2 * lq + part;
          t.a[i] = buf_load<raw_t>(rs, k < d.rows ? co[j] + k * ESZ : OOB, (uint32_t)(d.row * ESZ));
        }
        t.m = buf_load<raw_t>(rs, d.mp + lq < nmb && d.rows > 0 ? co[j] + lq * ESZ : OOB, (uint32_t)(d.mp * ESZ));
        return t;
      };
      auto re = [](raw_t v) -> double {
        if constexpr (C64) return (double)__uint_as_float(v.x);
        else return __hiloint2double((int)v.y, (int)v.x);
      };
      auto im = [](raw_t v) -> double {
        if constexpr (C64) return (double)__uint_as_float(v.y);
        else return __hiloint2double((int)v.w, (int)v.z);
      };
      auto swap = [](raw_t v) -> raw_t {               // the neighbouring lane's value
#pragma unroll
        for (int i = 0; i < (int)(sizeof(raw_t) / 4); ++i)
          v[i] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v[i], 0xB1, 0xF, 0xF, true);
        return v;
      };
      // W of a chunk for this lane's row: steps 0..3 its own rows, step 4 the multipole rows
      struct Fac { d2_t v[5]; };
      auto factor = [&](const Desc& d, u4_t ri) -> Fac {
        Fac x;
        const int r = min(l16, max(d.rows - 1, 0)), len = l16 < d.rows ? (int)ri.y : 0;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const int t = 8 * (s >> 1) + 2 * lq + (s & 1) - r;
          const bool ok = t >= 0 && t < len;
          const double2 v = coef[(int)ri.x + (ok ? t : 0)];
          x.v[s] = d2_t{ok ? v.x : 0.0, ok ? -v.y : 0.0};
        }
        const double2 v = cvec[d.row + r];
        const bool ok = len > 0 && (int)ri.z - d.mp == lq;
        x.v[4] = d2_t{ok ? v.x : 0.0, ok ? v.y : 0.0};
        return x;
      };
      auto rinfo = [&](const Desc& d) -> u4_t { return ((const u4_t*)a.rowinfo)[d.row + min(l16, max(d.rows - 1, 0))]; };
      const uint32_t sgn = part == 0 ? 0x80000000u : 0u;
      auto neg = [&](double x) -> double { return __hiloint2double(__double2hiint(x) ^ (int)sgn, __double2loint(x)); };
      Desc d = desc(wr);
      Tile t[R];
#pragma unroll
      for (int j = 0; j < R; ++j) t[j] = load(d, j);
      Fac f = factor(d, rinfo(d));
      lds_barrier();                                   // LDS of the previous phase is free
      for (int ck = wr; ck < a.n_chunk + wr; ck += 4) {  // (the same count for every wavefront)
        const Desc dn = desc(ck + 4);
        const u4_t rin = rinfo(dn);
        d4_t yacc[CTW];
        static_for<0, CTW>([&](auto jc) {
          constexpr int j = decltype(jc)::value;
          const Tile c = t[j % R];
          t[j % R] = j + R < CTW ? load(d, j + R) : load(dn, j + R - CTW);
          d4_t y{0, 0, 0, 0};
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const raw_t o = swap(c.a[i]);
            const double vr = re(c.a[i]), vi = im(c.a[i]), xr = re(o), xi = im(o);
            y = mfma(f.v[2 * i].x, part ? xi : vr, y);
            y = mfma(f.v[2 * i].y, neg(part ? xr : vi), y);
            y = mfma(f.v[2 * i + 1].x, part ? vi : xr, y);
            y = mfma(f.v[2 * i + 1].y, neg(part ? vr : xi), y);
          }
          y = mfma(f.v[4].x, part ? im(c.m) : re(c.m), y);
          y = mfma(f.v[4].y, neg(part ? re(c.m) : im(c.m)), y);
          yacc[j] = y;
          __builtin_amdgcn_sched_barrier(0);
        });
        d = dn;
        f = factor(dn, rin);
        contract(yacc, wr, ng);
      }
    }
    if (a.n_s > 0 && a.n_chunk == 0) {
      const int lane = lane_id(), l16 = lane & 15, lq = lane >> 4, c8 = l16 >> 1, part = l16 & 1;
      const int ldw = uni(pi.ldw), np = (a.n_s + KC - 1) / KC;
      const auto rs = make_rsrc((const char*)(a.ws + uni(pi.ws_off) + (long)gbase * nb * ldw), (uint32_t)((long)ng * nb * ldw * 16));
      uint32_t vo[DL2];
#pragma unroll
      for (int t = 0; t < DL2; ++t) vo[t] = unit_off(lane, t, ng, ldw, 0, false);
      uint32_t adr[4];
#pragma unroll
      for (int s = 0; s < 4; ++s)
        adr[s] = lq * NCB * 1024 + c8 * 64 + ((s ^ (((c8 >> 2) & 1) + 2 * (lq & 1))) * 16) + part * 8;
      auto issue2 = [&](int p) {
#pragma unroll
        for (int t = 0; t < DL2; ++t) {
          const int b = w + NW * t;
          unsigned char* dst = smem + (b < 4 * NCB ? (p % 3) * C::P2_B + b * 1024 : 3 * C::P2_B);
          lds_load16(rs, dst, p * KC + unit_k(lane, t, false) < a.n_s ? vo[t] : OOB, (uint32_t)(p * KC * 16));
        }
      };
      lds_barrier();
      issue2(0);
      issue2(1);                                       // (panels past the last row: out of range, no memory touched)
      for (int p = 0; p < np; ++p) {
        wait_vm<DL2>();                                // panel p landed, p + 1 may fly
        lds_barrier();                                 // (every wavefront is past panel p - 1, whose
        issue2(p + 2);                                 //  buffer takes panel p + 2)
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
      wait_vm<0>();
    }
  };

  for (int gbase = g0; gbase < g1; gbase += NG) {
    const int ng = min(NG, g1 - gbase);
    if (rb0 == 0) sparse_rows(gbase, ng);
    // ================= dense rows: blocks of 64 =================
    const int lane = lane_id(), l16 = lane & 15, lq = lane >> 4, c8 = l16 >> 1, part = l16 & 1;
    const int r_lo = max(rb0 - 1, 0) * BM, r_hi = min(nd, (rb1 - 1) * BM);
    const auto mrs = make_rsrc(mbase + (long)gbase * nb * nmb * ESZ, (uint32_t)((long)ng * nb * nmb * ESZ));
    uint32_t voff[DL];
#pragma unroll
    for (int t = 0; t < DL; ++t) voff[t] = unit_off(lane, t, ng, nmb, a.n_s, C64);
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
    // the panel of k [r0 + p KC, + KC) into its buffer; k at or past N_d read zero
    auto panel_at = [&](int p) -> unsigned char* { return smem + (p % 3 == 0 ? C::EOFF : (size_t)(p % 3 - 1) * C::PANEL_B); };
    auto issue = [&](int r0, int p) {
      const int kc = r0 + p * KC;
      unsigned char* pb = panel_at(p);
#pragma unroll
      for (int t = 0; t < DL; ++t) {
        const int b = w + NW * t;
        unsigned char* dst = !C::TRASH || b < C::NBLK ? pb + b * 1024 : smem + C::EOFF + C::PANEL_B;
        uint32_t vo = voff[t];
        if (kc + KC > nd && kc + unit_k(lane, t, C64) >= nd) vo = OOB;
        lds_load16(mrs, dst, vo, (uint32_t)(kc * ESZ));
      }
    };
    // the factor of panel p for this wavefront's 16 rows of the block (row tiles rotate over the wavefronts, so that
    // the short and the full ones meet every SIMD in turn): lane (l16, lq) takes k = 4 lq .. 4 lq + 3 of row l16
    auto row_tile = [&](int r0) { return (w + r0 / BM) & 3; };
    struct Fac { u4_t r0, r1, i0, i1; };
    const uint32_t f_lane = (uint32_t)((l16 * ldu + 4 * lq) * 8);
    auto load_f = [&](int r0, int p) -> Fac {
      const double* fp = Ug + (long)(r0 + 16 * row_tile(r0)) * ldu;   // (16 rows: within the factor's padded order)
      const auto rr = make_rsrc(fp, (uint32_t)(16 * ldu * 8)), ri = make_rsrc(fp + plane, (uint32_t)(16 * ldu * 8));
      const uint32_t so = (uint32_t)((r0 + p * KC) * 8);
      return Fac{buf_load<u4_t>(rr, f_lane, so), buf_load<u4_t>(rr, f_lane + 16, so), buf_load<u4_t>(ri, f_lane, so),
                 buf_load<u4_t>(ri, f_lane + 16, so)};
    };
    Fac f, fn;
    if (r_lo < r_hi) {
      __syncthreads();                                 // LDS of the previous phase is free
      issue(r_lo, 0);
      f = load_f(r_lo, 0);
    }
    for (int r0 = r_lo; r0 < r_hi; r0 += BM) {
      const int wr = row_tile(r0);
      const int rw = r0 + 16 * wr;                     // this wavefront's first row
      const int np = (nd - r0 + KC - 1) / KC;          // K panels (r0 is a multiple of KC)
      // panels before this one meet only zeros of the triangular factor in this wavefront's rows
      const int pact = rw < nd ? wr : np;
      d4_t yacc[CTW];
#pragma unroll
      for (int j = 0; j < CTW; ++j) yacc[j] = d4_t{0, 0, 0, 0};
      issue(r0, 1);
      wait_vm<DL>();
      lds_barrier();
      // requests of iteration p: the next panel's factor, then the raw panel two ahead (so that waiting for the
      // former leaves the latter in flight); at its end panel p + 1 has landed for every wavefront. Past the last
      // panel the requests go on (that factor again; loads whose every offset is out of range touch no memory): with
      // the same loads in flight on every path the compiler's own waits can count them
      auto request = [&](int p) {
        fn = load_f(r0, min(p + 1, np - 1));
        issue(r0, p + 2);
      };
      auto finish = [&]() {
        wait_vm<DL>();
        f = fn;
        lds_barrier();
      };
      int p = 0;
      for (; p < min(pact, np); ++p) {
        request(p);
        finish();
      }
      for (; p < np; ++p) {
        request(p);
        const unsigned char* pb = panel_at(p);
        const int klim = nd - (r0 + p * KC) - 4 * lq;  // (complex64: a unit may straddle N_d)
        auto lo = [](u4_t v) { return __hiloint2double((int)v.y, (int)v.x); };
        auto hi = [](u4_t v) { return __hiloint2double((int)v.w, (int)v.z); };
        const double fr[4] = {lo(f.r0), hi(f.r0), lo(f.r1), hi(f.r1)}, fi[4] = {lo(f.i0), hi(f.i0), lo(f.i1), hi(f.i1)};
        // operands D column tiles ahead of their products (an LDS read outlasts two products)
        constexpr int D = CTW >= 2 ? 4 : 2;
        auto bload = [&](int s, int hj) -> double {
          const int h = hj >= CTW, j = h ? hj - CTW : hj;
          double x = rd(pb + (h ? adr[s] ^ PFLIP : adr[s]) + j * 512);
          if (C64 && s >= klim) x = 0.0;
          return x;
        };
        constexpr int N = 8 * CTW;                     // products of a panel: (step, Re / Im of the factor, tile)
        double b[D + 1];
#pragma unroll
        for (int i = 0; i < D; ++i) b[i] = bload(i / (2 * CTW), i % (2 * CTW));
        static_for<0, N>([&](auto ic) {
          constexpr int i = decltype(ic)::value, s = i / (2 * CTW), hj = i % (2 * CTW);
          constexpr int i2 = i + D;
          if constexpr (i2 < N) b[i2 % (D + 1)] = bload(i2 / (2 * CTW), i2 % (2 * CTW));
          if constexpr (hj >= CTW) {
            const double x = __hiloint2double(__double2hiint(b[i % (D + 1)]) ^ (int)sgn, __double2loint(b[i % (D + 1)]));
            yacc[hj - CTW] = mfma(fi[s], x, yacc[hj - CTW]);
          } else {
            yacc[hj] = mfma(fr[s], b[i % (D + 1)], yacc[hj]);
          }
          __builtin_amdgcn_sched_barrier(0);
        });
        finish();
      }
      wait_vm<0>();                                    // the panels past the end, before their buffers are reused
      lds_barrier();
      // the next block's first panel and factor are requested before this block is contracted
      if (r0 + BM < r_hi) {
        issue(r0 + BM, 0);
        f = load_f(r0 + BM, 0);
      }
      contract(yacc, wr, ng);
    }
  }

  // ---- the item's Gram tiles to its slot (tiles left out by the band mask: zeros) ----
  const int lane = lane_id();
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
