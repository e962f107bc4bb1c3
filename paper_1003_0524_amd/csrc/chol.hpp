// Dense Cholesky of the (Schur-updated) blocks E(q) = L22 L22^H of every q, FP64, lower triangle in place, one block
// column of 64 at a time (left-looking): chol_update_kernel brings the 64-row tiles of the column up to date (and
// factors the diagonal tile), chol_solve_kernel solves the tiles below it.
//
// Bound by the FP64 matrix cores in the middle of the factorisation, by the diagonal tile's serial chain (about
// 28 us a column) and by few tiles at its end. All tiles of all q of a column are one launch: one workgroup per q
// for the whole factorisation, its products on the vector cores, left 112 of the 256 CUs idle with 144 q and waited
// for the largest: 144 matrices of order 372-944 (ZnO-like) 18.9 -> 3.5 ms, 64 of order 310
// (Si-like) 2.4 -> 0.43 ms.
// Left-looking: a tile is read and written once, where a right-looking update would rewrite the whole trailing
// matrix (1 GB here, four times the memory-side cache) per column.
#pragma once
#include "common.hpp"
#include "tile.hpp"
#include "wide.hpp"

namespace exc {

struct CholArgs {
  double2* A;             // per-q matrices (column-major, leading dimension lda)
  const int64_t* a_off;
  const int32_t* nd;
  const int32_t* lda;
  int32_t n_ch;
  const double* schur;    // [n_ch] (per q: [n_q][n_ch]) or nullptr
  int32_t schur_qs;       // n_ch when the channel blocks depend on q, else 0
  int* info;              // [n_q] first failing pivot (1-based), 0 = ok (zero at the start)
  int32_t jb;             // block column
};

constexpr int kCholBlock = 64;

// (re, im)[m][n] += sum_k conj(a[m][k]) b[n][k] over four k: a the lane's value of row m = l16,
// b that of n = l16, k = lane group (+ the caller's step)
__device__ __forceinline__ void chol_mac(d4_t& re, d4_t& im, d2_t a, d2_t b) {
  re = mfma(a.x, b.x, re);
  im = mfma(a.x, b.y, im);
  re = mfma(a.y, b.y, re);
  im = mfma(a.y, -b.x, im);
}

// The tile of rows [64 (jb + y), + 64) of block column jb of q = blockIdx.x: C = A - L_i L_j^H over the columns
// before it. Four wavefronts of 16 rows; panels of eight columns (64 rows of the tile, 64 of the block column's own
// rows; a 1 KB load brings 64 rows of one column) go global -> LDS three ahead. Rows are the N of the products: a
// lane group's 16 lanes hold 16 consecutive rows, so tiles move in 256-byte runs.
__global__ __launch_bounds__(256, 2) void chol_update_kernel(CholArgs a) {
  constexpr int KC = 8, NBUF = 4, PANEL_B = 2 * KC * 1024, DP = kCholBlock + 1;
  constexpr size_t LDS_B = (size_t)NBUF * PANEL_B > (size_t)kCholBlock * DP * 16 ? (size_t)NBUF * PANEL_B
                                                                                : (size_t)kCholBlock * DP * 16;
  constexpr uint32_t OOB = 0xFFFFFFF0u;
  __shared__ __align__(1024) unsigned char smem[LDS_B];
  const int q = blockIdx.x, n = uni(a.nd[q]), lda = uni(a.lda[q]);
  const int j0 = a.jb * kCholBlock, i0 = j0 + (int)blockIdx.y * kCholBlock;
  if (i0 >= n) return;                                 // uniform
  double2* A = a.A + uni(a.a_off[q]);
  const int tid = threadIdx.x, lane = tid & 63, w = uni(tid >> 6), l16 = lane & 15, lq = lane >> 4;
  const int np = j0 / KC;
  const uint32_t vo[2] = {i0 + lane < n ? (uint32_t)(i0 + lane) * 16 : OOB, j0 + lane < n ? (uint32_t)(j0 + lane) * 16 : OOB};
  // panel p: loads of wavefront w are columns 4 (w & 1) .. + 3 of the tile's rows (w < 2) or the block column's
  auto issue = [&](int p) {
    const auto rs = make_rsrc(A + (long)min(p, np - 1) * KC * lda, (uint32_t)(KC * lda * 16));
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int k = 4 * (w & 1) + t;
      lds_load16(rs, smem + (p % NBUF) * PANEL_B + ((w >> 1) * KC + k) * 1024,
                 p < np ? (w < 2 ? vo[0] : vo[1]) : OOB, (uint32_t)(k * lda * 16));
    }
  };
  d4_t re[4], im[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) re[t] = im[t] = d4_t{0, 0, 0, 0};
  if (np > 0) {
    issue(0);
    issue(1);
    issue(2);
    for (int p = 0; p < np; ++p) {
      wait_vm<8>();                                    // panel p landed, two more may fly
      lds_barrier();                                   // (every wavefront is past panel p - 1)
      issue(p + 3);
      const d2_t* own = (const d2_t*)(smem + (p % NBUF) * PANEL_B) + 16 * w + l16;
      const d2_t* col = (const d2_t*)(smem + (p % NBUF) * PANEL_B + KC * 1024) + l16;
#pragma unroll
      for (int s = 0; s < KC / 4; ++s) {
        const d2_t b = own[(4 * s + lq) * 64];
        d2_t x[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) x[t] = col[(4 * s + lq) * 64 + 16 * t];
#pragma unroll
        for (int t = 0; t < 4; ++t) chol_mac(re[t], im[t], x[t], b);
      }
    }
    wait_vm<0>();                                      // (the panels past the end)
    lds_barrier();
  }
  if (blockIdx.y > 0) {
    const int row = i0 + 16 * w + l16;
    if (row < n && np > 0) {
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          double2* c = A + row + (long)(j0 + 16 * t + lq + 4 * e) * lda;
          *c = make_double2(c->x - re[t][e], c->y - im[t][e]);
        }
    }
    return;
  }

  // ---- the diagonal tile: factored in LDS (past the matrix's order: the identity), 16 columns at a time ----
  d2_t* D = (d2_t*)smem;                               // [64][DP]
  const int nb = min(kCholBlock, n - j0);
  {
    const int r = 16 * w + l16;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int c = 16 * t + lq + 4 * e;
        d2_t v{r == c ? 1.0 : 0.0, 0.0};
        if (r < nb && c <= r) {
          const double2 x = A[j0 + r + (long)(j0 + c) * lda];
          v = d2_t{x.x - re[t][e], x.y - im[t][e]};
          if (r == c && a.schur && j0 + c < a.n_ch) v.x -= a.schur[(long)q * a.schur_qs + j0 + c];
        }
        D[r * DP + c] = v;
      }
  }
  __syncthreads();
  int failed = 0;
  for (int c0 = 0; c0 < kCholBlock; c0 += 16) {
    if (w == 0) {
      // lane = row: the 16 x 16 block and the rows below it, column by column in registers
      const int r = lane;
      d2_t x[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) x[j] = D[r * DP + c0 + j];
      auto bcast = [&](double v, int from) -> double {
        return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), from),
                                __builtin_amdgcn_readlane(__double2loint(v), from));
      };
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        double d = bcast(x[j].x, c0 + j);
        if (!(d > 0.0)) {
          if (!failed) failed = j0 + c0 + j + 1;
          d = 1.0;
        }
        d = sqrt(d);
        x[j] = r == c0 + j ? d2_t{d, 0.0} : d2_t{x[j].x / d, x[j].y / d};
#pragma unroll
        for (int m = j + 1; m < 16; ++m) {
          const double lr = bcast(x[j].x, c0 + m), li = bcast(x[j].y, c0 + m);
          x[m].x -= x[j].x * lr + x[j].y * li;
          x[m].y -= x[j].y * lr - x[j].x * li;
        }
      }
#pragma unroll
      for (int j = 0; j < 16; ++j)
        if (r >= c0 + j) D[r * DP + c0 + j] = x[j];
    }
    __syncthreads();
    // the columns after them: lane = row, a wavefront takes every fourth column
    if (c0 + 16 < kCholBlock) {
      const int r = lane;
      d2_t x[16];
#pragma unroll
      for (int p = 0; p < 16; ++p) x[p] = D[r * DP + c0 + p];
      for (int c = c0 + 16 + w; c < kCholBlock; c += 4) {
        d2_t v = D[r * DP + c];
#pragma unroll
        for (int p = 0; p < 16; ++p) {
          const d2_t l = D[c * DP + c0 + p];
          v.x -= x[p].x * l.x + x[p].y * l.y;
          v.y -= x[p].y * l.x - x[p].x * l.y;
        }
        if (r >= c) D[r * DP + c] = v;
      }
      __syncthreads();
    }
  }
  for (int c = w; c < nb; c += 4)
    if (lane < nb && lane >= c) {
      const d2_t v = D[lane * DP + c];
      A[j0 + lane + (long)(j0 + c) * lda] = make_double2(v.x, v.y);
    }
  if (tid == 0 && failed && a.info[q] == 0) a.info[q] = failed;
}

// X L_jj^H = C for the 64 rows from 64 (jb + 1 + y) of block column jb, 16 rows per wavefront and 16 columns at a
// time: X_b by substitution against the diagonal block L_bb, then C_c -= X_b L_cb^H for the blocks after it on the
// matrix cores. The accumulator layout of the products is their operand layout (lane group lq, element e: column
// lq + 4 e), so the rows stay in registers from their load to their store; in the substitution the lane group of column
// j passes it to the others, which subtract it from their columns. (Products with the inverted diagonal block are
// shorter, but their residual grows with the block's condition: 80 functions, 16 of them with an inverse of 1e4, take
// E - L L^H to twice the bound that substitution keeps to within a hundredth of. The time is the same, 8.5 ms for a
// context of the ZnO-like workload.)
__global__ __launch_bounds__(256) void chol_solve_kernel(CholArgs a) {
  __shared__ d2_t Ld[4][16][16];                       // diagonal blocks: [block][column][row], rows >= column
  const int q = blockIdx.x, n = uni(a.nd[q]), lda = uni(a.lda[q]);
  const int j0 = a.jb * kCholBlock, i0 = j0 + ((int)blockIdx.y + 1) * kCholBlock;
  if (i0 >= n) return;                                 // uniform
  const int lane = threadIdx.x & 63, w = uni((int)threadIdx.x >> 6), l16 = lane & 15, lq = lane >> 4;
  double2* A = a.A + uni(a.a_off[q]);
  const int row = i0 + 16 * w + l16;
  auto ld = [](const double2* p) -> d2_t { return *(const d2_t*)p; };
  d4_t re[4], im[4];
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const d2_t v = ld(A + min(row, n - 1) + (long)(j0 + 16 * t + lq + 4 * e) * lda);
      re[t][e] = v.x;
      im[t][e] = v.y;
    }
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int c = threadIdx.x >> 4, r = threadIdx.x & 15;
    Ld[b][c][r] = ld(A + j0 + 16 * b + r + (long)(j0 + 16 * b + c) * lda);
  }
  __syncthreads();
  if (i0 + 16 * w >= n) return;                        // uniform per wavefront; no barrier below
#pragma unroll
  for (int b = 0; b < 4; ++b) {
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int je = j >> 2, jq = j & 3;
      const double d = Ld[b][j][j].x;
      const double xr = __shfl(re[b][je] / d, 16 * jq + l16), xi = __shfl(im[b][je] / d, 16 * jq + l16);
#pragma unroll
      for (int e = je; e < 4; ++e) {
        const d2_t l = Ld[b][j][lq + 4 * e];
        const double sr = re[b][e] - (xr * l.x + xi * l.y), si = im[b][e] - (xi * l.x - xr * l.y);
        if (e > je || lq > jq) {
          re[b][e] = sr;
          im[b][e] = si;
        } else if (lq == jq) {
          re[b][e] = xr;
          im[b][e] = xi;
        }
      }
    }
    if (row < n) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        A[row + (long)(j0 + 16 * b + lq + 4 * e) * lda] = make_double2(re[b][e], im[b][e]);
    }
#pragma unroll
    for (int c = b + 1; c < 4; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        chol_mac(re[c], im[c], ld(A + j0 + 16 * c + l16 + (long)(j0 + 16 * b + lq + 4 * e) * lda),
                 d2_t{-re[b][e], -im[b][e]});
  }
}

}  // namespace exc
