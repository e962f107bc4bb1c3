// Back-transform of V^x(k) to the LAPW basis (Sec. III.A, eq. "APW trafo"):
//   V_GG = Z V Z^H,  Z = S c  (n_G x n_b, S the overlap matrix, c the eigenvectors).
//
// Two launches on FP64 MFMA in 16 x 16 tiles: bt_left_kernel forms T = Z V (n_G x n_b), bt_gram_kernel, a wavefront
// per tile, the lower triangle of the n_G x n_G product T Z^H (V is Hermitian, so the product is: the tile above the
// diagonal is written as the conjugate of the one below). Complex blocks are built from four real 16x16x4 products;
// operands come straight from Z, V and T (L2-resident, n_b <= 128) into registers, the next 16 values of n requested
// before the products of these. Rows of C lie along the lanes, so the lower tile is stored in runs of 256 contiguous
// bytes. Small tiles, so that the stores of some wavefronts overlap the products of others.
//
// Output bytes bound it for n_b < ~40 (the half product has n_b / 4 flop per output byte against the FP64 ridge of
// ~14), the matrix cores beyond. n_G = 2000, n_b = 100 (64 MB out, 1.6 GFLOP, 24 us at the matrix cores' rate): T on
// the vector cores, an element per thread, 17 -> 8 us; the whole square in 64 x 64 tiles of four wavefronts 68 -> 34 us
// (the lower triangle in 32 x 32 tiles of one wavefront: 40 us).
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

#include "common.hpp"

namespace exc {

// re + i im += a b over four values of k, a the lane's value of the A block (row l % 16, k = l / 16), b that of the
// B block; CONJ: conj(a) b
template <bool CONJ>
__device__ __forceinline__ void bt_mac(d4_t& re, d4_t& im, d2_t a, d2_t b) {
  const double ay = CONJ ? a.y : -a.y;
  re = mfma(a.x, b.x, re);
  im = mfma(a.x, b.y, im);
  re = mfma(ay, b.y, re);
  im = mfma(-ay, b.x, im);
}

// T[g + n * nG] = sum_m Z[g + m * nG] V[m + n * nb] for 16 g (blockIdx.x) and 16 n (blockIdx.y): D[n][g]. Four
// wavefronts take a quarter of m each (at most 32: every load in flight at once) and add up in LDS.
__global__ __launch_bounds__(256) void bt_left_kernel(const double2* __restrict__ Z, const double2* __restrict__ V,
                                                      int nG, int nb, double2* __restrict__ T) {
  __shared__ double red[3][8][64];
  const int lane = threadIdx.x & 63, w = uni((int)threadIdx.x >> 6), l16 = lane & 15, kq = lane >> 4;
  const int g = (int)blockIdx.x * 16 + l16, n = (int)blockIdx.y * 16 + l16;
  const int kw = ((nb + 15) >> 4) * 4, m0 = w * kw;    // this wavefront's m: [m0, m0 + kw)
  const double2 *zp = Z + min(g, nG - 1), *vp = V + (long)min(n, nb - 1) * nb;
  d4_t re{0, 0, 0, 0}, im{0, 0, 0, 0};
  d2_t z[8], v[8];
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const int m = m0 + 4 * s + kq;
    const bool ok = 4 * s < kw && m < nb;
    const d2_t x = *(const d2_t*)(zp + (long)(ok ? m : 0) * nG), y = *(const d2_t*)(vp + (ok ? m : 0));
    z[s] = d2_t{ok ? x.x : 0.0, ok ? x.y : 0.0};
    v[s] = d2_t{ok ? y.x : 0.0, ok ? y.y : 0.0};
  }
#pragma unroll
  for (int s = 0; s < 8; ++s) bt_mac<false>(re, im, v[s], z[s]);
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (w > 0) {
      red[w - 1][i][lane] = re[i];
      red[w - 1][4 + i][lane] = im[i];
    }
  __syncthreads();
  if (w > 0 || g >= nG) return;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    double x = re[i], y = im[i];
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      x += red[u][i][lane];
      y += red[u][4 + i][lane];
    }
    const int c = (int)blockIdx.y * 16 + kq + 4 * i;
    if (c < nb) T[g + (long)c * nG] = make_double2(x, y);
  }
}

// C[b + a * nG] = sum_n T[b + n * nG] conj(Z[a + n * nG]) for the 16 x 16 tiles of rows b >= columns a, and their
// mirror images: D[a][b] with the A operand conj(Z) and the B operand T, so that lane l holds D[l / 16 + 4 i][l % 16].
__global__ __launch_bounds__(64, 4) void bt_gram_kernel(const double2* __restrict__ T, const double2* __restrict__ Z,
                                                        int nG, int nb, double2* __restrict__ C) {
  const int lane = threadIdx.x, l16 = lane & 15, kq = lane >> 4;
  const auto rz = make_rsrc(Z, (uint32_t)((long)nG * nb * 16)), rt = make_rsrc(T, (uint32_t)((long)nG * nb * 16));
  const long nt = (nG + 15) / 16;
  for (long tile = blockIdx.x; tile < nt * (nt + 1) / 2; tile += gridDim.x) {
    long tb = (long)((sqrt(8.0 * (double)tile + 1.0) - 1.0) * 0.5);
    while (tb * (tb + 1) / 2 > tile) --tb;
    while ((tb + 1) * (tb + 2) / 2 <= tile) ++tb;
    const int ta = uni((int)(tile - tb * (tb + 1) / 2));
    const int a0 = ta * 16, b = uni((int)tb) * 16 + l16;
    // (rows past n_G: the last one again, not stored; n >= nb: past the buffers' ends, zeros)
    const uint32_t oz = (uint32_t)(min(a0 + l16, nG - 1) + (long)kq * nG) * 16;
    const uint32_t ot = (uint32_t)(min(b, nG - 1) + (long)kq * nG) * 16;
    d4_t re{0, 0, 0, 0}, im{0, 0, 0, 0};
    struct Chunk { d2_t z[4], t[4]; };                 // 16 values of n
    auto load = [&](Chunk& c, int n0) {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const uint32_t o = (uint32_t)(n0 + 4 * s) * (uint32_t)nG * 16;
        c.z[s] = buf_load<d2_t>(rz, oz + o, 0);
        c.t[s] = buf_load<d2_t>(rt, ot + o, 0);
      }
    };
    Chunk c0, c1;
    load(c0, 0);
    int n0 = 0;
    for (; n0 + 16 <= nb; n0 += 16) {
      load(c1, n0 + 16);
#pragma unroll
      for (int s = 0; s < 4; ++s) bt_mac<true>(re, im, c0.z[s], c0.t[s]);
      c0 = c1;
    }
    // the last chunk's steps of four (none of them empty)
    if (n0 < nb) bt_mac<true>(re, im, c0.z[0], c0.t[0]);
    if (n0 + 4 < nb) bt_mac<true>(re, im, c0.z[1], c0.t[1]);
    if (n0 + 8 < nb) bt_mac<true>(re, im, c0.z[2], c0.t[2]);
    if (n0 + 12 < nb) bt_mac<true>(re, im, c0.z[3], c0.t[3]);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int a = a0 + kq + 4 * e;
      if (a < nG && b < nG) {
        C[b + (long)a * nG] = make_double2(re[e], im[e]);
        if (ta != (int)tb) C[a + (long)b * nG] = make_double2(re[e], -im[e]);
      }
    }
  }
}

}  // namespace exc
