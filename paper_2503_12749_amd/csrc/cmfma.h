// Complex tile products on the FP32 matrix cores, shared by the pair-moment
// sums and the joint-distribution box contractions.
//
// A 128 x 128 complex tile C += A B^T over a slab of kSlab samples, with the
// four real planes of the operands in LDS as [sample][row] (A re, A im) and
// [sample][col] (B re, B im), each row kTile floats.  v_mfma_f32_32x32x2f32
// takes lane l's A[l % 32][l / 32] and B[l / 32][l % 32], so every fragment
// is one LDS float per lane; output register r of lane l is element
// (8 (r / 4) + 4 (l / 32) + r % 4, l % 32) of a 32 x 32 block.  Wave
// (wi, wj) owns rows [64 wi, 64 wi + 64) and columns [64 wj, 64 wj + 64):
//   Re += Ar Br^T - Ai Bi^T,   Im += Ar Bi^T + Ai Br^T.
#pragma once

#include <hip/hip_runtime.h>

namespace mp {

namespace cmfma {

typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int kTile = 128;  // rows and columns of the complex tile
constexpr int kSlab = 32;   // samples per slab

__device__ __attribute__((always_inline)) inline void zero(f32x16 (&accR)[2][2],
                                                            f32x16 (&accI)[2][2]) {
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        accR[a][b][q] = 0.f;
        accI[a][b][q] = 0.f;
      }
}

// One slab (are, aim, bre, bim point at [kSlab][kTile] planes in LDS), for the block
// products that `mask` names: bit 4 t + 2 a + b for samples 2 t, 2 t + 1 and the wave's
// 32 x 32 block (a, b).  The next samples' fragments are read ahead of the products.
__device__ __attribute__((always_inline)) inline void slab_masked(
    const float* are, const float* aim, const float* bre, const float* bim, int wi, int wj, int lane,
    uint64_t mask, f32x16 (&accR)[2][2], f32x16 (&accI)[2][2]) {
  const int lr = lane & 31, lh = lane >> 5;
  const float* pa[2] = {are + lh * kTile + 64 * wi + lr, aim + lh * kTile + 64 * wi + lr};
  const float* pb[2] = {bre + lh * kTile + 64 * wj + lr, bim + lh * kTile + 64 * wj + lr};
  float x[2][2], y[2][2], nx[2][2], ny[2][2];
  auto read = [&](int t, float(&u)[2][2], float(&v)[2][2]) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        u[c][a] = pa[c][2 * t * kTile + 32 * a];
        v[c][a] = pb[c][2 * t * kTile + 32 * a];
      }
  };
  read(0, x, y);
#pragma unroll
  for (int t = 0; t < kSlab / 2; ++t) {
    if (t + 1 < kSlab / 2) read(t + 1, nx, ny);
    const uint32_t m = (uint32_t)(mask >> (4 * t));
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b)
        if (m & (1u << (2 * a + b))) {
          accR[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[0][a], y[0][b], accR[a][b], 0, 0, 0);
          accI[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[0][a], y[1][b], accI[a][b], 0, 0, 0);
          accR[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(-x[1][a], y[1][b], accR[a][b], 0, 0, 0);
          accI[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[1][a], y[0][b], accI[a][b], 0, 0, 0);
        }
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        x[c][a] = nx[c][a];
        y[c][a] = ny[c][a];
      }
  }
}

// Three-product form of one slab: P1 += Ar Br^T, P2 += Ai Bi^T,
// P3 += (Ar + Ai)(Br + Bi)^T, so that Re = P1 - P2 and Im = P3 - P1 - P2.  The
// fragments of four samples are read ahead of the products, two samples' at a time
// (ds_read2st64, whose offsets span the planes: no address arithmetic).
__device__ __attribute__((always_inline)) inline void slab3(const float* are, const float* aim,
                                                             const float* bre, const float* bim,
                                                             int wi, int wj, int lane,
                                                             f32x16 (&p1)[2][2], f32x16 (&p2)[2][2],
                                                             f32x16 (&p3)[2][2]) {
  const int lr = lane & 31, lh = lane >> 5;
  int oa[2] = {lh * kTile + 64 * wi + lr, lh * kTile + 64 * wi + lr + 32};
  int ob[2] = {lh * kTile + 64 * wj + lr, lh * kTile + 64 * wj + lr + 32};
#pragma unroll
  for (int a = 0; a < 2; ++a) asm("" : "+v"(oa[a]), "+v"(ob[a]));  // an address each
  float x[2][2][2], y[2][2][2], nx[2][2][2], ny[2][2][2];  // [step][re, im][block]
  auto read = [&](int t, float(&u)[2][2][2], float(&v)[2][2][2]) {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int g = 0; g < 2; ++g) {
        u[g][0][a] = are[oa[a] + 2 * (t + g) * kTile];
        v[g][0][a] = bre[ob[a] + 2 * (t + g) * kTile];
        u[g][1][a] = aim[oa[a] + 2 * (t + g) * kTile];
        v[g][1][a] = bim[ob[a] + 2 * (t + g) * kTile];
      }
  };
  read(0, x, y);
#pragma unroll
  for (int t = 0; t < kSlab / 2; t += 2) {
    if (t + 2 < kSlab / 2) read(t + 2, nx, ny);
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
          p1[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[g][0][a], y[g][0][b], p1[a][b], 0, 0, 0);
          p2[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[g][1][a], y[g][1][b], p2[a][b], 0, 0, 0);
          p3[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(
              x[g][0][a] + x[g][1][a], y[g][0][b] + y[g][1][b], p3[a][b], 0, 0, 0);
        }
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int a = 0; a < 2; ++a) {
          x[g][c][a] = nx[g][c][a];
          y[g][c][a] = ny[g][c][a];
        }
  }
}

// Tile row and column of output register q of 32 x 32 block (a, b).
__device__ __attribute__((always_inline)) inline int out_row(int wi, int a, int q, int lane) {
  return 64 * wi + 32 * a + 8 * (q >> 2) + 4 * (lane >> 5) + (q & 3);
}
__device__ __attribute__((always_inline)) inline int out_col(int wj, int b, int lane) {
  return 64 * wj + 32 * b + (lane & 31);
}

}  // namespace cmfma

}  // namespace mp
