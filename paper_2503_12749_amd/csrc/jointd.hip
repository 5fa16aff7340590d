// Joint distribution of d = 3 or 4 bin counts (main text, higher-dimensional
// binning; eq. General_GCP with the projector of eq. projection_op), and the
// inverse DFT of every joint grid (d = 2 included).
//
// Per sample the generating function on the grid theta_b = 2 pi k_b / K_b is
//   chi(theta) = cosh(n + sum_b X_b) / cosh(n),   X_b = n_b (e^{i theta_b} - 1)
//              = e^{c1} prod_b e^{X_b} + e^{c2} prod_b e^{-X_b},
// with c1 = -log(1 + e^{-2n}) and c2 = -2n - log(1 + e^{-2n}) (written for
// either sign of n as in the one-distribution path): two rank-1 tensors over
// the d bins.  The first is below e^kLogEps for every sample of a chunk
// outside a box around theta = 0, the second outside a box around theta =
// pi; each box half-width is the chunk's maximum of the samples' exact
// per-axis bounds.  Inside a box the sum of a term over a sub-ensemble's
// samples is a complex contraction over samples,
//   S[(k_1 .. k_{d-1}), k_d] = sum_s A_s[(k_1 .. k_{d-1})] B_s[k_d],
//   A_s = prod_{b<d} f_{s,b}(k_b),   B_s = f_{s,d}(k_d),
// from per-sample factor tables f: e^{+-X_b} times e^{-i theta_b m_lo_b} (the
// window shift), the second term's factors scaled by e^{-2 Re n_b}, and the
// term's constant shared equally by the d factors so that every factor stays
// within the FP32 range.  The contraction runs on the FP32 matrix cores for
// the FP32 and split paths and with FP64 FMAs for the FP64 path.
//
// Kernels per chunk: jointd_occupations (n_b, c1, c2 per sample),
// record_bands (the box half-widths), jointd_factors (the tables of both terms inside their boxes),
// jointd_sum_f32 / jointd_sum_f64 (acc[s][k_1]..[k_d] += S, one launch per
// term, so each accumulator element has one writer per launch).  Finalize:
// the d-dimensional inverse DFT one axis at a time over the nonzero entries
// of each line, per sub-ensemble, folded into the mean and sigma_T with
// Welford's update.
#include <hip/hip_runtime.h>

#include "chi.h"
#include "cmfma.h"
#include "common.h"

namespace mp {

namespace {

constexpr int kJD = 4;  // largest d of this path
constexpr int kAxisMaxK = 4096;  // longest line of the inverse DFT (two-bin windows)

typedef __attribute__((ext_vector_type(4))) float f32x4;
using cmfma::f32x16;

struct JointDParams {
  int M;
  int64_t ldm, E, e0, ns;
  int est, d;
  int n_runs;
  int run_lo[MP_MAX_RUNS], run_hi[MP_MAX_RUNS], run_bin[MP_MAX_RUNS];
  int m_lo[kJD], K[kJD], Kp[kJD];  // window, grid, factor-table row stride
  int64_t s_first;
  int64_t cells;     // prod K_b
  int64_t rows_max;  // prod_{b<d-1} K_b
  int rec;           // doubles per sample record: 2 d + 2
  int64_t tab[2][kJD];  // element offset of each factor table (term, axis)
};

__global__ void band_init(int* band) {
  if (threadIdx.x < 2 * kJD) band[threadIdx.x] = -1;
}

// Per sample (a wave, or a row of 16 lanes; the first lane writes): the record (Re n_b, Im n_b for b < d,
// c1, c2; c2 = -inf for +P, both NaN for a sample that is not finite).
// record_bands then sets the box half-widths
// band[term * 4 + b] (atomic max; -1 = term absent).
// PART: the bin sums come from the occupation-fused GEMM's partials (slots in
// run order) instead of the propagated amplitudes C.
template <typename CT, bool PART, int G>
__device__ inline void jointd_sample(const JointDParams& p, const CT* __restrict__ C,
                                     const float* __restrict__ part,
                                     const double* __restrict__ nglob, double* __restrict__ rec,
                                     int64_t k, int gl) {
  const int64_t ldc = 2 * p.ldm;
  const CT* ca = PART ? nullptr : C + k * ldc;
  const CT* cb = PART ? nullptr : C + (p.E + k) * ldc;
  double nr[kJD] = {0.0, 0.0, 0.0, 0.0}, ni[kJD] = {0.0, 0.0, 0.0, 0.0};
  int slot0 = 0;
  for (int q = 0; q < p.n_runs; ++q) {
    double re, im;
    if constexpr (PART) {
      const int nblk = run_blocks(p.run_lo[q], p.run_hi[q]);
      run_sum_partials<G>(part, p.E, slot0, nblk, k, gl, re, im);
      slot0 += nblk;
    } else {
      run_sum<CT, G>(ca, cb, p.ldm, p.run_lo[q], p.run_hi[q], gl, re, im);
    }
#pragma unroll
    for (int b = 0; b < kJD; ++b)
      if (b == p.run_bin[q]) {
        nr[b] += re;
        ni[b] += im;
      }
  }
  if (gl != 0) return;
  const double n = nglob[k];
  double* r = rec + k * p.rec;
  bool sums_finite = true;
#pragma unroll
  for (int b = 0; b < kJD; ++b)
    if (b < p.d) {
      r[2 * b] = nr[b];
      r[2 * b + 1] = ni[b];
      sums_finite = sums_finite && isfinite(nr[b]) && isfinite(ni[b]);
    }
  double c1 = 0.0, c2 = -INFINITY;
  if (p.est != MP_PLUS_P)
    parity_log_weights(n, sums_finite && isfinite(n), c1, c2);
  else if (!sums_finite)
    c1 = c2 = __builtin_nan("");
  r[2 * p.d] = c1;
  r[2 * p.d + 1] = c2;
}

template <typename CT, bool PART, int G>
__global__ __launch_bounds__(256) void jointd_occupations(JointDParams p, const CT* __restrict__ C,
                                                          const float* __restrict__ part,
                                                          const double* __restrict__ nglob,
                                                          double* __restrict__ rec) {
  constexpr int S = 256 / G;  // samples of a workgroup at a time
  const int64_t base = (int64_t)blockIdx.x * (S * kOccPerWave) + threadIdx.x / G;
  for (int j = 0; j < kOccPerWave; ++j) {
    const int64_t k = base + S * j;
    if (k >= p.E) return;
    jointd_sample<CT, PART, G>(p, C, part, nglob, rec, k, threadIdx.x % G);
  }
}

// Box of a term: half-widths h_b and widths w_b = min(2 h_b + 1, K_b); false
// if the term is absent on some axis (then no sample reaches e^kLogEps).
__device__ inline bool term_box(const JointDParams& p, const int* band, int tau, int (&h)[kJD],
                                int (&w)[kJD]) {
  bool ok = true;
#pragma unroll
  for (int b = 0; b < kJD; ++b) {
    h[b] = 0;
    w[b] = 1;
    if (b < p.d) {
      h[b] = band[tau * kJD + b];
      ok &= h[b] >= 0;
      w[b] = min(2 * h[b] + 1, p.K[b]);
    }
  }
  return ok;
}

// Grid index of box point j on axis b of term tau.
__device__ inline int box_index(const JointDParams& p, int tau, int b, int h, int j) {
  const int K = p.K[b];
  const int c = tau == 0 ? 0 : K / 2;
  return ((c - h + j) % K + K) % K;
}

// Factor f_{s,b}(j) of term tau for chunk sample k and box point j < w_b:
// e^{+-X_b(theta) + share (- 2 Re n_b for the second term)} e^{-i theta m_lo},
// stored in the path's precision (re plane, then im plane).
template <typename CT>
__global__ __launch_bounds__(256) void jointd_factors(JointDParams p, const double* __restrict__ rec,
                                                      const int* __restrict__ band,
                                                      CT* __restrict__ tables) {
  const int tau = blockIdx.y / p.d, b = blockIdx.y % p.d;
  int h[kJD], w[kJD];
  if (!term_box(p, band, tau, h, w)) return;
  const int Kp = p.Kp[b];
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t k = idx / Kp;
  const int j = (int)(idx - k * Kp);
  if (k >= p.E || j >= w[b]) return;
  const double* r = rec + k * p.rec;
  const double R = r[2 * b], I = r[2 * b + 1];
  double fr = 0.0, fi = 0.0;
  const double cterm = tau == 0 ? r[2 * p.d] : r[2 * p.d + 1];
  if (cterm != -INFINITY) {  // NaN weights are evaluated: they must reach the sums
    double share = cterm;
    if (tau == 1)
      for (int q = 0; q < p.d; ++q) share += 2.0 * r[2 * q];
    share /= p.d;
    const int K = p.K[b];
    const int kg = box_index(p, tau, b, h[b], j);
    constexpr double kTwoPi = 6.283185307179586476925286766559;
    const double th = kTwoPi * (double)kg / (double)K;
    const double sh = sin(0.5 * th);
    const double cm1 = -2.0 * sh * sh, sn = sin(th);
    const double xr = cm1 * R - sn * I, xi = cm1 * I + sn * R;
    const int64_t red = (((int64_t)kg * (int64_t)p.m_lo[b]) % K + K) % K;
    const double thl = kTwoPi * (double)red / (double)K;
    // FP64 tables take FP64 exp / sincos, FP32 tables FP32 ones (phase
    // reduced in FP64 first)
    constexpr bool kF64 = sizeof(CT) == 8;
    if (tau == 0)
      cis_exp<kF64>(xr + share, xi - thl, fr, fi);
    else
      cis_exp<kF64>(-xr - 2.0 * R + share, -xi - thl, fr, fi);
  }
  CT* t = tables + p.tab[tau][b];
  t[k * Kp + j] = (CT)fr;
  t[p.E * Kp + k * Kp + j] = (CT)fi;
}

// Chunk-local sample range [k0, k1) of sub-ensemble s.
__device__ inline void segment(const JointDParams& p, int64_t s, int64_t& k0, int64_t& k1) {
  const int64_t lo = s * p.ns - p.e0, hi = (s + 1) * p.ns - p.e0;
  k0 = lo > 0 ? lo : 0;
  k1 = hi < p.E ? hi : p.E;
}

// Box point indices (j_0 .. j_{d-2}) of flattened row r (last axis fastest).
__device__ inline void row_point(const JointDParams& p, const int (&w)[kJD], int64_t r,
                                 int (&j)[kJD]) {
#pragma unroll
  for (int b = kJD - 1; b >= 0; --b) {
    j[b] = 0;
    if (b < p.d - 1) {
      j[b] = (int)(r % w[b]);
      r /= w[b];
    }
  }
}

// acc[s] cell of box row r and box column c of term tau.
__device__ inline int64_t cell_of(const JointDParams& p, int tau, const int (&h)[kJD],
                                  const int (&w)[kJD], int64_t r, int c) {
  int j[kJD];
  row_point(p, w, r, j);
  int64_t flat = 0;
#pragma unroll
  for (int b = 0; b < kJD; ++b)
    if (b < p.d - 1) flat = flat * p.K[b] + box_index(p, tau, b, h[b], j[b]);
  return flat * p.K[p.d - 1] + box_index(p, tau, p.d - 1, h[p.d - 1], c);
}

// acc[s] cell of box point indices j (row axes) and box column c of term tau.
__device__ inline int64_t cell_from(const JointDParams& p, int tau, const int (&h)[kJD],
                                    const int (&j)[kJD], int c) {
  int64_t flat = 0;
#pragma unroll
  for (int b = 0; b < kJD; ++b)
    if (b < p.d - 1) flat = flat * p.K[b] + box_index(p, tau, b, h[b], j[b]);
  return flat * p.K[p.d - 1] + box_index(p, tau, p.d - 1, h[p.d - 1], c);
}

// Row widths of the FP32 box contraction: the last row axis (d - 2) padded
// to a multiple of 4, so that the four consecutive rows a thread stages
// share their other axes and take four aligned consecutive table entries.
__device__ inline void padded_widths(const JointDParams& p, const int (&w)[kJD], int (&wp)[kJD]) {
#pragma unroll
  for (int b = 0; b < kJD; ++b) wp[b] = b == p.d - 2 ? (w[b] + 3) & ~3 : w[b];
}

// Product over the row axes of one sample's factors (complex).
template <typename CT>
__device__ inline void row_factor(const JointDParams& p, int tau, const CT* __restrict__ tables,
                                  int64_t k, const int (&j)[kJD], double& ar, double& ai) {
  ar = 1.0;
  ai = 0.0;
#pragma unroll
  for (int b = 0; b < kJD - 1; ++b)
    if (b < p.d - 1) {
      const CT* t = tables + p.tab[tau][b] + k * p.Kp[b] + j[b];
      const double fr = (double)t[0], fi = (double)t[p.E * p.Kp[b]];
      const double nr = ar * fr - ai * fi;
      ai = ar * fi + ai * fr;
      ar = nr;
    }
}

// Workgroup -> (sub-ensemble, row tile, column tile) of a box of nrows rows; false
// for workgroups past it (the grid covers the largest possible box).  Row tiles
// from the box's centre outwards, all sub-ensembles and columns of one before the next:
// the samples reach the tiles in the middle most, and a launch of few turns ends
// sooner when its longest workgroups start first (jointd_sum_f32, 1280 workgroups of
// 128^3 points on 512 places: 10.1 ms in grid order, 8.2 ms so).
__device__ inline bool sum_item(const JointDParams& p, int tile, int64_t nrows, int64_t& s,
                                int64_t& rt, int& ct) {
  const int ctn = (p.K[p.d - 1] + tile - 1) / tile;
  const int64_t per_sub = (p.rows_max + tile - 1) / tile * ctn;
  const int64_t n_s = gridDim.x / per_sub, nt = (nrows + tile - 1) / tile;
  const int64_t item = blockIdx.x;
  ct = (int)(item % ctn);
  s = p.s_first + item / ctn % n_s;
  const int64_t rank = item / ctn / n_s;
  rt = nt / 2 + (rank & 1 ? -(rank + 1) / 2 : rank / 2);
  return rank < nt;
}

constexpr int PT = 128;  // box rows / columns per FP32 tile
constexpr int PK = 32;   // samples per slab
static_assert(PT == cmfma::kTile && PK == cmfma::kSlab, "tile shape of the shared MFMA core");

// FP32 matrix cores, the 4-product complex scheme of v_mfma_f32_32x32x2f32
// (lane l supplies A[l % 32][l / 32] and B[l / 32][l % 32]; output register
// r of lane l is element (8 (r / 4) + 4 (l / 32) + r % 4, l % 32)); wave
// (wi, wj) owns a 64 x 64 block of the 128 x 128 complex tile.  The row
// operand (the product of the row axes' factors) is formed in FP32 while a
// slab is staged, from 16-byte loads of the last row axis and the column
// axis and scalar loads of the others, all issued a slab ahead (loads behind
// branches had waited for each other, and cost as much as the products).  The
// box is the chunk's largest; most samples reach only part of it.  While a slab
// is staged the largest magnitude of every sample's 32-row and 32-column block
// is taken, and the product of a block is formed only for the sample pairs that
// reach e^kLogEps in it (about half of them for three bins of 100 modes with
// 24 photons each): what is left out is below the threshold that bounds the
// box.  Bound by the FP32 matrix cores (72 % busy), then by the staging between
// their products.  1e5 samples on 128^3 points, two full boxes, per term: 14.5 ms
// before, 14.4 with the block test alone, 10.1 with the loads ahead as well,
// 8.2 with the order of sum_item.  D = 4 spills 51 registers around the loads and gains all the
// same: counts of 2e4 samples on 48^4 points 41.7 ms before, 35.4 now; 2000 on 32^4
// 1.41 and 0.78 ms.
template <int D>
__global__ __launch_bounds__(256, 2) void jointd_sum_f32(JointDParams p, int tau,
                                                        const float* __restrict__ tables,
                                                        const int* __restrict__ band,
                                                        double* __restrict__ acc) {
  __shared__ __attribute__((aligned(16))) float lds[4][PK][PT];  // A re, A im, B re, B im
  __shared__ float big[2][PK][4];  // largest |re|, |im| of a sample's 32-row (column) block
  int h[kJD], w[kJD], wp[kJD];
  if (!term_box(p, band, tau, h, w)) return;
  padded_widths(p, w, wp);
  int64_t nrows = 1;  // a multiple of 4
#pragma unroll
  for (int b = 0; b < D - 1; ++b) nrows *= wp[b];
  const int ncols = w[D - 1];
  int64_t s, rt;
  int ct;
  if (!sum_item(p, PT, nrows, s, rt, ct) || ct * PT >= ncols) return;
  int64_t k0, k1;
  segment(p, s, k0, k1);
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int wi = wave >> 1, wj = wave & 1;
  const int lc = (tid & 31) * 4, lrow = tid >> 5;

  // the thread's rows r0 .. r0 + 3 share axes 0 .. d-3 and take entries
  // jl .. jl + 3 (jl a multiple of 4) of the last row axis
  const int64_t r0 = rt * PT + lc;
  const bool rvalid = r0 < nrows;
  int jr[kJD];
  row_point(p, wp, rvalid ? r0 : 0, jr);
  constexpr int al = D - 2, bl = D - 1;
  const int jl = jr[al], wl = w[al];
  const float* tl = tables + p.tab[tau][al];
  const int64_t tl_im = p.E * p.Kp[al];
  const float* tb = tables + p.tab[tau][bl];
  const int64_t tb_im = p.E * p.Kp[bl];
  const int c0 = ct * PT + lc;
  const int cl = c0 < ncols ? c0 : 0;  // cl + 3 < Kp (both multiples of 4)

  // A slab's loads (clamped addresses, no branches around them) are in flight while the
  // slab before it is multiplied; what is out of range is selected away when they are used.
  f32x4 lre[4], lim[4], bre[4], bim[4];
  float fr[al][4], fi[al][4];  // factors of axes 0 .. d-3
  auto load = [&](int64_t kb) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int64_t k = min(kb + lrow + 8 * u, k1 - 1);
#pragma unroll
      for (int b = 0; b < al; ++b) {
        const float* t = tables + p.tab[tau][b] + k * p.Kp[b] + jr[b];
        fr[b][u] = t[0];
        fi[b][u] = t[p.E * p.Kp[b]];
      }
      lre[u] = *(const f32x4*)(tl + k * p.Kp[al] + jl);
      lim[u] = *(const f32x4*)(tl + tl_im + k * p.Kp[al] + jl);
      bre[u] = *(const f32x4*)(tb + k * p.Kp[bl] + cl);
      bim[u] = *(const f32x4*)(tb + tb_im + k * p.Kp[bl] + cl);
    }
  };
  // planes of samples kb + lrow + 8 u: the thread's rows, then its columns
  auto row_values = [&](int64_t kb, int u, f32x4& re, f32x4& im) {
    const bool kv = kb + lrow + 8 * u < k1 && rvalid;
    float pr = 1.f, pi = 0.f;
#pragma unroll
    for (int b = 0; b < al; ++b) {
      const float nr = pr * fr[b][u] - pi * fi[b][u];
      pi = pr * fi[b][u] + pi * fr[b][u];
      pr = nr;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      // table entries past the box width are never written: select, not multiply
      const bool av = kv && jl + e < wl;
      re[e] = av ? pr * lre[u][e] - pi * lim[u][e] : 0.f;
      im[e] = av ? pr * lim[u][e] + pi * lre[u][e] : 0.f;
    }
  };
  auto col_values = [&](int64_t kb, int u, f32x4& re, f32x4& im) {
    const bool kv = kb + lrow + 8 * u < k1;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool bv = kv && c0 + e < ncols;
      re[e] = bv ? bre[u][e] : 0.f;
      im[e] = bv ? bim[u][e] : 0.f;
    }
  };

  // the bits of the largest magnitude over eight neighbouring threads (32 rows or columns)
  // of one sample; a NaN's bits are above every number's
  auto block_max = [&](f32x4 re, f32x4 im) {
    uint32_t m = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      m = max(m, max(__float_as_uint(re[e]) & 0x7FFFFFFFu, __float_as_uint(im[e]) & 0x7FFFFFFFu));
    m = max(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0xB1, 0xF, 0xF, false));   // lane ^ 1
    m = max(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x4E, 0xF, 0xF, false));   // lane ^ 2
    m = max(m, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)m, 0x141, 0xF, 0xF, false));  // 7 - lane
    return __uint_as_float(m);
  };
  // a block product whose cells are all below e^kLogEps: |a b| <= 2 max max
  const float least = 0.5f * 1.0530617e-20f;

  f32x16 accR[2][2], accI[2][2];
  cmfma::zero(accR, accI);

  load(k0);
  for (int64_t kb = k0; kb < k1; kb += PK) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      f32x4 v[4];
      row_values(kb, u, v[0], v[1]);
      col_values(kb, u, v[2], v[3]);
#pragma unroll
      for (int pl = 0; pl < 4; ++pl) *(f32x4*)&lds[pl][lrow + 8 * u][lc] = v[pl];
      const float ma = block_max(v[0], v[1]), mb = block_max(v[2], v[3]);
      if ((tid & 7) == 0) {
        big[0][lrow + 8 * u][(tid & 31) >> 3] = ma;
        big[1][lrow + 8 * u][(tid & 31) >> 3] = mb;
      }
    }
    __syncthreads();
    if (kb + PK < k1) load(kb + PK);
    // lane 4 t + 2 a + b: samples 2 t, 2 t + 1, the wave's block (a, b)
    const int t2 = (lane >> 2) * 2, ra = 2 * wi + ((lane >> 1) & 1), cb = 2 * wj + (lane & 1);
    const bool need = !(big[0][t2][ra] * big[1][t2][cb] < least) ||
                      !(big[0][t2 + 1][ra] * big[1][t2 + 1][cb] < least);
    cmfma::slab_masked(&lds[0][0][0], &lds[1][0][0], &lds[2][0][0], &lds[3][0][0], wi, wj, lane,
                       __ballot(need), accR, accI);
  }

  double* as = acc + 2 * s * p.cells;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int q = 0; q < 16; ++q) {
        const int64_t gr = rt * PT + cmfma::out_row(wi, a, q, lane);
        const int gc = ct * PT + cmfma::out_col(wj, b, lane);
        if (gr < nrows && gc < ncols) {
          int j[kJD];
          row_point(p, wp, gr, j);
          if (j[al] < wl) {
            double* o = as + 2 * cell_from(p, tau, h, j, gc);
            o[0] += accR[a][b][q];
            o[1] += accI[a][b][q];
          }
        }
      }
}

constexpr int QT = 64;  // box rows / columns per FP64 tile
constexpr int QK = 16;  // samples per slab

// FP64 FMAs: thread (ty, tx) owns rows ty + 16 u and columns tx + 16 v of a
// 64 x 64 complex tile; per sample Re += ar br, Re -= ai bi, Im += ar bi,
// Im += ai br.
__global__ __launch_bounds__(256) void jointd_sum_f64(JointDParams p, int tau,
                                                     const double* __restrict__ tables,
                                                     const int* __restrict__ band,
                                                     double* __restrict__ acc) {
  __shared__ double lds[4][QK][QT];
  int h[kJD], w[kJD];
  if (!term_box(p, band, tau, h, w)) return;
  int64_t nrows = 1;
#pragma unroll
  for (int b = 0; b < kJD - 1; ++b)
    if (b < p.d - 1) nrows *= w[b];
  const int ncols = w[p.d - 1];
  int64_t s, rt;
  int ct;
  if (!sum_item(p, QT, nrows, s, rt, ct) || ct * QT >= ncols) return;
  int64_t k0, k1;
  segment(p, s, k0, k1);
  const int tid = threadIdx.x, ty = tid >> 4, tx = tid & 15;
  const int lc = (tid & 15) * 4, lrow = tid >> 4;
  int jr[4][kJD];
  bool rv[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int64_t r = rt * QT + lc + e;
    rv[e] = r < nrows;
    row_point(p, w, rv[e] ? r : 0, jr[e]);
  }
  const int bl = p.d - 1;
  const double* tb = tables + p.tab[tau][bl];
  const int64_t tb_im = p.E * p.Kp[bl];
  const int c0 = ct * QT + lc;
  double re[4][4], im[4][4];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int v = 0; v < 4; ++v) re[u][v] = im[u][v] = 0.0;

  for (int64_t kb = k0; kb < k1; kb += QK) {
    __syncthreads();
    const int64_t k = kb + lrow;
    const bool kv = k < k1;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      double ar = 0.0, ai = 0.0;
      if (kv && rv[e]) row_factor<double>(p, tau, tables, k, jr[e], ar, ai);
      lds[0][lrow][lc + e] = ar;
      lds[1][lrow][lc + e] = ai;
      const bool cv = kv && c0 + e < ncols;
      lds[2][lrow][lc + e] = cv ? tb[k * p.Kp[bl] + c0 + e] : 0.0;
      lds[3][lrow][lc + e] = cv ? tb[tb_im + k * p.Kp[bl] + c0 + e] : 0.0;
    }
    __syncthreads();
    for (int kk = 0; kk < QK; ++kk) {
      double xr[4], xi[4], yr[4], yi[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        xr[u] = lds[0][kk][ty + 16 * u];
        xi[u] = lds[1][kk][ty + 16 * u];
        yr[u] = lds[2][kk][tx + 16 * u];
        yi[u] = lds[3][kk][tx + 16 * u];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          re[u][v] = fma(xr[u], yr[v], re[u][v]);
          re[u][v] = fma(-xi[u], yi[v], re[u][v]);
          im[u][v] = fma(xr[u], yi[v], im[u][v]);
          im[u][v] = fma(xi[u], yr[v], im[u][v]);
        }
    }
  }
  double* as = acc + 2 * s * p.cells;
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t gr = rt * QT + ty + 16 * u;
      const int gc = ct * QT + tx + 16 * v;
      if (gr < nrows && gc < ncols) {
        double* o = as + 2 * cell_of(p, tau, h, w, gr, gc);
        o[0] += re[u][v];
        o[1] += im[u][v];
      }
    }
}

// ---------------------------------------------------------------- finalize

// DFT along one axis of a grid, out[.., l, ..] = sum_k in[.., k, ..] e^{-2 pi i k l / K},
// in two short steps per line: with K = A B, k = B a + b and l = l1 + A l2,
//   Z[l1][b] = e^{-2 pi i b l1 / K} sum_a in[B a + b] e^{-2 pi i a l1 / A},
//   out[l1 + A l2] = sum_b Z[l1][b] e^{-2 pi i b l2 / B}:
// A + B products per point instead of K (A: the largest divisor up to 16 and
// sqrt(K); a K without one takes the sum directly, A = 1, over the k where a
// line is not zero).  A thread forms several outputs of a sum from one pass
// over its terms (OUT of the second sum): a term times its step twiddle per output, a
// chain of at most 16 rotations from an exact twiddle.  A workgroup holds G lines in LDS,
// neighbours along the contiguous dimension, one padding element per B so that
// both steps read without bank conflicts; step 1 works in place.  Workgroups
// whose lines are all zero (outside the boxes) write zeros.  Bound by the FP64
// operations and the L2 traffic about equally; one line or two per workgroup
// with K products per point, one sub-ensemble per launch, took 153 us per axis
// and sub-ensemble for 128^3 points and 111 us for 1024^2 (now 36 and 49 us).
//
// in and out hold `subs` grids: blockIdx.y for the inner axes; on the last
// axis a workgroup takes its lines of every sub-ensemble in order, and the
// value times `scale` is folded into the running mean (P_re, P_im) and sum of
// squared deviations (m2) with Welford's update.
struct AxisParams {
  int K, A, B, G, GP;  // GP: lines' LDS stride (odd)
  int out;             // outputs per thread of the second sum: 8 or 1
  int64_t n_lines, stride, cells;
  double scale;
  int s0, subs;
};
constexpr int kAxisA = 16;    // longest first sum
constexpr int kAxisPoints = 2048;  // points per workgroup (G lines), where K allows
// Small grids are bound by the latency of a workgroup instead: a workgroup then holds as few
// lines as leave kAxisGroups workgroups (of at least 128 points), and where the second sum
// has less than 128 items of eight outputs a thread forms one output, of terms loaded four
// at a time, and the first sum is at most four long.  Three launches and one
// sub-ensemble, by 2048 points and eight outputs against so: 64 x 64 points 31 and 20 us, 97 x 89
// 52 and 20, 256 x 256 56 and 22, 24^3 37 and 24, 4 x 4 x 500 49 and 29; at 512 x 512 the
// rule changes nothing (63 us), and one output a thread would take longer.
constexpr int kAxisGroups = 256;
constexpr int kAxisMaxSubs = 1024;  // sub-ensembles per launch

// x / d for 0 <= x < 2^22 and 1 <= d: the FP32 estimate is at most one off
__device__ inline int fast_div(int x, int d, float inv_d) {
  int q = (int)((float)x * inv_d);
  const int r = x - q * d;
  return q + (r >= d ? 1 : 0) - (r < 0 ? 1 : 0);
}

template <bool LAST, int OUT>
__global__ __launch_bounds__(256) void jointd_axis(AxisParams p, const double* __restrict__ in,
                                                   double* __restrict__ out,
                                                   double* __restrict__ P_re,
                                                   double* __restrict__ P_im,
                                                   double* __restrict__ m2) {
  typedef __attribute__((ext_vector_type(2), aligned(8))) double d2u;  // in: any FP64 address
  typedef __attribute__((ext_vector_type(2))) double d2;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  const int K = p.K, A = p.A, B = p.B, G = p.G, GP = p.GP;
  d2* buf = (d2*)smem;                  // (K + A) x GP
  d2* tw = buf + (int64_t)(K + A) * GP;  // e^{-2 pi i q / B}, q < B
  d2* twa = tw + B;                      // e^{-2 pi i q / A}, q < A
  d2* twk = twa + A;                     // A > 1: e^{-2 pi i q / K}, q < B
  int* nzb = (int*)(twk + (A > 1 ? B : 0));  // any line nonzero at k = b mod B
  const int tid = threadIdx.x;
  const int64_t L0 = (int64_t)blockIdx.x * G;
  const int nl = p.n_lines - L0 < G ? (int)(p.n_lines - L0) : G;
  const float inv_k = 1.0f / (float)K, inv_b = 1.0f / (float)B, inv_g = 1.0f / (float)G;
  for (int i = tid; i < B + A + (A > 1 ? B : 0); i += 256) {
    const int q = i < B ? i : (i < B + A ? i - B : i - B - A);
    double sw, cw;
    sincospi(-2.0 * ((double)q / (i < B ? B : (i < B + A ? A : K))), &sw, &cw);
    tw[i] = d2{cw, sw};
  }
  // first element of line g (its elements are p.stride apart)
  auto line_base = [&](int g) {
    const int64_t L = L0 + g, outer = L / p.stride;
    return outer * (int64_t)K * p.stride + (L - outer * p.stride);
  };
  const int s_lo = LAST ? 0 : (int)blockIdx.y, s_hi = LAST ? p.subs : s_lo + 1;
  for (int s = s_lo; s < s_hi; ++s) {
    const d2u* src = (const d2u*)in + (int64_t)s * p.cells;
    for (int i = tid; i < B; i += 256) nzb[i] = 0;
    __syncthreads();  // also: the previous sub-ensemble's lines are consumed
    bool any = false;
    for (int i = tid; i < K * G; i += 256) {
      int k, g;
      if constexpr (LAST) {  // stride 1: lanes along the line
        g = fast_div(i, K, inv_k);
        k = i - g * K;
      } else {
        k = fast_div(i, G, inv_g);
        g = i - k * G;
      }
      d2 v = {0.0, 0.0};
      if (g < nl) v = src[LAST ? (L0 + g) * K + k : line_base(g) + k * p.stride];
      const int a = fast_div(k, B, inv_b);
      buf[(k + a) * GP + g] = v;
      if (v.x != 0.0 || v.y != 0.0) {  // a NaN counts as nonzero
        any = true;
        nzb[k - a * B] = 1;
      }
    }
    any = __syncthreads_or(any);
    if (any && A > 1) {
      for (int it = tid; it < B * G; it += 256) {
        const int b = fast_div(it, G, inv_g), g = it - b * G;
        d2* x = buf + b * GP + g;
        const int pitch = (B + 1) * GP;
        double zr[kAxisA], zi[kAxisA];
#pragma unroll
        for (int u = 0; u < kAxisA; ++u) zr[u] = zi[u] = 0.0;
        for (int a = 0; a < A; ++a) {
          const d2 v = x[a * pitch], w = twa[a];
          double vr = v.x, vi = v.y;
#pragma unroll
          for (int u = 0; u < kAxisA; ++u) {
            if (u >= A) break;
            zr[u] += vr;
            zi[u] += vi;
            const double t = fma(vr, w.x, -(vi * w.y));
            vi = fma(vr, w.y, vi * w.x);
            vr = t;
          }
        }
        const d2 wk = twk[b];
        double wr = 1.0, wi = 0.0;
#pragma unroll
        for (int u = 0; u < kAxisA; ++u) {
          if (u >= A) break;
          x[u * pitch] = d2{fma(zr[u], wr, -(zi[u] * wi)), fma(zr[u], wi, zi[u] * wr)};
          const double t = fma(wr, wk.x, -(wi * wk.y));
          wi = fma(wr, wk.y, wi * wk.x);
          wr = t;
        }
      }
      __syncthreads();
    }
    const int AG = A * G, nj = (B + OUT - 1) / OUT;
    const float inv_ag = 1.0f / (float)AG, inv_a = 1.0f / (float)A;
    for (int it = tid; it < AG * nj; it += 256) {
      const int j = fast_div(it, AG, inv_ag), r = it - j * AG;
      int l1, g;
      if constexpr (LAST) {
        g = fast_div(r, A, inv_a);
        l1 = r - g * A;
      } else {
        l1 = fast_div(r, G, inv_g);
        g = r - l1 * G;
      }
      double sr[OUT], si[OUT];
#pragma unroll
      for (int u = 0; u < OUT; ++u) sr[u] = si[u] = 0.0;
      if (any) {
        const d2* z = buf + l1 * (B + 1) * GP + g;
        const int l0 = j * OUT;  // < B
        int q = 0;               // b l0 mod B
        if constexpr (OUT == 1) {
          // four terms at a time, their loads together; those past B count as zero
          for (int b = 0; b < B; b += 4) {
            d2 v[4], w[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              v[e] = z[min(b + e, B - 1) * GP];
              w[e] = tw[q];
              q += l0;
              q -= q >= B ? B : 0;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const double xr = b + e < B ? v[e].x : 0.0, xi = b + e < B ? v[e].y : 0.0;
              sr[0] += fma(xr, w[e].x, -(xi * w[e].y));
              si[0] += fma(xr, w[e].y, xi * w[e].x);
            }
          }
        } else {
          for (int b = 0; b < B; ++b) {
            if (nzb[b]) {
              const d2 v = z[b * GP], w0 = tw[q], w = tw[b];
              double vr = fma(v.x, w0.x, -(v.y * w0.y)), vi = fma(v.x, w0.y, v.y * w0.x);
#pragma unroll
              for (int u = 0; u < OUT; ++u) {
                sr[u] += vr;
                si[u] += vi;
                const double t = fma(vr, w.x, -(vi * w.y));
                vi = fma(vr, w.y, vi * w.x);
                vr = t;
              }
            }
            q += l0;
            q -= q >= B ? B : 0;
          }
        }
      }
      if (g >= nl) continue;
      const int64_t base = LAST ? (L0 + g) * K : line_base(g);
#pragma unroll
      for (int u = 0; u < OUT; ++u) {
        const int l2 = j * OUT + u;
        if (l2 >= B) break;
        const int64_t cell = base + (l1 + A * l2) * p.stride;
        if constexpr (!LAST) {
          ((d2*)out)[(int64_t)s * p.cells + cell] = d2{sr[u], si[u]};
        } else {
          const double vr = sr[u] * p.scale, vi = si[u] * p.scale;
          const int n = p.s0 + s;
          if (n == 0) {
            P_re[cell] = vr;
            if (P_im) P_im[cell] = vi;
            m2[cell] = 0.0;
          } else {
            const double mean = P_re[cell];
            const double dr = vr - mean;
            const double nm = mean + dr / (n + 1);
            P_re[cell] = nm;
            if (P_im) P_im[cell] += (vi - P_im[cell]) / (n + 1);
            m2[cell] += dr * (vr - nm);
          }
        }
      }
    }
    __syncthreads();
  }
}

__global__ void jointd_sigma(int64_t cells, int n_sub, double* __restrict__ sigma) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= cells) return;
  sigma[i] = n_sub > 1 ? sqrt(sigma[i] / (n_sub - 1) / n_sub) : __builtin_nan("");
}

int64_t round_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }

// Shape of the DFT along axis a of a K[0] x .. x K[d - 1] grid.
AxisParams axis_params(int32_t d, const int32_t* K, int a, int64_t cells) {
  AxisParams p{};
  p.K = K[a];
  p.stride = 1;
  for (int b = a + 1; b < d; ++b) p.stride *= K[b];
  p.cells = cells;
  p.n_lines = cells / p.K;
  p.G = 1;
  while (p.G < 64 && 2 * p.G * p.K <= kAxisPoints) p.G *= 2;
  while (p.G > 1 && (p.n_lines + p.G - 1) / p.G < kAxisGroups && p.G * p.K >= 256) p.G /= 2;
  for (p.out = 8;; p.out = 1) {
    p.A = 1;
    for (int f = 2; f <= (p.out == 8 ? kAxisA : 4) && f * f <= p.K; ++f)
      if (p.K % f == 0) p.A = f;
    p.B = p.K / p.A;
    if (p.out == 1 || p.G * p.A * ((p.B + 7) / 8) >= 128) break;
  }
  p.GP = p.G == 1 ? 1 : p.G + 1;
  return p;
}

size_t axis_lds(const AxisParams& p) {
  return (size_t)(p.K + p.A) * p.GP * 16 + (size_t)(p.A + p.B + (p.A > 1 ? p.B : 0)) * 16 +
         (size_t)p.B * 4;
}
// the largest: one line of a prime K below kAxisMaxK
constexpr int kAxisMaxLds = (kAxisMaxK + 1) * 16 + (kAxisMaxK + 1) * 16 + kAxisMaxK * 4;
static_assert(kAxisMaxLds <= 160 * 1024, "LDS of a workgroup");

// Workspace layout of a chunk: band ints, per-sample records, factor tables
// (FP64 elements for the FP64 path, FP32 otherwise).
size_t layout(JointDParams& p, size_t elem) {
  int64_t off = 256;  // band
  off += round_up(p.E * p.rec * 8, 256);
  int64_t tab = 0;
  for (int tau = 0; tau < 2; ++tau)
    for (int b = 0; b < p.d; ++b) {
      p.tab[tau][b] = tab;
      tab += 2 * p.E * p.Kp[b];
    }
  return (size_t)off + (size_t)tab * elem;
}

bool fill_params(JointDParams& p, int32_t M, int64_t E, int32_t d, const int32_t* bin_of_mode,
                 const int32_t* m_lo, const int32_t* K, int64_t ns, int64_t e0) {
  p.M = M;
  p.ldm = ld_modes(M);
  p.E = E;
  p.e0 = e0;
  p.ns = ns;
  p.d = d;
  p.rec = 2 * d + 2;
  p.cells = 1;
  p.rows_max = 1;
  for (int b = 0; b < d; ++b) {
    p.m_lo[b] = m_lo ? m_lo[b] : 0;
    p.K[b] = K[b];
    p.Kp[b] = (int)round_up(K[b], 4);
    p.cells *= K[b];
    // the FP32 contraction pads the last row axis to a multiple of 4
    if (b < d - 1) p.rows_max *= b == d - 2 ? round_up(K[b], 4) : K[b];
  }
  p.s_first = e0 / ns;
  p.n_runs = 0;
  if (!bin_of_mode) return true;
  for (int j = 0; j < M;) {
    const int b = bin_of_mode[j];
    int j2 = j + 1;
    while (j2 < M && bin_of_mode[j2] == b) ++j2;
    if (b >= 0) {
      if (p.n_runs >= MP_MAX_RUNS) return false;
      p.run_lo[p.n_runs] = j;
      p.run_hi[p.n_runs] = j2;
      p.run_bin[p.n_runs] = b;
      ++p.n_runs;
    }
    j = j2;
  }
  return true;
}

}  // namespace

mp_status record_bands_launch(const double* rec, int64_t E, int d, const int32_t* K,
                              int band_stride, int* band, hipStream_t stream);

size_t jointd_workspace(int32_t d, const int32_t* K, int64_t E) {
  JointDParams p{};
  fill_params(p, 1, E, d, nullptr, nullptr, K, 1, 0);
  return layout(p, 8);
}

// Two buffers of one grid per sub-ensemble in flight: as many as fit 64 MiB,
// at least one (grids beyond 2^21 cells run one sub-ensemble per launch and
// fill the chip with it).
size_t jointd_finalize_workspace(int32_t d, const int32_t* K, int32_t n_sub) {
  int64_t cells = 1;
  for (int b = 0; b < d; ++b) cells *= K[b];
  const int64_t one = round_up(cells * 16, 256);
  int64_t subs = (64ll << 20) / (2 * one);
  subs = subs < n_sub ? subs : n_sub;
  subs = subs < kAxisMaxSubs ? subs : kAxisMaxSubs;
  return (size_t)(256 + 2 * one * (subs > 1 ? subs : 1));
}

// part != nullptr: the bin sums come from the occupation-fused GEMM's partials
// (runs in the order fill_params builds them) and C is unused.
mp_status jointd_launch(int32_t M, int64_t E, const void* C, const double* n, mp_precision prec,
                        mp_estimator est, int32_t d, const int32_t* bin_of_mode,
                        const int32_t* m_lo, const int32_t* K, int32_t n_sub, int64_t ns,
                        int64_t e0, double* acc, void* ws, size_t ws_bytes, hipStream_t stream,
                        const float* part) {
  MP_CHECK_ARG(d >= 3 && d <= kJD, MP_ERR_UNSUPPORTED,
               "mp_binned_counts: joint distributions need d <= %d (d = %d)", kJD, d);
  for (int b = 0; b < d; ++b)
    MP_CHECK_ARG(K[b] >= 1 && K[b] <= 1024, MP_ERR_UNSUPPORTED,
                 "mp_binned_counts: joint windows of d >= 3 need 1 <= K <= 1024 (K[%d] = %d)", b, K[b]);
  JointDParams p{};
  int64_t cells = 1;
  for (int b = 0; b < d; ++b) cells *= K[b];
  MP_CHECK_ARG(cells < 0x7fffffff, MP_ERR_UNSUPPORTED,
               "mp_binned_counts: joint grid of %lld cells exceeds 2^31 - 1", (long long)cells);
  MP_CHECK_ARG(fill_params(p, M, E, d, bin_of_mode, m_lo, K, ns, e0), MP_ERR_UNSUPPORTED,
               "mp_binned_counts: bins form more than %d contiguous mode runs", MP_MAX_RUNS);
  p.est = est;
  const int64_t s_last = (e0 + E - 1) / ns;
  MP_CHECK_ARG(s_last < n_sub, MP_ERR_SHAPE,
               "mp_binned_counts: samples [%lld, %lld) exceed n_sub * samples_per_sub = %lld",
               (long long)e0, (long long)(e0 + E), (long long)n_sub * ns);
  const size_t need = layout(p, prec == MP_FP64 ? 8 : 4);
  MP_CHECK_ARG(ws && ws_bytes >= need, MP_ERR_WORKSPACE,
               "mp_binned_counts: workspace of %zu bytes needed, %zu given", need, ws_bytes);
  const int tile = prec == MP_FP64 ? QT : PT;
  const int64_t items = (s_last - p.s_first + 1) * ((p.rows_max + tile - 1) / tile) *
                        ((K[d - 1] + tile - 1) / tile);
  MP_CHECK_ARG(items < 0x7fffffff, MP_ERR_UNSUPPORTED,
               "mp_binned_counts: the joint grid of %lld workgroups is too large", (long long)items);
  int* band = (int*)ws;
  double* rec = (double*)((char*)ws + 256);
  void* tables = (char*)ws + 256 + round_up(E * p.rec * 8, 256);
  hipLaunchKernelGGL(band_init, dim3(1), dim3(64), 0, stream, band);
  // rows of 16 lanes also for the partials, of which a run has few (amplitudes, 1e5 samples
  // of three bins of 100 modes: 144 us, 186 us by waves)
  const bool rows = part || short_runs(M, p.n_runs, elem_bytes_c(prec), kRowBytesOcc);
  const int64_t per = kOccPerWave * (rows ? 16 : 4);
  auto occ = [&](auto kernel, auto* c) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)((E + per - 1) / per)), dim3(256), 0, stream, p, c, part,
                       n, rec);
  };
  if (part)
    occ(jointd_occupations<float, true, 16>, (const float*)nullptr);
  else if (prec == MP_FP64)
    occ(rows ? jointd_occupations<double, false, 16> : jointd_occupations<double, false, 64>,
        (const double*)C);
  else
    occ(rows ? jointd_occupations<float, false, 16> : jointd_occupations<float, false, 64>,
        (const float*)C);
  int kp_max = 0;
  for (int b = 0; b < d; ++b) kp_max = p.Kp[b] > kp_max ? p.Kp[b] : kp_max;
  const dim3 fgrid((unsigned)((E * kp_max + 255) / 256), (unsigned)(2 * d));
  const mp_status sb = record_bands_launch(rec, E, d, K, kJD, band, stream);
  if (sb != MP_OK) return sb;
  if (prec == MP_FP64) {
    hipLaunchKernelGGL(jointd_factors<double>, fgrid, dim3(256), 0, stream, p, rec, band,
                       (double*)tables);
    for (int tau = 0; tau < 2; ++tau)
      hipLaunchKernelGGL(jointd_sum_f64, dim3((unsigned)items), dim3(256), 0, stream, p, tau,
                         (const double*)tables, band, acc);
  } else {
    hipLaunchKernelGGL(jointd_factors<float>, fgrid, dim3(256), 0, stream, p, rec, band,
                       (float*)tables);
    for (int tau = 0; tau < 2; ++tau)
      hipLaunchKernelGGL((p.d == 3 ? jointd_sum_f32<3> : jointd_sum_f32<4>), dim3((unsigned)items),
                         dim3(256), 0, stream, p, tau, (const float*)tables, band, acc);
  }
  MP_HIP_LAUNCH_CHECK("mp_binned_counts joint (d >= 3) launch");
  return MP_OK;
}

mp_status jointd_finalize(int32_t d, const int32_t* K, int32_t n_sub, int64_t ns,
                          const double* acc, double* P_re, double* P_im, double* sigma, void* ws,
                          size_t ws_bytes, hipStream_t stream) {
  // one sub-ensemble at a time needs the least; a larger workspace
  // (jointd_finalize_workspace with the run's n_sub) takes several per launch
  const size_t need = jointd_finalize_workspace(d, K, 1);
  MP_CHECK_ARG(ws && ws_bytes >= need, MP_ERR_WORKSPACE,
               "mp_counts_finalize: workspace of %zu bytes needed, %zu given", need, ws_bytes);
  const int kmax = d == 2 ? kAxisMaxK : 1024;
  for (int b = 0; b < d; ++b)
    MP_CHECK_ARG(K[b] >= 1 && K[b] <= kmax, MP_ERR_UNSUPPORTED,
                 "mp_counts_finalize: joint windows of %d bins need 1 <= K <= %d (K[%d] = %d)", d,
                 kmax, b, K[b]);
  static bool lds_set = false;
  if (!lds_set) {
    for (const void* k : {(const void*)jointd_axis<false, 8>, (const void*)jointd_axis<true, 8>,
                          (const void*)jointd_axis<false, 1>, (const void*)jointd_axis<true, 1>}) {
      const hipError_t e =
          hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kAxisMaxLds);
      MP_CHECK_ARG(e == hipSuccess, MP_ERR_HIP, "mp_counts_finalize: %s", hipGetErrorString(e));
    }
    lds_set = true;
  }
  int64_t cells = 1;
  for (int b = 0; b < d; ++b) cells *= K[b];
  MP_CHECK_ARG(cells < 0x7fffffff, MP_ERR_UNSUPPORTED,
               "mp_counts_finalize: joint grid of %lld cells exceeds 2^31 - 1", (long long)cells);
  const int64_t one = round_up(cells * 16, 256);
  const int64_t fit = ((int64_t)ws_bytes - 256) / (2 * one);
  int batch = (int)(fit < n_sub ? fit : n_sub);
  batch = batch < kAxisMaxSubs ? batch : kAxisMaxSubs;
  double* buf[2] = {(double*)((char*)ws + 256), (double*)((char*)ws + 256 + batch * one)};
  AxisParams axis[kJD];
  for (int a = 0; a < d; ++a) axis[a] = axis_params(d, K, a, cells);
  for (int s = 0; s < n_sub; s += batch) {
    const double* src = acc + 2 * (int64_t)s * cells;
    for (int a = 0; a < d; ++a) {
      AxisParams& p = axis[a];
      p.s0 = s;
      p.subs = n_sub - s < batch ? n_sub - s : batch;
      p.scale = 1.0 / ((double)cells * (double)ns);
      double* dst = buf[a & 1];
      const unsigned groups = (unsigned)((p.n_lines + p.G - 1) / p.G);
      if (a == d - 1)
        hipLaunchKernelGGL((p.out == 8 ? jointd_axis<true, 8> : jointd_axis<true, 1>), dim3(groups), dim3(256), axis_lds(p), stream, p, src,
                           (double*)nullptr, P_re, P_im, sigma);
      else
        hipLaunchKernelGGL((p.out == 8 ? jointd_axis<false, 8> : jointd_axis<false, 1>),
                           dim3(groups, (unsigned)p.subs), dim3(256),
                           axis_lds(p), stream, p, src, dst, (double*)nullptr, (double*)nullptr,
                           (double*)nullptr);
      src = dst;
    }
  }
  hipLaunchKernelGGL(jointd_sigma, dim3((unsigned)((cells + 255) / 256)), dim3(256), 0, stream,
                     cells, n_sub, sigma);
  MP_HIP_LAUNCH_CHECK("mp_counts_finalize joint (d >= 3) launch");
  return MP_OK;
}

}  // namespace mp
