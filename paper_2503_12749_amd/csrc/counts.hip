// Grouped photon-count observables: occupations, matrix-P parity weight and
// characteristic function (fused), deterministic sub-ensemble reduction, and
// the FP64 inverse DFT to P(m) with the sub-ensemble error sigma_T.
//
// Paper, eq. c-number-variable: per sample the pattern observable is
// G(m) = g0(n_S, m) prod_i n_i^c_i e^{-n_i} / c_i!, with
// g0 = (1 + pi_m e^{2 (n_S - n)}) / (1 + e^{-2n}).  Summed over the patterns of
// each bin (multinomial theorem) and over all counts with weights z_b^m_b,
//     chi(z) = (e^X + e^{-X - 2n}) / (1 + e^{-2n}) = cosh(n + X) / cosh(n),
//     X = sum_b n_b (z_b - 1),
// so the count distribution of the ensemble is the inverse DFT of the mean
// chi on z = e^{2 pi i k / K}.  Each evaluation also carries the window shift
// z^{-m_lo}, and both terms are formed as exp(real exponent) * cis(phase)
// with the exponent shifted by -log(1 + e^{-2|n|}) so that nothing overflows
// for either sign of n.  The positive-P variant (Appendix A) drops g0: chi = e^X.
//
// Sub-ensembles (Appendix A): samples g in [s N_S, (s+1) N_S) form
// sub-ensemble s; P is the mean of the sub-ensemble estimates and sigma_T
// their standard deviation over sqrt(N_R).
#include <hip/hip_runtime.h>

#include <mutex>
#include <vector>

#include "chi.h"
#include "common.h"

namespace mp {

constexpr int kSBlk = 64;        // least samples per workgroup of the fused kernel
constexpr int kSBlkMax = 256;
constexpr int kCountThreads = 512;
constexpr int kEpt = 4;          // accumulator entries per thread tested at a time
constexpr int kMaxDist = MP_MAX_BINS + 1;
struct CountsParams {
  int M;
  int64_t ldm;
  int64_t E;        // samples in the chunk
  int64_t e0;       // global index of the chunk's first sample
  int64_t ns;       // samples per sub-ensemble
  int d;
  int mode;         // mp_bin_mode
  int est;          // mp_estimator
  int n_runs;
  int run_lo[MP_MAX_RUNS], run_hi[MP_MAX_RUNS], run_bin[MP_MAX_RUNS];
  int n_dist;
  int dist_src[kMaxDist];  // bin index feeding each distribution, -1 = total
  int m_lo[kMaxDist], K[kMaxDist];
  int off[kMaxDist + 1];   // entry offsets (prefix sums of K)
  int entries;
  // block -> (sub-ensemble, tile) arithmetic
  int64_t s_first, s_last;
  int t_first, t_mid, t_last, n_mid;
  int sblk;         // samples per workgroup, kSBlk .. kSBlkMax
};

__host__ __device__ inline int64_t sub_lo(const CountsParams& p, int64_t s) {
  int64_t a = s * p.ns;
  return a > p.e0 ? a : p.e0;
}
__host__ __device__ inline int64_t sub_hi(const CountsParams& p, int64_t s) {
  int64_t a = (s + 1) * p.ns, b = p.e0 + p.E;
  return a < b ? a : b;
}

// Block b -> sub-ensemble s and global sample range [lo, hi).
__device__ inline void block_samples(const CountsParams& p, int b, int64_t& s, int64_t& lo,
                                     int64_t& hi) {
  int tile;
  if (b < p.t_first) {
    s = p.s_first;
    tile = b;
  } else {
    b -= p.t_first;
    if (b < p.n_mid * p.t_mid) {
      s = p.s_first + 1 + b / p.t_mid;
      tile = b % p.t_mid;
    } else {
      s = p.s_last;
      tile = b - p.n_mid * p.t_mid;
    }
  }
  const int64_t a = sub_lo(p, s), z = sub_hi(p, s);
  lo = a + (int64_t)tile * p.sblk;
  hi = lo + p.sblk < z ? lo + p.sblk : z;
}

// Sources of a workgroup's bin sums for counts_fused: the propagated amplitudes
// C (mp_propagate) or the per-block partials of the occupation-fused GEMM.
// bin_sums leaves nb[i][b] of the samples lo + i (chunk-local k0 + i), i < nsmp,
// in LDS for every bin b < d, behind a barrier; red is LDS scratch.
typedef __attribute__((ext_vector_type(2))) double d2;

template <typename CT, int G>
struct FromC {
  const CT* C;
  // G lanes per sample over its modes: a wave, or a row of 16 (four samples at a time)
  __device__ inline void bin_sums(const CountsParams& p, int64_t k0, int nsmp,
                                  d2 (*nb)[kMaxDist], d2*) const {
    const int gl = threadIdx.x % G;
    const int64_t ldc = 2 * p.ldm;
    for (int i = threadIdx.x / G; i < nsmp; i += kCountThreads / G) {
      const int64_t k = k0 + i;
      if (gl == 0)
        for (int b = 0; b < p.d; ++b) nb[i][b] = d2{0.0, 0.0};
      for (int q = 0; q < p.n_runs; ++q) {
        double re, im;
        run_sum<CT, G>(C + k * ldc, C + (p.E + k) * ldc, p.ldm, p.run_lo[q], p.run_hi[q], gl, re, im);
        if (gl == 0) nb[i][p.run_bin[q]] += d2{re, im};
      }
    }
    __syncthreads();
  }
};

struct FromPartials {
  const float* part;  // FusedOut layout, E = p.E
  // lane per sample, so that the 16-byte partials of neighbouring samples share their
  // lines (a wave per sample with lanes over slots read each line eight times over);
  // the waves share out a run's slots
  __device__ inline void bin_sums(const CountsParams& p, int64_t k0, int nsmp,
                                  d2 (*nb)[kMaxDist], d2* red) const {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int groups = (nsmp + 63) / 64, split = kCountThreads / 64 / ((p.sblk + 63) / 64);
    const int g = wave / split, w = wave % split;
    const int i = 64 * g + lane;
    for (int e = threadIdx.x; e < nsmp * p.d; e += kCountThreads) nb[e / p.d][e % p.d] = d2{0.0, 0.0};
    int slot0 = 0;
    for (int q = 0; q < p.n_runs; ++q) {
      const int nblk = run_blocks(p.run_lo[q], p.run_hi[q]);
      d2 s = {0.0, 0.0};
      if (g < groups && i < nsmp)
#pragma unroll 4
        for (int t = w; t < nblk; t += split) {
          const float4 v = *(const float4*)(part + ((int64_t)(slot0 + t) * p.E + k0 + i) * 4);
          s += d2{(double)v.x + (double)v.z, (double)v.y + (double)v.w};
        }
      red[threadIdx.x] = s;
      __syncthreads();
      if (threadIdx.x < nsmp) {
        const int at = (threadIdx.x / 64) * split * 64 + lane;
        d2 t = red[at];
        for (int u = 1; u < split; ++u) t += red[at + 64 * u];
        nb[threadIdx.x][p.run_bin[q]] += t;
      }
      __syncthreads();
      slot0 += nblk;
    }
    if (p.n_runs == 0) __syncthreads();
  }
};

// Phase 1: the samples' bin occupations (Src), and their two parity weights.
// Phase 2: the characteristic function on the window grid, summed over the
// workgroup's samples.  A term is evaluated only where its exact log-magnitude
// exceeds kLogEps, which for large occupations leaves the grid points near
// theta = 0 (first term) and pi (second): the grid points where no sample of the
// workgroup can reach it, by a bound from the samples' least Re n_q and largest
// |Im n_q|, are dropped up front, the others listed in LDS, and the threads take
// that list times groups of the samples, so that every lane has work (with a
// fixed grid point per thread, 256 of 1408 points active at M = 1000 kept one or
// two of four waves busy).  The groups' sums meet in LDS in order.
// Bound by phase 1's loads (from C: 16 bytes per mode and sample) and the
// exponentials of phase 2.  1e5 samples of M = 1000 from FP32 C, 1408 points:
// 341 us against 569 us with 64 samples per 256 threads and fixed points;
// 65536 samples of M = 8000 from partials, 4160 points: 60 against 376 us.
template <typename Src, bool F64>
__global__ __launch_bounds__(kCountThreads) void counts_fused(CountsParams p, Src src,
                                                              const double* __restrict__ nglob,
                                                              double* __restrict__ partials) {
  __shared__ d2 s_nb[kSBlkMax][kMaxDist];
  __shared__ d2 s_c[kSBlkMax];  // log-weights; the second -inf where the partner underflows
  __shared__ d2 s_red[kCountThreads];
  __shared__ int s_list[kCountThreads * kEpt];
  __shared__ int s_wcnt[kCountThreads / 64];
  __shared__ double s_bound[kMaxDist][4];  // least Re, largest |Im|, largest c1, c2 + 2 Re
  __shared__ int s_all;
  int64_t sub, lo, hi;
  block_samples(p, blockIdx.x, sub, lo, hi);
  const int nsmp = (int)(hi - lo);
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;

  if (tid == 0) s_all = 0;
  src.bin_sums(p, lo - p.e0, nsmp, s_nb, s_red);
  if (tid < nsmp) {
    if (p.n_dist > p.d) {  // the total over the bins
      d2 t = {0.0, 0.0};
      for (int b = 0; b < p.d; ++b) t += s_nb[tid][b];
      s_nb[tid][p.d] = t;
    }
    const double n = nglob[lo - p.e0 + tid];
    bool finite = p.est == MP_PLUS_P || isfinite(n);
    double mx = 0.0;
    for (int q = 0; q < p.n_dist; ++q) {
      const d2 v = s_nb[tid][q];
      finite = finite && isfinite(v.x) && isfinite(v.y);
      const double a = sqrt(v.x * v.x + v.y * v.y);
      mx = a > mx ? a : mx;
    }
    d2 c;
    if (p.est == MP_PLUS_P) {
      c = d2{finite ? 0.0 : __builtin_nan(""), -INFINITY};
    } else {
      double c1, c2;
      parity_log_weights(n, finite, c1, c2);
      // |e^{-X}| <= e^{2 |n_b|}: skip the parity partner when it underflows
      c = d2{c1, 2.0 * mx + c2 < -800.0 ? -INFINITY : c2};
    }
    s_c[tid] = c;
    if (!finite) s_all = 1;  // a sample that is not finite reaches every grid point
  }
  __syncthreads();
  for (int q = wave; q < p.n_dist; q += kCountThreads / 64) {
    double r = INFINITY, i = 0.0, a = -INFINITY, b = -INFINITY;
    for (int k = lane; k < nsmp; k += 64) {
      const d2 v = s_nb[k][q], c = s_c[k];
      r = fmin(r, v.x);
      i = fmax(i, fabs(v.y));
      a = fmax(a, c.x);
      b = fmax(b, c.y + 2.0 * v.x);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      r = fmin(r, __shfl_xor(r, off, 64));
      i = fmax(i, __shfl_xor(i, off, 64));
      a = fmax(a, __shfl_xor(a, off, 64));
      b = fmax(b, __shfl_xor(b, off, 64));
    }
    if (lane == 0) {
      s_bound[q][0] = r;
      s_bound[q][1] = i;
      s_bound[q][2] = a;
      s_bound[q][3] = b;
    }
  }
  __syncthreads();

  constexpr double kTwoPi = 6.283185307179586476925286766559;
  const bool all = s_all != 0;
  auto dist_of = [&](int e) {
    int q = 0;
    while (q + 1 < p.n_dist && e >= p.off[q + 1]) ++q;
    return q;
  };
  double* out = partials + (int64_t)blockIdx.x * p.entries * 2;
  for (int base = 0; base < p.entries; base += kCountThreads * kEpt) {
    // the grid points that some sample may reach, in order
    int count = 0;
#pragma unroll
    for (int u = 0; u < kEpt; ++u) {
      const int e = base + u * kCountThreads + tid;
      bool in = false;
      if (e < p.entries) {
        const int q = dist_of(e);
        const double th = kTwoPi * (double)(e - p.off[q]) / (double)p.K[q];
        // in FP32 with a margin of 1: |log-magnitudes| that matter are below 2^13 times a
        // few ulps, and the bound only has to include every point that the exact test takes
        const float sh = sinf((float)(0.5 * th)), ch = cosf((float)(0.5 * th));
        const double one_minus = 2.0 * (double)sh * sh, one_plus = 2.0 * (double)ch * ch;
        const double sn = 2.0 * fabs((double)sh * ch);
        const double* bd = s_bound[q];
        const double slack = 1.0 + 1e-5 * (fabs(bd[0]) + bd[1]);
        in = all || bd[2] - one_minus * bd[0] + sn * bd[1] + slack > kLogEps ||
             bd[3] - one_plus * bd[0] + sn * bd[1] + slack > kLogEps;
        if (!in) {
          out[2 * (int64_t)e] = 0.0;
          out[2 * (int64_t)e + 1] = 0.0;
        }
      }
      const unsigned long long mask = __ballot(in);
      if (lane == 0) s_wcnt[wave] = __popcll(mask);
      __syncthreads();
      int at = count;
#pragma unroll
      for (int w = 0; w < kCountThreads / 64; ++w) {
        at += w < wave ? s_wcnt[w] : 0;
        count += s_wcnt[w];
      }
      if (in) s_list[at + __popcll(mask & ((1ull << lane) - 1ull))] = e;
      __syncthreads();
    }
    for (int a0 = 0; a0 < count; a0 += kCountThreads) {
      // `groups` threads per listed point, each with every groups-th sample
      const int na = count - a0 < kCountThreads ? count - a0 : kCountThreads;
      int groups = 1;
      while (2 * groups * na <= kCountThreads && groups < nsmp) groups *= 2;
      const int g = tid / na, ai = tid - g * na;
      d2 sum = {0.0, 0.0};
      int e = 0;
      if (g < groups) {
        e = s_list[a0 + ai];
        const int q = dist_of(e), K = p.K[q], kk = e - p.off[q];
        const double th = kTwoPi * (double)kk / (double)K;
        double sn, cs;
        sincos(th, &sn, &cs);
        const double sh = sin(0.5 * th);
        const double cm1 = -2.0 * sh * sh;  // cos(th) - 1 without cancellation
        const int64_t red = ((int64_t)kk * (int64_t)p.m_lo[q]) % K;
        const double thl = kTwoPi * (double)red / (double)K;  // th * m_lo reduced mod 2 pi
        for (int i = g; i < nsmp; i += groups) {
          const d2 v = s_nb[i][q], c = s_c[i];
          // log-magnitudes of the two terms are xr + c1 and c2 - xr; a term
          // below e^kLogEps is skipped (a NaN one is kept: it must reach the sums)
          // (fused in this order: partials of few bits reach rounding ties of the FP32 terms at
          // theta = pi/2 and 3 pi/2)
          const double xr = fma(cm1, v.x, -(sn * v.y));
          const bool t1 = !(xr + c.x <= kLogEps), t2 = c.y != -INFINITY && !(c.y - xr <= kLogEps);
          if (!(t1 || t2)) continue;
          const double xi = fma(sn, v.x, cm1 * v.y);
          double tr, ti;
          if (t1) {
            cis_exp<F64>(xr + c.x, xi - thl, tr, ti);
            sum += d2{tr, ti};
          }
          if (t2) {
            cis_exp<F64>(c.y - xr, -xi - thl, tr, ti);
            sum += d2{tr, ti};
          }
        }
      }
      s_red[tid] = sum;
      __syncthreads();
      if (tid < na) {
        for (int u = 1; u < groups; ++u) sum += s_red[tid + u * na];
        out[2 * (int64_t)e] = sum.x;
        out[2 * (int64_t)e + 1] = sum.y;
      }
      __syncthreads();
    }
  }
}

// acc[s] += sum over the tiles of s of the partials, in tile order.
__global__ void counts_reduce(CountsParams p, const double* __restrict__ partials,
                              double* __restrict__ acc) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= p.entries) return;
  const int64_t s = p.s_first + blockIdx.y;
  int b0, nt;
  if (s == p.s_first) {
    b0 = 0;
    nt = p.t_first;
  } else if (s == p.s_last) {
    b0 = p.t_first + p.n_mid * p.t_mid;
    nt = p.t_last;
  } else {
    b0 = p.t_first + (int)(s - p.s_first - 1) * p.t_mid;
    nt = p.t_mid;
  }
  double re = 0.0, im = 0.0;
  for (int t = 0; t < nt; ++t) {
    const double* src = partials + ((int64_t)(b0 + t) * p.entries + e) * 2;
    re += src[0];
    im += src[1];
  }
  double* dst = acc + (s * (int64_t)p.entries + e) * 2;
  dst[0] += re;
  dst[1] += im;
}

// ---------------------------------------------------------------- joint, d = 2

// Joint distribution of two bins.  Per sample the generating function
// factorises,
//     chi(z1, z2) = e^{c1} u1(z1) u2(z2) + e^{c2} v1(z1) v2(z2),
//     u_b = e^{X_b} z_b^{-m_lo_b},  v_b = e^{-X_b} z_b^{-m_lo_b},
// so the sum over a sub-ensemble is a sum of rank-1 outer products.  For
// theta in [0, pi] the exponent of |u_b| is
//     f_b(theta) = -(1 - cos theta) Re n_b + |sin theta| |Im n_b|
// (v_b: the same about theta = pi, plus 2 Re n_b), which rises to its maximum
// at tan theta* = |Im n_b| / Re n_b and then falls monotonically.  Each sample
// gets, per term and bin, the half-width of the band around theta = 0 (u) or
// pi (v) outside which its term is below e^-46 (~1e-20) for every value of the
// other bin; the chunk's band is the maximum over its samples.  Terms outside
// the band are bounded by that threshold, not approximated.


struct Joint2Params {
  int M;
  int64_t ldm, E, e0, ns;
  int est;
  int n_runs;
  int run_lo[MP_MAX_RUNS], run_hi[MP_MAX_RUNS], run_bin[MP_MAX_RUNS];
  int m_lo[2], K[2];
  int64_t s_first, s_last;
};

// Per-sample record (G lanes per sample, the first writes): n1, n2 (complex),
// c1, c2 (c2 = -inf for +P; both NaN for a sample that is not finite).
// record_bands then sets the chunk's bands
// band[0..3] = u1, u2, v1, v2 half-widths (atomic max, -1 = empty).
// PART: the bin sums come from the occupation-fused GEMM's partials (slots in
// run order) instead of the propagated amplitudes C.
template <typename CT, bool PART, int G>
__device__ inline void joint2_sample(const Joint2Params& p, const CT* __restrict__ C,
                                     const float* __restrict__ part,
                                     const double* __restrict__ nglob, double* __restrict__ rec,
                                     int64_t k, int gl) {
  const int64_t ldc = 2 * p.ldm;
  const CT* ca = PART ? nullptr : C + k * ldc;
  const CT* cb = PART ? nullptr : C + (p.E + k) * ldc;
  double R1 = 0.0, I1 = 0.0, R2 = 0.0, I2 = 0.0;
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
    const bool first = p.run_bin[q] == 0;
    R1 += first ? re : 0.0;
    I1 += first ? im : 0.0;
    R2 += first ? 0.0 : re;
    I2 += first ? 0.0 : im;
  }
  if (gl != 0) return;
  const double n = nglob[k];
  const bool sums_finite = isfinite(R1) && isfinite(I1) && isfinite(R2) && isfinite(I2);
  double c1 = 0.0, c2 = -INFINITY;
  if (p.est != MP_PLUS_P)
    parity_log_weights(n, sums_finite && isfinite(n), c1, c2);
  else if (!sums_finite)
    c1 = c2 = __builtin_nan("");
  double* r = rec + k * 6;
  r[0] = R1;
  r[1] = I1;
  r[2] = R2;
  r[3] = I2;
  r[4] = c1;
  r[5] = c2;
}

template <typename CT, bool PART, int G>
__global__ __launch_bounds__(256) void joint2_occupations(Joint2Params p, const CT* __restrict__ C,
                                                          const float* __restrict__ part,
                                                          const double* __restrict__ nglob,
                                                          double* __restrict__ rec) {
  constexpr int S = 256 / G;  // samples of a workgroup at a time
  const int64_t base = (int64_t)blockIdx.x * (S * kOccPerWave) + threadIdx.x / G;
  for (int j = 0; j < kOccPerWave; ++j) {
    const int64_t k = base + S * j;
    if (k >= p.E) return;
    joint2_sample<CT, PART, G>(p, C, part, nglob, rec, k, threadIdx.x % G);
  }
}

__global__ void joint2_band_init(int* band) {
  if (threadIdx.x < 4) band[threadIdx.x] = -1;
}

// Box half-widths from the per-sample records (layout of record_band): block
// row blockIdx.y = tau d + b, samples strided over its threads, the workgroup's maximum,
// then one atomic maximum per workgroup into band[tau * band_stride + b].  At most
// kBandBlocks workgroups per row: with one atomic per wave of one sample a thread the kernel
// waited for them to take turns at a row's word (1e5 samples, three bins: 118 us, now
// 41 us; two bins: 89 us, now 22 us).
constexpr int kBandBlocks = 128;
__global__ __launch_bounds__(256) void record_bands(const double* __restrict__ rec, int64_t E,
                                                    int d, int K0, int K1, int K2, int K3,
                                                    int band_stride, int* __restrict__ band) {
  __shared__ int top[4];
  const int tau = blockIdx.y / d, b = blockIdx.y % d;
  const int K = b == 0 ? K0 : (b == 1 ? K1 : (b == 2 ? K2 : K3));
  int h = -1;
  for (int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x; k < E; k += (int64_t)gridDim.x * 256)
    h = max(h, record_band(rec + k * (2 * d + 2), d, tau, b, K));
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) h = max(h, __shfl_xor(h, off, 64));
  if ((threadIdx.x & 63) == 0) top[threadIdx.x >> 6] = h;
  __syncthreads();
  if (threadIdx.x == 0)
    atomicMax(&band[tau * band_stride + b], max(max(top[0], top[1]), max(top[2], top[3])));
}

mp_status record_bands_launch(const double* rec, int64_t E, int d, const int32_t* K,
                              int band_stride, int* band, hipStream_t stream) {
  const int64_t full = (E + 255) / 256, blocks = full < kBandBlocks ? full : kBandBlocks;
  hipLaunchKernelGGL(record_bands, dim3((unsigned)blocks, (unsigned)(2 * d)), dim3(256), 0,
                     stream, rec, E, d, K[0], d > 1 ? K[1] : 1, d > 2 ? K[2] : 1,
                     d > 3 ? K[3] : 1, band_stride, band);
  MP_HIP_LAUNCH_CHECK("mp_binned_counts box bounds launch");
  return MP_OK;
}

// One axis point of a tile: the grid angle's cos - 1 and sin, the window shift,
// and whether the point lies in the term's band.
struct Joint2Point {
  double cm1, sn, thl;
  bool in;
};

__device__ inline Joint2Point joint2_point(int k, int K, int m_lo, bool in) {
  constexpr double kTwoPi = 6.283185307179586476925286766559;
  const double th = kTwoPi * (double)k / (double)K;
  const double sh = sin(0.5 * th);
  const int64_t red = ((int64_t)k * (int64_t)m_lo) % K;
  return {-2.0 * sh * sh, sin(th), kTwoPi * (double)red / (double)K, in};
}

// e^{sign X(theta) + c} z^{-m_lo}, X = n (e^{i theta} - 1)
template <bool F64>
__device__ inline void joint2_factor(const Joint2Point& q, double R, double I, double c,
                                     double sign, double& fr, double& fi) {
  // (fused in this order, see counts_fused)
  const double xr = fma(q.cm1, R, -(q.sn * I)), xi = fma(q.cm1, I, q.sn * R);
  cis_exp<F64>(fma(sign, xr, c), fma(sign, xi, -q.thl), fr, fi);
}

typedef __attribute__((ext_vector_type(4))) double f64x4;
constexpr int kJWaves = 8;  // each takes every eighth group of four samples

// acc[s][k1][k2] += sum over the chunk's samples of sub-ensemble s of the
// band-limited outer products, on the FP64 matrix cores: v_mfma_f64_16x16x4f64
// takes A[l % 16][l / 16] and B[l / 16][l % 16] from lane l, so a lane forms the
// factors of its sample (l / 16 of a group of four) at three points of either
// axis straight into the operand registers and a wave adds a tile of 16 JB x 16 JB
// complex cells (JB = 3: 48 x 48, 36 products), without LDS or a barrier in the loop; the eight waves'
// sums are added through LDS in wave order at the end.  Output register r of
// lane l is row l / 16 + 4 r, column l % 16 of a block.  Tiles start at the
// corner of each term's box (grid z = term; tiles past the box return), so a
// box of about 2 x 70 points takes nine of them; boxes that meet (small
// grids) are tiled on the grid instead, each tile adding both terms, so that a
// cell has one writer either way.  Bound by the FP64 products and the factors'
// exponentials about equally (they run beside each other, two waves per SIMD).
// 16 x 16 tiles with both factors in LDS and plain FMAs evaluated every factor
// nine times and took 6852 us for 1e5 samples of M = 1000 in ten sub-ensembles
// on 1024 x 1024 windows (now 1126 us).
template <bool F64, int JB>
__global__ __launch_bounds__(64 * kJWaves, 1) void joint2_accumulate(
    Joint2Params p, const double* __restrict__ rec, const int* __restrict__ band,
    double* __restrict__ acc) {
  constexpr int kJT = 16 * JB;  // tile side
  __shared__ double red[kJT][kJT][2];
  const int K1 = p.K[0], K2 = p.K[1];
  int h1[2], h2[2];
  bool on[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {
    h1[t] = band[2 * t];
    h2[t] = band[2 * t + 1];
    on[t] = h1[t] >= 0 && h2[t] >= 0;
  }
  // boxes about 0 and about K / 2 share a cell where they meet on both axes
  const bool meet = on[0] && on[1] && h1[0] + h1[1] >= K1 / 2 && h2[0] + h2[1] >= K2 / 2;
  const int only = (int)blockIdx.z;  // the term of this workgroup, unless the boxes meet
  const int tiles2 = (K2 + kJT - 1) / kJT;
  const int i0 = (int)(blockIdx.x / tiles2) * kJT, j0 = (int)(blockIdx.x % tiles2) * kJT;
  int org1 = 0, org2 = 0, w1 = K1, w2 = K2;  // origin and extent of the tiled region
  if (meet) {
    if (only == 1) return;
  } else {
    if (!on[only]) return;
    w1 = min(2 * h1[only] + 1, K1);
    w2 = min(2 * h2[only] + 1, K2);
    org1 = ((only ? K1 / 2 : 0) - h1[only] + K1) % K1;
    org2 = ((only ? K2 / 2 : 0) - h2[only] + K2) % K2;
  }
  if (i0 >= w1 || j0 >= w2) return;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, lr = lane & 15, lh = lane >> 4;
  const int64_t s = p.s_first + blockIdx.y;
  int64_t lo = s * p.ns, hi = (s + 1) * p.ns;
  lo = lo > p.e0 ? lo : p.e0;
  hi = hi < p.e0 + p.E ? hi : p.e0 + p.E;

  f64x4 re[JB][JB], im[JB][JB];
#pragma unroll
  for (int a = 0; a < JB; ++a)
#pragma unroll
    for (int b = 0; b < JB; ++b) re[a][b] = im[a][b] = f64x4{0.0, 0.0, 0.0, 0.0};
  for (int t = meet ? 0 : only; t <= (meet ? 1 : only); ++t) {
    Joint2Point q1[JB], q2[JB];
#pragma unroll
    for (int b = 0; b < JB; ++b) {
      const int i = i0 + 16 * b + lr, j = j0 + 16 * b + lr;
      const int k1 = (org1 + i) % K1, k2 = (org2 + j) % K2;
      q1[b] = joint2_point(k1, K1, p.m_lo[0],
                           i < w1 && circ_dist(k1, t ? K1 / 2 : 0, K1) <= h1[t]);
      q2[b] = joint2_point(k2, K2, p.m_lo[1],
                           j < w2 && circ_dist(k2, t ? K2 / 2 : 0, K2) <= h2[t]);
    }
    const double sign = t == 0 ? 1.0 : -1.0;
    for (int64_t g = lo + 4 * wave; g < hi; g += 4 * kJWaves) {
      const bool mine = g + lh < hi;
      const double* r = rec + ((mine ? g + lh : lo) - p.e0) * 6;
      const double R1 = r[0], I1 = r[1], R2 = r[2], I2 = r[3];
      const double cterm = t == 0 ? r[4] : r[5];
      // the product's log-magnitude at the band centre (c, or c + 2 Re n_1
      // + 2 Re n_2 for the second term) is shared evenly between the two
      // factors, so neither overflows while the other underflows in FP32
      const double share = 0.5 * (cterm + (t == 0 ? 0.0 : 2.0 * (R1 + R2)));
      const bool ok = mine && cterm != -INFINITY;
      double xr[JB], xi[JB], yr[JB], yi[JB];
#pragma unroll
      for (int b = 0; b < JB; ++b) {
        xr[b] = xi[b] = yr[b] = yi[b] = 0.0;
        if (ok && q1[b].in)
          joint2_factor<F64>(q1[b], R1, I1, share - (t == 0 ? 0.0 : 2.0 * R1), sign, xr[b], xi[b]);
        if (ok && q2[b].in)
          joint2_factor<F64>(q2[b], R2, I2, share - (t == 0 ? 0.0 : 2.0 * R2), sign, yr[b], yi[b]);
      }
#pragma unroll
      for (int a = 0; a < JB; ++a)
#pragma unroll
        for (int b = 0; b < JB; ++b) {
          re[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(xr[a], yr[b], re[a][b], 0, 0, 0);
          im[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(xr[a], yi[b], im[a][b], 0, 0, 0);
          re[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(-xi[a], yi[b], re[a][b], 0, 0, 0);
          im[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(xi[a], yr[b], im[a][b], 0, 0, 0);
        }
    }
  }
  for (int w = 0; w < kJWaves; ++w) {
    if (wave == w) {
#pragma unroll
      for (int a = 0; a < JB; ++a)
#pragma unroll
        for (int b = 0; b < JB; ++b)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            double* o = red[16 * a + lh + 4 * r][16 * b + lr];
            o[0] = (w == 0 ? 0.0 : o[0]) + re[a][b][r];
            o[1] = (w == 0 ? 0.0 : o[1]) + im[a][b][r];
          }
    }
    __syncthreads();
  }
  for (int e = tid; e < kJT * kJT; e += 64 * kJWaves) {
    const int i = i0 + e / kJT, j = j0 + e % kJT;
    const double ar = red[e / kJT][e % kJT][0], ai = red[e / kJT][e % kJT][1];
    if (i < w1 && j < w2 && (ar != 0.0 || ai != 0.0)) {
      const int k1 = (org1 + i) % K1, k2 = (org2 + j) % K2;
      double* dst = acc + ((int64_t)s * K1 * K2 + (int64_t)k1 * K2 + k2) * 2;
      dst[0] += ar;
      dst[1] += ai;
    }
  }
}

// Tile of joint2_accumulate: the largest with at least 512 workgroups (two per
// CU) over the whole grid, so that small grids of few sub-ensembles still
// spread over the chip; a larger tile evaluates fewer factors (2 JB per lane
// for 4 JB^2 products).  JB = 3 spills in the FP64 form.
template <bool F64, int JB>
static void joint2_launch_tile(const Joint2Params& p, unsigned nst, const double* rec,
                               const int* band, double* acc, hipStream_t stream) {
  constexpr int T = 16 * JB;
  const int64_t tiles = (int64_t)((p.K[0] + T - 1) / T) * ((p.K[1] + T - 1) / T);
  if constexpr (JB > 1) {
    if (tiles * nst < 512)
      return joint2_launch_tile<F64, JB - 1>(p, nst, rec, band, acc, stream);
  }
  hipLaunchKernelGGL((joint2_accumulate<F64, JB>), dim3((unsigned)tiles, nst, 2),
                     dim3(64 * kJWaves), 0, stream, p, rec, band, acc);
}

// part != nullptr: the bin sums come from the occupation-fused GEMM's partials
// (runs in the order built here, as fused_runs builds them) and C is unused.
mp_status joint2_launch(int32_t M, int64_t E, const void* C, const double* n, mp_precision prec,
                        mp_estimator est, const int32_t* bin_of_mode, const int32_t* m_lo,
                        const int32_t* K, int32_t n_sub, int64_t ns, int64_t e0, double* acc,
                        void* ws, size_t ws_bytes, hipStream_t stream, const float* part) {
  Joint2Params p{};
  p.M = M;
  p.ldm = ld_modes(M);
  p.E = E;
  p.e0 = e0;
  p.ns = ns;
  p.est = est;
  p.n_runs = 0;
  for (int j = 0; j < M;) {
    const int b = bin_of_mode[j];
    int j2 = j + 1;
    while (j2 < M && bin_of_mode[j2] == b) ++j2;
    if (b >= 0) {
      MP_CHECK_ARG(p.n_runs < MP_MAX_RUNS, MP_ERR_UNSUPPORTED,
                   "mp_binned_counts: bins form more than %d contiguous mode runs", MP_MAX_RUNS);
      p.run_lo[p.n_runs] = j;
      p.run_hi[p.n_runs] = j2;
      p.run_bin[p.n_runs] = b;
      ++p.n_runs;
    }
    j = j2;
  }
  for (int b = 0; b < 2; ++b) {
    p.m_lo[b] = m_lo[b];
    p.K[b] = K[b];
  }
  p.s_first = e0 / ns;
  p.s_last = (e0 + E - 1) / ns;
  MP_CHECK_ARG(p.s_last < n_sub, MP_ERR_SHAPE,
               "mp_binned_counts: samples [%lld, %lld) exceed n_sub * samples_per_sub = %lld",
               (long long)e0, (long long)(e0 + E), (long long)n_sub * ns);
  const size_t need = 256 + (size_t)E * 48;
  MP_CHECK_ARG(ws && ws_bytes >= need, MP_ERR_WORKSPACE,
               "mp_binned_counts: workspace of %zu bytes needed, %zu given", need, ws_bytes);
  int* band = (int*)ws;
  double* rec = (double*)((char*)ws + 256);
  hipLaunchKernelGGL(joint2_band_init, dim3(1), dim3(64), 0, stream, band);
  // rows of 16 lanes also for the partials, of which a run has few (1.15e5 samples of
  // M = 223: 22 us, 72 us by waves)
  const bool rows = part || short_runs(M, p.n_runs, elem_bytes_c(prec), kRowBytesOcc);
  const int64_t per = kOccPerWave * (rows ? 16 : 4);
  auto occ = [&](auto kernel, auto* c) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)((E + per - 1) / per)), dim3(256), 0, stream, p, c, part,
                       n, rec);
  };
  if (part)
    occ(joint2_occupations<float, true, 16>, (const float*)nullptr);
  else if (prec == MP_FP64)
    occ(rows ? joint2_occupations<double, false, 16> : joint2_occupations<double, false, 64>,
        (const double*)C);
  else
    occ(rows ? joint2_occupations<float, false, 16> : joint2_occupations<float, false, 64>,
        (const float*)C);
  MP_HIP_LAUNCH_CHECK("mp_binned_counts joint occupations launch");
  const mp_status sb = record_bands_launch(rec, E, 2, K, 2, band, stream);
  if (sb != MP_OK) return sb;
  const unsigned nst = (unsigned)(p.s_last - p.s_first + 1);
  if (prec == MP_FP64)
    joint2_launch_tile<true, 2>(p, nst, rec, band, acc, stream);
  else
    joint2_launch_tile<false, 3>(p, nst, rec, band, acc, stream);
  MP_HIP_LAUNCH_CHECK("mp_binned_counts joint accumulate launch");
  return MP_OK;
}

// ---------------------------------------------------------------- finalize

struct FinalParams {
  int n_dist;
  int K[kMaxDist];
  int off[kMaxDist + 1];
  int tile_off[kMaxDist + 1];  // first workgroup of each distribution
  int entries;
  int n_sub;
  int group;  // sub-ensembles per sweep over the terms, at most kFinSubs
  double inv_ns;
};

// Inverse DFT of every sub-ensemble and the statistics over them.  A
// workgroup owns kFinL output points of one distribution.  It walks the terms
// kFinThreads at a time: each thread loads one term of `group` sub-ensembles
// (coalesced), the terms that are zero in all of them (the grid points the
// counting kernels skip: at M = 8000 all but a few hundred of 4160) are
// dropped by a ballot prefix sum, and the rest go to LDS with their index.
// The threads, kFinL points by kFinPhases phases of that list, then form each
// twiddle e^{-2 pi i (t l mod K) / K} once for the group from two tables (64
// and K / 64 entries; one product, two roundings) and add 4 FMAs per term and
// sub-ensemble.  Bound by those FMAs on dense accumulators and by the loads
// (every workgroup reads all terms, from L2) on sparse ones.  kFinL = 16: 260
// workgroups at K = 4160, two per CU.  One output point per workgroup with one
// sincospi per term and sub-ensemble took 1837 us for windows of 4 x 2176 and
// 4352 points and 15 sub-ensembles and 476 us for 4160 points and 8 (now 87
// and 28 us).
constexpr int kFinL = 16, kFinPhases = 32, kFinSubs = 6, kFinThreads = kFinL * kFinPhases;
constexpr int kFinMaxK = 65536;

__global__ __launch_bounds__(kFinThreads) void counts_finalize(FinalParams p,
                                                               const double* __restrict__ acc,
                                                               double* __restrict__ P_re,
                                                               double* __restrict__ P_im,
                                                               double* __restrict__ sigma) {
  typedef __attribute__((ext_vector_type(2), aligned(8))) double d2u;  // acc: any FP64 address
  typedef __attribute__((ext_vector_type(2))) double d2;
  constexpr int kWaves = kFinThreads / 64;
  __shared__ d2 tw_hi[kFinMaxK / 64 + 1], tw_lo[64];
  __shared__ d2 xs[kFinThreads][kFinSubs];
  __shared__ uint32_t ts[kFinThreads];
  __shared__ d2 red[kWaves][kFinSubs][kFinL];
  __shared__ int wcnt[kWaves];
  int q = 0;
  while (q + 1 < p.n_dist && (int)blockIdx.x >= p.tile_off[q + 1]) ++q;
  const int K = p.K[q];
  const int tid = threadIdx.x, li = tid & (kFinL - 1), phase = tid / kFinL;
  const int wave = tid >> 6, lane = tid & 63;
  const int lo = ((int)blockIdx.x - p.tile_off[q]) * kFinL + li;
  const uint32_t l = (uint32_t)(lo < K ? lo : K - 1);
  const float inv_k = 1.0f / (float)K;
  for (int i = tid; i <= (K - 1) / 64; i += kFinThreads) {
    double sw, cw;
    sincospi(-2.0 * ((double)(64 * i) / K), &sw, &cw);
    tw_hi[i] = d2{cw, sw};
  }
  if (tid < 64) {
    double sw, cw;
    sincospi(-2.0 * ((double)tid / K), &sw, &cw);
    tw_lo[tid] = d2{cw, sw};
  }
  double mean_r = 0.0, mean_i = 0.0, m2 = 0.0;
  for (int s0 = 0; s0 < p.n_sub; s0 += p.group) {
    const int sc = p.n_sub - s0 < p.group ? p.n_sub - s0 : p.group;
    const d2u* a = (const d2u*)acc + (int64_t)s0 * p.entries + p.off[q];
    double ar[kFinSubs], ai[kFinSubs];
#pragma unroll
    for (int u = 0; u < kFinSubs; ++u) ar[u] = ai[u] = 0.0;
    for (int t0 = 0; t0 < K; t0 += kFinThreads) {
      const int t = t0 + tid;
      d2 x[kFinSubs];
      bool nz = false;  // a NaN counts as nonzero
#pragma unroll
      for (int u = 0; u < kFinSubs; ++u) {
        x[u] = d2{0.0, 0.0};
        if (u < sc && t < K) x[u] = a[(int64_t)u * p.entries + t];
        nz |= x[u].x != 0.0 || x[u].y != 0.0;
      }
      const unsigned long long mask = __ballot(nz);
      __syncthreads();  // the previous terms are consumed
      if (lane == 0) wcnt[wave] = __popcll(mask);
      __syncthreads();
      int base = 0, count = 0;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        base += w < wave ? wcnt[w] : 0;
        count += wcnt[w];
      }
      if (nz) {
        const int at = base + __popcll(mask & ((1ull << lane) - 1ull));
        ts[at] = (uint32_t)t;
#pragma unroll
        for (int u = 0; u < kFinSubs; ++u)
          if (u < sc) xs[at][u] = x[u];
      }
      __syncthreads();
      for (int i = phase; i < count; i += kFinPhases) {
        // t l < 2^32 (K <= 65536); its quotient by K is below 65536 and its FP32
        // estimate at most one off
        const uint32_t tl = ts[i] * l;
        int r = (int)(tl - (uint32_t)((float)tl * inv_k) * (uint32_t)K);
        r += r < 0 ? K : 0;
        r -= r >= K ? K : 0;
        const d2 h = tw_hi[r >> 6], g = tw_lo[r & 63];
        const double wr = fma(h.x, g.x, -(h.y * g.y)), wi = fma(h.x, g.y, h.y * g.x);
#pragma unroll
        for (int u = 0; u < kFinSubs; ++u)
          if (u < sc) {
            const d2 v = xs[i][u];
            ar[u] = fma(v.x, wr, fma(-v.y, wi, ar[u]));
            ai[u] = fma(v.x, wi, fma(v.y, wr, ai[u]));
          }
      }
    }
    // the four phases of a wave, then the waves, in a fixed order
#pragma unroll
    for (int u = 0; u < kFinSubs; ++u) {
      ar[u] += __shfl_xor(ar[u], 16, 64);
      ai[u] += __shfl_xor(ai[u], 16, 64);
      ar[u] += __shfl_xor(ar[u], 32, 64);
      ai[u] += __shfl_xor(ai[u], 32, 64);
      if (lane < kFinL) red[wave][u][li] = d2{ar[u], ai[u]};
    }
    __syncthreads();
    if (tid < kFinSubs * kFinL) {
      const int u = tid / kFinL;
      d2 s = red[0][u][li];
#pragma unroll 2
      for (int w = 1; w < kWaves; ++w) s += red[w][u][li];
      red[0][u][li] = d2{s.x * p.inv_ns / K, s.y * p.inv_ns / K};
    }
    __syncthreads();
    if (tid < kFinL) {  // Welford's update over the sub-ensembles
      for (int u = 0; u < sc; ++u) {
        const d2 v = red[0][u][li];
        const double dr = v.x - mean_r;
        mean_r += dr / (s0 + u + 1);
        mean_i += (v.y - mean_i) / (s0 + u + 1);
        m2 += dr * (v.x - mean_r);
      }
    }
    __syncthreads();
  }
  if (tid < kFinL && lo < K) {
    const int e = p.off[q] + lo;
    P_re[e] = mean_r;
    if (P_im) P_im[e] = mean_i;
    sigma[e] = p.n_sub > 1 ? sqrt(m2 / (p.n_sub - 1) / p.n_sub) : __builtin_nan("");
  }
}

size_t jointd_workspace(int32_t d, const int32_t* K, int64_t E);
size_t jointd_finalize_workspace(int32_t d, const int32_t* K, int32_t n_sub);
mp_status jointd_launch(int32_t M, int64_t E, const void* C, const double* n, mp_precision prec,
                        mp_estimator est, int32_t d, const int32_t* bin_of_mode,
                        const int32_t* m_lo, const int32_t* K, int32_t n_sub, int64_t ns,
                        int64_t e0, double* acc, void* ws, size_t ws_bytes, hipStream_t stream,
                        const float* part);
mp_status jointd_finalize(int32_t d, const int32_t* K, int32_t n_sub, int64_t ns,
                          const double* acc, double* P_re, double* P_im, double* sigma, void* ws,
                          size_t ws_bytes, hipStream_t stream);

size_t finalize_workspace(int32_t d, mp_bin_mode mode, const int32_t* K, int32_t n_sub) {
  if (mode == MP_JOINT && d >= 2) return jointd_finalize_workspace(d, K, n_sub);
  return 0;
}

// ---------------------------------------------------------------- host side

static int64_t entries_of(int d, mp_bin_mode mode, const int32_t* K) {
  if (mode == MP_JOINT) {
    int64_t e = 1;
    for (int b = 0; b < d; ++b) e *= K[b];
    return e;
  }
  int nd = d + (mode == MP_MARGINALS_AND_TOTAL ? 1 : 0);
  int64_t e = 0;
  for (int q = 0; q < nd; ++q) e += K[q];
  return e;
}

int64_t acc_entries(int32_t d, mp_bin_mode mode, const int32_t* K) {
  if (!K || d < 1 || d > MP_MAX_BINS) return -1;
  return entries_of(d, mode, K);
}

// Fills the tiling part of the parameters for workgroups of `sblk` samples;
// returns the number of workgroups.  Workspace sizes are those of kSBlk.
static int64_t plan_tiles(CountsParams& p, int sblk) {
  p.sblk = sblk;
  p.s_first = p.e0 / p.ns;
  p.s_last = (p.e0 + p.E - 1) / p.ns;
  auto tiles = [&](int64_t s) { return (int)((sub_hi(p, s) - sub_lo(p, s) + p.sblk - 1) / p.sblk); };
  p.t_first = tiles(p.s_first);
  p.t_mid = (int)((p.ns + p.sblk - 1) / p.sblk);
  p.n_mid = p.s_last > p.s_first + 1 ? (int)(p.s_last - p.s_first - 1) : 0;
  p.t_last = p.s_last != p.s_first ? tiles(p.s_last) : 0;
  return (int64_t)p.t_first + (int64_t)p.n_mid * p.t_mid + p.t_last;
}

// Contiguous mode runs of the bins (modes with bin -1 are skipped); false if
// there are more than MP_MAX_RUNS.
static bool fill_runs(CountsParams& p, int32_t M, const int32_t* bin_of_mode) {
  p.n_runs = 0;
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

size_t binned_workspace(int32_t d, mp_bin_mode mode, const int32_t* K, int64_t E, int32_t n_sub,
                        int64_t ns, int64_t e0) {
  if (!K || d < 1 || d > MP_MAX_BINS || E < 1 || ns < 1 || e0 < 0) return 0;
  if (mode == MP_JOINT && d == 2) return 256 + (size_t)E * 48;
  if (mode == MP_JOINT && d >= 3) return jointd_workspace(d, K, E);
  CountsParams p{};
  p.E = E;
  p.e0 = e0;
  p.ns = ns;
  const int64_t blocks = plan_tiles(p, kSBlk);
  return (size_t)blocks * (size_t)entries_of(d, mode, K) * 16;
}

// Parameters of a d = 1, marginal or marginal + total accumulation.
static mp_status setup_counts(CountsParams& p, const char* who, int32_t M, int64_t E, int32_t d,
                              const int32_t* bin_of_mode, mp_bin_mode mode, const int32_t* m_lo,
                              const int32_t* K, int32_t n_sub, int64_t ns, int64_t e0,
                              mp_estimator est, int64_t& blocks) {
  p.M = M;
  p.ldm = ld_modes(M);
  p.E = E;
  p.e0 = e0;
  p.ns = ns;
  p.d = d;
  p.mode = mode;
  p.est = est;
  if (!fill_runs(p, M, bin_of_mode)) {
    set_error("%s: bins form more than %d contiguous mode runs", who, MP_MAX_RUNS);
    return MP_ERR_UNSUPPORTED;
  }
  p.n_dist = mode == MP_JOINT ? 1 : d + (mode == MP_MARGINALS_AND_TOTAL ? 1 : 0);
  p.off[0] = 0;
  for (int q = 0; q < p.n_dist; ++q) {
    p.dist_src[q] = q < d ? q : -1;
    p.m_lo[q] = m_lo[q];
    p.K[q] = K[q];
    p.off[q + 1] = p.off[q] + K[q];
  }
  p.entries = p.off[p.n_dist];
  blocks = plan_tiles(p, kSBlk);
  if (p.s_last >= n_sub) {
    set_error("%s: samples [%lld, %lld) exceed n_sub * samples_per_sub = %lld", who,
              (long long)e0, (long long)(e0 + E), (long long)n_sub * ns);
    return MP_ERR_SHAPE;
  }
  if (blocks >= 0x7FFFFFFF) {
    set_error("%s: chunk too large", who);
    return MP_ERR_UNSUPPORTED;
  }
  return MP_OK;
}

// Samples per workgroup of counts_fused: two workgroups run per CU, so the chunk's
// sub-ensembles are cut into just under 512 r equal tiles, r the least that keeps
// them within kSBlkMax samples (more per workgroup share the search for active grid
// points and write fewer partials, 16 bytes per entry each, read back by
// counts_reduce); short chunks keep kSBlk.  1e5 samples of M = 1000 in ten
// sub-ensembles: 341 us with 510 workgroups of 197, 369 us with 790 of 128 (a
// second turn half empty).
static int counts_block(const CountsParams& p) {
  const int64_t subs = p.s_last - p.s_first + 1, len = p.ns < p.E ? p.ns : p.E;
  for (int64_t r = 1;; ++r) {
    const int64_t tiles = 512 * r / subs;
    if (tiles < 1) continue;
    const int64_t s = (len + tiles - 1) / tiles;
    if (s <= kSBlkMax) return s < kSBlk ? kSBlk : (int)s;
  }
}

// Runs counts_fused and counts_reduce.
template <typename Src, bool F64>
static mp_status counts_go(const char* who, CountsParams& p, Src src, const double* n, double* part,
                           double* acc, hipStream_t stream) {
  const int64_t blocks = plan_tiles(p, counts_block(p));
  hipLaunchKernelGGL((counts_fused<Src, F64>), dim3((unsigned)blocks), dim3(kCountThreads), 0, stream,
                     p, src, n, part);
  const int ns_touched = (int)(p.s_last - p.s_first + 1);
  hipLaunchKernelGGL(counts_reduce, dim3((p.entries + 255) / 256, ns_touched), dim3(256), 0, stream,
                     p, (const double*)part, acc);
  const hipError_t e = hipGetLastError();
  MP_CHECK_ARG(e == hipSuccess, MP_ERR_HIP, "%s counts launch: %s", who, hipGetErrorString(e));
  return MP_OK;
}

mp_status binned_counts_launch(int32_t M, int64_t E, const void* C, const double* n,
                               mp_precision prec, mp_estimator est, int32_t d,
                               const int32_t* bin_of_mode, mp_bin_mode mode, const int32_t* m_lo,
                               const int32_t* K, int32_t n_sub, int64_t ns, int64_t e0,
                               double* acc, void* ws, size_t ws_bytes, hipStream_t stream) {
  if (mode == MP_JOINT && d == 2)
    return joint2_launch(M, E, C, n, prec, est, bin_of_mode, m_lo, K, n_sub, ns, e0, acc, ws,
                         ws_bytes, stream, nullptr);
  if (mode == MP_JOINT && d >= 3)
    return jointd_launch(M, E, C, n, prec, est, d, bin_of_mode, m_lo, K, n_sub, ns, e0, acc, ws,
                         ws_bytes, stream, nullptr);
  MP_CHECK_ARG(mode != MP_JOINT || d == 1, MP_ERR_UNSUPPORTED,
               "mp_binned_counts: joint distributions need d <= 4 (d = %d)", d);
  CountsParams p{};
  int64_t blocks = 0;
  const mp_status st = setup_counts(p, "mp_binned_counts", M, E, d, bin_of_mode, mode, m_lo, K,
                                    n_sub, ns, e0, est, blocks);
  if (st != MP_OK) return st;
  const size_t need = (size_t)blocks * (size_t)p.entries * 16;
  MP_CHECK_ARG(ws && ws_bytes >= need, MP_ERR_WORKSPACE,
               "mp_binned_counts: workspace of %zu bytes needed, %zu given", need, ws_bytes);
  auto go = [&](auto src, auto f64) {
    return counts_go<decltype(src), decltype(f64)::value>("mp_binned_counts", p, src, n, (double*)ws,
                                                          acc, stream);
  };
  const bool rows = short_runs(M, p.n_runs, elem_bytes_c(prec), kRowBytesCounts);
  if (prec == MP_FP64)
    return rows ? go(FromC<double, 16>{(const double*)C}, std::true_type{})
                : go(FromC<double, 64>{(const double*)C}, std::true_type{});
  return rows ? go(FromC<float, 16>{(const float*)C}, std::false_type{})
              : go(FromC<float, 64>{(const float*)C}, std::false_type{});
}

mp_status gemm_fused_launch(int32_t M, int64_t E, const void* packed, mp_precision prec,
                            const void* ab, const FusedOut& fo, hipStream_t stream);

// Workspace of mp_propagate_counts: the GEMM's partials (slots x E x 16 B),
// then the counts kernel's per-block partials.
static void propagate_counts_sizes(const CountsParams& p, int64_t blocks, size_t& part_bytes,
                                   size_t& total) {
  int slot_off[MP_MAX_RUNS];
  const int64_t slots = fused_slots(p.n_runs, p.run_lo, p.run_hi, slot_off);
  part_bytes = ((size_t)slots * (size_t)p.E * 16 + 255) / 256 * 256;
  total = part_bytes + (size_t)blocks * (size_t)p.entries * 16;
}

// Runs of a bin partition for the fused partials of a joint distribution of
// d >= 2 bins: maximal ranges of modes with one bin >= 0, in mode order (the
// order in which the joint paths walk them).
static mp_status fused_runs(int32_t M, const int32_t* bin_of_mode, FusedOut& fo) {
  fo.n_runs = 0;
  for (int j = 0; j < M;) {
    const int b = bin_of_mode[j];
    int j2 = j + 1;
    while (j2 < M && bin_of_mode[j2] == b) ++j2;
    if (b >= 0) {
      MP_CHECK_ARG(fo.n_runs < MP_MAX_RUNS, MP_ERR_UNSUPPORTED,
                   "mp_propagate_counts: bins form more than %d contiguous mode runs", MP_MAX_RUNS);
      fo.run_lo[fo.n_runs] = j;
      fo.run_hi[fo.n_runs] = j2;
      ++fo.n_runs;
    }
    j = j2;
  }
  fused_slots(fo.n_runs, fo.run_lo, fo.run_hi, fo.slot_off);
  return MP_OK;
}

static size_t joint_part_bytes(const FusedOut& fo, int64_t E) {
  const int64_t slots = fo.n_runs ? fo.slot_off[fo.n_runs - 1] +
                                        run_blocks(fo.run_lo[fo.n_runs - 1], fo.run_hi[fo.n_runs - 1])
                                  : 0;
  return ((size_t)slots * (size_t)E * 16 + 255) / 256 * 256;
}

size_t propagate_counts_workspace(int32_t M, int64_t E, int32_t d, const int32_t* bin_of_mode,
                                  mp_bin_mode mode, const int32_t* K, int32_t n_sub, int64_t ns,
                                  int64_t e0) {
  if (mode == MP_JOINT && d >= 2) {  // the partials, then the joint path's workspace
    FusedOut fo{};
    if (fused_runs(M, bin_of_mode, fo) != MP_OK) return 0;
    return joint_part_bytes(fo, E) + binned_workspace(d, mode, K, E, n_sub, ns, e0);
  }
  CountsParams p{};
  std::vector<int32_t> m_lo(MP_MAX_BINS + 1, 0);
  int64_t blocks = 0;
  if (setup_counts(p, "mp_propagate_counts_workspace", M, E, d, bin_of_mode, mode, m_lo.data(), K,
                   n_sub, ns, e0, MP_MATRIX_P, blocks) != MP_OK)
    return 0;
  size_t part_bytes, total;
  propagate_counts_sizes(p, blocks, part_bytes, total);
  return total;
}

// The occupation-fused GEMM's output description for a chunk of E samples:
// the runs of the bin partition, their slots, and the partials at the start of
// ws (the counts kernel's per-block partials follow them).
mp_status fused_out_setup(int32_t M, int64_t E, int32_t d, const int32_t* bin_of_mode,
                          mp_bin_mode mode, const int32_t* m_lo, const int32_t* K, int32_t n_sub,
                          int64_t ns, int64_t e0, mp_estimator est, void* ws, size_t ws_bytes,
                          FusedOut& fo) {
  if (mode == MP_JOINT && d >= 2) {
    fo = FusedOut{};
    const mp_status sr = fused_runs(M, bin_of_mode, fo);
    if (sr != MP_OK) return sr;
    const size_t total =
        joint_part_bytes(fo, E) + binned_workspace(d, mode, K, E, n_sub, ns, e0);
    MP_CHECK_ARG(ws && ws_bytes >= total, MP_ERR_WORKSPACE,
                 "mp_propagate_counts: workspace of %zu bytes needed, %zu given", total, ws_bytes);
    fo.part = (float*)ws;
    fo.E = E;
    return MP_OK;
  }
  CountsParams p{};
  int64_t blocks = 0;
  const mp_status st = setup_counts(p, "mp_propagate_counts", M, E, d, bin_of_mode, mode, m_lo, K,
                                    n_sub, ns, e0, est, blocks);
  if (st != MP_OK) return st;
  size_t part_bytes, total;
  propagate_counts_sizes(p, blocks, part_bytes, total);
  MP_CHECK_ARG(ws && ws_bytes >= total, MP_ERR_WORKSPACE,
               "mp_propagate_counts: workspace of %zu bytes needed, %zu given", total, ws_bytes);
  fo = FusedOut{};
  fo.part = (float*)ws;
  fo.E = E;
  fo.n_runs = p.n_runs;
  for (int q = 0; q < p.n_runs; ++q) {
    fo.run_lo[q] = p.run_lo[q];
    fo.run_hi[q] = p.run_hi[q];
  }
  fused_slots(p.n_runs, fo.run_lo, fo.run_hi, fo.slot_off);
  return MP_OK;
}

// Counts from the partials an occupation-fused GEMM left at the start of ws
// (laid out by fused_out_setup with the same arguments).  The fused GEMM runs
// in FP32 or a split precision, so the joint paths take their FP32 factor
// tables.
mp_status counts_from_partials_launch(int32_t M, int64_t E, const double* n, mp_estimator est,
                                      int32_t d, const int32_t* bin_of_mode, mp_bin_mode mode,
                                      const int32_t* m_lo, const int32_t* K, int32_t n_sub,
                                      int64_t ns, int64_t e0, double* acc, void* ws,
                                      size_t ws_bytes, hipStream_t stream) {
  if (mode == MP_JOINT && d >= 2) {
    // the joint paths read the bin sums from the partials; their own
    // workspace follows them
    FusedOut fo{};
    const mp_status sr = fused_runs(M, bin_of_mode, fo);
    if (sr != MP_OK) return sr;
    const size_t pb = joint_part_bytes(fo, E);
    MP_CHECK_ARG(ws && ws_bytes >= pb, MP_ERR_WORKSPACE,
                 "mp_propagate_counts: workspace of %zu bytes needed, %zu given", pb, ws_bytes);
    void* jws = (char*)ws + pb;
    const size_t jbytes = ws_bytes - pb;
    return d == 2 ? joint2_launch(M, E, nullptr, n, MP_FP32, est, bin_of_mode, m_lo, K, n_sub, ns,
                                  e0, acc, jws, jbytes, stream, (const float*)ws)
                  : jointd_launch(M, E, nullptr, n, MP_FP32, est, d, bin_of_mode, m_lo, K, n_sub,
                                  ns, e0, acc, jws, jbytes, stream, (const float*)ws);
  }
  CountsParams p{};
  int64_t blocks = 0;
  const mp_status st = setup_counts(p, "mp_propagate_counts", M, E, d, bin_of_mode, mode, m_lo, K,
                                    n_sub, ns, e0, est, blocks);
  if (st != MP_OK) return st;
  size_t part_bytes, total;
  propagate_counts_sizes(p, blocks, part_bytes, total);
  MP_CHECK_ARG(ws && ws_bytes >= total, MP_ERR_WORKSPACE,
               "mp_propagate_counts: workspace of %zu bytes needed, %zu given", total, ws_bytes);
  return counts_go<FromPartials, false>("mp_propagate_counts", p, FromPartials{(const float*)ws}, n,
                                        (double*)((char*)ws + part_bytes), acc, stream);
}

mp_status propagate_counts_launch(int32_t M, int64_t E, mp_precision prec, mp_estimator est,
                                  const void* ab, const double* n, const void* packed, int32_t d,
                                  const int32_t* bin_of_mode, mp_bin_mode mode,
                                  const int32_t* m_lo, const int32_t* K, int32_t n_sub,
                                  int64_t ns, int64_t e0, double* acc, void* ws, size_t ws_bytes,
                                  hipStream_t stream) {
  FusedOut fo;
  mp_status st = fused_out_setup(M, E, d, bin_of_mode, mode, m_lo, K, n_sub, ns, e0, est, ws,
                                 ws_bytes, fo);
  if (st != MP_OK) return st;
  if (fo.n_runs > 0 && (st = gemm_fused_launch(M, E, packed, prec, ab, fo, stream)) != MP_OK)
    return st;
  return counts_from_partials_launch(M, E, n, est, d, bin_of_mode, mode, m_lo, K, n_sub, ns, e0,
                                     acc, ws, ws_bytes, stream);
}

// One distribution through the bilinear form alpha^T W beta (W packed by
// bilinear_pack_launch; the mode set S is inside W): the GEMM's partials cover
// one run of all M input modes, which the d = 1 counting kernels then read.
mp_status gemm_bilinear_launch(int32_t M, int64_t E, const void* packed, mp_precision prec,
                               const void* ab, const FusedOut& fo, hipStream_t stream);

mp_status propagate_counts_bilinear_launch(int32_t M, int64_t E, mp_precision prec,
                                           mp_estimator est, const void* ab, const double* n,
                                           const void* packed, const int32_t* m_lo,
                                           const int32_t* K, int32_t n_sub, int64_t ns,
                                           int64_t e0, double* acc, void* ws, size_t ws_bytes,
                                           hipStream_t stream) {
  const std::vector<int32_t> all(M, 0);
  FusedOut fo;
  mp_status st = fused_out_setup(M, E, 1, all.data(), MP_JOINT, m_lo, K, n_sub, ns, e0, est, ws,
                                 ws_bytes, fo);
  if (st != MP_OK) return st;
  if ((st = gemm_bilinear_launch(M, E, packed, prec, ab, fo, stream)) != MP_OK) return st;
  return counts_from_partials_launch(M, E, n, est, 1, all.data(), MP_JOINT, m_lo, K, n_sub, ns,
                                     e0, acc, ws, ws_bytes, stream);
}

// ---------------------------------------------------------------- no-allocation variant

// Scratch of mp_propagate_counts_noalloc: the occupation-fused GEMM's
// per-block partials followed by the counting kernel's per-tile partials, in
// a device array that every GPU the library runs on holds from module load to
// process exit.  In host code the array's name is only a stand-in for the
// symbol, never a device address: the address is looked up once per device
// (with that device current) and kept, and only that address reaches kernels.
// Each call writes every scratch byte it later reads (the GEMM epilogue every
// (slot, sample) partial of the chunk, the counting kernel every entry of its
// tile), so nothing has to start at zero and the previous call's contents are
// never read.  Calls that overlap on one GPU share the array and race.
static __device__ __align__(256) unsigned char scratch[MP_NOALLOC_SCRATCH_BYTES];

constexpr int kMaxScratchDevices = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_addr[kMaxScratchDevices];

static mp_status scratch_of_current_device(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) {
    set_error("mp_propagate_counts_noalloc: hipGetDevice: %s", hipGetErrorString(e));
    return MP_ERR_HIP;
  }
  if (dev < 0 || dev >= kMaxScratchDevices) {
    set_error("mp_propagate_counts_noalloc: device %d beyond the %d supported", dev,
              kMaxScratchDevices);
    return MP_ERR_UNSUPPORTED;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || p == nullptr) {
      set_error("mp_propagate_counts_noalloc: hipGetSymbolAddress of the scratch array: %s",
                hipGetErrorString(e));
      return MP_ERR_HIP;
    }
    g_scratch_addr[dev] = p;
  }
  *out = g_scratch_addr[dev];
  return MP_OK;
}

// mp_propagate_counts with the library's scratch as its workspace; arguments
// validated by the caller as for mp_propagate_counts.  Sizes are checked before
// any HIP call.
mp_status propagate_counts_noalloc_launch(int32_t M, int64_t E, mp_precision prec,
                                          mp_estimator est, const void* ab, const double* n,
                                          const void* packed, int32_t d,
                                          const int32_t* bin_of_mode, mp_bin_mode mode,
                                          const int32_t* m_lo, const int32_t* K, int32_t n_sub,
                                          int64_t ns, int64_t e0, double* acc,
                                          hipStream_t stream) {
  MP_CHECK_ARG(mode != MP_JOINT || d == 1, MP_ERR_UNSUPPORTED,
               "mp_propagate_counts_noalloc: joint distributions of %d bins are not supported "
               "(use mp_propagate_counts)", d);
  const size_t need = propagate_counts_workspace(M, E, d, bin_of_mode, mode, K, n_sub, ns, e0);
  MP_CHECK_ARG(need > 0, MP_ERR_UNSUPPORTED,
               "mp_propagate_counts_noalloc: bins form more than %d contiguous mode runs",
               MP_MAX_RUNS);
  MP_CHECK_ARG(need <= (size_t)MP_NOALLOC_SCRATCH_BYTES, MP_ERR_WORKSPACE,
               "mp_propagate_counts_noalloc: this chunk needs %zu bytes of scratch, more than "
               "the library's %zu (split the chunk, or pass a workspace to "
               "mp_propagate_counts)", need, (size_t)MP_NOALLOC_SCRATCH_BYTES);
  void* ws = nullptr;
  const mp_status st = scratch_of_current_device(&ws);
  if (st != MP_OK) return st;
  return propagate_counts_launch(M, E, prec, est, ab, n, packed, d, bin_of_mode, mode, m_lo, K,
                                 n_sub, ns, e0, acc, ws, (size_t)MP_NOALLOC_SCRATCH_BYTES, stream);
}

mp_status counts_finalize_launch(int32_t d, mp_bin_mode mode, const int32_t* K, int32_t n_sub,
                                 int64_t ns, const double* acc, double* P_re, double* P_im,
                                 double* sigma, void* ws, size_t ws_bytes, hipStream_t stream) {
  if (mode == MP_JOINT && d >= 2)
    return jointd_finalize(d, K, n_sub, ns, acc, P_re, P_im, sigma, ws, ws_bytes, stream);
  FinalParams p{};
  p.n_dist = mode == MP_JOINT ? 1 : d + (mode == MP_MARGINALS_AND_TOTAL ? 1 : 0);
  p.off[0] = 0;
  for (int q = 0; q < p.n_dist; ++q) {
    p.K[q] = K[q];
    p.off[q + 1] = p.off[q] + K[q];
    p.tile_off[q + 1] = p.tile_off[q] + (K[q] + kFinL - 1) / kFinL;
  }
  p.entries = (int)entries_of(d, mode, K);
  p.n_sub = n_sub;
  p.inv_ns = 1.0 / (double)ns;
  // equal groups of at most kFinSubs sub-ensembles
  const int groups = (n_sub + kFinSubs - 1) / kFinSubs;
  p.group = (n_sub + groups - 1) / groups;
  hipLaunchKernelGGL(counts_finalize, dim3(p.tile_off[p.n_dist]), dim3(kFinThreads), 0, stream, p,
                     acc, P_re, P_im, sigma);
  MP_HIP_LAUNCH_CHECK("mp_counts_finalize launch");
  return MP_OK;
}


// ---------------------------------------------------------------- finiteness

__global__ void zero_i64(int64_t* p) {
  if (threadIdx.x == 0) *p = 0;
}

// Grid-stride count of non-finite entries: one atomic add per wave into the cleared
// counter, or, as one workgroup (`alone`, up to kFiniteAlone values: a launch less),
// their sum through LDS.
constexpr int64_t kFiniteAlone = 32768;

__global__ __launch_bounds__(1024) void count_nonfinite(const double* __restrict__ x, int64_t n,
                                                        bool alone, int64_t* __restrict__ count) {
  __shared__ int64_t part[16];
  int64_t c = 0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    c += isfinite(x[i]) ? 0 : 1;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off, 64);
  if (!alone) {
    if ((threadIdx.x & 63) == 0 && c != 0)
      atomicAdd((unsigned long long*)count, (unsigned long long)c);
    return;
  }
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < (int)blockDim.x / 64; ++w) c += part[w];
    *count = c;
  }
}

mp_status check_finite_launch(const double* x, int64_t n, int64_t* scratch, int64_t* n_bad,
                              hipStream_t stream) {
  if (n <= kFiniteAlone) {
    hipLaunchKernelGGL(count_nonfinite, dim3(1), dim3(1024), 0, stream, x, n, true, scratch);
  } else {
    hipLaunchKernelGGL(zero_i64, dim3(1), dim3(64), 0, stream, scratch);
    const int64_t blocks = (n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096;
    hipLaunchKernelGGL(count_nonfinite, dim3((unsigned)blocks), dim3(256), 0, stream, x, n, false,
                       scratch);
  }
  MP_HIP_LAUNCH_CHECK("mp_check_finite launch");
  int64_t c = 0;
  hipError_t e = hipMemcpyAsync(&c, scratch, sizeof(c), hipMemcpyDeviceToHost, stream);
  if (e == hipSuccess) e = hipStreamSynchronize(stream);
  if (e != hipSuccess) {
    set_error("mp_check_finite: %s", hipGetErrorString(e));
    return MP_ERR_HIP;
  }
  if (n_bad) *n_bad = c;
  if (c != 0) {
    set_error("mp_check_finite: %lld of %lld values are NaN or infinite", (long long)c,
              (long long)n);
    return MP_ERR_NONFINITE;
  }
  return MP_OK;
}

// ---------------------------------------------------------------- per-sample observables

// Occupation of every distribution for every sample of the chunk:
// nq[(k n_dist + q) 2 + {0, 1}] = (Re, Im) n_q of chunk sample k, by G lanes per
// sample (64: one sample per wave at a time; 16: four).  Lane gl < n_dist of the group
// adds up distribution gl over the bin runs and writes it.  Bound by memory from
// some 50 modes on, below that by the chain of loads and reductions over a sample's
// runs.  FP32, one run of 14 modes, 1.2e5 samples: 13 us (56 us by waves with LDS
// shuffles); six of 14: 39 us (234); one of 1000, 4e4 samples: 110 us, 5.8 TB/s (123).
template <typename CT, int G>
__global__ __launch_bounds__(256) void occupations_kernel(CountsParams p, const CT* __restrict__ C,
                                                          double* __restrict__ nq) {
  constexpr int S = 64 / G;  // samples per wave at a time
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int gl = lane % G;
  const int64_t ldc = 2 * p.ldm;
  int src = -2;  // bin of this lane's distribution, -1 = all
#pragma unroll
  for (int q = 0; q < kMaxDist; ++q)
    if (q == gl && q < p.n_dist) src = p.dist_src[q];
  for (int j = 0; j < kOccPerWave; ++j) {
    const int64_t k0 = ((int64_t)blockIdx.x * (4 * kOccPerWave) + 4 * j + wave) * S;
    if (k0 >= p.E) return;
    int64_t k = k0 + lane / G;
    const bool valid = k < p.E;
    if (!valid) k = k0;
    double vr = 0.0, vi = 0.0;
    for (int q = 0; q < p.n_runs; ++q) {
      double re, im;
      run_sum<CT, G>(C + k * ldc, C + (p.E + k) * ldc, p.ldm, p.run_lo[q], p.run_hi[q], gl, re, im);
      if (src == -1 || src == p.run_bin[q]) {
        vr += re;
        vi += im;
      }
    }
    if (valid && src != -2) {
      double* o = nq + (k * p.n_dist + gl) * 2;
      o[0] = vr;
      o[1] = vi;
    }
  }
}

struct SampleStatParams {
  int64_t E, e0, ns;   // chunk size, first global sample, samples per sub-ensemble
  int64_t s_first;     // first sub-ensemble the chunk touches
  int n_dist;
  int est;             // mp_estimator
  int kmax;            // moments
  int q, m, n_bins;    // histogram: distribution, count, bins
  int per;             // histogram: samples per thread
  double o_min, inv_width;
};

// Normally ordered moments (eq. moment with the parity-projected weights):
// per sample n_q^k, times tanh(n) for odd k on the matrix-P path (+P: 1).
// Block (s, q): the chunk's samples of sub-ensemble s_first + blockIdx.x,
// summed in a fixed order (strided per thread, then over the waves) and added to
// acc[s][q][k - 1] (re, im).  Bound by the chain of a thread's samples where there
// are few workgroups, then by the reductions over their waves: the least threads, 64 to
// 1024, that leave a thread four samples, 256 where more than 512 workgroups fill the CUs
// (1e5 samples, one bin: 22 us in sub-ensembles of 1e4, 43 us with 256 threads; 8 us in
// sub-ensembles of 100, 17 us with 1024 threads; 1e6 samples, nine bins, 1e4: 127 and 151 us).
constexpr int kMomentThreads = 1024;
__global__ __launch_bounds__(kMomentThreads) void moments_kernel(SampleStatParams p,
                                                                 const double* __restrict__ n,
                                                                 const double* __restrict__ nq,
                                                                 double* __restrict__ acc) {
  __shared__ double red[kMomentThreads / 64][MP_MAX_MOMENTS][2];
  const int64_t s = p.s_first + blockIdx.x;
  const int q = blockIdx.y;
  int64_t lo = s * p.ns, hi = (s + 1) * p.ns;
  lo = lo > p.e0 ? lo : p.e0;
  hi = hi < p.e0 + p.E ? hi : p.e0 + p.E;
  double sr[MP_MAX_MOMENTS], si[MP_MAX_MOMENTS];
#pragma unroll
  for (int o = 0; o < MP_MAX_MOMENTS; ++o) sr[o] = si[o] = 0.0;
  for (int64_t g = lo + threadIdx.x; g < hi; g += blockDim.x) {
    const int64_t k = g - p.e0;
    const double zr = nq[(k * p.n_dist + q) * 2], zi = nq[(k * p.n_dist + q) * 2 + 1];
    double w = 1.0;  // +P
    if (p.est != MP_PLUS_P) {
      const double nk = n[k];
      w = isfinite(nk) ? tanh(nk) : __builtin_nan("");
    }
    double pr = 1.0, pi = 0.0;
#pragma unroll
    for (int o = 0; o < MP_MAX_MOMENTS; ++o) {
      if (o < p.kmax) {
        const double tr = pr * zr - pi * zi;
        pi = pr * zi + pi * zr;
        pr = tr;
        const double f = (o & 1) ? 1.0 : w;  // order o + 1 odd -> weight w
        sr[o] += f * pr;
        si[o] += f * pi;
      }
    }
  }
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 0; o < MP_MAX_MOMENTS; ++o)
    if (o < p.kmax) {
      const double tr = wave_sum(sr[o]), ti = wave_sum(si[o]);
      if (lane == 0) {
        red[wave][o][0] = tr;
        red[wave][o][1] = ti;
      }
    }
  __syncthreads();
  if ((int)threadIdx.x < 2 * p.kmax) {
    const int o = threadIdx.x >> 1, c = threadIdx.x & 1;
    double t = 0.0;
    for (int w = 0; w < (int)blockDim.x / 64; ++w) t += red[w][o][c];
    acc[((s * p.n_dist + q) * p.kmax + o) * 2 + c] += t;
  }
}

// Per-sample count observable of distribution q at count m (eq.
// c-number-variable for one bin: g0 n_q^m e^{-n_q} / m!, with g0 formed as in
// counts_fused; +P: n_q^m e^{-n_q} / m!), real part, in n_bins equal bins from o_min.
// Bin of chunk sample k (0: below the range, n_bins + 1: above it or not finite).
__device__ inline int64_t histogram_bin(const SampleStatParams& p, const double* __restrict__ n,
                                        const double* __restrict__ nq, int64_t k) {
  const double zr = nq[(k * p.n_dist + p.q) * 2], zi = nq[(k * p.n_dist + p.q) * 2 + 1];
  const double mag = sqrt(zr * zr + zi * zi);
  // log(n_q^m / m!) as (real, phase); 0^0 = 1
  double lr, lp;
  if (p.m == 0) {
    lr = 0.0;
    lp = 0.0;
  } else if (mag == 0.0) {
    lr = -INFINITY;
    lp = 0.0;
  } else {
    lr = p.m * log(mag);
    lp = p.m * atan2(zi, zr);
  }
  lr -= lgamma((double)p.m + 1.0);
  double G;
  if (p.est == MP_PLUS_P) {
    G = exp(lr - zr) * cos(lp - zi);
  } else {
    const double nn = n[k];
    const double L = log1p(exp(-2.0 * fabs(nn)));
    const double c1 = (nn >= 0.0 ? 0.0 : 2.0 * nn) - L;
    const double c2 = (nn >= 0.0 ? -2.0 * nn : 0.0) - L;
    const double par = (p.m & 1) ? -1.0 : 1.0;
    G = exp(lr - zr + c1) * cos(lp - zi) + par * exp(lr + zr + c2) * cos(lp + zi);
  }
  if (!isfinite(zr) || !isfinite(zi) || (p.est != MP_PLUS_P && !isfinite(n[k])))
    G = __builtin_nan("");
  if (!(G == G) || G - G != 0.0) return p.n_bins + 1;  // not finite
  const double x = (G - p.o_min) * p.inv_width;
  return x < 0.0 ? 0 : (x >= (double)p.n_bins ? p.n_bins + 1 : (int64_t)x + 1);
}

// ONE: a sample per thread, each added by itself.  Else a workgroup counts its 256 per
// samples in LDS and adds its bins once, where the bins fit and the samples are of one
// sub-ensemble.  Counts are whole numbers, so both give the same sums.  One FP64 atomic per
// sample is bound by the turns at the few bins that are hit (1e5 samples, 100 bins: 58 us,
// 9 us counted in LDS); histogram_launch has the rule.
constexpr int kHistBins = 4096;
template <bool ONE>
__global__ __launch_bounds__(256) void histogram_kernel(SampleStatParams p, const double* __restrict__ n,
                                                        const double* __restrict__ nq,
                                                        double* __restrict__ hist) {
  if constexpr (ONE) {
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= p.E) return;
    atomicAdd(hist + (p.e0 + k) / p.ns * (p.n_bins + 2) + histogram_bin(p, n, nq, k), 1.0);
  } else {
    __shared__ int counts[kHistBins];
    const int64_t k0 = (int64_t)blockIdx.x * (256 * p.per);
    const int64_t k1 = k0 + 256 * p.per < p.E ? k0 + 256 * p.per : p.E;
    const int64_t s = (p.e0 + k0) / p.ns;
    const bool local = p.n_bins + 2 <= kHistBins && s == (p.e0 + k1 - 1) / p.ns;
    if (local) {
      for (int i = threadIdx.x; i < p.n_bins + 2; i += 256) counts[i] = 0;
      __syncthreads();
    }
    for (int64_t k = k0 + threadIdx.x; k < k1; k += 256) {
      const int64_t b = histogram_bin(p, n, nq, k);
      if (local)
        atomicAdd(&counts[b], 1);
      else
        atomicAdd(hist + (p.e0 + k) / p.ns * (p.n_bins + 2) + b, 1.0);
    }
    if (!local) return;
    __syncthreads();
    for (int i = threadIdx.x; i < p.n_bins + 2; i += 256)
      if (counts[i] != 0) atomicAdd(hist + s * (p.n_bins + 2) + i, (double)counts[i]);
  }
}

// Mean over sub-ensembles of scale * acc[s][v] / samples_per_sub and sigma_T =
// sd of its real part over the sub-ensembles / sqrt(n_sub) (NaN for one).
__global__ __launch_bounds__(256) void subensemble_stats_kernel(int n_sub, int64_t n_vals, int ncomp,
                                                                double scale,
                                                                const double* __restrict__ acc,
                                                                double* __restrict__ mean,
                                                                double* __restrict__ sigma) {
  const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (v >= n_vals) return;
  double m[2] = {0.0, 0.0};
  for (int s = 0; s < n_sub; ++s)
    for (int c = 0; c < ncomp; ++c) m[c] += acc[((int64_t)s * n_vals + v) * ncomp + c] * scale;
  for (int c = 0; c < ncomp; ++c) {
    m[c] /= n_sub;
    mean[v * ncomp + c] = m[c];
  }
  double ss = 0.0;
  for (int s = 0; s < n_sub; ++s) {
    const double dlt = acc[((int64_t)s * n_vals + v) * ncomp] * scale - m[0];
    ss += dlt * dlt;
  }
  sigma[v] = n_sub > 1 ? sqrt(ss / (n_sub - 1) / n_sub) : NAN;
}

mp_status occupations_launch(int32_t M, int64_t E, const void* C, mp_precision prec, int32_t d,
                             const int32_t* bin_of_mode, mp_bin_mode mode, double* nq,
                             hipStream_t stream) {
  CountsParams p{};
  p.M = M;
  p.ldm = ld_modes(M);
  p.E = E;
  p.d = d;
  p.mode = mode;
  if (!fill_runs(p, M, bin_of_mode)) {
    set_error("mp_occupations: bins form more than %d contiguous mode runs", MP_MAX_RUNS);
    return MP_ERR_UNSUPPORTED;
  }
  p.n_dist = d + (mode == MP_MARGINALS_AND_TOTAL ? 1 : 0);
  for (int q = 0; q < p.n_dist; ++q) p.dist_src[q] = q < d ? q : -1;
  const bool row = short_runs(M, p.n_runs, elem_bytes_c(prec), kRowBytesOcc);
  const int64_t per = 4 * kOccPerWave * (row ? 4 : 1);
  const dim3 grid((unsigned)((E + per - 1) / per));
  auto go = [&](auto kernel, auto* c) {
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, p, c, nq);
  };
  if (prec == MP_FP64)
    go(row ? occupations_kernel<double, 16> : occupations_kernel<double, 64>, (const double*)C);
  else
    go(row ? occupations_kernel<float, 16> : occupations_kernel<float, 64>, (const float*)C);
  MP_HIP_LAUNCH_CHECK("mp_occupations launch");
  return MP_OK;
}

mp_status moments_launch(int64_t E, const double* n, const double* nq, int32_t n_dist,
                         int32_t kmax, mp_estimator est, int64_t ns, int64_t e0, double* acc,
                         hipStream_t stream) {
  SampleStatParams p{};
  p.E = E;
  p.e0 = e0;
  p.ns = ns;
  p.s_first = e0 / ns;
  p.n_dist = n_dist;
  p.est = est;
  p.kmax = kmax;
  const int64_t n_touched = (e0 + E - 1) / ns - p.s_first + 1, len = ns < E ? ns : E;
  int threads = 64;
  const int most = n_touched * n_dist > 512 ? 256 : kMomentThreads;
  while (threads < most && threads * 4 < len) threads *= 2;
  hipLaunchKernelGGL(moments_kernel, dim3((unsigned)n_touched, (unsigned)n_dist), dim3(threads), 0,
                     stream, p, n, nq, acc);
  MP_HIP_LAUNCH_CHECK("mp_moments_accumulate launch");
  return MP_OK;
}

mp_status histogram_launch(int64_t E, const double* n, const double* nq, int32_t n_dist, int32_t q,
                           int32_t m, mp_estimator est, double o_min, double width,
                           int32_t n_bins, int64_t ns, int64_t e0, double* hist,
                           hipStream_t stream) {
  SampleStatParams p{};
  p.E = E;
  p.e0 = e0;
  p.ns = ns;
  p.n_dist = n_dist;
  p.est = est;
  p.q = q;
  p.m = m;
  p.n_bins = n_bins;
  p.o_min = o_min;
  p.inv_width = 1.0 / width;
  // Samples per thread, as E leaves some 256 workgroups.  Short sub-ensembles take one: few
  // workgroups would lie in one, and the atomics are spread over as many histograms (1e5
  // samples, 200 bins, by a sample each and by workgroup: 8.5 and 11 us at 100 samples a
  // sub-ensemble, 11.0 and 9.6 at 1000; 1e6 samples: 41 and 55 at 500, 63 and 44 at 3000).  So do
  // bins that do not fit where a thread has one sample anyway
  p.per = E < 2 * 65536 ? 1 : (E >= 8 * 65536 ? 8 : (int)(E / 65536));
  const bool one = ns < 768 || ns < 256 * p.per || (p.per == 1 && (int64_t)n_bins + 2 > kHistBins);
  if (one) p.per = 1;
  hipLaunchKernelGGL((one ? histogram_kernel<true> : histogram_kernel<false>),
                     dim3((unsigned)((E + 256 * p.per - 1) / (256 * p.per))), dim3(256), 0, stream, p,
                     n, nq, hist);
  MP_HIP_LAUNCH_CHECK("mp_observable_histogram launch");
  return MP_OK;
}

mp_status subensemble_stats_launch(int32_t n_sub, int64_t ns, int64_t n_vals, int32_t ncomp,
                                   double scale, const double* acc, double* mean, double* sigma,
                                   hipStream_t stream) {
  hipLaunchKernelGGL(subensemble_stats_kernel, dim3((unsigned)((n_vals + 255) / 256)), dim3(256), 0,
                     stream, n_sub, n_vals, ncomp, scale / (double)ns, acc, mean, sigma);
  MP_HIP_LAUNCH_CHECK("mp_subensemble_stats launch");
  return MP_OK;
}

}  // namespace mp
