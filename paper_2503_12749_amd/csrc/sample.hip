// Phase-space amplitudes of squeezed vacuum inputs.
//
// Paper, main text: a squeezed input is a real coherent-state integral with
// the even weight xi(alpha); with the unnormalised +P kernel the density
// matrix is reproduced by a real Gaussian pair per mode with variances
// sinh r cosh r and covariance sinh^2 r, and the parity-projected
// distribution (Omega_00 = 1) is sampled the same way.  Two independent
// normals give the pair exactly:
//     alpha = c+ w1 + c- w2,  beta = c+ w1 - c- w2,
//     c+ = sqrt(e^{2r} - 1) / 2,  c- = sqrt(1 - e^{-2r}) / 2.
//
// Noise: one Philox4x64-10 block (Salmon et al., SC'11) per (sample, mode
// pair) with counter (g, p, net, 0) and key (seed, 0); Box-Muller on words
// (0,1) for mode 2p and (2,3) for mode 2p+1.
//
// A wavefront takes its samples one or two at a time: lanes stride over mode
// pairs, so each sample's column (contiguous over modes) is written with
// coalesced stores, and n = alpha . beta is summed over the wave at its
// end.  Networks of at most 64 modes share a wave between several samples.  The FP64
// path evaluates Box-Muller with the library's FP64 log and sincos; the FP32
// and split paths evaluate it by short FP64 series and round the radius and
// the angle's sine and cosine to FP32 once (no systematic error beyond that
// rounding).
#include <hip/hip_runtime.h>

#include <type_traits>

#include "common.h"

namespace mp {

constexpr uint64_t kMul0 = 0xD2E7470EE14C6C93ull, kMul1 = 0xCA5A826395121157ull;
constexpr uint64_t kWeyl0 = 0x9E3779B97F4A7C15ull, kWeyl1 = 0xBB67AE8584CAA73Bull;

// Full 128-bit product of two 64-bit words from four 32 x 32 -> 64
// multiply-adds: a b = p00 + (a0 b1 + a1 b0) 2^32 + a1 b1 2^64.  The form is left to
// the compiler: wave-uniform operands run on the scalar unit, and the vector form adds
// 64-bit words without carry masks.  A hand-written carry chain of four adds has about
// five moves less, but gfx950 wants two wait states between a carry and its reader, which
// cost more (65536 samples of M = 8000: 2.75 ms with them, 2.60 without the chain).
__device__ inline void mulhilo64(uint64_t a, uint64_t b, uint64_t& hi, uint64_t& lo) {
  const uint32_t a0 = (uint32_t)a, a1 = (uint32_t)(a >> 32);
  const uint32_t b0 = (uint32_t)b, b1 = (uint32_t)(b >> 32);
  const uint64_t p00 = (uint64_t)a0 * b0;
  const uint64_t t1 = (uint64_t)a0 * b1 + (p00 >> 32);
  const uint64_t t2 = (uint64_t)a1 * b0 + (uint32_t)t1;
  hi = (uint64_t)a1 * b1 + (t1 >> 32) + (t2 >> 32);
  lo = (t2 << 32) | (uint32_t)p00;
}

// a ^ b ^ c, one v_bitop3_b32 per half
__device__ inline uint64_t xor3(uint64_t a, uint64_t b, uint64_t c) {
  const uint32_t lo = __builtin_amdgcn_bitop3_b32((uint32_t)a, (uint32_t)b, (uint32_t)c, 0x96);
  const uint32_t hi = __builtin_amdgcn_bitop3_b32((uint32_t)(a >> 32), (uint32_t)(b >> 32),
                                                  (uint32_t)(c >> 32), 0x96);
  return ((uint64_t)hi << 32) | lo;
}

// Rounds `from` .. 9 on lane-dependent words; k0, k1 are round 0's keys.
__device__ inline void philox_rounds(int from, uint64_t& c0, uint64_t& c1, uint64_t& c2,
                                     uint64_t& c3, uint64_t k0, uint64_t k1) {
#pragma unroll
  for (int round = from; round < 10; ++round) {
    uint64_t hi0, lo0, hi1, lo1;
    mulhilo64(kMul0, c0, hi0, lo0);
    mulhilo64(kMul1, c2, hi1, lo1);
    c0 = xor3(hi1, c1, k0 + (uint64_t)round * kWeyl0);
    c1 = lo1;
    c2 = xor3(hi0, c3, k1 + (uint64_t)round * kWeyl1);
    c3 = lo0;
  }
}

// Philox4x64-10 with counter (g, p, net, 0) and key (seed, 0) for a
// wave-uniform g: what the first three rounds compute without the lane's p.
struct PhiloxHead {
  uint64_t c0, m2, a, b, lo;
};
__device__ inline PhiloxHead philox_head(uint64_t g, uint64_t net, uint64_t seed) {
  uint64_t hi, lo;
  PhiloxHead h;
  // round 0: (g, p, net, 0) -> (hi1 ^ p ^ k0, lo1, hi0 ^ k1, lo0)
  mulhilo64(kMul1, net, hi, lo);
  h.c0 = hi ^ seed;  // ^ p
  const uint64_t c1 = lo;
  mulhilo64(kMul0, g, hi, lo);
  const uint64_t c2 = hi, c3 = lo;
  // round 1: c0 depends on the lane, c2 does not
  h.m2 = c3 ^ kWeyl1;  // c2' = hi0 ^ c3 ^ k1
  mulhilo64(kMul1, c2, hi, lo);
  const uint64_t d0 = hi ^ c1 ^ (seed + kWeyl0), d1 = lo;
  // round 2: c0 = d0 uniform, c2 on the lane
  mulhilo64(kMul0, d0, hi, lo);
  h.a = d1 ^ (seed + 2 * kWeyl0);  // c0'' = hi1 ^ c1 ^ k0
  h.b = hi ^ (2 * kWeyl1);         // c2'' = hi0 ^ k1 ^ c3
  h.lo = lo;                       // c3''
  return h;
}
__device__ inline void philox_lane(const PhiloxHead& h, uint32_t p, uint64_t seed, uint64_t& c0,
                                   uint64_t& c1, uint64_t& c2, uint64_t& c3) {
  uint64_t hi, lo;
  mulhilo64(kMul0, h.c0 ^ p, hi, lo);  // round 1
  c2 = hi ^ h.m2;
  c3 = lo;
  mulhilo64(kMul1, c2, hi, lo);  // round 2
  c0 = hi ^ h.a;
  c1 = lo;
  c2 = c3 ^ h.b;
  c3 = h.lo;
  philox_rounds(3, c0, c1, c2, c3, seed, 0);
}

__device__ inline void box_muller(uint64_t xe, uint64_t xo, double& w1, double& w2) {
  const double u = (double)((xe >> 11) + 1ull) * 0x1p-53;
  const double v = (double)(xo >> 11) * 0x1p-53;
  const double rho = sqrt(-2.0 * log(u));
  double s, c;
  sincos(2.0 * M_PI * v, &s, &c);
  w1 = rho * c;
  w2 = rho * s;
}

// The same transform for the paths that store FP32 or split 16-bit
// amplitudes.  Both parts are evaluated in FP64 by short series and rounded to
// FP32 once, so the amplitudes carry only that rounding: a library FP32
// logarithm was measured to bias -ln u by about +4e-8 on average, which biases
// every photon number the same way (the radius) and does not average out.
//   radius: u = m 2^k with m in [sqrt(1/2), sqrt(2)), s = (m - 1) / (m + 1)
//     (|s| <= 0.172), ln m = 2 atanh s = 2 s (1 + s^2/3 + ... + s^12/13),
//     the first omitted term below 1.3e-12 relative;
//   angle: 2 pi v = pi x 2^-52 (x = xo >> 11); the top two bits of x give the
//     quarter turn q, the other 51 the fraction f in [0, 1/2) with
//     angle = q pi/2 + pi f, and f >= 1/4 is reflected to g = 1/2 - f (sine
//     and cosine swap), exactly on the integer; sin and cos of pi g in
//     [0, pi/4] from their Taylor series to t^13 and t^12 (first omitted terms
//     below 3e-14 and 4e-13).
//
// fma_const: a b + c with the constant c in scalar registers (left to itself the
// compiler copies each coefficient of a series to a vector register first).
__device__ inline double fma_const(double a, double b, double c) {
  double d;
  asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(c));
  return d;
}

__device__ inline double neg_log_unit(double u) {
  int k;
  double m = frexp(u, &k);  // u = m 2^k, m in [1/2, 1)
  if (m < 0.70710678118654752440) {
    m *= 2.0;
    k -= 1;
  }
  // s = (m - 1) / (m + 1): hardware reciprocal refined by two Newton steps
  const double d = m + 1.0;
  double rd = __builtin_amdgcn_rcp(d);
  rd = fma(rd, fma(-d, rd, 1.0), rd);
  rd = fma(rd, fma(-d, rd, 1.0), rd);
  const double s = (m - 1.0) * rd;
  const double s2 = s * s;
  double p = 1.0 / 13.0;
  p = fma_const(p, s2, 1.0 / 11.0);
  p = fma_const(p, s2, 1.0 / 9.0);
  p = fma_const(p, s2, 1.0 / 7.0);
  p = fma_const(p, s2, 1.0 / 5.0);
  p = fma_const(p, s2, 1.0 / 3.0);
  p = fma(p, s2, 1.0);
  constexpr double kLn2 = 0.69314718055994530942;
  return -fma((double)k, kLn2, 2.0 * s * p);
}

__device__ inline void sincos_eighth(double t, double& s, double& c) {
  const double t2 = t * t;
  double ps = 1.0 / 6227020800.0;  // 1/13!
  ps = fma_const(ps, t2, -1.0 / 39916800.0);
  ps = fma_const(ps, t2, 1.0 / 362880.0);
  ps = fma_const(ps, t2, -1.0 / 5040.0);
  ps = fma_const(ps, t2, 1.0 / 120.0);
  ps = fma_const(ps, t2, -1.0 / 6.0);
  ps = fma(ps, t2, 1.0);
  double pc = 1.0 / 479001600.0;  // 1/12!
  pc = fma_const(pc, t2, -1.0 / 3628800.0);
  pc = fma_const(pc, t2, 1.0 / 40320.0);
  pc = fma_const(pc, t2, -1.0 / 720.0);
  pc = fma_const(pc, t2, 1.0 / 24.0);
  pc = fma(pc, t2, -0.5);
  pc = fma(pc, t2, 1.0);
  s = t * ps;
  c = pc;
}

__device__ inline void box_muller_f32(uint64_t xe, uint64_t xo, float& w1, float& w2) {
  const double u = (double)((xe >> 11) + 1ull) * 0x1p-53;
  const float rho = sqrtf((float)(2.0 * neg_log_unit(u)));  // two unbiased roundings
  const uint64_t x = xo >> 11;
  const uint32_t q = (uint32_t)(x >> 51);
  const uint64_t fx = x & ((1ull << 51) - 1ull);  // f = fx 2^-52
  const bool upper = (fx >> 50) != 0;              // f >= 1/4
  const uint64_t gx = upper ? (1ull << 51) - fx : fx;  // g 2^52, at most 2^50: exact in FP64
  constexpr double kPi = 3.14159265358979323846;
  double s, c;
  sincos_eighth((double)gx * (0x1p-52 * kPi), s, c);
  const float sf = (float)(upper ? c : s);  // sin(pi f), cos(pi f)
  const float cf = (float)(upper ? s : c);
  const float cq = (q & 1u) ? -sf : cf;  // cos(q pi/2 + pi f) for q = 0, 1
  const float sq = (q & 1u) ? cf : sf;
  const float sign = (q & 2u) ? -1.0f : 1.0f;  // q = 2, 3: half a turn more
  w1 = rho * (sign * cq);
  w2 = rho * (sign * sq);
}

__device__ inline uint16_t bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ inline float bf16_val(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }

// Stores the amplitudes of modes (2p, 2p+1) of one column in the storage
// precision and returns the stored values (hi + lo for the split forms).
__device__ inline void store_pair_f64(void* ab, uint32_t off, double x0, double x1) {
  typedef __attribute__((ext_vector_type(2))) double d2;
  *(d2*)((double*)ab + off) = d2{x0, x1};
}

// FP16(a0 b0 + c0) in the low half, FP16(a1 b1 + c1) in the high half (NEG: - c), each
// rounded once from the exact sum (v_fma_mix), as the FP16 forms have always stored
// their amplitudes; from the FP32 value they would be rounded twice.  Written out so
// that no instance of the kernel gets the other form.  The waits cover the partial
// register writes.
template <bool NEG>
__device__ inline uint32_t fma_f16x2(float a0, float b0, float c0, float a1, float b1, float c1) {
  uint32_t h;
  if constexpr (NEG)
    asm("v_fma_mixlo_f16 %0, %1, %2, -%3\n\ts_nop 1\n\t"
        "v_fma_mixhi_f16 %0, %4, %5, -%6\n\ts_nop 1"
        : "=&v"(h) : "v"(a0), "v"(b0), "v"(c0), "v"(a1), "v"(b1), "v"(c1));
  else
    asm("v_fma_mixlo_f16 %0, %1, %2, %3\n\ts_nop 1\n\t"
        "v_fma_mixhi_f16 %0, %4, %5, %6\n\ts_nop 1"
        : "=&v"(h) : "v"(a0), "v"(b0), "v"(c0), "v"(a1), "v"(b1), "v"(c1));
  return h;
}
__device__ inline float f16_low(uint32_t h) {
  return (float)__builtin_bit_cast(_Float16, (uint16_t)h);
}
__device__ inline float f16_high(uint32_t h) {
  return (float)__builtin_bit_cast(_Float16, (uint16_t)(h >> 16));
}

// Split storage: element j of a column sits at 64 (j / 32) + j % 32 (hi) and
// 32 further (lo); off is the hi position of the even mode 2p, whose partner
// 2p + 1 shares its block.  h: the FP16 values (fma_f16x2; FP16 forms only).
template <int PREC>
__device__ inline void store_pair_f32(void* ab, uint32_t off, float x0, float x1, uint32_t h, double& y0,
                                      double& y1) {
  if constexpr (PREC == MP_FP32) {
    typedef __attribute__((ext_vector_type(2))) float f2;
    *(f2*)((float*)ab + off) = f2{x0, x1};
    y0 = x0;
    y1 = x1;
  } else if constexpr (PREC == MP_SPLIT_BF16) {
    // x - hi is exact in FP32 (at most 16 significant bits remain)
    const uint16_t h0 = bf16_rne(x0), h1 = bf16_rne(x1);
    const uint16_t l0 = bf16_rne(x0 - bf16_val(h0)), l1 = bf16_rne(x1 - bf16_val(h1));
    uint16_t* q = (uint16_t*)ab;
    *(uint32_t*)(q + off) = (uint32_t)h0 | ((uint32_t)h1 << 16);
    *(uint32_t*)(q + off + 32) = (uint32_t)l0 | ((uint32_t)l1 << 16);
    y0 = (double)bf16_val(h0) + (double)bf16_val(l0);
    y1 = (double)bf16_val(h1) + (double)bf16_val(l1);
  } else if constexpr (PREC == MP_SPLIT1T_FP16) {
    // one FP16 value per entry
    *(uint32_t*)((uint16_t*)ab + off) = h;
    y0 = f16_low(h);
    y1 = f16_high(h);
  } else {
    const float h0 = f16_low(h), h1 = f16_high(h);
    typedef __attribute__((ext_vector_type(2))) _Float16 h2;
    const h2 l = {(_Float16)(x0 - h0), (_Float16)(x1 - h1)};
    uint16_t* q = (uint16_t*)ab;
    *(uint32_t*)(q + off) = h;
    *(h2*)(q + off + 32) = l;
    y0 = (double)h0 + (double)(float)l.x;
    y1 = (double)h1 + (double)(float)l.y;
  }
}

// Two values as e4m3 codes (first in the low byte) by the hardware pack
// conversion, which rounds to nearest even and gives e4m3_rne's codes for
// every input below 448 in magnitude (checked over 4e6 inputs, every rounding
// tie and the subnormal range included); inputs are clamped to +-448 first,
// e4m3_rne's saturation.  One instruction instead of e4m3_rne's integer
// sequence, in a kernel bound by its ALU work.
__device__ inline uint16_t e4m3_pair(float x0, float x1) {
  x0 = fminf(fmaxf(x0, -448.0f), 448.0f);
  x1 = fminf(fmaxf(x1, -448.0f), 448.0f);
  return (uint16_t)(__builtin_amdgcn_cvt_pk_fp8_f32(x0, x1, 0, false) & 0xFFFF);
}

// MP_SPLIT1T_FP16 storage: mode j of storage column c (column pairs, each
// 32-mode block holding the pair's two runs of 32 values side by side).
__device__ inline int64_t split1t_offset(int64_t c, int64_t j, int64_t ldm) {
  return (c >> 1) * 2 * ldm + 64 * (j >> 5) + (j & 31) + (c & 1) * 32;
}

// Per-mode coefficients of a mode pair in the arithmetic of the path.
template <bool F64>
struct PairCoef;
template <>
struct PairCoef<true> { double p0, m0, p1, m1; };
template <>
struct PairCoef<false> { float p0, m0, p1, m1; };

// c+ = sqrt(e^{2r} - 1) / 2, c- = sqrt(1 - e^{-2r}) / 2 of modes 2p and 2p + 1;
// zero on padding.
template <bool F64>
__device__ inline PairCoef<F64> pair_coef(const double* __restrict__ r, int64_t p, int M) {
  double c[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int u = 0; u < 2; ++u)
    if (2 * p + u < M) {
      const double ru = r[2 * p + u];
      c[2 * u] = 0.5 * sqrt(expm1(2.0 * ru));
      c[2 * u + 1] = 0.5 * sqrt(-expm1(-2.0 * ru));
    }
  if constexpr (F64)
    return {c[0], c[1], c[2], c[3]};
  else
    return {(float)c[0], (float)c[1], (float)c[2], (float)c[3]};
}

// Amplitudes of mode pair p of chunk sample k from its four Philox words, stored;
// returns their share of n.
template <int PREC>
__device__ inline double sample_pair(int M, int64_t ldm, int64_t E, void* __restrict__ ab, int64_t k,
                                     int p, uint64_t c0, uint64_t c1, uint64_t c2, uint64_t c3,
                                     const PairCoef<PREC == MP_FP64>& cf) {
  const int64_t j0 = 2 * p;
  // column stride ldm (FP64, FP32) or 2 ldm (split, hi and lo interleaved);
  // the T-split form stores column pairs, beta from E2 on.  The columns' bases
  // are wave-uniform in sample_kernel, the lane's part of the address 32 bits.
  typedef std::conditional_t<PREC == MP_FP64, double,
                             std::conditional_t<PREC == MP_FP32, float, uint16_t>> Elem;
  constexpr bool kPair = PREC == MP_SPLIT1T_FP16 || PREC == MP_SPLIT1T_F8;
  Elem *pa, *pb;
  uint32_t off;
  if constexpr (PREC == MP_FP64 || PREC == MP_FP32) {
    pa = (Elem*)ab + k * ldm;
    pb = (Elem*)ab + (E + k) * ldm;
    off = (uint32_t)j0;
  } else {
    pa = (Elem*)ab + (kPair ? split1t_offset(k, 0, ldm) : k * 2 * ldm);
    pb = (Elem*)ab + (kPair ? split1t_offset(split1t_half(E) + k, 0, ldm) : (E + k) * 2 * ldm);
    off = 64u * ((uint32_t)j0 >> 5) + ((uint32_t)j0 & 31u);
  }
  if constexpr (PREC == MP_FP64) {
    double w1 = 0.0, w2 = 0.0, w3 = 0.0, w4 = 0.0;
    if (j0 < M) box_muller(c0, c1, w1, w2);
    if (j0 + 1 < M) box_muller(c2, c3, w3, w4);
    const double t0 = cf.m0 * w2, t1 = cf.m1 * w4;
    const double a0 = fma(cf.p0, w1, t0), b0 = fma(cf.p0, w1, -t0);
    const double a1 = fma(cf.p1, w3, t1), b1 = fma(cf.p1, w3, -t1);
    store_pair_f64(pa, off, a0, a1);
    store_pair_f64(pb, off, b0, b1);
    return a0 * b0 + a1 * b1;
  } else {
    float w1 = 0.0f, w2 = 0.0f, w3 = 0.0f, w4 = 0.0f;
    if (j0 < M) box_muller_f32(c0, c1, w1, w2);
    if (j0 + 1 < M) box_muller_f32(c2, c3, w3, w4);
    // written as FMAs: left to contraction, alpha and beta of a pair could round
    // different products first, and instances of the kernel differ
    const float t0 = cf.m0 * w2, t1 = cf.m1 * w4;
    const float a0 = fmaf(cf.p0, w1, t0), b0 = fmaf(cf.p0, w1, -t0);
    const float a1 = fmaf(cf.p1, w3, t1), b1 = fmaf(cf.p1, w3, -t1);
    // the pair forms store the FP16 operand (and then its e4m3 copy)
    constexpr int SP = PREC == MP_SPLIT1T_F8 ? MP_SPLIT1T_FP16 : PREC;
    uint32_t ha = 0, hb = 0;
    if constexpr (PREC != MP_FP32 && PREC != MP_SPLIT_BF16) {
      ha = fma_f16x2<false>(cf.p0, w1, t0, cf.p1, w3, t1);
      hb = fma_f16x2<true>(cf.p0, w1, t0, cf.p1, w3, t1);
    }
    double ya0, ya1, yb0, yb1;
    store_pair_f32<SP>(pa, off, a0, a1, ha, ya0, ya1);
    store_pair_f32<SP>(pb, off, b0, b1, hb, yb0, yb1);
    if constexpr (PREC == MP_SPLIT1T_F8) {
      // e4m3 copies of the stored FP16 values, after the FP16 part
      const int64_t e2 = split1t_half(E);
      uint8_t* b8 = (uint8_t*)ab + 4 * e2 * ldm;
      uint8_t *qa = b8 + pair8_offset(k, 0, ldm), *qb = b8 + pair8_offset(e2 + k, 0, ldm);
      const uint32_t off8 = 128u * ((uint32_t)j0 >> 6) + ((uint32_t)j0 & 63u);
      // lanes 2q and 2q + 1 hold modes 4q' .. 4q' + 3 of a 64-mode block:
      // the even lane stores the four codes as one word
      const uint32_t ca = e4m3_pair((float)ya0, (float)ya1);
      const uint32_t cb = e4m3_pair((float)yb0, (float)yb1);
      const uint32_t na = (uint32_t)__shfl_xor((int)ca, 1, 64);
      const uint32_t nb = (uint32_t)__shfl_xor((int)cb, 1, 64);
      if ((p & 1) == 0) {
        *(uint32_t*)(qa + off8) = ca | (na << 16);
        *(uint32_t*)(qb + off8) = cb | (nb << 16);
      }
      if ((E & 1) && k == E - 1) {
        *(uint16_t*)(qa + off8 + 64) = 0;
        *(uint16_t*)(qb + off8 + 64) = 0;
      }
    }
    if constexpr (kPair) {
      // odd E: the last sample (even k) shares its pairs with the padding
      // columns E and E2 + E, which the GEMM reads; they hold zeros
      if ((E & 1) && k == E - 1) {
        double z0, z1;
        store_pair_f32<SP>(pa, off + 32, 0.0f, 0.0f, 0u, z0, z1);
        store_pair_f32<SP>(pb, off + 32, 0.0f, 0.0f, 0u, z0, z1);
      }
    }
    return ya0 * yb0 + ya1 * yb1;
  }
}

// Each wavefront owns `per_wave` (even) consecutive samples and takes them two
// at a time.  The coefficients of coef_pairs() mode pairs at a time sit in LDS,
// formed once for the workgroup's 8 per_wave samples (expm1 and square roots in
// FP64; formed once per four samples they were a tenth of the kernel's time).
// The sample index is wave-uniform (v_readfirstlane), which leaves the Philox
// products whose operands do not depend on the lane yet, both of round 1 and
// one of rounds 2 and 3, to the scalar unit: 4 of 20.  Bound by the vector
// ALU: Philox (64-bit multiply-adds at half rate) and the FP64 series about
// equally.  65536 samples of M = 8000: 2.60 ms (3.17 GB written, the
// FP8-correction form) against 3.68 ms with per-wave coefficients and
// the sample index in a vector register.
constexpr int kSampleWaves = 8, kSampleMax = 4;
template <int PREC>
constexpr int coef_pairs() { return PREC == MP_FP64 ? 1024 : 2048; }  // 32 KB

template <int PREC>
__global__ __launch_bounds__(64 * kSampleWaves) void sample_kernel(
    int M, int64_t ldm, int64_t g0, int64_t E, int per_wave, const double* __restrict__ r,
    uint64_t seed, uint32_t net, void* __restrict__ ab, double* __restrict__ n_out) {
  constexpr bool F64 = PREC == MP_FP64;
  constexpr int PB = coef_pairs<PREC>();
  __shared__ PairCoef<F64> coef[PB];
  __shared__ double n_sum[kSampleWaves][kSampleMax];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t k0 = (wide_block() * kSampleWaves + wave) * per_wave;
  const int64_t left = E - k0;
  const int nk = left < per_wave ? (left < 0 ? 0 : (int)left) : per_wave;
  const int pairs = (int)(ldm / 2);
  for (int p0 = 0; p0 < pairs; p0 += PB) {
    const int np = pairs - p0 < PB ? pairs - p0 : PB;  // a multiple of 64
    if (p0 > 0) __syncthreads();
    for (int i = threadIdx.x; i < np; i += 64 * kSampleWaves)
      coef[i] = pair_coef<F64>(r, p0 + i, M);
    __syncthreads();
    for (int s = 0; s < nk; s += 2) {
      double n0 = 0.0, n1 = 0.0;
      const bool two = s + 1 < nk;
      const PhiloxHead h0 = philox_head((uint64_t)(g0 + k0 + s), net, seed);
      const PhiloxHead h1 = philox_head((uint64_t)(g0 + k0 + s + 1), net, seed);
      for (int i = lane; i < np; i += 64) {
        const PairCoef<F64> cf = coef[i];
        uint64_t c0, c1, c2, c3, sd = seed;
        // the round keys are formed from the seed by the scalar unit on every pass: kept
        // across the loop they would not fit the scalar registers
        asm volatile("" : "+s"(sd));
        philox_lane(h0, (uint32_t)(p0 + i), sd, c0, c1, c2, c3);
        n0 += sample_pair<PREC>(M, ldm, E, ab, k0 + s, p0 + i, c0, c1, c2, c3, cf);
        if (two) {
          asm volatile("" : "+s"(sd));
          philox_lane(h1, (uint32_t)(p0 + i), sd, c0, c1, c2, c3);
          n1 += sample_pair<PREC>(M, ldm, E, ab, k0 + s + 1, p0 + i, c0, c1, c2, c3, cf);
        }
      }
      n0 = wave_sum(n0);
      n1 = wave_sum(n1);
      if (lane == 0) {
        n_sum[wave][s] = (p0 > 0 ? n_sum[wave][s] : 0.0) + n0;
        if (two) n_sum[wave][s + 1] = (p0 > 0 ? n_sum[wave][s + 1] : 0.0) + n1;
      }
    }
  }
  if (lane == 0)
    for (int s = 0; s < nk; ++s) n_out[k0 + s] = n_sum[wave][s];
}

// Networks of at most kSmallModes modes: `lps` lanes (a power of two, 2 .. 32,
// at least the number of mode pairs) per sample, 64 / lps samples per wave, so
// that the lanes are not idle beside the few pairs; the padding modes of the
// samples are then cleared by the whole wave.  1e4 samples of M = 16 in FP64:
// 14 us against 44 us with one sample per wave at a time.
constexpr int kSmallModes = 64;
constexpr int kSmallLd = kLdAlign;  // their row stride

template <int PREC>
__global__ __launch_bounds__(256) void sample_small(int M, int64_t ldm, int64_t g0, int64_t E,
                                                    int lps, const double* __restrict__ r,
                                                    uint64_t seed, uint32_t net,
                                                    void* __restrict__ ab,
                                                    double* __restrict__ n_out) {
  constexpr bool F64 = PREC == MP_FP64;
  const int lane = threadIdx.x & 63, p = lane & (lps - 1);
  const int64_t k = (wide_block() * 256 + threadIdx.x) / lps;
  const bool valid = k < E;
  const PairCoef<F64> cf = pair_coef<F64>(r, p, M);
  double n = 0.0;
  if (valid) {
    uint64_t c0 = (uint64_t)(g0 + k), c1 = (uint64_t)p, c2 = net, c3 = 0;
    philox_rounds(0, c0, c1, c2, c3, seed, 0);
    n = sample_pair<PREC>(M, ldm, E, ab, k, p, c0, c1, c2, c3, cf);
  }
  for (int off = lps >> 1; off > 0; off >>= 1) n += __shfl_xor(n, off, 64);
  if (valid && p == 0) n_out[k] = n;
  // the padding modes [2 lps, ldm) of the wave's samples by the whole wave, in storage
  // order: pieces V of `bytes` bytes from base on, where a sample (or the two of a pair, or
  // the hi and lo values of one: SIDES) has runs of RUN modes in turn.  The wave's pieces
  // are whole samples or pairs, so a lane's modes are the same on every turn
  const int64_t k0 = k - lane / lps;
  auto clear = [&](auto piece, auto run, auto sides, char* base, uint32_t bytes) {
    typedef decltype(piece) V;
    constexpr uint32_t RUN = decltype(run)::value, SIDES = decltype(sides)::value;
    constexpr uint32_t el = F64 ? 8 : (PREC == MP_FP32 ? 4 : (sizeof(V) == 4 ? 1 : 2));
    constexpr uint32_t turn = 64 * sizeof(V), group = SIDES * kSmallLd;
    static_assert(turn % (group * el) == 0, "whole samples");
    const uint32_t e = lane * (uint32_t)sizeof(V) / el % group;
    if (e / (RUN * SIDES) * RUN + e % RUN < 2u * lps) return;
    for (uint32_t o = lane * sizeof(V); o < bytes; o += turn) *(V*)(base + o) = V{};
  };
  typedef __attribute__((ext_vector_type(2))) uint64_t u64x2;
  constexpr bool kPair = PREC == MP_SPLIT1T_FP16 || PREC == MP_SPLIT1T_F8;
  const int64_t half = kPair ? split1t_half(E) : E, left = half - k0;
  if (left <= 0) return;
  const uint32_t nc = left < 64 / lps ? (uint32_t)left : 64u / lps;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int64_t c0 = (h * half + k0) * kSmallLd;
    if constexpr (F64 || PREC == MP_FP32) {
      constexpr uint32_t sz = F64 ? 8 : 4;
      clear(u64x2{}, std::integral_constant<uint32_t, kSmallLd>{}, std::integral_constant<uint32_t, 1>{},
            (char*)ab + c0 * sz, nc * kSmallLd * sz);
    } else {
      // runs of 32 16-bit values: the hi and the lo ones of a column (split), or the two
      // columns of a pair (T-split; the first column of a wave and of either half is even)
      constexpr uint32_t sz = kPair ? 2 : 4;
      clear((uint64_t)0, std::integral_constant<uint32_t, 32>{}, std::integral_constant<uint32_t, 2>{},
            (char*)ab + c0 * sz, nc * kSmallLd * sz);
      if constexpr (PREC == MP_SPLIT1T_F8)
        clear((uint32_t)0, std::integral_constant<uint32_t, 64>{}, std::integral_constant<uint32_t, 2>{},
              (char*)ab + 4 * half * kSmallLd + c0, nc * kSmallLd);
    }
  }
}

template <int PREC>
static mp_status sample_go(int32_t M, int64_t g0, int64_t E, const double* r, uint64_t seed,
                           uint32_t net, void* ab, double* n_out, hipStream_t stream) {
  const int64_t ldm = ld_modes(M);
  int64_t blocks, lps = 2;
  // four samples per wave (a workgroup's 32 share the coefficients) once that leaves
  // at least 2048 workgroups, eight per CU: fewer idle the chip in their last turn
  const int64_t per_wave = E >= 2048 * 4 * kSampleWaves ? 4 : 2;
  if (M <= kSmallModes) {
    while (2 * lps < M) lps *= 2;
    blocks = (E * lps + 255) / 256;
  } else {
    blocks = (E + kSampleWaves * per_wave - 1) / (kSampleWaves * per_wave);
  }
  if (blocks > 0x7FFFFFFF) {
    set_error("mp_sample: E too large for one launch");
    return MP_ERR_UNSUPPORTED;
  }
  if (M <= kSmallModes)
    hipLaunchKernelGGL(sample_small<PREC>, wide_grid(blocks), dim3(256), 0, stream, M, ldm, g0,
                       E, (int)lps, r, seed, net, ab, n_out);
  else
    hipLaunchKernelGGL(sample_kernel<PREC>, wide_grid(blocks), dim3(64 * kSampleWaves), 0, stream, M,
                       ldm, g0, E, (int)per_wave, r, seed, net, ab, n_out);
  MP_HIP_LAUNCH_CHECK("mp_sample launch");
  return MP_OK;
}

mp_status sample_launch(int32_t M, int64_t g0, int64_t E, const double* r, uint64_t seed,
                        uint32_t net, mp_precision prec, void* ab, double* n_out,
                        hipStream_t stream) {
  switch (prec) {
    case MP_FP64: return sample_go<MP_FP64>(M, g0, E, r, seed, net, ab, n_out, stream);
    case MP_FP32: return sample_go<MP_FP32>(M, g0, E, r, seed, net, ab, n_out, stream);
    case MP_SPLIT_BF16: return sample_go<MP_SPLIT_BF16>(M, g0, E, r, seed, net, ab, n_out, stream);
    case MP_SPLIT_FP16:
    case MP_SPLIT1_FP16:  // the same split sample layout
      return sample_go<MP_SPLIT_FP16>(M, g0, E, r, seed, net, ab, n_out, stream);
    case MP_SPLIT1T_FP16:
      return sample_go<MP_SPLIT1T_FP16>(M, g0, E, r, seed, net, ab, n_out, stream);
    case MP_SPLIT1T_F8: return sample_go<MP_SPLIT1T_F8>(M, g0, E, r, seed, net, ab, n_out, stream);
    default: set_error("mp_sample: unknown precision %d", (int)prec); return MP_ERR_ARG;
  }
}

}  // namespace mp
