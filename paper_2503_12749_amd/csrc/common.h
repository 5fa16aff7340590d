// Internal helpers of libmpgbs: status reporting, layout arithmetic, and the
// small device utilities shared by the kernels of this library.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdint>
#include <cstdio>

#include "../../include/mpgbs.h"

namespace mp {

// Thread-local message of the last failed call (see mp_last_error).
void set_error(const char* fmt, ...);
void clear_error();

#define MP_CHECK_ARG(cond, code, ...)      \
  do {                                     \
    if (!(cond)) {                         \
      ::mp::set_error(__VA_ARGS__);        \
      return code;                         \
    }                                      \
  } while (0)

#define MP_HIP_LAUNCH_CHECK(what)                                                  \
  do {                                                                             \
    hipError_t e_ = hipGetLastError();                                             \
    if (e_ != hipSuccess) {                                                        \
      ::mp::set_error("%s: %s", what, hipGetErrorString(e_));                      \
      return MP_ERR_HIP;                                                           \
    }                                                                              \
  } while (0)

constexpr int kLdAlign = 128;  // mode padding (GEMM tile multiple)

// Output of the occupation-fused GEMM: per (slot, sample) the partial sums of
// alpha'_j beta'_j over the modes of one bin run inside one 128-mode block.
// Run q owns the slots slot_off[q] + (block - run_lo[q] / 128) for the blocks
// it touches.  Each slot holds, per sample, (re, im) from the wave with the
// Re rows of alpha' and (re, im) from the wave with the Im rows: four floats
// at part[(slot * E + sample) * 4].
struct FusedOut {
  float* part;
  int64_t E;
  int n_runs;
  int run_lo[MP_MAX_RUNS], run_hi[MP_MAX_RUNS], slot_off[MP_MAX_RUNS];
};

// One network of a grouped split-precision GEMM launch.
struct GroupNet {
  const uint16_t* A;  // packed [Re T; Im T], hi and lo interleaved in 32-blocks
  const uint16_t* B;  // sampled amplitudes, hi and lo interleaved in 32-blocks
  float* C;
  int64_t ldm, ncols;
  int kmodes;  // modes multiplied through (k_modes)
  float out_scale;
  int f8_scale_a;  // MP_SPLIT1T_F8: block scale of the FP8 product's A operand
  FusedOut fo;  // the occupation-fused epilogue's output (C unused then)
};

// Modes that a GEMM multiplies through (propagate.hip).
int k_modes(int32_t M, int depth = 64);

// Slots of the fused partials for a set of runs; fills slot_off and returns
// the total.
inline int64_t fused_slots(int n_runs, const int* run_lo, const int* run_hi, int* slot_off) {
  int64_t s = 0;
  for (int q = 0; q < n_runs; ++q) {
    slot_off[q] = (int)s;
    s += (run_hi[q] - 1) / 128 - run_lo[q] / 128 + 1;
  }
  return s;
}

inline int64_t ld_modes(int32_t M) { return ((int64_t)M + kLdAlign - 1) / kLdAlign * kLdAlign; }

inline size_t elem_bytes_ab(mp_precision p) {
  switch (p) {
    case MP_FP64: return 8;
    case MP_FP32: return 4;
    case MP_SPLIT1T_FP16: return 2;  // one FP16 value (storage columns: split1t_half)
    case MP_SPLIT1T_F8: return 3;    // one FP16 value and its e4m3 copy
    default: return 4;  // hi + lo values of 2 bytes each
  }
}

inline size_t elem_bytes_c(mp_precision p) { return p == MP_FP64 ? 8 : 4; }

inline bool valid_prec(int p) { return p >= MP_FP64 && p <= MP_SPLIT1T_F8; }

// Storage columns per half of the MP_SPLIT1T_FP16 and MP_SPLIT1T_F8 sample
// operands: E rounded up to even, so that the beta columns start a column pair.
__host__ __device__ inline int64_t split1t_half(int64_t E) { return E + (E & 1); }

// Precisions whose sample operand is stored in column pairs (split1t_half).
inline bool pair_columns(mp_precision p) { return p == MP_SPLIT1T_FP16 || p == MP_SPLIT1T_F8; }

// Columns of the sample operand: 2 E, or the storage columns of the pair forms.
inline int64_t ab_columns(int64_t E, mp_precision p) {
  return pair_columns(p) ? 2 * split1t_half(E) : 2 * E;
}

// x in OCP e4m3 (4 exponent bits, bias 7, 3 mantissa bits; no infinities,
// 0x7F and 0xFF are NaN), rounded to nearest even; magnitudes of 448, the
// largest finite value, and above give 448.
__host__ __device__ inline uint8_t e4m3_rne(float x) {
  uint32_t u;
  __builtin_memcpy(&u, &x, 4);
  const uint32_t sign = (u >> 24) & 0x80u, a = u & 0x7FFFFFFFu;
  if (a >= 0x43E00000u) return (uint8_t)(sign | 0x7Eu);  // |x| >= 448
  if (a >= 0x3C800000u) {                                // |x| >= 2^-6: normal
    const uint32_t r = a + 0x7FFFFu + ((a >> 20) & 1u);  // keep 3 mantissa bits
    const uint32_t v = (((r >> 23) - 120u) << 3) | ((r >> 20) & 7u);
    return (uint8_t)(sign | v);
  }
  // subnormal: multiples of 2^-9 (code 8 is 2^-6, the smallest normal)
  const float m = __builtin_fabsf(x) * 512.0f;  // exact, below 8
  uint32_t q = (uint32_t)m;
  const float f = m - (float)q;
  if (f > 0.5f || (f == 0.5f && (q & 1u))) ++q;
  return (uint8_t)(sign | q);
}

// Scale exponent of the e4m3 remainder of a prescaled FP16 operand: with the
// prescale 2^e of fp16 T (|T_ij| <= 1, so |x| <= 2^e) the remainder x - hi is
// at most one unit in the last place of hi, 2^(e - 10), and 2^(18 - e) maps
// it to at most 256 (e4m3 reaches 448).
__host__ __device__ inline int e4m3_lo_scale_exp(int e) { return 18 - e; }

// Byte offset of entry j of row (or storage column) r in an e4m3 operand
// stored in pairs: rows 2q and 2q + 1 share, for each 64-deep block, one
// 128-byte line (row 2q's 64 bytes, then row 2q + 1's).
__host__ __device__ inline int64_t pair8_offset(int64_t r, int64_t j, int64_t ldm) {
  return (r >> 1) * 2 * ldm + 128 * (j >> 6) + 64 * (r & 1) + (j & 63);
}

// The i-th word to read of the `bytes` at p (any address) to touch each of their 128-byte
// lines: an aligned 4-byte word that lies wholly inside them, null past the last.
__host__ __device__ inline const char* touch_word(const void* p, int64_t bytes, int64_t i) {
  const char* q = (const char*)(((uintptr_t)p + 3) & ~(uintptr_t)3) + 128 * i;
  return q + 4 <= (const char*)p + bytes ? q : nullptr;
}

// A grid of `blocks` workgroups in two dimensions, each with its number in wide_block();
// those past the last have to end by themselves.  A launch counts its threads along a
// dimension in 32 bits: beyond 2^32 it runs only what is left of them, without an error.
inline dim3 wide_grid(int64_t blocks) {
  const int64_t x = blocks < (1 << 22) ? blocks : 1 << 22;  // of at most 512 threads
  return dim3((unsigned)x, (unsigned)((blocks + x - 1) / x));
}
__device__ inline int64_t wide_block() { return (int64_t)blockIdx.y * gridDim.x + blockIdx.x; }

// v of the lane that the DPP control names, for both halves of a double.
template <int CTRL>
__device__ inline double dpp_f64(double v) {
  const int2 w = __builtin_bit_cast(int2, v);
  return __builtin_bit_cast(double, make_int2(__builtin_amdgcn_mov_dpp(w.x, CTRL, 0xF, 0xF, true),
                                              __builtin_amdgcn_mov_dpp(w.y, CTRL, 0xF, 0xF, true)));
}

// Sums over the G = 16 or 64 neighbouring lanes of a lane's group, in every lane, on
// the cross-lane paths of the vector unit (an LDS shuffle per step waits some 100
// cycles, in a chain of six).
template <int G>
__device__ inline double group_sum(double v) {
  static_assert(G == 16 || G == 64, "a row of 16 lanes or the wave");
  v += dpp_f64<0xB1>(v);   // lane ^ 1
  v += dpp_f64<0x4E>(v);   // lane ^ 2
  v += dpp_f64<0x141>(v);  // 7 - lane of 8: the other four
  v += dpp_f64<0x140>(v);  // 15 - lane of 16: the other eight
  if constexpr (G == 64) {
    // rows (0, 1) and (2, 3) exchanged, then the wave's halves
    const int2 w = __builtin_bit_cast(int2, v);
    const auto x = __builtin_amdgcn_permlane16_swap(w.x, w.x, false, false);
    const auto y = __builtin_amdgcn_permlane16_swap(w.y, w.y, false, false);
    v = __builtin_bit_cast(double, make_int2(x[0], y[0])) +
        __builtin_bit_cast(double, make_int2(x[1], y[1]));
    const int2 u = __builtin_bit_cast(int2, v);
    const auto c = __builtin_amdgcn_permlane32_swap(u.x, u.x, false, false);
    const auto d = __builtin_amdgcn_permlane32_swap(u.y, u.y, false, false);
    v = __builtin_bit_cast(double, make_int2(c[0], d[0])) +
        __builtin_bit_cast(double, make_int2(c[1], d[1]));
  }
  return v;
}
__device__ inline double wave_sum(double v) { return group_sum<64>(v); }

}  // namespace mp
