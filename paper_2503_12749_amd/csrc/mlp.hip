// Small MLP surrogate: forward, mean-squared-error backward and Adam, as
// plain HIP kernels.  The network maps sweep parameters to moments of the
// binned count distribution that the matrix-P method produces; it is trained
// on method outputs and screens parameter sweeps, with the method itself
// checking its picks (see the Python driver).
//
// Layout: layer l maps width[l] -> width[l+1] with y = x W_l + b_l, W_l stored
// row-major (width[l] rows, width[l+1] columns), then b_l; the layers are
// concatenated in one FP32 parameter vector.  The forward and backward passes
// read the weights from a BF16 copy of that vector (FP32 accumulation); Adam
// updates the FP32 master copy and refreshes the BF16 one.  Hidden layers use
// SiLU, the last layer is linear.  All reductions are in a fixed order (no
// floating-point atomics), so a training run is reproducible bit for bit.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "common.h"

namespace mp {

__device__ inline float bf16f(uint16_t h) { return __uint_as_float(((uint32_t)h) << 16); }
__device__ inline uint16_t to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// 1 / (1 + e^-z): e^-z as 2^t with the rounding of t = -z log2(e) carried along
// to first order, the reciprocal refined once; both within an ulp or two of
// FP32.  Below -88.7 e^-z overflows and the quotient is 0.  A NaN z may give any
// value here: every use multiplies by z.
__device__ inline float sigmoidf(float z) {
  constexpr float kLog2e = 1.44269502f, kLog2eLo = 1.92596299e-8f, kLn2 = 0.693147182f;
  const float x = fminf(fmaxf(z, -88.72f), 88.72f);
  const float t = -x * kLog2e;
  const float dt = fmaf(-x, kLog2e, -t) - x * kLog2eLo;
  float e = __builtin_amdgcn_exp2f(t);
  e = fmaf(e, dt * kLn2, e);
  const float d = 1.0f + e;
  float r = __builtin_amdgcn_rcpf(d);
  r = fmaf(fmaf(-d, r, 1.0f), r, r);
  return z < -88.72f ? 0.0f : r;
}

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(8))) float f32x8;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef f32x4 f32x4u __attribute__((aligned(4)));
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((address_space(3))) void lds_void;

// The network as the kernels see it.
struct MlpNet {
  int L, batch;
  int width[MP_MLP_MAX_LAYERS + 1];
  int64_t off[MP_MLP_MAX_LAYERS];   // layer l's weights in the parameter vector
  int64_t z[MP_MLP_MAX_LAYERS];     // Z_l (later dZ_l) and A_l in the workspace (floats)
  int64_t a[MP_MLP_MAX_LAYERS];
  int vec[MP_MLP_MAX_LAYERS];       // 8 weights from any column on stay in the vector
  int pitch;                        // of an LDS operand row (bf16 values)
};

// Prediction (no gradients): one layer, A = SiLU(X W + b) (the last layer linear),
// 64 x 64 tiles of four waves with v_mfma_f32_32x32x16_bf16 on the three BF16 terms
// of X, staging K chunks in LDS: X as three BF16 planes [row][k] and W
// transposed as [col][k] (rows padded by 16 bytes: the 16-byte fragment reads of
// 16 consecutive rows hit distinct banks).  Lane l holds X[l % 32][8 (l / 32) + e],
// W[8 (l / 32) + e][l % 32] (e = 0..7) of a 16-deep step; output register r is row
// 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32 of the wave's block.  mlp_rows
// below would take less time here too, but sums in another order, and predictions
// are handed out in double precision: they keep their values to the last bit.
constexpr int MLP_T = 64, MLP_THREADS = 256;

// KC: depth of a staged K chunk (mlp_forward has the rule).  Bound by the
// latency of a chunk: its loads are all issued before the first is used, and the deeper
// chunk takes a quarter of the turns.  512 rows, layers of 5, 208, 55, 307, 51 and 8:
// 11.2 us a layer of more than 32 inputs (20.4 us with 32-deep chunks loaded as used).
template <int KC>
__global__ __launch_bounds__(MLP_THREADS) void mlp_layer(const float* __restrict__ Aop,
                                                     const uint16_t* __restrict__ W16, int R,
                                                     int K, int N, const float* __restrict__ bias,
                                                     float* __restrict__ Act, int silu) {
  constexpr int KP = KC + 8, kPer = MLP_T * KC / MLP_THREADS;  // values of X and of W per thread
  extern __shared__ __attribute__((aligned(16))) uint16_t mlp_layer_lds[];
  uint16_t(*sA)[MLP_T][KP] = (uint16_t(*)[MLP_T][KP])mlp_layer_lds;
  uint16_t(*sB)[KP] = (uint16_t(*)[KP])(mlp_layer_lds + 3 * MLP_T * KP);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r0 = blockIdx.x * MLP_T, n0 = blockIdx.y * MLP_T;
  const int wr = (wave >> 1) * 32, wc = (wave & 1) * 32;
  const int lr = lane & 31, lh = lane >> 5;
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
  for (int k0 = 0; k0 < K; k0 += KC) {
    float x[kPer];
    uint16_t w[kPer];
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int e = threadIdx.x + i * MLP_THREADS;
      const int r = min(r0 + e / KC, R - 1), k = min(k0 + e % KC, K - 1);
      x[i] = Aop[(int64_t)r * K + k];
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int e = threadIdx.x + i * MLP_THREADS;  // coalesced along n
      const int k = min(k0 + e / MLP_T, K - 1), n = min(n0 + e % MLP_T, N - 1);
      w[i] = W16[(int64_t)k * N + n];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int e = threadIdx.x + i * MLP_THREADS, r = e / KC, k = e % KC;
      const float v = (r0 + r < R && k0 + k < K) ? x[i] : 0.0f;
      const uint16_t h = to_bf16(v);
      const float x1 = v - bf16f(h);
      const uint16_t m = to_bf16(x1);
      sA[0][r][k] = h;
      sA[1][r][k] = m;
      sA[2][r][k] = to_bf16(x1 - bf16f(m));
    }
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int e = threadIdx.x + i * MLP_THREADS, k = e / MLP_T, n = e % MLP_T;
      sB[n][k] = (k0 + k < K && n0 + n < N) ? w[i] : (uint16_t)0;
    }
    __syncthreads();
    const int depth = min(KC, (K - k0 + 15) & ~15);  // past it are zeros
    for (int ks = 0; ks < depth; ks += 16) {
      const int kk = ks + 8 * lh;
      const bf16x8 b = *(const bf16x8*)&sB[wc + lr][kk];
      // small terms first
#pragma unroll
      for (int t = 2; t >= 0; --t) {
        const bf16x8 a = *(const bf16x8*)&sA[t][wr + lr][kk];
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
      }
    }
  }
  const int col = n0 + wc + lr;
  if (col >= N) return;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = r0 + wr + 8 * (r >> 2) + 4 * lh + (r & 3);
    if (row >= R) continue;
    const int64_t o = (int64_t)row * N + col;
    const float z = acc[r] + bias[col];
    Act[o] = silu ? z * (1.0f / (1.0f + expf(-z))) : z;
  }
}

// Products with the BF16 weights run on the BF16 matrix cores: the FP32
// operand x is split into three BF16 terms, x = h + m + l (each the rounded
// remainder of the previous), so that h W + m W + l W carries x to FP32
// precision (24 bits) and each product of BF16 values is exact in the FP32
// accumulation.
//
// A workgroup of eight waves takes kMlpRows rows of the batch through the whole
// network: every layer's forward product, then the loss, its gradient and every
// layer's input-gradient product.  The rows' activations never leave
// LDS between layers (three BF16 planes [row][k], split once when they are
// formed); the weights come from L2, straight into the operand registers of
// v_mfma_f32_16x16x32_bf16 (lane l: A[l % 16][8 (l / 16) + e], B[8 (l / 16) + e]
// [l % 16], e = 0..7; output register r is row 4 (l / 16) + r, column l % 16).
// A pass covers 256 columns: two groups of 128 by four parts of the 32-deep steps
// (wave = 4 group + part).  A lane owns the eight neighbours n0 + 8 (l % 16) + f of
// its group, so that every weight load is 16 bytes:
//   forward:  B[k][n] = W[k][n], one load per k brings the eight columns (then an
//     8 x 8 transpose in registers);
//   backward: B[k][n] = W[n][k], one load per column brings its eight k.
// Rows start on any 2-byte address.  The parts' sums meet in LDS ((0 + 2) + (1 + 3)),
// from where a thread takes eight neighbouring columns of one row for the
// elementwise work, so that its loads and stores are wide too.
// Bound by the latency from layer to layer and by the instructions and weight
// loads of the few CUs that a batch fills (16 at batch 256).  With 32 columns per
// wave and all k, a 256 x 256 forward layer's 4-byte weight loads took 11500 cycles
// and its scattered stores 4000; a launch per layer and pass over 64 x 64 tiles,
// each staging both operands through LDS element by element, took 31 us per forward
// and 26 us per backward 256 x 256 layer at batch 256 (all seven products of a
// training step take 38 us now).  The sums of four passes (widths up to 1024) do not all
// fit: 31 of 256 registers spill.
constexpr int kMlpRows = 16, kMlpWaves = 8, kMlpThreads = 64 * kMlpWaves;
constexpr int kMlpGroup = 128, kMlpParts = 4, kMlpPass = 256;
constexpr int kMlpPasses = 1024 / kMlpPass;                   // widths are at most 1024
constexpr int kMlpSumRow = kMlpGroup + 4;                     // pitch of the sums (floats)
constexpr int kMlpSums = 4 * kMlpRows * kMlpSumRow;           // [group][2][row][column]

// The lane's weights of a 32-deep step, 8 lh .. + 7 of its rows k0 .. + 31, for the
// eight columns from n (columns past N repeat others, their products are never stored; rows
// past K repeat the last one and are zeroed): b[e] = row e's eight columns forward, b[f] =
// column f's eight rows backward.
template <bool VEC>
__device__ inline u32x4 mlp_run(const uint16_t* W, uint32_t at, int n, int N) {
  typedef u32x4 u32x4u __attribute__((aligned(2)));
  // at: below 2^20, a 32-bit byte offset from the layer's uniform base
  if constexpr (VEC) return *(const u32x4u*)((const char*)W + 2u * at);
  u32x4 v;  // n: the run's place in its row of N values
#pragma unroll
  for (int d = 0; d < 4; ++d) {
    const int e0 = n + 2 * d < N ? 2 * d : N - 1 - n, e1 = n + 2 * d + 1 < N ? 2 * d + 1 : N - 1 - n;
    v[d] = W[at + e0] | (uint32_t)W[at + e1] << 16;
  }
  return v;
}

template <bool VEC, bool FWD>
__device__ inline void mlp_step(const uint16_t* W, int K, int N, int k0, int n, int lh,
                                u32x4 (&b)[8]) {
  const int k = k0 + 8 * lh;
  const bool whole = k0 + 32 <= K;
  if constexpr (FWD) {
    const int c = n < N ? n : (N - 1) & ~7;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int row = whole || k + e < K ? k + e : K - 1;
      b[e] = mlp_run<VEC>(W, (uint32_t)(row * N + c), c, N);
    }
    if (!whole)
#pragma unroll
      for (int e = 0; e < 8; ++e) b[e] = k + e < K ? b[e] : u32x4{0, 0, 0, 0};
  } else {
    const int q = whole || k < K ? k : (K - 1) & ~7;
#pragma unroll
    for (int f = 0; f < 8; ++f) {
      const int row = n + f < N ? n + f : N - 1;
      b[f] = mlp_run<VEC>(W, (uint32_t)(row * K + q), q, K);
    }
    if (!whole)
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const uint32_t keep = (k + 2 * d < K ? 0xFFFFu : 0u) | (k + 2 * d + 1 < K ? 0xFFFF0000u : 0u);
#pragma unroll
        for (int f = 0; f < 8; ++f) b[f][d] &= keep;
      }
  }
}

// c[f] = operand (planes, this part's steps of k < K) x B for the lane's eight columns from
// n; the next step's weights are loaded ahead of the products.
template <bool VEC, bool FWD>
__device__ inline void mlp_product(const uint16_t* W, int K, int N, int n, int part,
                                   const uint16_t* planes, int plane, int pitch, int lane,
                                   f32x4 (&c)[8]) {
  const uint16_t* ap = planes + (lane & 15) * pitch + 8 * (lane >> 4);
  auto products = [&](int k0, const u32x4(&b)[8]) {
    bf16x8 a[3];
#pragma unroll
    for (int t = 0; t < 3; ++t) a[t] = *(const bf16x8*)(ap + t * plane + k0);
#pragma unroll
    for (int f = 0; f < 8; ++f) {
      u32x4 w = b[f];
      if constexpr (FWD)  // column f of the 8 rows: low or high halves of two rows per word
#pragma unroll
        for (int d = 0; d < 4; ++d)
          w[d] = __builtin_amdgcn_perm(b[2 * d + 1][f / 2], b[2 * d][f / 2],
                                       f & 1 ? 0x07060302u : 0x05040100u);
#pragma unroll
      for (int t = 2; t >= 0; --t)  // small terms first
        c[f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t], __builtin_bit_cast(bf16x8, w), c[f], 0,
                                                       0, 0);
    }
  };
  constexpr int kNext = 32 * kMlpParts;
  u32x4 b0[8], b1[8];
  int k0 = 32 * part;
  if (k0 < K) mlp_step<VEC, FWD>(W, K, N, k0, n, lane >> 4, b0);
  while (k0 < K) {
    if (k0 + kNext < K) mlp_step<VEC, FWD>(W, K, N, k0 + kNext, n, lane >> 4, b1);
    products(k0, b0);
    k0 += kNext;
    if (k0 >= K) break;
    if (k0 + kNext < K) mlp_step<VEC, FWD>(W, K, N, k0 + kNext, n, lane >> 4, b0);
    products(k0, b1);
    k0 += kNext;
  }
}

__global__ __launch_bounds__(kMlpThreads) void mlp_rows(MlpNet p, const uint16_t* __restrict__ w16,
                                                        const float* __restrict__ params,
                                                        const float* __restrict__ X,
                                                        const float* __restrict__ Y,
                                                        float* __restrict__ ws,
                                                        double* __restrict__ part) {
  extern __shared__ __attribute__((aligned(16))) uint16_t planes[];  // [3][kMlpRows][pitch]
  __shared__ double red[kMlpWaves];
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lh = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int group = wave / kMlpParts, pq = wave % kMlpParts;
  const int64_t first = wide_block() * kMlpRows;
  if (first >= p.batch) return;
  const int row0 = (int)first;
  const int plane = kMlpRows * p.pitch;
  float* sums = (float*)(planes + 3 * plane);
  // elementwise work: row m of the block, columns pass + n8 .. + 7
  const int m = tid >> 5, n8 = 8 * (tid & 31);
  const bool valid = row0 + m < p.batch;

  // operand values of columns n .. n + 7 of row m
  auto put = [&](int n, const float (&x)[8]) {
    uint16_t* o = planes + m * p.pitch + n;
    f32x8 v;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = x[e];
#pragma unroll
    for (int t = 0; t < 3; ++t) {
      const bf16x8 h = __builtin_convertvector(v, bf16x8);
      *(bf16x8*)(o + t * plane) = h;
      v -= __builtin_convertvector(h, f32x8);
    }
  };
  // eight values of a row of N from column n on: 16-byte accesses where they all exist
  auto get8 = [&](const float* src, int n, int N, float (&x)[8]) {
    if (n + 8 <= N) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const f32x4 v = *(const f32x4u*)(src + n + 4 * h);
#pragma unroll
        for (int e = 0; e < 4; ++e) x[4 * h + e] = v[e];
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = n + e < N ? src[n + e] : 0.0f;
    }
  };
  auto set8 = [&](float* dst, int n, int N, const float (&x)[8]) {
    if (n + 8 <= N) {
#pragma unroll
      for (int h = 0; h < 2; ++h)
        *(f32x4u*)(dst + n + 4 * h) = f32x4{x[4 * h], x[4 * h + 1], x[4 * h + 2], x[4 * h + 3]};
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (n + e < N) dst[n + e] = x[e];
    }
  };
  // one layer's product: z[ps] = row m, columns 256 ps + n8 .. + 7.  Every wave is past its
  // reads of the operand when it returns.
  float z[kMlpPasses][8];
  auto layer = [&](auto fwd, const uint16_t* W, int K, int N, int vec) {
    constexpr bool FWD = decltype(fwd)::value;
#pragma unroll
    for (int ps = 0; ps < kMlpPasses; ++ps) {
      if (ps * kMlpPass >= N) break;
      const int n0 = ps * kMlpPass + kMlpGroup * group;
      f32x4 a[8];
#pragma unroll
      for (int f = 0; f < 8; ++f) a[f] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (n0 < N) {
        if (vec)
          mlp_product<true, FWD>(W, K, N, n0 + 8 * lr, pq, planes, plane, p.pitch, lane, a);
        else
          mlp_product<false, FWD>(W, K, N, n0 + 8 * lr, pq, planes, plane, p.pitch, lane, a);
      }
      if (ps > 0) __syncthreads();  // the previous pass's sums are read
      // rows 4 lh + r, eight columns: parts 2 and 3 leave their sums, 0 and 1 add theirs
      float* o = sums + ((group * 2 + (pq & 1)) * kMlpRows + 4 * lh) * kMlpSumRow + 8 * lr;
#pragma unroll
      for (int turn = 0; turn < 2; ++turn) {
        if ((pq < 2) == (turn == 1)) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              f32x4* q = (f32x4*)(o + r * kMlpSumRow + 4 * h);
              f32x4 v = {a[4 * h][r], a[4 * h + 1][r], a[4 * h + 2][r], a[4 * h + 3][r]};
              if (turn == 1) v += *q;
              *q = v;
            }
        }
        __syncthreads();
      }
      const float* s0 = sums + ((n8 / kMlpGroup) * 2 * kMlpRows + m) * kMlpSumRow + n8 % kMlpGroup;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const f32x4 v = *(const f32x4*)(s0 + 4 * h) +
                        *(const f32x4*)(s0 + kMlpRows * kMlpSumRow + 4 * h);
#pragma unroll
        for (int e = 0; e < 4; ++e) z[ps][4 * h + e] = v[e];
      }
    }
  };

  // Touch every 128-byte line of the weights (one 4-byte direct-to-LDS load each, into a
  // sink behind the sums that nothing reads): they arrive in this XCD's L2 while the first
  // layers run, instead of one memory latency per layer.
  {
    const int64_t n = p.off[p.L - 1] + (int64_t)(p.width[p.L - 1] + 1) * p.width[p.L];
    lds_void* sink = (lds_void*)(sums + kMlpSums);
    const char* q;
    for (int64_t i = tid; (q = touch_word(w16, 2 * n, i)) != nullptr; i += kMlpThreads)
      __builtin_amdgcn_global_load_lds((const void*)q, sink, 4, 0, 0);
  }
  for (int n = n8; n < ((p.width[0] + 31) & ~31); n += kMlpPass) {
    float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (valid) get8(X + (int64_t)(row0 + m) * p.width[0], n, p.width[0], x);
    put(n, x);
  }
  __syncthreads();

  double loss = 0.0;
  for (int l = 0; l < p.L; ++l) {
    const int K = p.width[l], N = p.width[l + 1];
    const float* bias = params + p.off[l] + (int64_t)K * N;
    const bool last = l + 1 == p.L;
    const int64_t row = (int64_t)(row0 + m) * N;
    layer(std::true_type{}, w16 + p.off[l], K, N, p.vec[l]);
#pragma unroll
    for (int ps = 0; ps < kMlpPasses; ++ps) {
      const int n = ps * kMlpPass + n8;
      if (n >= ((N + 31) & ~31)) break;
      float x[8];  // the next operand: activations, or dY; zero past N and past the batch
      get8(bias, n, N, x);
#pragma unroll
      for (int e = 0; e < 8; ++e) z[ps][e] += x[e];
      if (!last) {
#pragma unroll
        for (int e = 0; e < 8; ++e) x[e] = z[ps][e] * sigmoidf(z[ps][e]);
        if (valid) {
          set8(ws + p.z[l] + row, n, N, z[ps]);
          set8(ws + p.a[l] + row, n, N, x);
        }
      } else {
        const float count = (float)((int64_t)p.batch * N);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float d = valid && n + e < N ? z[ps][e] - Y[row + n + e] : 0.0f;
          loss += (double)d * d;
          x[e] = 2.0f * d / count;
        }
        if (valid) set8(ws + p.z[l] + row, n, N, x);
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = valid && n + e < N ? x[e] : 0.0f;
      put(n, x);
    }
    __syncthreads();
  }
  for (int l = p.L - 1; l > 0; --l) {
    const int K = p.width[l + 1], N = p.width[l];  // dZ_l (rows x K) times W_l^T
    float* zs = ws + p.z[l - 1] + (int64_t)(row0 + m) * N;
    layer(std::false_type{}, w16 + p.off[l], K, N, p.vec[l]);
#pragma unroll
    for (int ps = 0; ps < kMlpPasses; ++ps) {
      const int n = ps * kMlpPass + n8;
      if (n >= ((N + 31) & ~31)) break;
      float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      if (valid) {
        get8(zs, n, N, x);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float sg = sigmoidf(x[e]);
          x[e] = z[ps][e] * (sg * (1.0f + x[e] * (1.0f - sg)));
        }
        set8(zs, n, N, x);  // dZ takes the place of Z
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = n + e < N ? x[e] : 0.0f;
      put(n, x);
    }
    __syncthreads();
  }
  // the rows' squared errors, in a fixed order
  loss = wave_sum(loss);
  if (lane == 0) red[wave] = loss;
  __syncthreads();
  if (tid == 0) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kMlpWaves; ++w) t += red[w];
    part[wide_block()] = t;
  }
}

// Weight and bias gradients of every layer in one launch, on the FP32 matrix
// cores (both operands are FP32 activations or gradients):
//   G[(I + 1) x O] = [X | 1]^T dZ,  rows i < I: dW, row I: db = sum_b dZ[b][.]
// which is the layer's slice of the gradient vector (W row-major, then b).
// v_mfma_f32_32x32x2f32 takes A[l % 32][l / 32] and B[l / 32][l % 32] from lane
// l: two batch rows of 32 neighbouring activations and of 32 gradients, loaded
// straight from memory.  A workgroup computes one 32 x 32 tile, its four waves
// a quarter of the batch each, added through LDS in wave order.  The last
// workgroup adds the loss partials.  Latency-bound at these sizes: a launch per
// layer over 64 x 64 tiles staged through LDS took 37 us per 256 x 256 layer at
// batch 256 (all layers together 7 us now).
struct MlpTiles {
  int first[MP_MLP_MAX_LAYERS + 1];  // first workgroup of each layer; then the loss's
};

__global__ __launch_bounds__(256) void mlp_grads(MlpNet p, MlpTiles tiles,
                                                 const float* __restrict__ X,
                                                 const float* __restrict__ ws,
                                                 float* __restrict__ grads,
                                                 const double* __restrict__ part, int n_part,
                                                 float* __restrict__ loss) {
  __shared__ float red[3][32 * 32];
  __shared__ double lred[4];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, lr = lane & 31, lh = lane >> 5;
  if ((int)blockIdx.x >= tiles.first[p.L]) {
    double t = 0.0;
    for (int i = tid; i < n_part; i += 256) t += part[i];
    t = wave_sum(t);
    if (lane == 0) lred[wave] = t;
    __syncthreads();
    if (tid == 0)
      *loss = (float)((lred[0] + lred[1] + lred[2] + lred[3]) /
                      (double)((int64_t)p.batch * p.width[p.L]));
    return;
  }
  int l = 0;
  while ((int)blockIdx.x >= tiles.first[l + 1]) ++l;
  const int I = p.width[l], O = p.width[l + 1], to = (O + 31) / 32;
  const int tile = (int)blockIdx.x - tiles.first[l];
  const int i = tile / to * 32 + lr, o = tile % to * 32 + lr;
  const float* in = l > 0 ? ws + p.a[l - 1] : X;
  const float* dz = ws + p.z[l];
  const int quarter = ((p.batch + 3) / 4 + 1) & ~1;
  const int b0 = wave * quarter, b1 = b0 + quarter < p.batch ? b0 + quarter : p.batch;
  f32x16 acc;
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
  // rows past the quarter and columns past the layer repeat the last ones; the
  // activations' values there are zeroed, the gradients' columns never stored
  const float* xp = in + (i < I ? i : I - 1);
  const float* dp = dz + (o < O ? o : O - 1);
  constexpr int S = 16;  // steps of two rows loaded together, one block ahead
  float x0[S], d0[S], x1[S], d1[S];
  auto fetch = [&](int b, float(&x)[S], float(&d)[S]) {
#pragma unroll
    for (int j = 0; j < S; ++j) {
      const int r = b + 2 * j + lh;
      const int64_t row = r < b1 ? r : b1 - 1;
      x[j] = xp[row * I];
      d[j] = dp[row * O];
    }
  };
  auto multiply = [&](int b, const float(&x)[S], const float(&d)[S]) {
#pragma unroll
    for (int j = 0; j < S; ++j) {
      const bool v = b + 2 * j + lh < b1;
      const float a = i == I ? 1.0f : x[j];
      acc = __builtin_amdgcn_mfma_f32_32x32x2f32(v && i <= I ? a : 0.0f, v ? d[j] : 0.0f, acc, 0, 0,
                                                  0);
    }
  };
  if (b0 < b1) {
    fetch(b0, x0, d0);
    for (int b = b0; b < b1; b += 4 * S) {
      fetch(b + 2 * S, x1, d1);
      multiply(b, x0, d0);
      fetch(b + 4 * S, x0, d0);
      multiply(b + 2 * S, x1, d1);
    }
  }
  if (wave > 0)
#pragma unroll
    for (int r = 0; r < 16; ++r) red[wave - 1][r * 64 + lane] = acc[r];
  __syncthreads();
  if (wave > 0 || o >= O) return;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int row = tile / to * 32 + 8 * (r >> 2) + 4 * lh + (r & 3);
    const float g = ((acc[r] + red[0][r * 64 + lane]) + red[1][r * 64 + lane]) + red[2][r * 64 + lane];
    if (row <= I) grads[p.off[l] + (int64_t)row * O + o] = g;
  }
}

__global__ void mlp_adam(int64_t n, float* __restrict__ p, const float* __restrict__ g,
                         float* __restrict__ m, float* __restrict__ v, uint16_t* __restrict__ p16,
                         float lr, float b1, float b2, float eps, float wd, float c1, float c2) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  // Adam with decoupled weight decay
  const float pi = p[i] - lr * ((mi / c1) / (sqrtf(vi / c2) + eps) + wd * p[i]);
  p[i] = pi;
  p16[i] = to_bf16(pi);
}

__global__ void mlp_round_bf16(int64_t n, const float* __restrict__ p, uint16_t* __restrict__ p16) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p16[i] = to_bf16(p[i]);
}

// ---------------------------------------------------------------- host side

static int64_t layer_offset(const mp_mlp_shape* s, int l) {
  int64_t off = 0;
  for (int k = 0; k < l; ++k) off += (int64_t)(s->width[k] + 1) * s->width[k + 1];
  return off;
}

int64_t mlp_param_count(const mp_mlp_shape* s) { return layer_offset(s, s->n_layers); }

static int64_t mlp_parts(int32_t batch) { return ((int64_t)batch + kMlpRows - 1) / kMlpRows; }

static int64_t act_elems(const mp_mlp_shape* s, int32_t batch) {
  // Z and A of every layer (Z becomes dZ in the backward pass), the loss partials (a double
  // per workgroup of mlp_rows) and their alignment
  int64_t e = 2 * mlp_parts(batch) + 2;
  for (int l = 0; l < s->n_layers; ++l) e += 2 * (int64_t)batch * s->width[l + 1];
  return e;
}

size_t mlp_workspace(const mp_mlp_shape* s, int32_t batch) {
  return (size_t)act_elems(s, batch) * 4 + 256;
}

// Layers and workspace offsets of a call; returns the LDS bytes.
static size_t mlp_net(const mp_mlp_shape* s, int32_t batch, MlpNet& p, int64_t* used) {
  p = MlpNet{};
  p.L = s->n_layers;
  p.batch = batch;
  int64_t cur = 0;
  int wmax = 0;
  for (int l = 0; l <= p.L; ++l) {
    p.width[l] = s->width[l];
    wmax = std::max(wmax, (int)s->width[l]);
  }
  for (int l = 0; l < p.L; ++l) {
    const int O = p.width[l + 1];
    p.off[l] = layer_offset(s, l);
    p.z[l] = cur;
    p.a[l] = cur + (int64_t)batch * O;
    cur += 2 * (int64_t)batch * O;
    // the longest run of 8 starts in the last weight row (its tail may reach into the
    // biases and the next layer, never past the vector); only networks of a few values
    // take single loads
    p.vec[l] = p.off[l] + (int64_t)(p.width[l] - 1) * O + (O + 7) / 8 * 8 <= mlp_param_count(s);
  }
  if (used) *used = cur;
  // 8 values of padding: the 16-byte operand reads of the 16 rows spread over the banks
  p.pitch = ((wmax + 31) & ~31) + 8;
  // the planes, the sums handed between parts, the sink
  return (size_t)3 * kMlpRows * p.pitch * 2 + (size_t)kMlpSums * 4 + 256;
}

static mp_status mlp_lds(const void* kernel, size_t lds) {
  if (lds <= 65536) return MP_OK;
  const hipError_t e =
      hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  MP_CHECK_ARG(e == hipSuccess, MP_ERR_HIP, "mlp: %s", hipGetErrorString(e));
  return MP_OK;
}

mp_status mlp_forward(const mp_mlp_shape* s, const uint16_t* w16, const float* params,
                      const float* X, int32_t batch, float* Y, void* ws, hipStream_t st) {
  float* cur = (float*)ws;
  const float* in = X;
  for (int l = 0; l < s->n_layers; ++l) {
    const int I = s->width[l], O = s->width[l + 1];
    const int64_t off = layer_offset(s, l);
    const bool last = l + 1 == s->n_layers;
    // one layer reads X while it writes: through the workspace, as Y may be X
    float* act = last && l > 0 ? Y : cur;
    cur += (int64_t)batch * O;
    const int64_t groups = (int64_t)((batch + MLP_T - 1) / MLP_T) * ((O + MLP_T - 1) / MLP_T);
    // the deep chunk's LDS leaves two workgroups per CU: from a full turn of them on, shallow
    // chunks overlap more (the sums are in the same order): layers of 5, 256, 256, 256 and 8,
    // 131072 rows: 848 us deep, 381 us shallow; 4096 rows 45 us deep, 91 us before deep chunks
    const int KC = I <= 32 || groups >= 512 ? 32 : 128;
    auto kernel = KC == 32 ? mlp_layer<32> : mlp_layer<128>;
    const size_t lds = (size_t)4 * MLP_T * (KC + 8) * 2;
    const mp_status r = mlp_lds((const void*)kernel, lds);
    if (r != MP_OK) return r;
    hipLaunchKernelGGL(kernel,
                       dim3((unsigned)((batch + MLP_T - 1) / MLP_T), (unsigned)((O + MLP_T - 1) / MLP_T)),
                       dim3(MLP_THREADS), lds, st, in, w16 + off, (int)batch, I, O,
                       params + off + (int64_t)I * O, act, last ? 0 : 1);
    in = act;
  }
  MP_HIP_LAUNCH_CHECK("mlp forward launch");
  if (s->n_layers == 1) {
    const hipError_t e =
        hipMemcpyAsync(Y, in, (size_t)batch * s->width[1] * 4, hipMemcpyDeviceToDevice, st);
    MP_CHECK_ARG(e == hipSuccess, MP_ERR_HIP, "mlp forward copy: %s", hipGetErrorString(e));
  }
  return MP_OK;
}

mp_status mlp_loss_grad(const mp_mlp_shape* s, const uint16_t* w16, const float* params,
                        const float* X, const float* Y, int32_t batch, float* grads, float* loss,
                        void* ws, hipStream_t st) {
  MlpNet p;
  int64_t used = 0;
  const size_t lds = mlp_net(s, batch, p, &used);
  const mp_status r = mlp_lds((const void*)mlp_rows, lds);
  if (r != MP_OK) return r;
  double* part = (double*)(((uintptr_t)((float*)ws + used) + 7) & ~(uintptr_t)7);
  const int n_part = (int)mlp_parts(batch);
  hipLaunchKernelGGL(mlp_rows, wide_grid(n_part), dim3(kMlpThreads), lds, st, p, w16, params, X,
                     Y, (float*)ws, part);
  MlpTiles t{};
  for (int l = 0; l < p.L; ++l)
    t.first[l + 1] = t.first[l] + (p.width[l] + 32) / 32 * ((p.width[l + 1] + 31) / 32);
  hipLaunchKernelGGL(mlp_grads, dim3((unsigned)(t.first[p.L] + 1)), dim3(256), 0, st, p, t, X,
                     (const float*)ws, grads, part, n_part, loss);
  MP_HIP_LAUNCH_CHECK("mlp backward launch");
  return MP_OK;
}

mp_status mlp_adam_launch(int64_t n, float* params, const float* grads, float* m, float* v,
                          uint16_t* w16, float lr, float b1, float b2, float eps, float wd,
                          int32_t step, hipStream_t st) {
  const float c1 = 1.0f - powf(b1, (float)step), c2 = 1.0f - powf(b2, (float)step);
  hipLaunchKernelGGL(mlp_adam, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, params,
                     grads, m, v, w16, lr, b1, b2, eps, wd, c1, c2);
  MP_HIP_LAUNCH_CHECK("mlp adam launch");
  return MP_OK;
}

mp_status mlp_round_launch(int64_t n, const float* params, uint16_t* w16, hipStream_t st) {
  hipLaunchKernelGGL(mlp_round_bf16, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n,
                     params, w16);
  MP_HIP_LAUNCH_CHECK("mlp round launch");
  return MP_OK;
}

}  // namespace mp
