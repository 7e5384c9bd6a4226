// The local policy update of a SAPO node (Algorithm 1, the PolicyGradient step; Sec. 4.2: GRPO without a
// KL term, asymmetric clipping, Adam with its default hyper-parameters): kernels, orchestration, C ABI.
//
// Values are fp32 on row-major buffers: master parameters, activations, gradients and the two Adam
// moments; the large GEMMs form their products from half-precision pairs on the matrix cores at fp32 accuracy
// (k_gemm_x3).  One update = forward pass over the whole training set with every layer's activations
// kept (HBM is large enough: about 80 KB per token and layer for the 0.5B shape), the clipped surrogate,
// the backward pass, one Adam step.  Every sum has a fixed order (atomics take integer maxima only), so an update is
// reproducible bit for bit.
#include <math.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <type_traits>
#include <vector>

#include "ranges.h"
#include "surrogate.h"
#include "train.h"

using namespace sapo;

#define T_CK(expr)                                                                                     \
  do {                                                                                                 \
    hipError_t e__ = (expr);                                                                           \
    if (e__ != hipSuccess)                                                                             \
      return set_error(SAPO_EHIP, "%s failed: %s (%s:%d)", #expr, hipGetErrorString(e__), __FILE__, __LINE__); \
  } while (0)

namespace {

// ---------------------------------------------------------------------------------------
// C[M, N] (ldc) = beta * C + op(A) op(B), fp32.  op(A) is M x K: A[m * lda + k], or A[k * lda + m] when
// TA; op(B) is K x N: B[k * ldb + n], or B[n * ldb + k] when TB.  64 x 64 tile per workgroup of 256
// threads, 4 x 4 outputs per thread, 16-deep k steps staged through LDS.  The three forms used:
//   y = x W^T (TA 0, TB 1), dx = dy W (0, 0), dW = dy^T x (1, 0).
// ---------------------------------------------------------------------------------------
constexpr int kTM = 64, kTN = 64, kTK = 16, kPitch = 68;

// Batched launches (blockIdx.z = batch b): with s = b / nh and h = b % nh the operands start at
// A + s a1 + h a2, B + s b1 + (h / bdiv) b2, C + s c1 + h c2 (elements).  nh = 1 and zeros: one GEMM.
struct Batch {
  int nh = 1, bdiv = 1;
  long a1 = 0, a2 = 0, b1 = 0, b2 = 0, c1 = 0, c2 = 0;
  int count = 1;
  // causal attention products (rows and columns are positions of one sequence): 1 = only output tiles with
  // column <= row are needed (scores, dP); 2 = op(A)[i][k] is zero for k > i, the k loop ends at the tile's last
  // row (P V, dS K); 3 = op(A)[j][k] is zero for k < j, the k loop starts at the tile's first row (dS^T Q, P^T dO)
  int causal = 0;
  // Segmented contraction (MFMA kernel only): K consists of K / kseg segments of kseg (a multiple of 16); segment g
  // reads op(A) from A + g sega and op(B) from B + g segb, indexed by k - g kseg.  With causal = 3 the skipped start
  // applies to every segment.  Used to add the query heads of a group up inside one GEMM, in head order.
  int kseg = 0;
  long sega = 0, segb = 0;
};
// Tile of a 1-D launch of nx * ny workgroups.  Workgroup ids are dealt round-robin to the 8 XCDs (each with its
// own L2), so XCD x = id % 8 takes the contiguous tile range [x per, (x + 1) per) and walks it in panels of 8
// tile rows, column by column: the ~100 workgroups an XCD runs at once then share 8 row blocks and a dozen
// column blocks through its L2 instead of streaming every block from the memory side.
__device__ __forceinline__ bool raster_tile(int nx, int ny, int& tx, int& ty) {
  const int nt = nx * ny, per = (nt + 7) >> 3;
  const int j = blockIdx.x >> 3, t = (blockIdx.x & 7) * per + j;
  if (j >= per || t >= nt) return false;
  const int panel = t / (8 * nx), w = t - panel * 8 * nx;
  const int rows = min(8, ny - panel * 8);
  ty = panel * 8 + w % rows;
  tx = w / rows;
  return true;
}
inline unsigned raster_grid(int nx, int ny) { return (unsigned)(((long)nx * ny + 7) / 8 * 8); }

__device__ __forceinline__ void batch_offsets(const Batch& bt, const float* __restrict__& A, const float* __restrict__& B,
                                              float* __restrict__& C) {
  const int b = blockIdx.z, s = b / bt.nh, h = b % bt.nh;
  A += s * bt.a1 + h * bt.a2;
  B += s * bt.b1 + (h / bt.bdiv) * bt.b2;
  C += s * bt.c1 + h * bt.c2;
}

template <int TA, int TB>
__global__ void __launch_bounds__(256) k_sgemm(const float* __restrict__ A, int lda, const float* __restrict__ B, int ldb,
                                               float* __restrict__ C, int ldc, int M, int N, int K, float beta, Batch bt) {
  __shared__ __align__(16) float As[kTK][kPitch];
  __shared__ __align__(16) float Bs[kTK][kPitch];
  batch_offsets(bt, A, B, C);
  const int tid = threadIdx.x, tx = tid & 15, ty = tid >> 4;
  const int m0 = blockIdx.y * kTM, n0 = blockIdx.x * kTN;
  float acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = 0.f;
  for (int k0 = 0; k0 < K; k0 += kTK) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = tid + 256 * i;
      {
        const int mm = TA ? (e & 63) : (e >> 4), kk = TA ? (e >> 6) : (e & 15);
        const int m = m0 + mm, k = k0 + kk;
        float v = 0.f;
        if (m < M && k < K) v = TA ? A[(size_t)k * lda + m] : A[(size_t)m * lda + k];
        As[kk][mm] = v;
      }
      {
        const int nn = TB ? (e >> 4) : (e & 63), kk = TB ? (e & 15) : (e >> 6);
        const int n = n0 + nn, k = k0 + kk;
        float v = 0.f;
        if (n < N && k < K) v = TB ? B[(size_t)n * ldb + k] : B[(size_t)k * ldb + n];
        Bs[kk][nn] = v;
      }
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < kTK; ++kk) {
      const float4 a = *(const float4*)&As[kk][ty * 4];
      const float4 b = *(const float4*)&Bs[kk][tx * 4];
      const float av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(av[i], bv[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = m0 + ty * 4 + i;
    if (m >= M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = n0 + tx * 4 + j;
      if (n >= N) continue;
      float* c = C + (size_t)m * ldc + n;
      *c = (beta != 0.f) ? fmaf(beta, *c, acc[i][j]) : acc[i][j];
    }
  }
}

// The same contraction on the matrix cores (v_mfma_f32_32x32x2_f32: fp32 operands, fp32 accumulation), for
// operands whose sizes and leading dimensions are multiples of 4 and whose bases are 16-byte aligned.
// 128 x 128 tile per workgroup, 4 waves of 64 x 64 (2 x 2 MFMA tiles), 16-deep k steps, two LDS buffers: the
// next step's operands are fetched into registers while the current step is multiplied.  LDS rows are k,
// 160 floats apart, so the two k rows a wave reads at once fall into disjoint banks.
constexpr int kGM = 128, kGK = 16, kGP = 160;
typedef float f32x16_t __attribute__((ext_vector_type(16)));

template <int TRANS>   // TRANS 0: src[row * ld + k] (k contiguous); 1: src[k * ld + row] (row contiguous)
__device__ __forceinline__ void gemm_fetch(const float* __restrict__ src, int ld, int row0, int n_rows, int k0, int K,
                                           float4 (&r)[2]) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int e = threadIdx.x + 256 * i;
    r[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (TRANS == 0) {
      const int row = row0 + (e >> 2), k = k0 + (e & 3) * 4;
      if (row < n_rows && k < K) r[i] = *(const float4*)(src + (size_t)row * ld + k);
    } else {
      const int k = k0 + (e >> 5), row = row0 + (e & 31) * 4;
      if (row < n_rows && k < K) r[i] = *(const float4*)(src + (size_t)k * ld + row);
    }
  }
}
template <int TRANS>
__device__ __forceinline__ void gemm_stage(float (*buf)[kGP], const float4 (&r)[2]) {
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int e = threadIdx.x + 256 * i;
    if (TRANS == 0) {
      const int row = e >> 2, k = (e & 3) * 4;
      buf[k][row] = r[i].x; buf[k + 1][row] = r[i].y; buf[k + 2][row] = r[i].z; buf[k + 3][row] = r[i].w;
    } else {
      *(float4*)&buf[e >> 5][(e & 31) * 4] = r[i];
    }
  }
}

template <int TA, int TB, int NARROW>   // NARROW: N <= 64, the four waves stack along M (32 rows x 64 columns each)
__global__ void __launch_bounds__(256) k_sgemm_mfma(const float* __restrict__ A, int lda, const float* __restrict__ B, int ldb,
                                                    float* __restrict__ C, int ldc, int M, int N, int K, float beta,
                                                    Batch bt) {
  __shared__ __align__(16) float As[2][kGK][kGP];
  __shared__ __align__(16) float Bs[2][kGK][kGP];
  batch_offsets(bt, A, B, C);
  const int wave = wave_index(threadIdx.x), lane = threadIdx.x & 63;
  int tx, ty;
  if (!raster_tile((N + kGM - 1) / kGM, (M + kGM - 1) / kGM, tx, ty)) return;
  const int m0 = ty * kGM, n0 = tx * kGM;
  constexpr int MI = NARROW ? 1 : 2;
  const int wm = NARROW ? wave * 32 : (wave >> 1) * 64, wn = NARROW ? 0 : (wave & 1) * 64;
  f32x16_t acc[MI][2];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  if (bt.causal == 1 && n0 > m0 + kGM - 1) return;   // the whole tile lies above the diagonal
  int t_begin = 0, nk = (K + kGK - 1) / kGK;
  if (bt.causal == 2) nk = min(nk, (m0 + kGM + kGK - 1) / kGK);
  if (bt.causal == 3) t_begin = min(m0 / kGK, nk - 1);
  // segmented contraction: step u is step seg_skip + u % per of segment u / per
  const int seg_steps = bt.kseg > 0 ? bt.kseg / kGK : 0;
  const int seg_skip = (seg_steps && bt.causal == 3) ? min(m0 / kGK, seg_steps - 1) : 0;
  const int per = seg_steps - seg_skip;
  if (seg_steps) { t_begin = 0; nk = (K / bt.kseg) * per; }
  float4 ra[2], rb[2];
  // op(A) rows are m: A is "k contiguous" unless TA; op(B) rows are n: B is "k contiguous" when TB
  auto fetch = [&](int u) {
    const float* Ag = A;
    const float* Bg = B;
    int k0 = u * kGK, Kb = K;
    if (seg_steps) {
      const int g = u / per;
      k0 = (seg_skip + u - g * per) * kGK;
      Ag += g * bt.sega;
      Bg += g * bt.segb;
      Kb = bt.kseg;
    }
    gemm_fetch<TA>(Ag, lda, m0, M, k0, Kb, ra);
    gemm_fetch<TB ? 0 : 1>(Bg, ldb, n0, N, k0, Kb, rb);
  };
  fetch(t_begin);
  gemm_stage<TA>(As[t_begin & 1], ra);
  gemm_stage<TB ? 0 : 1>(Bs[t_begin & 1], rb);
  __syncthreads();
  for (int t = t_begin; t < nk; ++t) {
    const int cur = t & 1;
    if (t + 1 < nk) fetch(t + 1);
#pragma unroll
    for (int kk = 0; kk < kGK; kk += 2) {
      const int kr = kk + (lane >> 5), c = lane & 31;
      const float b0 = Bs[cur][kr][wn + c], b1 = Bs[cur][kr][wn + 32 + c];
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        const float a = As[cur][kr][wm + i * 32 + c];
        acc[i][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b0, acc[i][0], 0, 0, 0);
        acc[i][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b1, acc[i][1], 0, 0, 0);
      }
    }
    if (t + 1 < nk) {
      gemm_stage<TA>(As[cur ^ 1], ra);
      gemm_stage<TB ? 0 : 1>(Bs[cur ^ 1], rb);
    }
    __syncthreads();
  }
  // accumulator v of lane l: row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32 of the 32 x 32 tile
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int n = n0 + wn + j * 32 + (lane & 31);
      if (n >= N) continue;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int m = m0 + wm + i * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
        if (m >= M) continue;
        float* c = C + (size_t)m * ldc + n;
        *c = (beta != 0.f) ? fmaf(beta, *c, acc[i][j][v]) : acc[i][j][v];
      }
    }
}

// ---------------------------------------------------------------------------------------
// The large GEMMs at fp32 accuracy on the half-precision matrix cores.  Every row of an operand (a row of op(A), a column of
// op(B): what one output's contraction runs along) is scaled by a power of two that brings its largest value into
// [2^14, 2^15), and a scaled value is taken as the sum of two halves: hi, the value rounded to nearest, and lo, the remainder
// rounded to nearest.  hi + lo is within 2^-23 of a value of at least 2^-17 of its row's largest and within 2^-40 of that
// largest for smaller ones.  A product is the three partial products hi lo, lo hi, hi hi, each exact in fp32; lo lo, below 2^-22
// of the product and of either sign, is dropped.  The output is scaled back by an exact power of two.  Three
// v_mfma_f32_32x32x16_f16 (32 cycles each) do the work of sixteen v_mfma_f32_32x32x2_f32 (64 cycles each).  What this replaces,
// values cut into three bf16 pieces without scales and six partial products, dropped products up to 2^-21 of one sign,
// took six, and 6 bytes a value instead of 4: 64 x 384 tokens of the 0.5B decoder 385 -> 264 ms an update, the products 287 -> 170
// (1.17 PFLOP/s executed, 1.48 in the largest), with smaller errors against 64 bits, since the sums take half as many roundings (64 x
// 384 tokens: gradient 1.5e-5 -> 8.5e-6, log-probs 1.36e-6 -> 1.24e-6; 3 x 65: 2.9e-6 -> 2.3e-6, 1.06e-6 -> 1.00e-6).
// That is NP = 3, the accuracy of three bf16 pieces.  With NP = 2 a value is rounded to bf16 and the remainder to bf16 (16
// significant bits, no scales: 7 % less time an update), the same three products; with NP = 1 the same kernels are a plain
// bf16 GEMM with fp32 accumulation (the value rounded to nearest).
//
// A row's largest value is kept as its bits without the sign, as integers order them (NaN above infinity above all others);
// whoever writes a tensor leaves the maxima of its rows, and packing it by rows those of its columns for the products
// that contract over the rows.  Maxima do not depend on the order they are taken in, so atomics leave the same bits.
//
// Operands are cut by k_pack_x3 into the order a workgroup stages them in: for every block of 128 rows and every 16-k step,
// [part][k half][row] entries of 8 values (16 bytes): one contiguous 2 KB x parts x 2 run per step, and the LDS image
// needs no rearrangement.  Rows and k are zero-padded to the blocks.  "Rows" are the M side of op(A) or the N side of op(B);
// k is the contraction.
// ---------------------------------------------------------------------------------------
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 halfx8_t __attribute__((ext_vector_type(8)));
// 16-byte entries as a plain vector type: with HIP's uint4 struct the compiler kept the kernel's prefetch registers
// in scratch memory (every load waited for at once, then re-read), 2.7x slower
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
union Frag8 { u32x4_t u; bf16x8_t v; halfx8_t h; };

__device__ __forceinline__ uint32_t max_u32_xor16(uint32_t v) {
  const lane_u32x2 r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return max((uint32_t)r[0], (uint32_t)r[1]);
}
__device__ __forceinline__ uint32_t max_u32_xor32(uint32_t v) {
  const lane_u32x2 r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return max((uint32_t)r[0], (uint32_t)r[1]);
}
__device__ __forceinline__ uint32_t abs_bits(float x) { return __float_as_uint(x) & 0x7FFFFFFFu; }
// the wave's largest, in every lane: four steps within 16 lanes by DPP, two between them
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true));    // lane ^ 1
  v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true));    // lane ^ 2
  v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xF, 0xF, true));   // mirrored within 8
  v = max(v, (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x140, 0xF, 0xF, true));   // mirrored within 16
  return max_u32_xor32(max_u32_xor16(v));
}
// Scale of a row whose largest value has the bits mx: 2^-row_exp(mx).  Rows below 2^-112 take the largest scale (their values,
// multiples of 2^-149, are then multiples of 2^-23); with an infinity or NaN in the row every output of it is one whatever
// the scale.
__device__ __forceinline__ int row_exp(uint32_t mx) {
  const int e = (int)(mx >> 23);
  return e == 255 ? 0 : max(e, 15) - 141;
}
__device__ __forceinline__ float row_scale(uint32_t mx) { return __uint_as_float((uint32_t)(127 - row_exp(mx)) << 23); }

__host__ __device__ constexpr int x3_parts(int NP) { return NP == 1 ? 1 : 2; }   // 16-bit values that a value is kept as
// 8 values (scaled: NP 3) as MFMA fragments
template <int NP> __device__ __forceinline__ void x3_cut(const float (&x)[8], float scale, Frag8 (&f)[x3_parts(NP)]) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    if constexpr (NP == 3) {
      const float y = x[e] * scale;
      const _Float16 hi = (_Float16)y;   // round to nearest even
      f[0].h[e] = hi;
      f[1].h[e] = (_Float16)(y - (float)hi);
    } else {
      const __bf16 hi = (__bf16)x[e];
      f[0].v[e] = hi;
      if constexpr (NP == 2) f[1].v[e] = (__bf16)(x[e] - (float)hi);
    }
  }
}

// entry (16 bytes) of (part, row, k / 8) in a packed operand with KB = padded K / 16 steps
__device__ __forceinline__ size_t x3_entry(int parts, int KB, int part, int row, int k8) {
  return ((((size_t)(row >> 7) * KB + (k8 >> 1)) * parts + part) * 2 + (k8 & 1)) * 128 + (row & 127);
}
template <int NP>
__device__ __forceinline__ void x3_store(u32x4_t* __restrict__ dst, int KB, int row, int k8, const float (&x)[8], float scale) {
  constexpr int PC = x3_parts(NP);
  Frag8 f[PC];
  x3_cut<NP>(x, scale, f);
#pragma unroll
  for (int pc = 0; pc < PC; ++pc) dst[x3_entry(PC, KB, pc, row, k8)] = f[pc].u;
}
// the row's scale (NP 3)
template <int NP> __device__ __forceinline__ float x3_scale(const uint32_t* __restrict__ mx, int row) {
  return NP < 3 ? 1.f : row_scale(mx[row]);
}
// Largest values of the 8 columns k0 .. k0 + 7 of each lane, over the wave's lanes with the same lane % C, into col_mx
template <int C> __device__ __forceinline__ void wave_column_max(uint32_t (&cm)[8], uint32_t* __restrict__ col_mx, int k0, int K) {
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    if constexpr (C == 4) cm[e] = max(cm[e], (uint32_t)__builtin_amdgcn_mov_dpp((int)cm[e], 0x124, 0xF, 0xF, true));   // rotated by 4 lanes of 16
    cm[e] = max_u32_xor32(max_u32_xor16(max(cm[e], (uint32_t)__builtin_amdgcn_mov_dpp((int)cm[e], 0x128, 0xF, 0xF, true))));   // by 8
  }
  const int r = (threadIdx.x & 63) / C;   // every such lane has all of them: number r leaves column k0 + r
  uint32_t v = cm[0];
#pragma unroll
  for (int e = 1; e < 8; ++e) v = r == e ? cm[e] : v;
  if (r < 8 && k0 + r < K) atomicMax(col_mx + k0 + r, v);
}
// src[row * ld + k]: one workgroup per (block of 128 rows, 8 k steps), everything a thread reads is in flight at once.  One and two
// pieces: thread (row, k half) takes 8 octets of its row, which every part is written of in longer runs (7 x 141 tokens of the 0.5B
// decoder, one piece: 7.6 us a launch on average, 8.8 in the order below).
template <int NP>
__global__ void __launch_bounds__(256) k_pack_x3(const float* __restrict__ src, int ld, int rows, int K, int /*rows_pad*/, int KB,
                                                 u32x4_t* __restrict__ dst, const uint32_t* /*row_mx*/, uint32_t* /*col_mx*/) {
  static_assert(NP < 3, "three pieces: k_pack_x3_max");
  const int row = blockIdx.x * 128 + (threadIdx.x >> 1), kh = threadIdx.x & 1;
  const float* rp = src + (size_t)row * ld;
  const bool vec = ((ld & 3) == 0) && ((((uintptr_t)src) & 15) == 0);
  const int kb0 = blockIdx.y * 8, n = min(KB - kb0, 8);
  if (vec && (kb0 + 8) * 16 <= K && (int)blockIdx.x * 128 + 128 <= rows) {
    float x[8][8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float* q = rp + (kb0 + i) * 16 + kh * 8;
      *(float4*)&x[i][0] = *(const float4*)q;
      *(float4*)&x[i][4] = *(const float4*)(q + 4);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) x3_store<NP>(dst, KB, row, (kb0 + i) * 2 + kh, x[i], 1.f);
    return;
  }
  for (int kb = kb0; kb < kb0 + n; ++kb) {
    const int k0 = kb * 16 + kh * 8;
    float x[8];
    if (row < rows && k0 + 8 <= K && vec) {
      *(float4*)&x[0] = *(const float4*)(rp + k0);
      *(float4*)&x[4] = *(const float4*)(rp + k0 + 4);
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) x[j] = (row < rows && k0 + j < K) ? rp[k0 + j] : 0.f;
    }
    x3_store<NP>(dst, KB, row, kb * 2 + kh, x, 1.f);
  }
}
// Three pieces, scaled by the rows' maxima row_mx: a lane holds one octet of k of 8 rows, so that the columns' maxima (into col_mx, if
// given) are mostly the lane's own.
__global__ void __launch_bounds__(256) k_pack_x3_max(const float* __restrict__ src, int ld, int rows, int K, int /*rows_pad*/, int KB,
                                                     u32x4_t* __restrict__ dst, const uint32_t* __restrict__ row_mx,
                                                     uint32_t* __restrict__ col_mx) {
  const int wave = wave_index(threadIdx.x), lane = threadIdx.x & 63, octet = (int)blockIdx.y * 16 + wave * 4 + (lane & 3), k0 = octet * 8;
  auto row_of = [&](int i) { return (int)blockIdx.x * 128 + (lane >> 2) + 16 * i; };
  const bool vec = ((ld & 3) == 0) && ((((uintptr_t)src) & 15) == 0);
  float x[8][8];
  if (vec && ((int)blockIdx.y + 1) * 128 <= K && ((int)blockIdx.x + 1) * 128 <= rows) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float* q = src + (size_t)row_of(i) * ld + k0;
      *(float4*)&x[i][0] = *(const float4*)q;
      *(float4*)&x[i][4] = *(const float4*)(q + 4);
    }
  } else if (vec && (K & 3) == 0) {   // outside: the last row, the last four k, taken out again; no branch between the loads
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float4 v = *(const float4*)(src + (size_t)min(row_of(i), rows - 1) * ld + min(k0 + 4 * h, K - 4));
        *(float4*)&x[i][4 * h] = row_of(i) < rows && k0 + 4 * h < K ? v : make_float4(0.f, 0.f, 0.f, 0.f);
      }
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float v = src[(size_t)min(row_of(i), rows - 1) * ld + min(k0 + j, K - 1)];
        x[i][j] = row_of(i) < rows && k0 + j < K ? v : 0.f;
      }
  }
  if (octet >= KB * 2) return;   // padded steps are a multiple of 4 (8 octets): the whole wave
#pragma unroll
  for (int i = 0; i < 8; ++i) x3_store<3>(dst, KB, row_of(i), octet, x[i], row_scale(row_mx[min(row_of(i), rows - 1)]));
  if (col_mx) {
    uint32_t cm[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      cm[j] = abs_bits(x[0][j]);
#pragma unroll
      for (int i = 1; i < 8; ++i) cm[j] = max(cm[j], abs_bits(x[i][j]));
    }
    wave_column_max<4>(cm, col_mx, k0, K);
  }
}
// src[k * ld + row] (rows contiguous): 64 rows x 64 k per workgroup through LDS
template <int NP>
__global__ void __launch_bounds__(256) k_pack_x3_t(const float* __restrict__ src, int ld, int rows, int K, int rows_pad, int KB,
                                                   u32x4_t* __restrict__ dst, const uint32_t* __restrict__ row_mx,
                                                   uint32_t* __restrict__ /*col_mx*/) {
  __shared__ float tile[64][65];
  const int r0 = blockIdx.x * 64, k0 = blockIdx.y * 64;
  for (int e = threadIdx.x; e < 64 * 64; e += 256) {
    const int kk = e >> 6, rr = e & 63;
    const int k = k0 + kk, row = r0 + rr;
    tile[kk][rr] = (row < rows && k < K) ? src[(size_t)k * ld + row] : 0.f;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < 64 * 8; e += 256) {
    const int rr = e & 63, kq = e >> 6;           // 8 groups of 8 k
    const int row = r0 + rr, k8 = (k0 >> 3) + kq;
    if (row >= rows_pad || k8 >= KB * 2) continue;
    float x[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = tile[kq * 8 + j][rr];
    x3_store<NP>(dst, KB, row, k8, x, x3_scale<NP>(row_mx, min(row, rows - 1)));
  }
}

// Maxima of the rows of a few matrices [rows, K], contiguous: a wave per row
constexpr int kRowMaxTasks = 100;
struct RowMaxTask { const float* src; uint32_t* out; int rows, K; unsigned first_block; };
struct RowMaxTasks { int n; RowMaxTask t[kRowMaxTasks]; };
static_assert(sizeof(RowMaxTasks) + 64 <= 4096, "kernel arguments");
__global__ void __launch_bounds__(256) k_row_max(RowMaxTasks tasks) {
  int ti = 0;
  for (int end = tasks.n; end - ti > 1;) {
    const int mid = (ti + end) >> 1;
    if (blockIdx.x >= tasks.t[mid].first_block) ti = mid; else end = mid;
  }
  const RowMaxTask t = tasks.t[ti];
  const int lane = threadIdx.x & 63, row = (int)(blockIdx.x - t.first_block) * 4 + wave_index(threadIdx.x);
  if (row >= t.rows) return;
  const float* p = t.src + (size_t)row * t.K;
  uint32_t mx = 0;
  if ((t.K & 3) == 0 && ((uintptr_t)t.src & 15) == 0) {
#pragma unroll 4
    for (int k = lane * 4; k < t.K; k += 256) {
      const float4 v = *(const float4*)(p + k);
      mx = max(max(max(mx, abs_bits(v.x)), max(abs_bits(v.y), abs_bits(v.z))), abs_bits(v.w));
    }
  } else {
    for (int k = lane; k < t.K; k += 64) mx = max(mx, abs_bits(p[k]));
  }
  mx = wave_max_u32(mx);
  if (lane == 0) t.out[row] = mx;
}

// k steps of 16 per stage of the packed GEMM: what keeps a stage at 32 .. 48 MFMAs per wave
__host__ __device__ constexpr int x3_stage(int NP) { return NP == 1 ? 4 : 2; }

__host__ __device__ constexpr int x3_tn_stage(int NP) { return NP == 1 ? 2 : 1; }   // of k_gemm_x3_tn

// The products go out smallest first: hi lo, lo hi, hi hi; one piece takes the last.
template <int NP> __device__ __forceinline__ constexpr int x3_terms() { return NP == 1 ? 1 : 3; }
__device__ constexpr int kTermA[3] = {0, 1, 0}, kTermB[3] = {1, 0, 0};
template <int NP> __device__ __forceinline__ f32x16_t x3_mfma(const Frag8& a, const Frag8& b, const f32x16_t& c) {
  if constexpr (NP == 3) return __builtin_amdgcn_mfma_f32_32x32x16_f16(a.h, b.h, c, 0, 0, 0);
  else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a.v, b.v, c, 0, 0, 0);
}

// One wave-wide 1 KiB copy global -> LDS / load into registers (base + lane offset), awaited with x3_wait; issued from inline
// assembly because the compiler would wait for a copy before any LDS read.
__device__ __forceinline__ void x3_dma(const char* base, unsigned off, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base) : "memory");
}
template <int IMM> __device__ __forceinline__ void x3_reg(u32x4_t& d, const char* base, unsigned off) {
  asm volatile("global_load_dwordx4 %0, %1, %2 offset:%3" : "=v"(d) : "v"(off), "s"(base), "n"(IMM) : "memory");
}
template <int N> __device__ __forceinline__ void x3_wait() {
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

// C tile of a wave: TJ x 4 MFMA tiles; accumulator v of lane l: row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32.  With
// NP 3 the operands' scales are taken out of the sums: amx, bmx are their rows' maxima.
template <bool full> __device__ __forceinline__ void x3_col_exps(int (&eb)[4], const uint32_t* __restrict__ bmx, int n, int N) {
#pragma unroll
  for (int j = 0; j < 4; ++j) eb[j] = row_exp(bmx[full ? n + j * 32 : min(n + j * 32, N - 1)]);
}
template <bool full> __device__ __forceinline__ void x3_row_exps(int (&ea)[4], const uint32_t* __restrict__ amx, int m, int M) {   // rows m .. m + 3
  if constexpr (full) {
    const u32x4_t a = *(const u32x4_t*)(amx + m);
#pragma unroll
    for (int u = 0; u < 4; ++u) ea[u] = row_exp(a[u]);
  } else {
#pragma unroll
    for (int u = 0; u < 4; ++u) ea[u] = row_exp(amx[min(m + u, M - 1)]);
  }
}
// A tile without rows or columns past the end is stored without a comparison per value, rows by scalar base addresses.
template <int NP, int TJ>
__device__ __forceinline__ void x3_store_tile(const f32x16_t (&acc)[TJ][4], float* C, const float* Cin, int ldc, int row0, int n0,
                                              int M, int N, float beta, const uint32_t* __restrict__ amx,
                                              const uint32_t* __restrict__ bmx) {
  const int lane = threadIdx.x & 63;
  auto store = [&](auto full_c, auto beta_c) __attribute__((always_inline)) {
    constexpr bool full = decltype(full_c)::value, add = decltype(beta_c)::value;
    const unsigned off = (unsigned)((lane >> 5) * 4 * ldc + n0 + (lane & 31)) * 4u;   // bytes behind the base of a row pair
    const int m_lane = (lane >> 5) * 4, n = n0 + (lane & 31);
    const ptrdiff_t d_in = (const char*)Cin - (const char*)C;
    int eb[4];
    if constexpr (NP == 3) x3_col_exps<full>(eb, bmx, n, N);
#pragma unroll
    for (int t = 0; t < TJ; ++t)
#pragma unroll
      for (int v4 = 0; v4 < 4; ++v4) {
        const int m0 = row0 + t * 32 + 8 * v4;
        char* base[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) base[u] = (char*)(C + (size_t)(m0 + u) * ldc);
        int ea[4];
        if constexpr (NP == 3) x3_row_exps<full>(ea, amx, m0 + m_lane, M);
        float old[4][4];
        if constexpr (add) {
#pragma unroll
          for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              old[u][j] = 0.f;
              if (full || (m0 + u + m_lane < M && n + j * 32 < N)) old[u][j] = *(const float*)(base[u] + d_in + off + j * 128);
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            float r = acc[t][j][4 * v4 + u];
            if constexpr (NP == 3) r = ldexpf(r, ea[u] + eb[j]);
            if constexpr (add) r = fmaf(beta, old[u][j], r);
            if (full || (m0 + u + m_lane < M && n + j * 32 < N)) *(float*)(base[u] + off + j * 128) = r;
          }
      }
  };
  const bool full = row0 + 32 * TJ <= M && n0 + 128 <= N;
  if (beta != 0.f) {
    if (full) store(std::true_type(), std::true_type()); else store(std::false_type(), std::true_type());
  } else {
    if (full) store(std::true_type(), std::false_type()); else store(std::false_type(), std::false_type());
  }
}

// C[M, N] = beta C + A B^T of two packed operands.  128 TJ x 128 tile, 4 waves of 32 TJ rows x all 128 columns.  The A
// pieces go from global memory straight into the registers of the one wave that uses them, two stages ahead; the B
// pieces, which all four waves read, through a three-stage LDS ring filled by direct-to-LDS copies.  With both operands
// staged through LDS by way of registers (what this replaces: waves of 64 x 64 or 128 x 64) the LDS moved 0.56 - 0.75 KB
// per MFMA, and a step's copies, which the compiler waits for in front of the LDS stores, sat at its end; now 0.31 KB.
// TJ = 2: two workgroups per compute unit; TJ = 1: three.
template <int NP, int TJ>
__global__ void __launch_bounds__(256, TJ == 2 ? 2 : 3) k_gemm_x3(const u32x4_t* __restrict__ Ap, const u32x4_t* __restrict__ Bp,
                                                                  float* C, const float* Cin, int ldc, int M, int N, int KB,
                                                                  float beta, int kb_split, size_t c_split,
                                                                  const uint32_t* __restrict__ amx, const uint32_t* __restrict__ bmx) {
  constexpr int PC = x3_parts(NP), H = x3_stage(NP), NF = H * PC;     // ring copies per wave and stage; fragments of a column block
  constexpr int PER = NF + NF * TJ;                // requests per wave and stage
  constexpr int kRing = 3;
  __shared__ u32x4_t ring[kRing * NF * 4 * 64];
  const int wave = wave_index(threadIdx.x), lane = threadIdx.x & 63;
  int tx, ty;
  const int n_rb = (M + kGM - 1) / kGM;            // row blocks of the packed operand
  if (!raster_tile((N + kGM - 1) / kGM, (n_rb + TJ - 1) / TJ, tx, ty)) return;
  // blockIdx.z takes the k steps [z kb_split, (z + 1) kb_split) and writes its own copy of C (split weight gradients)
  const int t0 = blockIdx.z * kb_split, nst = (min(KB, t0 + kb_split) - t0) / H;
  C += (size_t)blockIdx.z * c_split;
  const int row_w = wave * 32 * TJ;                // this wave's rows of the tile
  // a tile's last row block may not exist: it repeats the previous one and is not stored
  const char* xbase = (const char*)(Ap + ((size_t)min(ty * TJ + (row_w >> 7), n_rb - 1) * KB + t0) * (PC * 256) + (row_w & 127));
  const char* wbase = (const char*)(Bp + ((size_t)tx * KB + t0) * (PC * 256) + wave * 32);
  const unsigned off = ((lane >> 5) * 128 + (lane & 31)) * 16;
  const unsigned lds0 =
      __builtin_amdgcn_readfirstlane((unsigned)(size_t)(const __attribute__((address_space(3))) void*)ring) + wave * 1024u;
  u32x4_t x[2][NF][TJ];
  f32x16_t acc[TJ][4];
#pragma unroll
  for (int t = 0; t < TJ; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[t][j][v] = 0.f;
  // fragment i = (k step of the stage) * PC + part: a 4 KiB step of the packed operand
  auto request_w = [&](int i, int st) { x3_dma(wbase + ((size_t)st * NF + i) * 4096, off, lds0 + ((st % kRing) * NF + i) * 4096u); };
  auto request_x = [&](u32x4_t (&dst)[TJ], int i, int st) {
    const char* b = xbase + ((size_t)st * NF + i) * 4096;
    x3_reg<0>(dst[0], b, off);
    if constexpr (TJ == 2) x3_reg<512>(dst[TJ - 1], b, off);
  };
#pragma unroll
  for (int p = 0; p < 2; ++p)
    if (p < nst) {
#pragma unroll
      for (int i = 0; i < NF; ++i) request_w(i, p);
#pragma unroll
      for (int i = 0; i < NF; ++i) request_x(x[p][i], i, p);
    }
  auto stage = [&](auto pc, int st) {
    constexpr int P = decltype(pc)::value;
    if (st + 1 < nst) x3_wait<PER>(); else x3_wait<0>();   // this wave's requests of stage st have landed ...
#pragma unroll
    for (int i = 0; i < NF; ++i)
#pragma unroll
      for (int t = 0; t < TJ; ++t) asm volatile("" : "+v"(x[P][i][t]));
    asm volatile("s_barrier" ::: "memory");                // ... and everybody's; stage st - 1 is consumed
    const bool more = st + 2 < nst;
    const u32x4_t* buf = ring + (st % kRing) * (NF * 4 * 64) + lane;
#pragma unroll
    for (int h = 0; h < H; ++h) {
      Frag8 b[4][PC];
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int q = 0; q < PC; ++q) b[j][q].u = buf[((h * PC + q) * 4 + j) * 64];
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
#pragma unroll
        for (int term = 3 - x3_terms<NP>(); term < 3; ++term)
#pragma unroll
          for (int t = 0; t < TJ; ++t) {
            Frag8 a; a.u = x[P][h * PC + kTermA[term]][t];
            acc[t][j] = x3_mfma<NP>(a, b[j][kTermB[term]], acc[t][j]);
          }
        if (h * 4 + j < NF) {   // the next-but-one stage's copies go out between the MFMAs, not in one burst
          __builtin_amdgcn_sched_barrier(0);
          if (more) request_w(h * 4 + j, st + 2);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      __builtin_amdgcn_s_setprio(0);
      __builtin_amdgcn_sched_barrier(0);
      if (more) {
#pragma unroll
        for (int q = 0; q < PC; ++q) request_x(x[P][h * PC + q], h * PC + q, st + 2);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  int st = 0;
  for (; st + 1 < nst; st += 2) {
    stage(std::integral_constant<int, 0>(), st);
    stage(std::integral_constant<int, 1>(), st + 1);
  }
  if (st < nst) stage(std::integral_constant<int, 0>(), st);
  x3_store_tile<NP, TJ>(acc, C, Cin, ldc, ty * kGM * TJ + row_w, tx * kGM, M, N, beta, amx, bmx);
}

// f(0), f(1), ... f(N - 1) with the index as a compile-time constant
template <typename F, int... I> __device__ __forceinline__ void each_of(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>()), ...);
}
template <int N, typename F> __device__ __forceinline__ void each(F&& f) { each_of(f, std::make_integer_sequence<int, N>()); }

// C[M, N] = beta C + A^T B with A [K, M] (lda) and B [K, N] (ldb) in fp32 as they lie (weight gradients: K counts tokens):
// the operands are cut into pieces on the way in.  Packing them first cost a read of 4 and a write and read of 2 NP bytes
// per value.  Same tile as k_gemm_x3; a wave reads the A values of its rows straight into registers (8 tokens of one row
// per lane: 128-byte runs), cuts them itself, and cuts a quarter of the B values for everybody, which go through two LDS
// buffers.  A stage's cuts are spread between the MFMAs of the stage before (the vector ALU works while the matrix core
// does), and a fragment's registers are requested again as soon as it is cut, a whole stage ahead.
template <int NP, int TJ>
__global__ void __launch_bounds__(256, TJ == 2 ? 2 : 3) k_gemm_x3_tn(const float* __restrict__ A, int lda, const float* __restrict__ B,
                                                                     int ldb, float* C, int ldc, int M, int N, int K, float beta,
                                                                     int k_split, size_t c_split, const uint32_t* __restrict__ amx,
                                                                     const uint32_t* __restrict__ bmx) {
  constexpr int PC = x3_parts(NP), H = x3_tn_stage(NP), kTasks = H * (TJ + 1), KS = 16 * H;
  __shared__ u32x4_t Bs[2][H * PC * 4 * 64];
  const int wave = wave_index(threadIdx.x), lane = threadIdx.x & 63, kh = lane >> 5, c = lane & 31;
  int tx, ty;
  if (!raster_tile((N + kGM - 1) / kGM, (M + kGM * TJ - 1) / (kGM * TJ), tx, ty)) return;
  const int k_begin = blockIdx.z * k_split;
  const StageRows rows(k_begin, min(K, k_begin + k_split), KS);
  const int nst = rows.nst;
  C += (size_t)blockIdx.z * c_split;
  const int row0 = ty * kGM * TJ + wave * 32 * TJ;
  // rows and columns past the end repeat the last one and are not stored
  unsigned arow[TJ];
#pragma unroll
  for (int t = 0; t < TJ; ++t) arow[t] = min(row0 + t * 32 + c, M - 1);
  const unsigned bcol = min(tx * kGM + wave * 32 + c, N - 1);
  unsigned aoff[TJ];   // byte offsets of the lane behind a token row's base
#pragma unroll
  for (int t = 0; t < TJ; ++t) aoff[t] = (unsigned)(kh * 8 * lda + arow[t]) * 4u;
  const unsigned boff = (unsigned)(kh * 8 * ldb + bcol) * 4u;
  float ascale[TJ];
#pragma unroll
  for (int t = 0; t < TJ; ++t) ascale[t] = x3_scale<NP>(amx, (int)arow[t]);
  const float bscale = x3_scale<NP>(bmx, (int)bcol);
  // Task i of a stage: fragment i % (TJ + 1) of k step i / (TJ + 1); the last fragment is the wave's part of B.
  float raw[kTasks][8];
  auto request = [&](auto ic, int s) __attribute__((always_inline)) {
    constexpr int i = decltype(ic)::value, h = i / (TJ + 1), t = i % (TJ + 1);
    const size_t k = rows.request(s) + h * 16;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if constexpr (t < TJ) raw[i][e] = *(const float*)((const char*)(A + (k + e) * lda) + aoff[t]);
      else raw[i][e] = *(const float*)((const char*)(B + (k + e) * ldb) + boff);
    }
  };
  Frag8 a[2][H][TJ][PC];
  auto cut = [&](auto ic, auto pc) __attribute__((always_inline)) {
    constexpr int i = decltype(ic)::value, h = i / (TJ + 1), t = i % (TJ + 1), p = decltype(pc)::value;
    if constexpr (t < TJ) {
      x3_cut<NP>(raw[i], ascale[t], a[p][h][t]);
    } else {
      Frag8 b[PC];
      x3_cut<NP>(raw[i], bscale, b);
#pragma unroll
      for (int q = 0; q < PC; ++q) Bs[p][((h * PC + q) * 4 + wave) * 64 + lane] = b[q].u;
    }
  };
  f32x16_t acc[TJ][4];
#pragma unroll
  for (int t = 0; t < TJ; ++t)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[t][j][v] = 0.f;
  auto stage = [&](auto pc, auto last_c, int s) __attribute__((always_inline)) {
    constexpr int P = decltype(pc)::value;
    constexpr bool last = decltype(last_c)::value;   // nothing follows: nothing is cut or requested
    const u32x4_t* buf = Bs[P] + lane;
    each<H * 4>([&](auto slot_c) __attribute__((always_inline)) {
      constexpr int slot = decltype(slot_c)::value, h = slot >> 2, j = slot & 3;
      Frag8 b[PC];
#pragma unroll
      for (int q = 0; q < PC; ++q) b[q].u = buf[((h * PC + q) * 4 + j) * 64];
#pragma unroll
      for (int term = 3 - x3_terms<NP>(); term < 3; ++term)
#pragma unroll
        for (int t = 0; t < TJ; ++t) acc[t][j] = x3_mfma<NP>(a[P][h][t][kTermA[term]], b[kTermB[term]], acc[t][j]);
      if constexpr (slot < kTasks && !last) {
        cut(slot_c, std::integral_constant<int, P ^ 1>());
        request(slot_c, s + 2);
        // one MFMA, then a few of the cut's instructions
#pragma unroll
        for (int m = 0; m < x3_terms<NP>() * TJ; ++m) {
          __builtin_amdgcn_sched_group_barrier(0x8, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x2, (NP == 3 ? 48 : 24) / (x3_terms<NP>() * TJ), 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    __syncthreads();
  };
  const std::integral_constant<int, 0> even;
  const std::integral_constant<int, 1> odd;
  // the first stage is the one that may be partial: tokens in front of it count as zero
  each<kTasks>([&](auto ic) __attribute__((always_inline)) {
    constexpr int i = decltype(ic)::value, h = i / (TJ + 1), t = i % (TJ + 1);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int i_row = h * 16 + kh * 8 + e;
      const size_t kc = rows.row(i_row);
      float v;
      if constexpr (t < TJ) v = A[kc * lda + arow[t]];
      else v = B[kc * ldb + bcol];
      raw[i][e] = rows.in(rows.k_first + i_row) ? v : 0.f;
    }
  });
  each<kTasks>([&](auto i) __attribute__((always_inline)) { cut(i, even); });
  if (rows.more()) each<kTasks>([&](auto i) __attribute__((always_inline)) { request(i, 1); });
  __syncthreads();
  int s = 0;
  for (; s + 1 < nst; s += 2) {
    stage(even, std::false_type(), s);
    stage(odd, std::false_type(), s + 1);
  }
  if (s < nst) stage(even, std::true_type(), s);
  x3_store_tile<NP, TJ>(acc, C, C, ldc, row0, tx * kGM, M, N, beta, amx, bmx);
}

// One operand of a packed GEMM: `rows` x K values at src[row * ld + k], or src[k * ld + row] when `trans`; the maxima of its
// rows, and where packing it by rows leaves those of its columns (both: NP 3 only).
struct X3Op { const float* src; int ld, rows, K; bool trans; const uint32_t* row_mx; uint32_t* col_mx; };
inline size_t x3_pack_bytes(int NP, size_t rows, size_t K) {
  return ((rows + 127) / 128 * 128) * ((K + 63) / 64 * 64) * 2 * x3_parts(NP);
}
inline int x3_steps(int K) { return (K + 63) / 64 * 4; }   // padded k steps: whole stages, whole waves of the packing
// left_out: rows (tokens) that the products at hand do without (PackedUpdate)
struct X3Bufs { void* a; void* b; size_t a_cap, b_cap; int NP; float* parts; size_t parts_cap; int left_out; };
__global__ void k_sum_parts(const float* __restrict__ part, int n_part, size_t n, float beta, const float* in, float* out);

hipError_t x3_pack(const X3Op& op, void* dst, size_t cap, int NP, hipStream_t st) {
  if (x3_pack_bytes(NP, op.rows, op.K) > cap) return hipErrorInvalidValue;
  const int rows_pad = (op.rows + 127) / 128 * 128, KB = x3_steps(op.K);
  const dim3 grid = op.trans ? dim3(rows_pad / 64, (KB * 16 + 63) / 64) : dim3(rows_pad / 128, (KB + 7) / 8);
  auto go = [&](auto kernel) {
    return launch(KID_MISC, kernel, grid, dim3(256), 0, st, op.src, op.ld, op.rows, op.K, rows_pad, KB, (u32x4_t*)dst, op.row_mx, op.col_mx);
  };
  if (NP == 3 && !op.row_mx) return hipErrorInvalidValue;
  if (op.trans) return NP == 3 ? go(k_pack_x3_t<3>) : NP == 2 ? go(k_pack_x3_t<2>) : go(k_pack_x3_t<1>);
  return NP == 3 ? go(k_pack_x3_max) : NP == 2 ? go(k_pack_x3<2>) : go(k_pack_x3<1>);
}
// Tile, grid and split of a product with `rows` x `cols` outputs and KB k steps in stages of `stage`, all_rows and all_KB of them had no
// row been left out (x3_split, x3_split_packed in ranges.h).
struct X3Grid { int TJ, splits, per_split; dim3 grid; };
X3Grid x3_grid(int NP, int rows, int cols, int KB, int all_rows, int all_KB, int stage, size_t parts_cap) {
  const X3Split s = x3_split_packed(NP, rows, cols, KB, all_rows, all_KB, stage, parts_cap);
  return X3Grid{s.TJ, s.parts, s.per_part, dim3(raster_grid((cols + kGM - 1) / kGM, (rows + kGM * s.TJ - 1) / (kGM * s.TJ)), 1, s.parts)};
}
hipError_t x3_sum_parts(const X3Bufs& bufs, int splits, size_t n, float beta, const float* Cin, float* C, hipStream_t st) {
  return launch(KID_MISC, k_sum_parts, dim3((unsigned)((n + 1023) / 1024)), dim3(256), 0, st, (const float*)bufs.parts, splits, n, beta,
                Cin, C);
}
// C[M, N] = beta C + op(A) op(B)^T-style product of two operands given row-wise over the same K; an operand packed earlier
// (a_packed, b_packed) is used as it is.  The tokens are A's rows, or (over_tokens) what is contracted over
hipError_t gemm_x3(const X3Op& A, const X3Op& B, float* C, const float* Cin, int ldc, float beta, const X3Bufs& bufs, hipStream_t st,
                   const void* b_packed = nullptr, bool split_ok = true, const void* a_packed = nullptr, bool over_tokens = false) {
  if (A.K != B.K || A.rows <= 0 || B.rows <= 0 || A.K <= 0 || (bufs.NP == 3 && (!A.row_mx || !B.row_mx))) return hipErrorInvalidValue;
  hipError_t e;
  if (!a_packed && (e = x3_pack(A, bufs.a, bufs.a_cap, bufs.NP, st)) != hipSuccess) return e;
  if (!b_packed && (e = x3_pack(B, bufs.b, bufs.b_cap, bufs.NP, st)) != hipSuccess) return e;
  const u32x4_t* pa_ = (const u32x4_t*)(a_packed ? a_packed : bufs.a);
  const u32x4_t* pb_ = (const u32x4_t*)(b_packed ? b_packed : bufs.b);
  const int KB = x3_steps(A.K);
  const int all_rows = over_tokens ? A.rows : A.rows + bufs.left_out, all_KB = over_tokens ? x3_steps(A.K + bufs.left_out) : KB;
  const X3Grid g = x3_grid(bufs.NP, A.rows, B.rows, KB, all_rows, all_KB, x3_stage(bufs.NP), split_ok && ldc == B.rows ? bufs.parts_cap : 0);
  float* out = g.splits > 1 ? bufs.parts : C;
  const size_t c_split = g.splits > 1 ? (size_t)A.rows * B.rows : 0;
  const float b_ = g.splits > 1 ? 0.f : beta;
  auto go = [&](auto kernel) {
    return launch(KID_GEMM_GENERIC, kernel, g.grid, dim3(256), 0, st, pa_, pb_, out, Cin, ldc, A.rows, B.rows, KB, b_, g.per_split, c_split,
                  A.row_mx, B.row_mx);
  };
  if (bufs.NP == 3) e = g.TJ == 2 ? go(k_gemm_x3<3, 2>) : go(k_gemm_x3<3, 1>);
  else if (bufs.NP == 2) e = g.TJ == 2 ? go(k_gemm_x3<2, 2>) : go(k_gemm_x3<2, 1>);
  else e = g.TJ == 2 ? go(k_gemm_x3<1, 2>) : go(k_gemm_x3<1, 1>);
  if (e != hipSuccess || g.splits == 1) return e;
  return x3_sum_parts(bufs, g.splits, (size_t)A.rows * B.rows, beta, Cin, C, st);
}
// C[M, N] = beta C + A^T B, A [K, M] and B [K, N] in fp32
hipError_t gemm_x3_tn(const float* A, int lda, const float* B, int ldb, float* C, int M, int N, int K, float beta,
                      const X3Bufs& bufs, hipStream_t st, const uint32_t* amx, const uint32_t* bmx) {   // maxima of their columns
  if (M <= 0 || N <= 0 || K <= 0 || (bufs.NP == 3 && (!amx || !bmx))) return hipErrorInvalidValue;
  const int KB = (K + 15) / 16;
  const X3Grid g = x3_grid(bufs.NP, M, N, KB, M, (K + bufs.left_out + 15) / 16, x3_tn_stage(bufs.NP), bufs.parts_cap);
  float* out = g.splits > 1 ? bufs.parts : C;
  const size_t c_split = g.splits > 1 ? (size_t)M * N : 0;
  const float b_ = g.splits > 1 ? 0.f : beta;
  auto go = [&](auto kernel) {
    return launch(KID_GEMM_GENERIC, kernel, g.grid, dim3(256), 0, st, A, lda, B, ldb, out, N, M, N, K, b_, g.per_split * 16, c_split,
                  amx, bmx);
  };
  hipError_t e;
  if (bufs.NP == 3) e = g.TJ == 2 ? go(k_gemm_x3_tn<3, 2>) : go(k_gemm_x3_tn<3, 1>);
  else if (bufs.NP == 2) e = g.TJ == 2 ? go(k_gemm_x3_tn<2, 2>) : go(k_gemm_x3_tn<2, 1>);
  else e = g.TJ == 2 ? go(k_gemm_x3_tn<1, 2>) : go(k_gemm_x3_tn<1, 1>);
  if (e != hipSuccess || g.splits == 1) return e;
  return x3_sum_parts(bufs, g.splits, (size_t)M * N, beta, C, C, st);
}

template <int TA, int TB>
hipError_t sgemm(const float* A, int lda, const float* B, int ldb, float* C, int ldc, int M, int N, int K, float beta,
                 hipStream_t st, const Batch& bt = Batch()) {
  if (M <= 0 || N <= 0 || K <= 0 || bt.count <= 0 || bt.count > 65535) return hipErrorInvalidValue;
  if (bt.kseg > 0 && (bt.kseg % kGK != 0 || K % bt.kseg != 0)) return hipErrorInvalidValue;
  const long strides = bt.a1 | bt.a2 | bt.b1 | bt.b2 | bt.sega | bt.segb;
  const bool aligned = ((M | N | K | lda | ldb) & 3) == 0 && (strides & 3) == 0 && (((uintptr_t)A | (uintptr_t)B) & 15) == 0;
  if (aligned && (long)M * N * bt.count >= 128 * 128) {
    const dim3 grid(raster_grid((N + kGM - 1) / kGM, (M + kGM - 1) / kGM), 1, bt.count);
    if (N <= 64)
      return launch(KID_GEMM_GENERIC, k_sgemm_mfma<TA, TB, 1>, grid, dim3(256), 0, st, A, lda, B, ldb, C, ldc, M, N, K, beta, bt);
    return launch(KID_GEMM_GENERIC, k_sgemm_mfma<TA, TB, 0>, grid, dim3(256), 0, st, A, lda, B, ldb, C, ldc, M, N, K, beta, bt);
  }
  if (bt.kseg > 0) return hipErrorInvalidValue;   // the vector-ALU kernel has no segmented contraction
  return launch(KID_GEMM_GENERIC, k_sgemm<TA, TB>, dim3((N + kTN - 1) / kTN, (M + kTM - 1) / kTM, bt.count), dim3(256), 0, st, A,
                lda, B, ldb, C, ldc, M, N, K, beta, bt);
}

__device__ __forceinline__ float block_sum256(float v, float* red) {
  v = wave_reduce_sum(v);
  __syncthreads();   // red may still be read from a previous call
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return red[0] + red[1] + red[2] + red[3];
}
__device__ __forceinline__ float block_max256(float v, float* red) {
  v = wave_reduce_max(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  return fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
}

// ---------------------------------------------------------------------------------------
// storage type <-> fp32 masters
// ---------------------------------------------------------------------------------------
__global__ void k_bf16_to_f32(const bf16* __restrict__ src, float* __restrict__ dst, size_t n) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) dst[i] = (float)src[i];
}
// Masters into the caller's tensors, a few launches for all of them (a conversion or copy per tensor: 218 launches, 3.4 ms on
// the 0.5B decoder with the gaps between them, 1.6 ms of kernels; now 0.8).  A block takes kExportBlock values of one tensor.
constexpr int kExportTasks = 96, kExportBlock = 4096;
struct ExportTask { const float* src; void* dst; size_t n; unsigned first_block, f32; };
struct ExportTasks { int n; ExportTask t[kExportTasks]; };
static_assert(sizeof(ExportTasks) + 64 <= 4096, "kernel arguments");
__global__ void __launch_bounds__(256) k_export(ExportTasks tasks) {
  int ti = 0;
  for (int end = tasks.n; end - ti > 1;) {
    const int mid = (ti + end) >> 1;
    if (blockIdx.x >= tasks.t[mid].first_block) ti = mid; else end = mid;
  }
  const ExportTask t = tasks.t[ti];
  const size_t i0 = (size_t)(blockIdx.x - t.first_block) * kExportBlock;
  const bool aligned = (((uintptr_t)t.src & 15) | ((uintptr_t)t.dst & (t.f32 ? 15 : 7))) == 0;
  if (aligned && i0 + kExportBlock <= t.n) {
    float4 v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = *(const float4*)(t.src + i0 + u * 1024 + threadIdx.x * 4);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const size_t i = i0 + u * 1024 + threadIdx.x * 4;
      if (t.f32) {
        *(float4*)((float*)t.dst + i) = v[u];
      } else {
        typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
        *(bf16x4*)((bf16*)t.dst + i) = bf16x4{(bf16)v[u].x, (bf16)v[u].y, (bf16)v[u].z, (bf16)v[u].w};
      }
    }
    return;
  }
  for (size_t i = i0 + threadIdx.x; i < t.n && i < i0 + kExportBlock; i += 256) {
    if (t.f32) ((float*)t.dst)[i] = t.src[i];
    else ((bf16*)t.dst)[i] = (bf16)t.src[i];
  }
}

// ---------------------------------------------------------------------------------------
// forward pieces
// ---------------------------------------------------------------------------------------
// token ids outside [0, V) are clamped into it (a caller's mistake must not become a wild access)
__device__ __forceinline__ int clamp_token(int t, int V) { return min(max(t, 0), V - 1); }

__global__ void __launch_bounds__(256) k_embed_rows(const int32_t* __restrict__ tokens, const float* __restrict__ embed,
                                                    float* __restrict__ h, int d, int V) {
  const size_t m = blockIdx.x;
  const float* src = embed + (size_t)clamp_token(tokens[m], V) * d;
  for (int i = threadIdx.x; i < d; i += 256) h[m * d + i] = src[i];
}

// Rows of the norms: a wave takes a row, a lane its float4s lane, lane + 64, ... (NV of them: d <= 256 NV); no
// workgroup-wide reduction, several rows in flight per compute unit.
constexpr int kNormMaxV = 8;
inline bool norm_rows_vectorised(int d) { return d % 4 == 0 && d <= 256 * kNormMaxV; }

// xn = h * rstd * gain, rstd = 1 / sqrt(mean(h^2) + eps).  Here a lane takes the values lane, lane + 64, ...: the squares are
// added as the workgroup-per-row kernel below adds them (four chains of every fourth block of 64, reduced one by one), so
// that rows of any width see the same rounding: with bf16 operands a last bit of rstd decides roundings downstream.
template <int NV, bool MX>   // MX: the rows' maxima as well
__global__ void __launch_bounds__(256) k_rmsnorm_fwd_rows(const float* __restrict__ h, const float* __restrict__ gain, float eps,
                                                          int M, int d, float* __restrict__ xn, float* __restrict__ rstd,
                                                          uint32_t* __restrict__ row_mx) {
  const int wave = wave_index(threadIdx.x), lane = threadIdx.x & 63;
  const size_t m = (size_t)blockIdx.x * 4 + wave;
  if (m >= (size_t)M) return;
  float x[4 * NV], ss[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 4 * NV; ++i) {
    const int f = lane + 64 * i;
    x[i] = f < d ? h[m * d + f] : 0.f;
    ss[i & 3] = fmaf(x[i], x[i], ss[i & 3]);
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) ss[c] = wave_reduce_sum(ss[c]);
  const float r = 1.0f / sqrtf((ss[0] + ss[1] + ss[2] + ss[3]) / (float)d + eps);
#pragma unroll
  for (int i = 0; i < 4 * NV; ++i) {
    const int f = lane + 64 * i;
    if constexpr (MX) x[i] = x[i] * r * (f < d ? gain[f] : 0.f);
    if (f < d) xn[m * d + f] = MX ? x[i] : x[i] * r * gain[f];
  }
  if (lane == 0) rstd[m] = r;
  if constexpr (MX) {
    uint32_t mx = 0;
#pragma unroll
    for (int i = 0; i < 4 * NV; ++i) mx = max(mx, abs_bits(x[i]));
    mx = wave_max_u32(mx);
    if (lane == 0) row_mx[m] = mx;
  }
}
// Backward of the norm and the gain's gradient in one pass over dxn and h (in two they took 209 us per norm at 24576 rows
// of 896, most of it in a kernel of 96 x 4 workgroups that walked 256 rows one after the other):
//   dh (+)= rstd * gain * dxn - rstd^3 * h * mean_j(dxn_j gain_j h_j),   part[block] = sum over the block's rows of
// dxn h rstd (kNormRows rows, each wave's in order, the four waves' sums in wave order)
constexpr int kNormRows = 32;
template <int NV, bool MX>   // MX: the rows' maxima as well
__global__ void __launch_bounds__(256) k_rmsnorm_bwd_rows(const float* __restrict__ dxn, const float* __restrict__ h,
                                                          const float* __restrict__ rstd, const float* __restrict__ gain, int M,
                                                          int d, float* __restrict__ dh, int accumulate, float* __restrict__ part,
                                                          uint32_t* __restrict__ row_mx) {
  __shared__ float4 red[4][NV * 64];
  const int wave = wave_index(threadIdx.x), lane = threadIdx.x & 63;
  float4 g[NV], dg[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int f = 4 * (lane + 64 * i);
    g[i] = f < d ? *(const float4*)(gain + f) : make_float4(0.f, 0.f, 0.f, 0.f);
    dg[i] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  const int m1 = min(M, ((int)blockIdx.x + 1) * kNormRows);
  for (int m = blockIdx.x * kNormRows + wave; m < m1; m += 4) {
    float4 x[NV], y[NV], o[NV];
    float dot = 0.f;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int f = 4 * (lane + 64 * i);
      const size_t at = (size_t)m * d + f;
      x[i] = o[i] = y[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (f < d) {
        x[i] = *(const float4*)(dxn + at);
        y[i] = *(const float4*)(h + at);
        if (accumulate) o[i] = *(const float4*)(dh + at);
      }
    }
#pragma unroll
    for (int i = 0; i < NV; ++i)
      dot = fmaf(x[i].x * g[i].x, y[i].x, fmaf(x[i].y * g[i].y, y[i].y, fmaf(x[i].z * g[i].z, y[i].z, fmaf(x[i].w * g[i].w, y[i].w, dot))));
    dot = wave_reduce_sum(dot);
    const float r = rstd[m], c = r * r * r * dot / (float)d;
    uint32_t mx = 0;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int f = 4 * (lane + 64 * i);
      dg[i].x = fmaf(x[i].x * y[i].x, r, dg[i].x); dg[i].y = fmaf(x[i].y * y[i].y, r, dg[i].y);
      dg[i].z = fmaf(x[i].z * y[i].z, r, dg[i].z); dg[i].w = fmaf(x[i].w * y[i].w, r, dg[i].w);
      if (f < d) {
        const float4 v = make_float4(o[i].x + (r * g[i].x * x[i].x - c * y[i].x), o[i].y + (r * g[i].y * x[i].y - c * y[i].y),
                                     o[i].z + (r * g[i].z * x[i].z - c * y[i].z), o[i].w + (r * g[i].w * x[i].w - c * y[i].w));
        *(float4*)(dh + (size_t)m * d + f) = v;
        if constexpr (MX) mx = max(max(max(mx, abs_bits(v.x)), max(abs_bits(v.y), abs_bits(v.z))), abs_bits(v.w));
      }
    }
    if constexpr (MX) {
      mx = wave_max_u32(mx);
      if (lane == 0) row_mx[m] = mx;
    }
  }
#pragma unroll
  for (int i = 0; i < NV; ++i) red[wave][lane + 64 * i] = dg[i];
  __syncthreads();
  for (int e = threadIdx.x; 4 * e < d; e += 256) {
    float4 s = red[0][e];
#pragma unroll
    for (int w = 1; w < 4; ++w) { s.x += red[w][e].x; s.y += red[w][e].y; s.z += red[w][e].z; s.w += red[w][e].w; }
    *(float4*)(part + (size_t)blockIdx.x * d + 4 * e) = s;
  }
}
// dgain = (accumulate: dgain +) the partial sums: 16 columns per workgroup, 16 threads per column take parts k, k + 16, ...;
// added in that order
__global__ void __launch_bounds__(256) k_gain_sum(const float* __restrict__ part, int n_part, int d, int accumulate,
                                                  float* __restrict__ dgain) {
  __shared__ float red[16][17];
  const int c = threadIdx.x & 15, k = threadIdx.x >> 4, i = blockIdx.x * 16 + c;
  float s = 0.f;
  if (i < d) {
#pragma unroll 8
    for (int p = k; p < n_part; p += 16) s += part[(size_t)p * d + i];
  }
  red[k][c] = s;
  __syncthreads();
  if (k == 0 && i < d) {
    for (int j = 1; j < 16; ++j) s += red[j][c];
    dgain[i] = accumulate ? dgain[i] + s : s;
  }
}

// The same for rows that do not come in float4s: one workgroup per row
__global__ void __launch_bounds__(256) k_rmsnorm_fwd(const float* __restrict__ h, const float* __restrict__ gain, float eps,
                                                     int d, float* __restrict__ xn, float* __restrict__ rstd) {
  __shared__ float red[4];
  const size_t m = blockIdx.x;
  float ss = 0.f;
  for (int i = threadIdx.x; i < d; i += 256) { const float v = h[m * d + i]; ss = fmaf(v, v, ss); }
  ss = block_sum256(ss, red);
  const float r = 1.0f / sqrtf(ss / (float)d + eps);
  if (threadIdx.x == 0) rstd[m] = r;
  for (int i = threadIdx.x; i < d; i += 256) xn[m * d + i] = h[m * d + i] * r * gain[i];
}
template <typename F> hipError_t with_norm_width(int d, F&& f) {   // f(number of float4s per lane)
  if (d <= 256) return f(std::integral_constant<int, 1>());
  if (d <= 512) return f(std::integral_constant<int, 2>());
  if (d <= 1024) return f(std::integral_constant<int, 4>());
  return f(std::integral_constant<int, kNormMaxV>());
}
hipError_t row_max(const float* x, int rows, int K, uint32_t* out, hipStream_t st) {   // of a matrix whose writer does not leave them
  RowMaxTasks t;
  t.n = 1;
  t.t[0] = RowMaxTask{x, out, rows, K, 0};
  return launch(KID_MISC, k_row_max, dim3((rows + 3) / 4), dim3(256), 0, st, t);
}
hipError_t rmsnorm_fwd(const float* h, const float* gain, float eps, int M, int d, float* xn, float* rstd, uint32_t* row_mx, hipStream_t st) {
  if (!norm_rows_vectorised(d)) {
    const hipError_t e = launch(KID_RMSNORM, k_rmsnorm_fwd, dim3(M), dim3(256), 0, st, h, gain, eps, d, xn, rstd);
    return e != hipSuccess || !row_mx ? e : row_max(xn, M, d, row_mx, st);
  }
  return with_norm_width(d, [&](auto nv) {
    constexpr int NV = decltype(nv)::value;
    return launch(KID_RMSNORM, row_mx ? k_rmsnorm_fwd_rows<NV, true> : k_rmsnorm_fwd_rows<NV, false>, dim3((M + 3) / 4), dim3(256), 0, st, h,
                  gain, eps, M, d, xn, rstd, row_mx);
  });
}

// Rotary embedding in place on the query and key heads of qkv[M, (Hq + 2 Hkv) hd]; position = pos[row], or row % T without it.
// dir = +1 rotates by the angle, -1 by its negative (the transpose: what the backward pass applies).
__global__ void k_rope(float* __restrict__ qkv, const float2* __restrict__ rope, int T, const int* __restrict__ pos, int n_rot_heads,
                       int hd, int row_len, float dir, size_t total) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= total) return;
  const int half = hd >> 1;
  const int i = (int)(idx % half);
  const int head = (int)((idx / half) % n_rot_heads);
  const size_t m = idx / ((size_t)half * n_rot_heads);
  const float2 cs = rope[(pos ? (size_t)pos[m] : m % T) * half + i];
  float* p = qkv + m * row_len + (size_t)head * hd + i;
  const float x1 = p[0], x2 = p[half], s = cs.y * dir;
  p[0] = x1 * cs.x - x2 * s;
  p[half] = x2 * cs.x + x1 * s;
}

// Causal grouped-query attention through batched GEMMs: scores[s, h] = Q_h K^T (T x T per sequence and
// query head), the row kernels below, out = P V.  Row r = (s * Hq + h) * T + i of the score buffer.
// k_softmax_causal: in place, p_ij = softmax_j(scale * s_ij) over j <= i, 0 for j > i; lse[r] = log sum_j exp(scale * s_ij).
__global__ void __launch_bounds__(64) k_softmax_causal(float* __restrict__ sc, float* __restrict__ lse, int T, float scale) {
  const size_t r = blockIdx.x;
  const int i = (int)(r % T), lane = threadIdx.x;
  float* row = sc + r * T;
  float mx = -INFINITY;
  for (int j = lane; j <= i; j += 64) mx = fmaxf(mx, row[j] * scale);
  mx = wave_reduce_max(mx);
  float sum = 0.f;
  for (int j = lane; j <= i; j += 64) sum += expf(row[j] * scale - mx);
  sum = wave_reduce_sum(sum);
  const float l = mx + logf(sum);
  if (lane == 0) lse[r] = l;
  for (int j = lane; j < T; j += 64) row[j] = (j <= i) ? expf(row[j] * scale - l) : 0.f;
}
// the same probabilities from kept log-sum-exps (backward pass): p_ij = exp(scale * s_ij - lse[r]), 0 for j > i
__global__ void k_probs_from_lse(float* __restrict__ sc, const float* __restrict__ lse, int T, float scale, size_t total) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= total) return;
  const size_t r = idx / T;
  const int j = (int)(idx % T), i = (int)(r % T);
  sc[idx] = (j <= i) ? expf(sc[idx] * scale - lse[r]) : 0.f;
}

__device__ __forceinline__ float swiglu(float g, float u) { return g / (1.0f + expf(-g)) * u; }
// act = silu(gate) * up from gu[M, 2F] (gate columns first).  Workgroup (x, y): columns of row y, four per thread where F
// allows it.
// row_mx, if given: the row's maximum.
__device__ __forceinline__ uint32_t abs_bits4(const float4& v) { return max(max(abs_bits(v.x), abs_bits(v.y)), max(abs_bits(v.z), abs_bits(v.w))); }
__global__ void k_swiglu_fwd4(const float* __restrict__ gu, float* __restrict__ act, int F, uint32_t* __restrict__ row_mx) {
  const int f = (blockIdx.x * 256 + threadIdx.x) * 4;
  uint32_t mx = 0;
  if (f < F) {
    const float* row = gu + (size_t)blockIdx.y * 2 * F + f;
    const float4 g = *(const float4*)row, u = *(const float4*)(row + F);
    float4 o;
    o.x = swiglu(g.x, u.x); o.y = swiglu(g.y, u.y); o.z = swiglu(g.z, u.z); o.w = swiglu(g.w, u.w);
    *(float4*)(act + (size_t)blockIdx.y * F + f) = o;
    mx = abs_bits4(o);
  }
  if (!row_mx) return;
  mx = wave_max_u32(mx);
  if ((threadIdx.x & 63) == 0) atomicMax(row_mx + blockIdx.y, mx);
}
// The same straight into the packed operand of the down projection, F % 64 == 0: act itself is not stored (the backward pass
// makes its other packed form again, k_swiglu_bwd_pack).  64 tokens x 64 features per workgroup, bound by its bytes.  us a
// layer of the 0.5B decoder for act and its packing before, and now: 21 x 301 tokens, one piece 61 + 39, 52 (5.9 TB/s).
template <int NP>
__global__ void __launch_bounds__(256) k_swiglu_fwd_pack(const float* __restrict__ gu, int M, int F, int KB, u32x4_t* __restrict__ dst,
                                                         uint32_t* /*row_mx*/) {
  static_assert(NP < 3, "three pieces: k_swiglu_fwd_pack_rows");
  const int f0 = blockIdx.x * 64, m0 = blockIdx.y * 64;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int c = (threadIdx.x & 7) * 8, m = m0 + (threadIdx.x >> 3) + 32 * i;
    float x[8];
    if (m < M) {
      const float* gp = gu + (size_t)m * 2 * F + f0 + c;
      float g[8], u[8];
      *(float4*)g = *(const float4*)gp; *(float4*)(g + 4) = *(const float4*)(gp + 4);
      *(float4*)u = *(const float4*)(gp + F); *(float4*)(u + 4) = *(const float4*)(gp + F + 4);
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = swiglu(g[e], u[e]);
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = 0.f;
    }
    x3_store<NP>(dst, KB, m, (f0 + c) >> 3, x, 1.f);
  }
}
// The same with three pieces, whose scales come from the rows' maxima: 4 tokens x all features per workgroup, whose threads keep their
// NI octets of act in registers between the maxima and the packing (NI 0: rows too wide for that are read twice).  A bound from
// gate's and up's maxima would need no row at once, but silu makes it as loose as gates are negative (2^20 with gates around -16).
// us a layer of the 0.5B decoder with rows read twice (8 tokens per workgroup) and now: 64 x 384 tokens 482, 338; 21 x 301 143, 90; 7 x
// 141 30, 12.5.
constexpr int kActRows = 4, kActStep = 512 / kActRows * 8;   // rows of a workgroup; features of its threads' one octet each
template <int NI>
__global__ void __launch_bounds__(512) k_swiglu_fwd_pack_rows(const float* __restrict__ gu, int M, int F, int KB, u32x4_t* __restrict__ dst,
                                                              uint32_t* __restrict__ row_mx) {
  constexpr int R = kActRows;
  __shared__ uint32_t red[8][R];
  const int wave = wave_index(threadIdx.x), lane = threadIdx.x & 63, r = lane % R, m = blockIdx.x * R + r, c0 = (wave * (64 / R) + lane / R) * 8;
  const float* row = gu + (size_t)min(m, M - 1) * 2 * F;
  auto act = [&](int f, float (&x)[8]) __attribute__((always_inline)) {
    float g[8], u[8];
    *(float4*)g = *(const float4*)(row + f); *(float4*)(g + 4) = *(const float4*)(row + f + 4);
    *(float4*)u = *(const float4*)(row + F + f); *(float4*)(u + 4) = *(const float4*)(row + F + f + 4);
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = m < M ? swiglu(g[e], u[e]) : 0.f;
  };
  float kept[NI ? NI : 1][8];
  uint32_t mx = 0;
  auto seen = [&](const float (&x)[8]) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < 8; ++e) mx = max(mx, abs_bits(x[e]));
  };
  if constexpr (NI > 0) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
      if (c0 + i * kActStep < F) { act(c0 + i * kActStep, kept[i]); seen(kept[i]); }
  } else {
#pragma unroll 2
    for (int f = c0; f < F; f += kActStep) { act(f, kept[0]); seen(kept[0]); }
  }
  mx = max(mx, (uint32_t)__builtin_amdgcn_mov_dpp((int)mx, 0x124, 0xF, 0xF, true));   // rotated by 4 lanes of 16
  mx = max(mx, (uint32_t)__builtin_amdgcn_mov_dpp((int)mx, 0x128, 0xF, 0xF, true));   // by 8
  mx = max_u32_xor32(max_u32_xor16(mx));
  if (lane < R) red[wave][lane] = mx;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 8; ++w) mx = max(mx, red[w][r]);
  if (threadIdx.x < R && m < M) row_mx[m] = mx;
  const float scale = row_scale(mx);
  if constexpr (NI > 0) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
      if (c0 + i * kActStep < F) x3_store<3>(dst, KB, m, (c0 + i * kActStep) >> 3, kept[i], scale);
  } else {
#pragma unroll 2
    for (int f = c0; f < F; f += kActStep) { act(f, kept[0]); x3_store<3>(dst, KB, m, f >> 3, kept[0], scale); }
  }
}
__global__ void k_swiglu_fwd(const float* __restrict__ gu, float* __restrict__ act, int F, size_t total) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= total) return;
  const size_t m = idx / F;
  const int f = (int)(idx % F);
  act[idx] = swiglu(gu[m * 2 * F + f], gu[m * 2 * F + F + f]);
}

// ---------------------------------------------------------------------------------------
// LM head rows.  Row r = (s, t) of the final-normed states predicts tokens[s, t + 1].  One workgroup per row
// of a chunk of logits: log-sum-exp, logp_new[s, t + 1] = z[target] - lse, the token's surrogate gradient
// w = d loss / d logp (it needs only this token's log-probs, its sequence's advantage and the number of
// masked tokens), then in place  logits <- d loss / d logits = w (onehot(target) - softmax).
// Rows whose target is not masked, and the last row of every sequence, become zero.
// ---------------------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_count_mask(const uint8_t* __restrict__ mask, size_t n, long long* __restrict__ out) {
  __shared__ int part[256];
  int c = 0;
  for (size_t i = threadIdx.x; i < n; i += 256) c += mask[i] != 0;
  part[threadIdx.x] = c;
  __syncthreads();
  if (threadIdx.x == 0) {
    long long t = 0;
    for (int j = 0; j < 256; ++j) t += part[j];
    *out = t;
  }
}
// Row k of `logits` belongs to token r = rows[k] of the batch (position r % T of sequence r / T), which predicts the
// masked token at r + 1 (the list holds exactly those rows).  In place: logits -> d loss / d logits.
// Two passes over the row, each in float4s: log-sum-exp on a running maximum, then the gradient (the second pass finds the
// row in the caches).  In three passes of single floats by 256 threads: 2.65 ms per chunk of 4352 x 151936 logits.
constexpr int kLogpThreads = 512;
__global__ void __launch_bounds__(kLogpThreads) k_logp_dlogits(float* __restrict__ logits, int V, const int* __restrict__ rows, int T,
                                                               const int32_t* __restrict__ tokens, const uint8_t* __restrict__ mask,
                                                               const float* __restrict__ logp_old, const float* __restrict__ adv,
                                                               float eps_low, float eps_high, const long long* __restrict__ n_masked,
                                                               float* __restrict__ logp_new, uint32_t* __restrict__ row_mx) {
  constexpr int NT = kLogpThreads;
  __shared__ float red_m[NT / 64], red_l[NT / 64];
  __shared__ uint32_t red_x[NT / 64];
  const int r = rows[blockIdx.x];
  const int t = r % T;
  float* z = logits + (size_t)blockIdx.x * V;
  const int V4 = (V & 3) == 0 ? V >> 2 : 0;   // rows of whole float4s (the buffer is aligned), else value by value
  if (t == T - 1 || !mask[r + 1]) {   // not in a well-formed list; uniform over the workgroup
    for (int v = threadIdx.x; v < V; v += NT) z[v] = 0.f;
    if (threadIdx.x == 0) row_mx[blockIdx.x] = 0;
    return;
  }
  float m = -INFINITY, l = 0.f;
  auto add = [&](float x) {
    if (x > m) { l = l * expf(m - x) + 1.f; m = x; } else { l += expf(x - m); }
  };
  if (V4) {
    for (int v0 = threadIdx.x; v0 < V4; v0 += 4 * NT) {
      float4 x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        x[u] = v0 + u * NT < V4 ? ((const float4*)z)[v0 + u * NT] : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
      float mx = m;
#pragma unroll
      for (int u = 0; u < 4; ++u) mx = fmaxf(mx, fmaxf(fmaxf(x[u].x, x[u].y), fmaxf(x[u].z, x[u].w)));
      if (mx == -INFINITY) continue;
      if (mx > m) { l *= expf(m - mx); m = mx; }
#pragma unroll
      for (int u = 0; u < 4; ++u) l += (expf(x[u].x - m) + expf(x[u].y - m)) + (expf(x[u].z - m) + expf(x[u].w - m));
    }
  } else {
    for (int v = threadIdx.x; v < V; v += NT) add(z[v]);
  }
  const float mw = wave_reduce_max(m);
  l = wave_reduce_sum(m == -INFINITY ? 0.f : l * expf(m - mw));
  if ((threadIdx.x & 63) == 0) { red_m[threadIdx.x >> 6] = mw; red_l[threadIdx.x >> 6] = l; }
  __syncthreads();
  float mx = red_m[0];
#pragma unroll
  for (int w = 1; w < NT / 64; ++w) mx = fmaxf(mx, red_m[w]);
  float sum = 0.f;
#pragma unroll
  for (int w = 0; w < NT / 64; ++w) sum += red_m[w] == -INFINITY ? 0.f : red_l[w] * expf(red_m[w] - mx);
  const float lse = mx + logf(sum);
  const int target = clamp_token(tokens[r + 1], V);
  const float lp = z[target] - lse;
  float rho; bool active;
  const float a = adv[r / T];
  surrogate_term(lp, logp_old[r + 1], a, eps_low, eps_high, rho, active);
  const float w = surrogate_dlogp(a, rho, active, *n_masked);
  __syncthreads();   // every thread has read z[target]
  if (threadIdx.x == 0) logp_new[r + 1] = lp;
  uint32_t gmax = 0;
  auto grad = [&](float x, int v) {
    const float g = w == 0.f ? 0.f : w * ((v == target ? 1.f : 0.f) - expf(x - lse));
    gmax = max(gmax, abs_bits(g));
    return g;
  };
  if (V4) {
    for (int v0 = threadIdx.x; v0 < V4; v0 += 4 * NT) {
      float4 x[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) x[u] = ((const float4*)z)[min(v0 + u * NT, V4 - 1)];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int v = v0 + u * NT;
        if (v < V4) ((float4*)z)[v] = make_float4(grad(x[u].x, 4 * v), grad(x[u].y, 4 * v + 1), grad(x[u].z, 4 * v + 2), grad(x[u].w, 4 * v + 3));
      }
    }
  } else {
    for (int v = threadIdx.x; v < V; v += NT) z[v] = grad(z[v], v);
  }
  gmax = wave_max_u32(gmax);
  if ((threadIdx.x & 63) == 0) red_x[threadIdx.x >> 6] = gmax;
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int w_ = 1; w_ < NT / 64; ++w_) gmax = max(gmax, red_x[w_]);
    row_mx[blockIdx.x] = gmax;
  }
}

// dst[k] = src[rows[k]] (gather; dst_mx[k] = src_mx[rows[k]] with it) or dst[rows[k]] = src[k] (scatter): rows of d floats, one
// workgroup per listed row
__global__ void __launch_bounds__(256) k_move_rows(const float* __restrict__ src, const int* __restrict__ rows, int d, int scatter,
                                                   float* __restrict__ dst, const uint32_t* __restrict__ src_mx,
                                                   uint32_t* __restrict__ dst_mx) {
  const size_t k = blockIdx.x, r = (size_t)rows[blockIdx.x];
  const float* a = src + (scatter ? k : r) * d;
  float* b = dst + (scatter ? r : k) * d;
  for (int i = threadIdx.x; i < d; i += 256) b[i] = a[i];
  if (src_mx && threadIdx.x == 0) dst_mx[k] = src_mx[r];
}
// out = beta in + sum over the parts, in part order (in may be out)
__global__ void k_sum_parts(const float* __restrict__ part, int n_part, size_t n, float beta, const float* in, float* out) {
  const size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4;
  if (i >= n) return;
  if (n % 4 != 0 || (((uintptr_t)out | (uintptr_t)in) & 15) != 0) {
    for (size_t k = i; k < min(i + 4, n); ++k) {
      float s = beta != 0.f ? beta * in[k] : 0.f;
      for (int p = 0; p < n_part; ++p) s += part[(size_t)p * n + k];
      out[k] = s;
    }
    return;
  }
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  if (beta != 0.f) {
    s = *(const float4*)(in + i);
    s.x *= beta; s.y *= beta; s.z *= beta; s.w *= beta;
  }
#pragma unroll 4
  for (int p = 0; p < n_part; ++p) {
    const float4 v = *(const float4*)(part + (size_t)p * n + i);
    s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
  }
  *(float4*)(out + i) = s;
}

// ---------------------------------------------------------------------------------------
// backward pieces
// ---------------------------------------------------------------------------------------
// RMSNorm: dh (+)= rstd * gain * dxn - rstd^3 * h * mean_j(dxn_j gain_j h_j); one workgroup per row.
__global__ void __launch_bounds__(256) k_rmsnorm_bwd(const float* __restrict__ dxn, const float* __restrict__ h,
                                                     const float* __restrict__ rstd, const float* __restrict__ gain, int d,
                                                     float* __restrict__ dh, int accumulate) {
  __shared__ float red[4];
  const size_t m = blockIdx.x;
  float dot = 0.f;
  for (int i = threadIdx.x; i < d; i += 256) dot = fmaf(dxn[m * d + i] * gain[i], h[m * d + i], dot);
  dot = block_sum256(dot, red);
  const float r = rstd[m];
  const float c = r * r * r * dot / (float)d;
  for (int i = threadIdx.x; i < d; i += 256) {
    const float g = r * gain[i] * dxn[m * d + i] - c * h[m * d + i];
    dh[m * d + i] = accumulate ? dh[m * d + i] + g : g;
  }
}
// d gain_i = sum_m dxn[m, i] h[m, i] rstd[m]: partial sums over blocks of 256 rows, then over the blocks in order
__global__ void __launch_bounds__(256) k_gain_grad_partial(const float* __restrict__ dxn, const float* __restrict__ h,
                                                           const float* __restrict__ rstd, int M, int d,
                                                           float* __restrict__ part) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= d) return;
  const int m0 = blockIdx.y * 256, m1 = min(M, m0 + 256);
  float s = 0.f;
  for (int m = m0; m < m1; ++m) s = fmaf(dxn[(size_t)m * d + i] * h[(size_t)m * d + i], rstd[m], s);
  part[(size_t)blockIdx.y * d + i] = s;
}
// column sums of x[M, N] over blocks of 256 rows (bias gradients); k_gain_grad_finish adds the blocks up in order
__global__ void __launch_bounds__(256) k_colsum_partial(const float* __restrict__ x, int M, int N, float* __restrict__ part) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= N) return;
  const int m0 = blockIdx.y * 256, m1 = min(M, m0 + 256);
  float s = 0.f;
  for (int m = m0; m < m1; ++m) s += x[(size_t)m * N + i];
  part[(size_t)blockIdx.y * N + i] = s;
}
__global__ void __launch_bounds__(256) k_gain_grad_finish(const float* __restrict__ part, int n_part, int d, int accumulate,
                                                          float* __restrict__ dgain) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= d) return;
  float s = 0.f;
  for (int p = 0; p < n_part; ++p) s += part[(size_t)p * d + i];
  dgain[i] = accumulate ? dgain[i] + s : s;
}

__device__ __forceinline__ void swiglu_grad(float g, float u, float da, float& dg, float& du) {
  const float sg = 1.0f / (1.0f + expf(-g));
  dg = da * u * sg * (1.0f + g * (1.0f - sg));
  du = da * g * sg;
}
__global__ void k_swiglu_bwd4(const float* __restrict__ dact, const float* __restrict__ gu, float* __restrict__ dgu, int F,
                              uint32_t* __restrict__ row_mx) {
  const int f = (blockIdx.x * 256 + threadIdx.x) * 4;
  uint32_t mx = 0;
  if (f < F) {
    const float* row = gu + (size_t)blockIdx.y * 2 * F + f;
    float* out = dgu + (size_t)blockIdx.y * 2 * F + f;
    const float4 g = *(const float4*)row, u = *(const float4*)(row + F), da = *(const float4*)(dact + (size_t)blockIdx.y * F + f);
    float4 dg, du;
    swiglu_grad(g.x, u.x, da.x, dg.x, du.x); swiglu_grad(g.y, u.y, da.y, dg.y, du.y);
    swiglu_grad(g.z, u.z, da.z, dg.z, du.z); swiglu_grad(g.w, u.w, da.w, dg.w, du.w);
    *(float4*)out = dg;
    *(float4*)(out + F) = du;
    mx = max(abs_bits4(dg), abs_bits4(du));
  }
  if (!row_mx) return;
  mx = wave_max_u32(mx);
  if ((threadIdx.x & 63) == 0) atomicMax(row_mx + blockIdx.y, mx);
}
// Maxima of d gate and d up by rows of tokens (of both) and by rows of features, and of act by rows of features, F % 64 == 0: the
// scales of k_swiglu_bwd_pack with three pieces, before it, since a column's is known when all rows are.  256 tokens x 64 features per
// workgroup, bound by its bytes: 64 x 384 tokens of the 0.5B decoder 310 us a layer (4.6 TB/s; two blocks of rows in flight instead of four
// 317), 21 x 301 86, 7 x 141 18.
struct SwigluMax { uint32_t *dgu_r, *dgu_c, *act_c; };
__global__ void __launch_bounds__(256) k_swiglu_bwd_max(const float* __restrict__ dact, const float* __restrict__ gu, int M, int F, SwigluMax mx) {
  const int c = (threadIdx.x & 7) * 8, f = blockIdx.x * 64 + c;
  uint32_t cg[8] = {}, cu[8] = {}, ca[8] = {};
#pragma unroll 4
  for (int i = 0; i < 8; ++i) {
    const int m = blockIdx.y * 256 + 32 * i + (threadIdx.x >> 3);
    uint32_t rm = 0;
    if (m < M) {
      const float *gp = gu + (size_t)m * 2 * F + f, *dp = dact + (size_t)m * F + f;
      float g[8], u[8], da[8];
      *(float4*)g = *(const float4*)gp; *(float4*)(g + 4) = *(const float4*)(gp + 4);
      *(float4*)u = *(const float4*)(gp + F); *(float4*)(u + 4) = *(const float4*)(gp + F + 4);
      *(float4*)da = *(const float4*)dp; *(float4*)(da + 4) = *(const float4*)(dp + 4);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float dg, du;
        swiglu_grad(g[e], u[e], da[e], dg, du);
        cg[e] = max(cg[e], abs_bits(dg));
        cu[e] = max(cu[e], abs_bits(du));
        ca[e] = max(ca[e], abs_bits(swiglu(g[e], u[e])));
        rm = max(max(rm, abs_bits(dg)), abs_bits(du));
      }
    }
    rm = max(rm, (uint32_t)__builtin_amdgcn_mov_dpp((int)rm, 0xB1, 0xF, 0xF, true));    // lane ^ 1
    rm = max(rm, (uint32_t)__builtin_amdgcn_mov_dpp((int)rm, 0x4E, 0xF, 0xF, true));    // lane ^ 2
    rm = max(rm, (uint32_t)__builtin_amdgcn_mov_dpp((int)rm, 0x141, 0xF, 0xF, true));   // lane ^ 7
    if (c == 0 && m < M) atomicMax(mx.dgu_r + m, rm);
  }
  wave_column_max<8>(cg, mx.dgu_c, f, F);
  wave_column_max<8>(cu, mx.dgu_c + F, f, F);
  wave_column_max<8>(ca, mx.act_c, f, F);
}
// The same straight into the packed operands of the two products that read it, F % 64 == 0: by rows of tokens (for the d input
// product) and by rows of features (for the weight gradients, which contract over the tokens); act, which the down
// projection's weight gradient contracts over the tokens, by rows of features as well.  Neither is stored in fp32.
// Bound by its bytes; 64 tokens x 64 features per workgroup, the tokens' octets for the second order through LDS.
// Before, dgu was written and read three times in fp32 (by the packing and, between its MFMAs, by the product over
// the tokens, which then took in twice its operands' bytes: 21 x 301 tokens, one piece, 297 us a layer at 0.37 PFLOP/s).
// act's packed form makes the pass longer (21 x 301 tokens, one piece 116 -> 122 us a layer) and the down projection's weight
// gradient shorter (112 -> 47).
template <int NP>
__global__ void __launch_bounds__(256) k_swiglu_bwd_pack(const float* __restrict__ dact, const float* __restrict__ gu, int M, int F,
                                                         int KB_rows, u32x4_t* __restrict__ by_rows, int KB_cols,
                                                         u32x4_t* __restrict__ by_cols, u32x4_t* __restrict__ act_by_cols,
                                                         SwigluMax mx) {
  __shared__ float tile[3][64][65];
  const int f0 = blockIdx.x * 64, m0 = blockIdx.y * 64;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = (threadIdx.x >> 3) + 32 * i, c = (threadIdx.x & 7) * 8, m = m0 + r;
    float dg[8], du[8], act[8];
    if (m < M) {
      const float *gp = gu + (size_t)m * 2 * F + f0 + c, *dp = dact + (size_t)m * F + f0 + c;
      float g[8], u[8], da[8];
      *(float4*)g = *(const float4*)gp; *(float4*)(g + 4) = *(const float4*)(gp + 4);
      *(float4*)u = *(const float4*)(gp + F); *(float4*)(u + 4) = *(const float4*)(gp + F + 4);
      *(float4*)da = *(const float4*)dp; *(float4*)(da + 4) = *(const float4*)(dp + 4);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        swiglu_grad(g[e], u[e], da[e], dg[e], du[e]);
        act[e] = swiglu(g[e], u[e]);   // the forward's value to the bit
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) dg[e] = du[e] = act[e] = 0.f;
    }
    const float scale = x3_scale<NP>(mx.dgu_r, min(m, M - 1));
    x3_store<NP>(by_rows, KB_rows, m, (f0 + c) >> 3, dg, scale);
    x3_store<NP>(by_rows, KB_rows, m, (F + f0 + c) >> 3, du, scale);
#pragma unroll
    for (int e = 0; e < 8; ++e) { tile[0][r][c + e] = dg[e]; tile[1][r][c + e] = du[e]; tile[2][r][c + e] = act[e]; }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    const int item = threadIdx.x + 256 * i, col = item & 63, oct = (item >> 6) & 7, which = item >> 9, k8 = (m0 >> 3) + oct;
    if (k8 >= KB_cols * 2) continue;
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = tile[which][oct * 8 + e][col];
    const int f = f0 + col;
    const int row = (which == 1 ? F : 0) + f;
    x3_store<NP>(which < 2 ? by_cols : act_by_cols, KB_cols, row, k8, x, x3_scale<NP>(which < 2 ? mx.dgu_c : mx.act_c, row));
  }
}
// dgu from dact: d gate = dact * up * sig(g) (1 + g (1 - sig(g))), d up = dact * silu(g)
__global__ void k_swiglu_bwd(const float* __restrict__ dact, const float* __restrict__ gu, float* __restrict__ dgu, int F,
                             size_t total) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= total) return;
  const size_t m = idx / F;
  const int f = (int)(idx % F);
  swiglu_grad(gu[m * 2 * F + f], gu[m * 2 * F + F + f], dact[idx], dgu[m * 2 * F + f], dgu[m * 2 * F + F + f]);
}

// ---------------------------------------------------------------------------------------
// Fused causal attention in fp32 on the matrix cores (v_mfma_f32_16x16x4_f32), for head dims 16, 32, 64, 128.
// A wave owns 16 positions of one (sequence, head) and walks the other side in tiles of 16; nothing of size
// T x T is stored.  Layouts of one 16x16x4 MFMA: A[m = lane % 16][k = lane / 16], B[k = lane / 16][n = lane % 16],
// D rows 4 (lane / 16) + v (v = 0..3), column lane % 16.  Two kinds of products:
//  * rows x rows over the head dim (scores, dP): both operands are read as float4 per lane - lane (r, g) takes
//    dims 16 w + 4 g + c of row r - and MFMA (w, c) contracts the dims {16 w + 4 g + c : g}: any assignment of dims
//    to k slots is fine as long as both operands use the same one;
//  * (head dim x positions) products over the 16 positions of the tile (P V, dS K, ...): the B operand of MFMA u
//    is the lane's own accumulator entry u of the tile just computed (position 4 g + u), the A operand is the
//    matching row of V / K / Q / dO, read as scalars (lanes along the head dim).
// qkv[M, q + 2 kv] holds rotated q, k and v; out[M, q]; lse[(s Hq + h) T + i].  A sequence is T rows; with `first` it is the rows
// first[s] .. first[s + 1] - 1 (at most T).
// ---------------------------------------------------------------------------------------
typedef float f32x4_t __attribute__((ext_vector_type(4)));

struct SeqRows { size_t row0; int n; };
__device__ __forceinline__ SeqRows seq_rows(const int* __restrict__ first, int s, int T) {
  if (!first) return SeqRows{(size_t)s * T, T};
  const int a = first[s];
  return SeqRows{(size_t)a, first[s + 1] - a};
}

template <int HD>
__device__ __forceinline__ void load_rows4(const float* __restrict__ base, size_t row_stride, int row, int g, float4 (&dst)[HD / 16]) {
#pragma unroll
  for (int w = 0; w < HD / 16; ++w) dst[w] = *(const float4*)(base + (size_t)row * row_stride + 16 * w + 4 * g);
}
__device__ __forceinline__ float f4c(const float4& v, int c) { return c == 0 ? v.x : c == 1 ? v.y : c == 2 ? v.z : v.w; }

// Rows = positions of `a`, 4 g + v; column = position of `b`, lane % 16: a b^T over the head dim, in CH chains.  Four chains have a
// quarter of the roundings at the sum's full size (the scores' rounding is most of the gradients' error where they lie hundreds
// apart; 16 sets with scores to 450: error against 64 bits 4.1e-4 -> 2.9e-4 of a tensor's largest entry).  With one and two pieces,
// whose operands' rounding is far larger and turns another last bit into another rounding downstream, one chain.
template <int HD, int CH>
__device__ __forceinline__ f32x4_t dot_rows(const float4 (&a)[HD / 16], const float4 (&b)[HD / 16]) {
  f32x4_t acc[CH];
#pragma unroll
  for (int i = 0; i < CH; ++i) acc[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int w = 0; w < HD / 16; ++w)
#pragma unroll
    for (int c = 0; c < 4; ++c)
      acc[c % CH] = __builtin_amdgcn_mfma_f32_16x16x4f32(f4c(a[w], c), f4c(b[w], c), acc[c % CH], 0, 0, 0);
  if constexpr (CH == 4) return (acc[0] + acc[1]) + (acc[2] + acc[3]);
  return acc[0];
}
// o (head dims x the 16 columns of lane % 16) += sum over the tile's positions 4 g + u of src[position][dim] * p[u];
// src rows start at `tile_base` (pointer to position 0 of the tile, this head's dims).  Which head dim an
// accumulator entry holds is free to choose (the rows of an MFMA are whatever its A operand's lanes supply):
//   head dims in multiples of 64: lane r supplies the dims 64 j + 4 r + c of a position as float4 loads, so
//     o[4 j + c][v] is dim 64 j + 16 g + 4 v + c;
//   otherwise lane r supplies dim 16 dt + r as scalars: o[dt][v] is dim 16 dt + 4 g + v.
// store_acc writes either arrangement out as float4 runs.
template <int HD>
__device__ __forceinline__ void accumulate_tile(const float* __restrict__ tile_base, size_t row_stride, int n_valid, int g, int r,
                                                const f32x4_t& p, f32x4_t (&o)[HD / 16]) {
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int pos = min(4 * g + u, n_valid - 1);   // rows past the end repeat the last one (their p is zero)
    const float* row = tile_base + (size_t)pos * row_stride;
    if constexpr (HD % 64 == 0) {
#pragma unroll
      for (int j = 0; j < HD / 64; ++j) {
        const float4 a = *(const float4*)(row + 64 * j + 4 * r);
#pragma unroll
        for (int c = 0; c < 4; ++c) o[4 * j + c] = __builtin_amdgcn_mfma_f32_16x16x4f32(f4c(a, c), p[u], o[4 * j + c], 0, 0, 0);
      }
    } else {
#pragma unroll
      for (int dt = 0; dt < HD / 16; ++dt) o[dt] = __builtin_amdgcn_mfma_f32_16x16x4f32(row[16 * dt + r], p[u], o[dt], 0, 0, 0);
    }
  }
}
template <int HD>
__device__ __forceinline__ void store_acc(float* __restrict__ row, const f32x4_t (&o)[HD / 16], int g, float mul) {
  if constexpr (HD % 64 == 0) {
#pragma unroll
    for (int j = 0; j < HD / 64; ++j)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        *(float4*)(row + 64 * j + 16 * g + 4 * v) =
            make_float4(o[4 * j][v] * mul, o[4 * j + 1][v] * mul, o[4 * j + 2][v] * mul, o[4 * j + 3][v] * mul);
  } else {
#pragma unroll
    for (int dt = 0; dt < HD / 16; ++dt)
      *(float4*)(row + 16 * dt + 4 * g) = make_float4(o[dt][0] * mul, o[dt][1] * mul, o[dt][2] * mul, o[dt][3] * mul);
  }
}

// Tiles of 16 positions, head dims in multiples of 64.  What bounded these kernels is the unit that returns loads from the L1:
// read as rows, four neighbouring lanes of a float4 load are in four rows, and it returned a lane a cycle, 64 instead of 16
// cycles per request (busy 60 - 69 % of the time, and all of the time that a compute unit had waves; the matrix cores
// 27 - 33 %), and most tiles were read twice, as rows and by columns.  Now a tile is read once, by columns - lane (r, g)
// holds chunk 16 j + r (4 dims) of the positions 4 g + u, 256 contiguous bytes per 16 lanes - which is the operand of the
// products over the positions, and goes through the wave's own LDS (chunks XORed with the row's low bits: free of bank
// conflicts both ways) for the products over the head dim; the next tile is on its way meanwhile.  Same products in the same
// order.  The grids deal the longest walks first: causal walks are 1 .. T / 16 tiles long, and with the tile index fastest
// the compute units had waves 62 % of the time.  Registers leave a SIMD four waves (forward), three (d queries) and two (d keys
// and values) at head dim 64, and two, one and one at head dim 128; limits for more spill.
// us per layer, forward / d queries / d keys and values, before and now:
//   14 heads of 64,  64 x 384 tokens: 329 / 415 / 686, 225 / 317 / 408;   21 x 301: 83 / 106 / 161, 58 / 77 / 100
//   12 heads of 128, 64 x 384 tokens: 490 / 701 / 1489, 384 / 680 / 905;   9 x 300: 76 / 105 / 183, 45 / 77 / 93
// Matrix cores busy over a launch, 64 x 384 tokens, heads of 64: 37 / 42 / 33 %, now 51 / 57 / 56 %; the rest is mostly the
// softmax's vector instructions, which a SIMD issues in turn with the MFMAs.
template <int HD> struct TileCols {
  f32x4_t x[4][HD / 64];
  unsigned off[4];   // bytes from the tile's first position to this lane's chunk of the positions 4 g + u
  __device__ __forceinline__ void stride(size_t row_stride, int g, int r) {
#pragma unroll
    for (int u = 0; u < 4; ++u) off[u] = (unsigned)((4 * g + u) * row_stride + 4 * r) * 4u;
  }
  // tile_base and n_valid are the same for the wave: a whole tile's requests need no address arithmetic
  __device__ __forceinline__ void load(const float* __restrict__ tile_base, size_t row_stride, int n_valid, int g, int r) {
    if (n_valid >= 16) {
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int j = 0; j < HD / 64; ++j) x[u][j] = *(const f32x4_t*)((const char*)tile_base + off[u] + 256 * j);
      return;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float* row = tile_base + (size_t)min(4 * g + u, n_valid - 1) * row_stride;   // rows past the end repeat the last one
#pragma unroll
      for (int j = 0; j < HD / 64; ++j) x[u][j] = *(const f32x4_t*)(row + 64 * j + 4 * r);
    }
  }
  // o += sum over the positions of this[position][dim] * p[position], as accumulate_tile
  __device__ __forceinline__ void accumulate(const f32x4_t& p, f32x4_t (&o)[HD / 16]) const {
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int j = 0; j < HD / 64; ++j)
#pragma unroll
        for (int c = 0; c < 4; ++c) o[4 * j + c] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u][j][c], p[u], o[4 * j + c], 0, 0, 0);
  }
  // as rows (load_rows4's layout), through the wave's 16 x HD floats at `area`
  __device__ __forceinline__ void rows(f32x4_t* area, int g, int r, float4 (&dst)[HD / 16]) const {
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int j = 0; j < HD / 64; ++j) area[(4 * g + u) * (HD / 4) + ((16 * j + r) ^ ((4 * g + u) & 7))] = x[u][j];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int w = 0; w < HD / 16; ++w) {
      const f32x4_t v = area[r * (HD / 4) + ((4 * w + g) ^ (r & 7))];
      dst[w] = make_float4(v[0], v[1], v[2], v[3]);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   // the next tile's values are not written before these are read
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
};
template <int HD> constexpr int tile_area() { return HD % 64 == 0 ? 16 * HD / 4 : 1; }   // float4s of LDS per wave and operand

template <int HD, int CH>
__global__ void __launch_bounds__(256, HD == 128 ? 2 : 1) k_tattn_fwd(const float* __restrict__ qkv, int T_max, const int* __restrict__ first, int hq, int hkv, float scale,
                                                   float* __restrict__ out, float* __restrict__ lse, uint32_t* __restrict__ row_mx) {
  const int wave = wave_index(threadIdx.x), lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int h = blockIdx.x, s = blockIdx.y, kvh = h / (hq / hkv);
  const int q0 = (((int)gridDim.z - 1 - (int)blockIdx.z) * 4 + wave) * 16;   // the longest walks first
  const SeqRows seq = seq_rows(first, s, T_max);
  const size_t row0 = seq.row0;
  const int T = seq.n;
  if (q0 >= T) return;
  const int qd = hq * HD, kvd = hkv * HD;
  const size_t rl = (size_t)qd + 2 * kvd;
  const float* base = qkv + row0 * rl;
  const float* qb = base + (size_t)h * HD;
  const float* kb = base + qd + (size_t)kvh * HD;
  const float* vb = kb + kvd;
  const int qi = min(q0 + r, T - 1);   // this lane's query (columns past T repeat the last one and are not stored)
  float4 qf[HD / 16];
  load_rows4<HD>(qb, rl, qi, g, qf);
  f32x4_t o[HD / 16];
#pragma unroll
  for (int dt = 0; dt < HD / 16; ++dt) o[dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float m_run = -INFINITY, l_run = 0.f;
  const int last = min(q0 + 15, T - 1);
  constexpr bool COLS = HD % 64 == 0;
  __shared__ f32x4_t area[4][tile_area<HD>()];
  TileCols<COLS ? HD : 64> kc, vc;
  if constexpr (COLS) {
    kc.stride(rl, g, r); vc.stride(rl, g, r);
    kc.load(kb, rl, min(16, T), g, r);
    vc.load(vb, rl, min(16, T), g, r);
  }
  for (int k0 = 0; k0 <= last; k0 += 16) {
    const int n_valid = min(16, T - k0), k1 = k0 + 16 <= last ? k0 + 16 : k0;   // the next tile (behind the last one: it again)
    float4 kf[HD / 16];
    if constexpr (COLS) {
      kc.rows(area[wave], g, r, kf);
      kc.load(kb + (size_t)k1 * rl, rl, min(16, T - k1), g, r);
    } else {
      load_rows4<HD>(kb, rl, min(k0 + r, T - 1), g, kf);
    }
    f32x4_t sc = dot_rows<HD, CH>(kf, qf);   // rows: keys k0 + 4 g + v; column: query qi
    float mx = -INFINITY;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int key = k0 + 4 * g + v;
      sc[v] = (key <= qi && key < T) ? sc[v] * scale : -INFINITY;
      mx = fmaxf(mx, sc[v]);
    }
    mx = max_xor32(max_xor16(mx));
    const float m_new = fmaxf(m_run, mx);        // finite: key 0 is visible to every query
    f32x4_t p;
    float ps = 0.f;
#pragma unroll
    for (int v = 0; v < 4; ++v) { p[v] = expf(sc[v] - m_new); ps += p[v]; }
    float alpha = 1.f;
    if (__builtin_amdgcn_ballot_w64(m_run != m_new) != 0) {   // the running maximum moved in some lane
      asm volatile("");   // a branch, not 16 selects
      alpha = expf(m_run - m_new);
#pragma unroll
      for (int dt = 0; dt < HD / 16; ++dt)
#pragma unroll
        for (int v = 0; v < 4; ++v) o[dt][v] *= alpha;
    }
    l_run = fmaf(l_run, alpha, ps);
    m_run = m_new;
    if constexpr (COLS) {
      vc.accumulate(p, o);
      vc.load(vb + (size_t)k1 * rl, rl, min(16, T - k1), g, r);
    } else {
      accumulate_tile<HD>(vb + (size_t)k0 * rl, rl, n_valid, g, r, p, o);
    }
  }
  l_run = sum_xor32(sum_xor16(l_run));
  const float inv = 1.0f / l_run;
  uint32_t mx = 0;
  if (row_mx) {
#pragma unroll
    for (int dt = 0; dt < HD / 16; ++dt)
#pragma unroll
      for (int v = 0; v < 4; ++v) mx = max(mx, abs_bits(o[dt][v] * inv));
    mx = max_u32_xor32(max_u32_xor16(mx));
  }
  if (q0 + r >= T) return;
  store_acc<HD>(out + (row0 + qi) * qd + (size_t)h * HD, o, g, inv);
  if (g == 0) {
    lse[((size_t)s * hq + h) * T_max + qi] = m_run + logf(l_run);
    if (row_mx) atomicMax(row_mx + row0 + qi, mx);   // the row's heads
  }
}

// Backward, queries: a wave owns 16 queries of one (sequence, head).  delta = dO . O; per key tile
//   p = exp(scale s - lse), dP = V dO^T, dS = scale p (dP - delta), dQ^T += K^T dS.
// Writes dq into dqkv's query columns and delta[(s Hq + h) T + i].
template <int HD, int CH>
__global__ void __launch_bounds__(256, HD == 64 ? 3 : 1) k_tattn_bwd_q(const float* __restrict__ qkv, const float* __restrict__ out,
                                                     const float* __restrict__ dout, const float* __restrict__ lse, int T_max,
                                                     const int* __restrict__ first, int hq, int hkv, float scale, float* __restrict__ dqkv, float* __restrict__ delta) {
  const int wave = wave_index(threadIdx.x), lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int h = blockIdx.x, s = blockIdx.y, kvh = h / (hq / hkv);
  const int q0 = (((int)gridDim.z - 1 - (int)blockIdx.z) * 4 + wave) * 16;   // the longest walks first
  const SeqRows seq = seq_rows(first, s, T_max);
  const size_t row0 = seq.row0;
  const int T = seq.n;
  if (q0 >= T) return;
  const int qd = hq * HD, kvd = hkv * HD;
  const size_t rl = (size_t)qd + 2 * kvd;
  const float* base = qkv + row0 * rl;
  const float* qb = base + (size_t)h * HD;
  const float* kb = base + qd + (size_t)kvh * HD;
  const float* vb = kb + kvd;
  const int qi = min(q0 + r, T - 1);
  float4 qf[HD / 16], dof[HD / 16], of[HD / 16];
  load_rows4<HD>(qb, rl, qi, g, qf);
  load_rows4<HD>(dout + row0 * qd + (size_t)h * HD, qd, qi, g, dof);
  load_rows4<HD>(out + row0 * qd + (size_t)h * HD, qd, qi, g, of);
  float dl = 0.f;
#pragma unroll
  for (int w = 0; w < HD / 16; ++w)
    dl += dof[w].x * of[w].x + dof[w].y * of[w].y + dof[w].z * of[w].z + dof[w].w * of[w].w;
  dl = sum_xor32(sum_xor16(dl));
  const size_t stat = ((size_t)s * hq + h) * T_max + qi;
  const float l = lse[stat];
  f32x4_t dq[HD / 16];
#pragma unroll
  for (int dt = 0; dt < HD / 16; ++dt) dq[dt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const int last = min(q0 + 15, T - 1);
  constexpr bool COLS = HD % 64 == 0;
  __shared__ f32x4_t area[4][2][tile_area<HD>()];
  TileCols<COLS ? HD : 64> kc, kn, vc;
  if constexpr (COLS) {
    kn.stride(rl, g, r); vc.stride(rl, g, r);
    kn.load(kb, rl, min(16, T), g, r);
    vc.load(vb, rl, min(16, T), g, r);
  }
  for (int k0 = 0; k0 <= last; k0 += 16) {
    const int n_valid = min(16, T - k0), k1 = k0 + 16 <= last ? k0 + 16 : k0;   // the next tile (behind the last one: it again)
    float4 kf[HD / 16], vf[HD / 16];
    if constexpr (COLS) {
      kc = kn;
      kc.rows(area[wave][0], g, r, kf);
      vc.rows(area[wave][1], g, r, vf);
      kn.load(kb + (size_t)k1 * rl, rl, min(16, T - k1), g, r);
      vc.load(vb + (size_t)k1 * rl, rl, min(16, T - k1), g, r);
    } else {
      load_rows4<HD>(kb, rl, min(k0 + r, T - 1), g, kf);
      load_rows4<HD>(vb, rl, min(k0 + r, T - 1), g, vf);
    }
    const f32x4_t sc = dot_rows<HD, CH>(kf, qf);    // rows: keys k0 + 4 g + v; column: query qi
    const f32x4_t dp = dot_rows<HD, CH>(vf, dof);   // dP[key][query] = v_key . dO_query
    f32x4_t ds;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int key = k0 + 4 * g + v;
      const float pv = (key <= qi && key < T) ? expf(sc[v] * scale - l) : 0.f;
      ds[v] = scale * pv * (dp[v] - dl);
    }
    if constexpr (COLS) kc.accumulate(ds, dq);
    else accumulate_tile<HD>(kb + (size_t)k0 * rl, rl, n_valid, g, r, ds, dq);
  }
  if (q0 + r >= T) return;
  store_acc<HD>(dqkv + (row0 + qi) * rl + (size_t)h * HD, dq, g, 1.0f);
  if (g == 0) delta[stat] = dl;
}

// Backward, keys and values: a wave owns 16 keys of one (sequence, KV head) and walks n_heads query heads of the group
// (part blockIdx.x / hkv of it) and the query tiles from its own on, in that fixed order; n_heads = 1 leaves one partial
// result per query head, which k_attn_bwd_finish adds in head order (all heads in one wave left the chip a fifth full:
// 840 waves of up to 7 x 19 dependent tiles at 21 x 301):
//   p = exp(scale s - lse_q), dV^T += dO^T p, dP = dO V^T, dS = scale p (dP - delta_q), dK^T += Q^T dS.
template <int HD, int CH>
__global__ void __launch_bounds__(256, HD == 64 ? 2 : 1) k_tattn_bwd_kv(const float* __restrict__ qkv, const float* __restrict__ dout,
                                                      const float* __restrict__ lse, const float* __restrict__ delta, int T_max,
                                                      const int* __restrict__ first, int hq, int hkv, float scale, int n_heads, float* __restrict__ dkv, size_t row_stride,
                                                      size_t part_stride) {
  const int wave = wave_index(threadIdx.x), lane = threadIdx.x & 63, r = lane & 15, g = lane >> 4;
  const int kvh = blockIdx.x % hkv, part = blockIdx.x / hkv, s = blockIdx.y, rep = hq / hkv;
  const int k0 = (blockIdx.z * 4 + wave) * 16;   // the longest walks first
  const SeqRows seq = seq_rows(first, s, T_max);
  const size_t row0 = seq.row0;
  const int T = seq.n;
  if (k0 >= T) return;
  const int qd = hq * HD, kvd = hkv * HD;
  const size_t rl = (size_t)qd + 2 * kvd;
  const float* base = qkv + row0 * rl;
  const float* kb = base + qd + (size_t)kvh * HD;
  const float* vb = kb + kvd;
  const int kj = min(k0 + r, T - 1);
  const bool key_ok = k0 + r < T;
  float4 kf[HD / 16], vf[HD / 16];
  load_rows4<HD>(kb, rl, kj, g, kf);
  load_rows4<HD>(vb, rl, kj, g, vf);
  f32x4_t dk[HD / 16], dv[HD / 16];
#pragma unroll
  for (int dt = 0; dt < HD / 16; ++dt) { dk[dt] = f32x4_t{0.f, 0.f, 0.f, 0.f}; dv[dt] = dk[dt]; }
  constexpr bool COLS = HD % 64 == 0;
  __shared__ f32x4_t area[4][2][tile_area<HD>()];
  for (int hh = 0; hh < n_heads; ++hh) {
    const int h = kvh * rep + part * n_heads + hh;
    const float* qb = base + (size_t)h * HD;
    const float* dob = dout + row0 * qd + (size_t)h * HD;
    const float* lse_h = lse + ((size_t)s * hq + h) * T_max;
    const float* del_h = delta + ((size_t)s * hq + h) * T_max;
    TileCols<COLS ? HD : 64> qc, qn, doc, don;
    if constexpr (COLS) {
      qn.stride(rl, g, r); don.stride(qd, g, r);
      qn.load(qb + (size_t)k0 * rl, rl, min(16, T - k0), g, r);
      don.load(dob + (size_t)k0 * qd, qd, min(16, T - k0), g, r);
    }
    for (int q0 = k0; q0 < T; q0 += 16) {
      const int n_valid = min(16, T - q0), q1 = q0 + 16 < T ? q0 + 16 : q0;   // the next tile (behind the last one: it again)
      float4 qf[HD / 16], dof[HD / 16];
      if constexpr (COLS) {
        qc = qn; doc = don;
        qc.rows(area[wave][0], g, r, qf);
        doc.rows(area[wave][1], g, r, dof);
        qn.load(qb + (size_t)q1 * rl, rl, min(16, T - q1), g, r);
        don.load(dob + (size_t)q1 * qd, qd, min(16, T - q1), g, r);
      } else {
        load_rows4<HD>(qb, rl, min(q0 + r, T - 1), g, qf);
        load_rows4<HD>(dob, qd, min(q0 + r, T - 1), g, dof);
      }
      const f32x4_t sc = dot_rows<HD, CH>(qf, kf);    // rows: queries q0 + 4 g + v; column: key kj
      const f32x4_t dp = dot_rows<HD, CH>(dof, vf);   // dP[query][key]
      f32x4_t pv, ds;
      float ls[4], de[4];
      if (n_valid == 16) {
#pragma unroll
        for (int v = 0; v < 4; ++v) { ls[v] = (lse_h + q0)[4 * g + v]; de[v] = (del_h + q0)[4 * g + v]; }
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v) { const int qc = min(q0 + 4 * g + v, T - 1); ls[v] = lse_h[qc]; de[v] = del_h[qc]; }
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int qi = q0 + 4 * g + v;
        const float pr = (key_ok && qi < T && kj <= qi) ? expf(sc[v] * scale - ls[v]) : 0.f;
        pv[v] = pr;
        ds[v] = scale * pr * (dp[v] - de[v]);
      }
      if constexpr (COLS) {
        doc.accumulate(pv, dv);
        qc.accumulate(ds, dk);
      } else {
        accumulate_tile<HD>(dob + (size_t)q0 * qd, qd, n_valid, g, r, pv, dv);
        accumulate_tile<HD>(qb + (size_t)q0 * rl, rl, n_valid, g, r, ds, dk);
      }
    }
  }
  if (!key_ok) return;
  float* krow = dkv + part * part_stride + (row0 + kj) * row_stride + (size_t)kvh * HD;
  store_acc<HD>(krow, dk, g, 1.0f);
  store_acc<HD>(krow + kvd, dv, g, 1.0f);
}

template <int HD, int CH>
hipError_t tattn_bwd(const float* qkv, const float* out, const float* dout, const float* lse, int S, int T, const int* first, size_t M,
                     int hq, int hkv, float scale, float* dqkv, float* delta, float* parts, hipStream_t st) {
  const unsigned tiles = (unsigned)((T + 63) / 64);
  hipError_t e = launch(KID_ATTN_GENERIC, k_tattn_bwd_q<HD, CH>, dim3(hq, S, tiles), dim3(256), 0, st, qkv, out, dout, lse, T, first, hq,
                        hkv, scale, dqkv, delta);
  if (e != hipSuccess) return e;
  const size_t qd = (size_t)hq * HD, kvd = (size_t)hkv * HD;
  if (parts)   // [query heads of a group][M rows][2 kvd]
    return launch(KID_ATTN_GENERIC, k_tattn_bwd_kv<HD, CH>, dim3(hq, S, tiles), dim3(256), 0, st, qkv, dout, lse, (const float*)delta, T,
                  first, hq, hkv, scale, 1, parts, 2 * kvd, M * 2 * kvd);
  return launch(KID_ATTN_GENERIC, k_tattn_bwd_kv<HD, CH>, dim3(hkv, S, tiles), dim3(256), 0, st, qkv, dout, lse, (const float*)delta, T,
                first, hq, hkv, scale, hq / hkv, dqkv + qd, qd + 2 * kvd, (size_t)0);
}
// The partial results of k_tattn_bwd_kv added in part order into dqkv's key and value columns, and the rotary embedding's
// transpose on the query and key columns.  One workgroup per row; a thread takes 4 rotation pairs or 4 value columns.
__global__ void __launch_bounds__(256) k_attn_bwd_finish(float* __restrict__ dqkv, const float* __restrict__ parts, int n_parts,
                                                         size_t part_stride, const float2* __restrict__ rope, int T, const int* __restrict__ pos,
                                                         int hq, int hkv, int hd, uint32_t* __restrict__ row_mx) {
  uint32_t mx = 0;
  auto seen = [&](const float4& v) { mx = max(max(max(mx, abs_bits(v.x)), max(abs_bits(v.y), abs_bits(v.z))), abs_bits(v.w)); };
  const size_t m = blockIdx.x;
  const int half = hd >> 1, qd = hq * hd, kvd = hkv * hd, quads = half >> 2;
  const size_t at = pos ? (size_t)pos[m] : m % T;   // the row's position
  float* row = dqkv + m * (size_t)(qd + 2 * kvd);
  const float* prow = parts + m * (size_t)(2 * kvd);
  auto sum = [&](int c) {   // column c of [dk | dv]
    float4 s = *(const float4*)(prow + c);
    for (int p = 1; p < n_parts; ++p) {
      const float4 v = *(const float4*)(prow + p * part_stride + c);
      s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    return s;
  };
  const int n_rot = (hq + hkv) * quads, n_all = n_rot + kvd / 4;
  for (int e = threadIdx.x; e < n_all; e += 256) {
    if (e >= n_rot) {
      const int c = kvd + 4 * (e - n_rot);
      const float4 v = sum(c);
      *(float4*)(row + qd + c) = v;
      seen(v);
      continue;
    }
    const int head = e / quads, i = 4 * (e % quads);
    float* p = row + head * hd + i;
    float4 a, b;
    if (head < hq) { a = *(const float4*)p; b = *(const float4*)(p + half); }
    else { a = sum((head - hq) * hd + i); b = sum((head - hq) * hd + i + half); }
    const float4* cs = (const float4*)(rope + at * half + i);
    const float4 c01 = cs[0], c23 = cs[1];   // (cos, sin) of four pairs
    const float4 lo = make_float4(a.x * c01.x + b.x * c01.y, a.y * c01.z + b.y * c01.w, a.z * c23.x + b.z * c23.y, a.w * c23.z + b.w * c23.w);
    const float4 hi = make_float4(b.x * c01.x - a.x * c01.y, b.y * c01.z - a.y * c01.w, b.z * c23.x - a.z * c23.y, b.w * c23.z - a.w * c23.w);
    *(float4*)p = lo;
    *(float4*)(p + half) = hi;
    seen(lo);
    seen(hi);
  }
  if (row_mx) {
    mx = wave_max_u32(mx);
    if ((threadIdx.x & 63) == 0) atomicMax(row_mx + m, mx);
  }
}

// Attention backward pieces (the contractions are batched GEMMs):
// delta[(s Hq + h) T + i] = dO_i . O_i over the head's dims; one wave per (s, i, h)
__global__ void __launch_bounds__(64) k_attn_delta(const float* __restrict__ dout, const float* __restrict__ out, int T, int hq,
                                                   int hd, float* __restrict__ delta) {
  const size_t b = blockIdx.x;            // (s * T + i) * hq + h
  const int h = (int)(b % hq);
  const size_t si = b / hq, s = si / T, i = si % T;
  const float* a = dout + (si * hq + h) * hd;
  const float* o = out + (si * hq + h) * hd;
  float d = 0.f;
  for (int e = threadIdx.x; e < hd; e += 64) d = fmaf(a[e], o[e], d);
  d = wave_reduce_sum(d);
  if (threadIdx.x == 0) delta[(s * hq + h) * T + i] = d;
}
// d(q . k)_ij = scale * p_ij (dP_ij - delta_i), in place over dP
__global__ void k_dscores(const float* __restrict__ prob, float* __restrict__ dp, const float* __restrict__ delta, int T,
                          float scale, size_t total) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= total) return;
  const float pr = prob[idx];   // zero above the diagonal, where dP was not computed
  dp[idx] = pr == 0.f ? 0.f : scale * pr * (dp[idx] - delta[idx / T]);
}

// Embedding rows: dE[tokens[m]] += dh[m], in the order of the rows for every token.  The rows are taken 4096 at a time:
// k_embed_order sorts a chunk's (token, row) pairs, k_embed_add gives every run of one token to a workgroup, which adds the
// run's rows in order, 8 of them on their way at a time, and adds the sum to the token's row of dE; the chunks follow
// each other on the stream.  (With one workgroup per class of tokens the most frequent token's rows were read, added to
// memory and waited for one after the other: 4.6 ms at 64 x 384 Zipf-distributed tokens.)
constexpr int kEmbedChunk = 4096;
__global__ void __launch_bounds__(1024) k_embed_order(const int32_t* __restrict__ tokens, int M, int V, int* __restrict__ order) {
  __shared__ unsigned long long key[kEmbedChunk];
  const int m0 = blockIdx.x * kEmbedChunk, n = min(M - m0, kEmbedChunk);
  for (int i = threadIdx.x; i < kEmbedChunk; i += 1024)
    key[i] = i < n ? ((unsigned long long)(unsigned)clamp_token(tokens[m0 + i], V) << 32) | (unsigned)i : ~0ull;
  for (int size = 2; size <= kEmbedChunk; size <<= 1)
    for (int step = size >> 1; step > 0; step >>= 1) {
      __syncthreads();
      for (int j = threadIdx.x; j < kEmbedChunk / 2; j += 1024) {
        const int lo = 2 * j - (j & (step - 1)), hi = lo + step;
        const unsigned long long a = key[lo], b = key[hi];
        if ((a > b) == ((lo & size) == 0)) { key[lo] = b; key[hi] = a; }
      }
    }
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += 1024) order[m0 + i] = (int)(unsigned)key[i];
}
// workgroup (x, y) of one wave: the run that starts at sorted position x, if one does, columns 256 y .. of it
__global__ void __launch_bounds__(64) k_embed_add(const int32_t* __restrict__ tokens, const int* __restrict__ order, int n,
                                                  const float* __restrict__ dh, int d, int V, float* __restrict__ dE) {
  const int x = blockIdx.x;
  const int tok = clamp_token(tokens[order[x]], V);
  if (x > 0 && clamp_token(tokens[order[x - 1]], V) == tok) return;
  int end = x + 1;
  while (end < n && clamp_token(tokens[order[end]], V) == tok) ++end;
  for (int c = blockIdx.y * 256 + threadIdx.x; c < min(d, ((int)blockIdx.y + 1) * 256); c += 64) {
    float s = 0.f;
    for (int p = x; p < end; p += 8) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = dh[(size_t)order[min(p + u, end - 1)] * d + c];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += p + u < end ? v[u] : 0.f;
    }
    dE[(size_t)tok * d + c] += s;
  }
}

// Adam (Kingma & Ba, Algorithm 1): c1 = 1 - beta1^t, c2 = 1 - beta2^t
__global__ void k_adam(float* __restrict__ theta, const float* __restrict__ g, float* __restrict__ m, float* __restrict__ v,
                       size_t n, float lr, float beta1, float beta2, float eps, float c1, float c2) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = beta1 * m[i] + (1.0f - beta1) * gi;
  const float vi = beta2 * v[i] + (1.0f - beta2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  theta[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

unsigned blocks256(size_t n) { return (unsigned)((n + 255) / 256); }

}  // namespace

// ---------------------------------------------------------------------------------------
// the trainer
// ---------------------------------------------------------------------------------------
struct sapo_trainer {
  sapo_model_config cfg;
  sapo_adam_config opt;
  int t = 0;                      // Adam steps taken
  int pieces = 3;                 // of the large GEMMs (NP there): 3 (fp32 accuracy), 2 (16 significant bits), 1 (bf16 operands)
  bool use_bias = false;          // the model has biases on its query / key / value projections (set_qkv_bias)
  int n_in = 0;                   // tensors of the input list; tensor n_in + l is layer l's bias vector
  int device = 0;
  size_t n_params = 0;
  float* theta = nullptr;         // [n_params] masters, tensors back to back in tensor-list order
  float* grad = nullptr;
  float* m = nullptr;
  float* v = nullptr;
  float2* rope = nullptr;         // [max_seq][hd / 2] (cos, sin)
  std::vector<size_t> off, len;   // per tensor
};

namespace {

struct Dims {
  size_t d, q, kv, nqkv, F, V;
  int L;
  explicit Dims(const sapo_model_config& c)
      : d(c.d_model), q((size_t)c.n_q_heads * c.head_dim), kv((size_t)c.n_kv_heads * c.head_dim), nqkv(q + 2 * kv), F(c.d_ff),
        V(c.vocab), L(c.n_layers) {}
};

int n_tensors_of(const sapo_model_config& c) { return 1 + 9 * c.n_layers + 1 + (c.tied_embeddings ? 0 : 1); }

void tensor_sizes(const sapo_model_config& c, std::vector<size_t>& len) {
  const Dims D(c);
  len.clear();
  len.push_back(D.V * D.d);
  for (int l = 0; l < D.L; ++l) {
    const size_t s[9] = {D.d, D.q * D.d, D.kv * D.d, D.kv * D.d, D.d * D.q, D.d, D.F * D.d, D.F * D.d, D.d * D.F};
    for (size_t x : s) len.push_back(x);
  }
  len.push_back(D.d);
  if (!c.tied_embeddings) len.push_back(D.V * D.d);
  for (int l = 0; l < D.L; ++l) len.push_back(D.nqkv);   // optional projection biases [bq | bk | bv] (zero and idle unless set)
}

// rows of logits held at once: about 2.5 GB (enough rows for the d-input GEMM of the head, whose output is only
// d_model wide, to fill the chip), a multiple of the GEMM tile
size_t lm_chunk_rows(const Dims& D, size_t M) {
  size_t r = ((size_t)5 << 29) / (D.V * sizeof(float)) / 128 * 128;
  if (r < 128) r = 128;
  return r < M ? r : M;
}

struct Arena {
  char* base;
  size_t off;
  template <typename T> T* take(size_t n) {
    off = (off + 255) & ~(size_t)255;
    T* p = base ? (T*)(base + off) : nullptr;
    off += n * sizeof(T);
    return p;
  }
};

// GEMMs with a long contraction whose output tiles do not fill the resident workgroups (the weight gradients; the
// head's d-input product: 238 tiles, contraction over the vocabulary) are split over the contraction into up to
// kMaxSplits parts that are added in part order; the buffer holds 8 parts of the largest layer matrix.
inline size_t split_parts_floats(const Dims& D) { return (size_t)8 * std::max((size_t)2 * D.F * D.d, (size_t)192 * 128 * 128); }
constexpr int kPieces = 3;   // the packed operands' buffers are sized for any

// the fused attention kernels need float4 rows: head dim 16 / 32 / 64 / 128 and row lengths that are multiples of 4
inline bool fused_attention(const sapo_model_config& c) {
  const int hd = c.head_dim;
  return (hd == 16 || hd == 32 || hd == 64 || hd == 128) && (c.n_q_heads * hd) % 4 == 0 && (c.n_kv_heads * hd) % 4 == 0;
}

struct LayerActs {
  float *h, *r1, *xn, *qkv, *lse, *ao, *h2, *r2, *xn2, *gu, *act;
};
// Maxima (bits) of the rows and columns of the products' operands: see k_gemm_x3
struct LayerMax {
  uint32_t *wqkv_r, *wo_r, *wgu_r, *wd_r;                   // weights by rows: written once per update
  uint32_t *wqkv_c, *wo_c, *wgu_c, *wd_c;                   // from here on taken by atomics, zeroed before a micro-batch
  uint32_t *xn_c, *ao_r, *ao_c, *xn2_c, *act_r, *act_c, *dh1_c, *dgu_r, *dgu_c, *dh2_c, *dqkv_r, *dqkv_c;
};
struct TrainPlan {
  std::vector<LayerMax> mx;
  uint32_t *xn_r, *dh_r, *dl_r, *xfc_r;            // by rows, written anew for every layer or chunk
  uint32_t *head_r, *head_c, *xfc_c, *dl_c;
  uint32_t* mx_zero;                                        // the atomics' ones, mx_zero_n of them (head_c lies in front of them: zeroed once per update)
  size_t mx_zero_n;
  std::vector<LayerActs> layer;
  bool packed_ffn;                              // the SwiGLU passes write packed operands (act of a layer is not kept)
  char* act_cols;                               // act of the layer at hand by rows of features
  float *h_last, *rf, *xf;                      // final residual rows, their rstd, final-normed rows
  float* xfc;                                   // the final-normed rows that predict a masked token, gathered
  int* eorder;                                  // a chunk's rows ordered by token (embedding gradient)
  int *mrows, *mpos, *mcount;                   // per micro-batch: those rows' indices (mpos: scratch, see PackedUpdate), their number
  int* first;                                   // packed rows: a sequence's first one
  float *dh, *dx, *dact, *dgu, *dao, *dqkv;     // backward temporaries (dgu: also its packed form by rows of features)
  float *delta, *prob, *dsc, *gpart, *logits, *logp_all, *loss;
  void* sur_ws;
  long long* n_masked;
  float* kparts;                                // partial products of the split weight-gradient GEMMs
  char *packa, *packb, *head_nt, *head_t;       // packed operands; the LM head packed once per update, both ways
  size_t packa_cap, packb_cap, head_cap, head_t_cap;
  size_t chunk;
  size_t bytes;
};

void make_plan(const sapo_model_config& c, size_t S, size_t T, size_t S_total, char* base, TrainPlan& p) {
  const Dims D(c);
  const size_t M = S * T;
  Arena A{base, 0};
  p.packed_ffn = D.F % 64 == 0 && (M + 127) / 128 * 2 <= 65535;
  p.layer.resize(D.L);
  for (int l = 0; l < D.L; ++l) {
    LayerActs& a = p.layer[l];
    a.h = A.take<float>(M * D.d);
    a.r1 = A.take<float>(M);
    a.xn = A.take<float>(M * D.d);
    a.qkv = A.take<float>(M * D.nqkv);
    a.lse = A.take<float>(S * c.n_q_heads * T);
    a.ao = A.take<float>(M * D.q);
    a.h2 = A.take<float>(M * D.d);
    a.r2 = A.take<float>(M);
    a.xn2 = A.take<float>(M * D.d);
    a.gu = A.take<float>(M * 2 * D.F);
    a.act = A.take<float>(p.packed_ffn ? 0 : M * D.F);
  }
  p.h_last = A.take<float>(M * D.d);
  p.rf = A.take<float>(M);
  p.xf = A.take<float>(M * D.d);
  p.xfc = A.take<float>(M * D.d);
  p.mrows = A.take<int>(S_total * T);
  p.eorder = A.take<int>(M);
  p.mpos = A.take<int>(2 * M);
  p.mcount = A.take<int>(2 * ((S_total + S - 1) / S));
  p.first = A.take<int>(S + 1);
  p.dh = A.take<float>(M * D.d);
  p.dx = A.take<float>(M * D.d);
  p.dact = A.take<float>(M * D.F);
  p.dgu = A.take<float>(std::max(M * 2 * D.F, x3_pack_bytes(kPieces, 2 * D.F, M) / sizeof(float)));
  p.act_cols = A.take<char>(p.packed_ffn ? x3_pack_bytes(kPieces, D.F, M) : 0);
  p.dao = A.take<float>(M * D.q);
  p.dqkv = A.take<float>(M * D.nqkv);
  p.delta = A.take<float>(S * c.n_q_heads * T);
  // T x T score matrices: only for head dims the fused attention kernels do not take
  const size_t n_tt = fused_attention(c) ? 0 : S * c.n_q_heads * T * T;
  p.prob = A.take<float>(n_tt);
  p.dsc = A.take<float>(n_tt);
  p.gpart = A.take<float>(std::max(((M + kNormRows - 1) / kNormRows) * D.d, ((M + 255) / 256) * std::max(D.d, D.nqkv)));
  p.chunk = lm_chunk_rows(D, M);
  p.logits = A.take<float>(p.chunk * D.V);
  p.logp_all = A.take<float>(S_total * T);   // log-probs of the whole training set (micro-batches fill their rows)
  p.loss = A.take<float>(4);
  p.n_masked = A.take<long long>(1);
  p.kparts = A.take<float>(split_parts_floats(D));
  // packed GEMM operands: the largest row-side (A) and column-side (B) operand of any GEMM of the update
  {
    const size_t R = p.chunk, twoF = 2 * D.F;
    const size_t a_shapes[][2] = {{M, D.d}, {M, D.q}, {M, D.F}, {M, twoF}, {M, D.nqkv}, {D.d, M}, {twoF, M}, {D.nqkv, M},
                                  {R, D.d}, {R, D.V}, {D.V, R}};
    const size_t b_shapes[][2] = {{D.nqkv, D.d}, {D.d, D.q}, {twoF, D.d}, {D.d, D.F}, {D.F, D.d}, {D.d, twoF},
                                  {D.d, M}, {D.q, D.d}, {D.q, M}, {D.d, D.nqkv}, {D.d, R}};
    p.packa_cap = p.packb_cap = 0;
    for (auto& sh : a_shapes) p.packa_cap = std::max(p.packa_cap, x3_pack_bytes(kPieces, sh[0], sh[1]));
    for (auto& sh : b_shapes) p.packb_cap = std::max(p.packb_cap, x3_pack_bytes(kPieces, sh[0], sh[1]));
    p.head_cap = x3_pack_bytes(kPieces, D.V, D.d);
    p.head_t_cap = x3_pack_bytes(kPieces, D.d, D.V);
    p.packa = A.take<char>(p.packa_cap);
    p.packb = A.take<char>(p.packb_cap);
    p.head_nt = A.take<char>(p.head_cap);
    p.head_t = A.take<char>(p.head_t_cap);
  }
  p.mx.resize(D.L);
  for (auto& m : p.mx) {
    m.wqkv_r = A.take<uint32_t>(D.nqkv); m.wo_r = A.take<uint32_t>(D.d); m.wgu_r = A.take<uint32_t>(2 * D.F); m.wd_r = A.take<uint32_t>(D.d);
  }
  for (uint32_t** r : {&p.xn_r, &p.dh_r, &p.dl_r, &p.xfc_r}) *r = A.take<uint32_t>(M);
  p.head_r = A.take<uint32_t>(D.V);
  p.head_c = A.take<uint32_t>(D.d);
  p.mx_zero = A.take<uint32_t>(1);
  const size_t zero0 = A.off;
  for (auto& m : p.mx) {
    m.wqkv_c = A.take<uint32_t>(D.d); m.wo_c = A.take<uint32_t>(D.q); m.wgu_c = A.take<uint32_t>(D.d); m.wd_c = A.take<uint32_t>(D.F);
    m.xn_c = A.take<uint32_t>(D.d); m.ao_r = A.take<uint32_t>(M); m.ao_c = A.take<uint32_t>(D.q); m.xn2_c = A.take<uint32_t>(D.d);
    m.act_r = A.take<uint32_t>(M); m.act_c = A.take<uint32_t>(D.F); m.dh1_c = A.take<uint32_t>(D.d); m.dgu_r = A.take<uint32_t>(M);
    m.dgu_c = A.take<uint32_t>(2 * D.F); m.dh2_c = A.take<uint32_t>(D.d); m.dqkv_r = A.take<uint32_t>(M); m.dqkv_c = A.take<uint32_t>(D.nqkv);
  }
  p.xfc_c = A.take<uint32_t>(D.d);
  p.dl_c = A.take<uint32_t>(D.V);
  p.mx_zero_n = (A.off - zero0) / sizeof(uint32_t) + 1;
  p.sur_ws = A.take<char>(g_surrogate_workspace_bytes());
  p.bytes = (A.off + 255) & ~(size_t)255;
}

int check_cfg(const sapo_model_config* c) {
  if (!c) return set_error(SAPO_EINVAL, "cfg is NULL");
  if (c->n_layers <= 0 || c->d_model <= 0 || c->n_q_heads <= 0 || c->n_kv_heads <= 0 || c->head_dim <= 0 || c->d_ff <= 0 ||
      c->vocab <= 0 || c->max_seq <= 0)
    return set_error(SAPO_EINVAL, "model sizes must be positive");
  if (c->n_q_heads % c->n_kv_heads != 0) return set_error(SAPO_ESHAPE, "n_q_heads must be a multiple of n_kv_heads");
  if (c->head_dim % 2 != 0 || c->head_dim > 128) return set_error(SAPO_ESHAPE, "head_dim must be even and at most 128");
  if (c->dtype != SAPO_DTYPE_F32 && c->dtype != SAPO_DTYPE_BF16) return set_error(SAPO_EINVAL, "unknown dtype");
  if (!(c->rms_eps > 0.f) || !(c->rope_theta > 0.f)) return set_error(SAPO_EINVAL, "rms_eps and rope_theta must be > 0");
  return SAPO_OK;
}

bool gain_tensor(const sapo_model_config& c, int i) {
  if (i == 0) return false;
  const int last_layer_tensor = 9 * c.n_layers;
  if (i <= last_layer_tensor) { const int k = (i - 1) % 9; return k == 0 || k == 5; }
  return i == last_layer_tensor + 1;
}

}  // namespace

extern "C" void sapo_trainer_destroy(sapo_trainer* tr) {
  if (!tr) return;
  (void)hipSetDevice(tr->device);
  for (void* p : {(void*)tr->theta, (void*)tr->grad, (void*)tr->m, (void*)tr->v, (void*)tr->rope})
    if (p) (void)hipFree(p);
  delete tr;
}

extern "C" int sapo_trainer_create(const sapo_model_config* cfg, const void* const* tensors, int n_tensors,
                                   const sapo_adam_config* opt, void* stream, sapo_trainer** out) {
  if (!out) return set_error(SAPO_EINVAL, "out is NULL");
  *out = nullptr;
  int rc = check_cfg(cfg);
  if (rc) return rc;
  if (!tensors) return set_error(SAPO_EINVAL, "tensors is NULL");
  if (n_tensors != n_tensors_of(*cfg))
    return set_error(SAPO_EINVAL, "n_tensors is %d, expected %d", n_tensors, n_tensors_of(*cfg));
  for (int i = 0; i < n_tensors; ++i)
    if (!tensors[i]) return set_error(SAPO_EINVAL, "tensor %d is NULL", i);
  sapo_adam_config o{1e-3f, 0.9f, 0.999f, 1e-8f};
  if (opt) o = *opt;
  if (!(o.lr > 0.f) || !(o.beta1 >= 0.f && o.beta1 < 1.f) || !(o.beta2 >= 0.f && o.beta2 < 1.f) || !(o.eps > 0.f))
    return set_error(SAPO_EINVAL, "Adam needs lr > 0, beta1 and beta2 in [0, 1), eps > 0");
  hipStream_t st = (hipStream_t)stream;
  sapo_trainer* tr = new sapo_trainer;
  tr->cfg = *cfg;
  tr->opt = o;
  (void)hipGetDevice(&tr->device);
  tensor_sizes(*cfg, tr->len);
  tr->off.resize(tr->len.size());
  size_t n = 0;
  for (size_t i = 0; i < tr->len.size(); ++i) { tr->off[i] = n; n += tr->len[i]; }
  tr->n_params = n;
  tr->n_in = n_tensors;
  auto bail = [&](int code) { sapo_trainer_destroy(tr); return code; };
  for (float** p : {&tr->theta, &tr->grad, &tr->m, &tr->v}) {
    hipError_t e = hipMalloc((void**)p, n * sizeof(float));
    if (e != hipSuccess) return bail(set_error(SAPO_EHIP, "hipMalloc of %zu bytes failed: %s", n * sizeof(float), hipGetErrorString(e)));
  }
  for (int i = 0; i < n_tensors; ++i) {
    float* dst = tr->theta + tr->off[i];
    hipError_t e;
    if (cfg->dtype == SAPO_DTYPE_F32 || gain_tensor(*cfg, i))
      e = hipMemcpyAsync(dst, tensors[i], tr->len[i] * sizeof(float), hipMemcpyDeviceToDevice, st);
    else
      e = launch(KID_MISC, k_bf16_to_f32, dim3(blocks256(tr->len[i])), dim3(256), 0, st, (const bf16*)tensors[i], dst, tr->len[i]);
    if (e != hipSuccess) return bail(set_error(SAPO_EHIP, "copy of tensor %d failed: %s", i, hipGetErrorString(e)));
  }
  for (float* p : {tr->grad, tr->m, tr->v}) {
    hipError_t e = g_fill_f32(p, 0.f, n, st);
    if (e != hipSuccess) return bail(set_error(SAPO_EHIP, "fill failed: %s", hipGetErrorString(e)));
  }
  {
    const size_t b0 = tr->off[n_tensors];   // the bias vectors start at zero
    hipError_t e = g_fill_f32(tr->theta + b0, 0.f, n - b0, st);
    if (e != hipSuccess) return bail(set_error(SAPO_EHIP, "fill failed: %s", hipGetErrorString(e)));
  }
  const int half = cfg->head_dim / 2;
  std::vector<float2> tab((size_t)cfg->max_seq * half);
  for (int pos = 0; pos < cfg->max_seq; ++pos)
    for (int i = 0; i < half; ++i) {
      const double ang = (double)pos * pow((double)cfg->rope_theta, -2.0 * i / cfg->head_dim);
      tab[(size_t)pos * half + i] = make_float2((float)cos(ang), (float)sin(ang));
    }
  hipError_t e = hipMalloc((void**)&tr->rope, tab.size() * sizeof(float2));
  if (e == hipSuccess) e = hipMemcpy(tr->rope, tab.data(), tab.size() * sizeof(float2), hipMemcpyHostToDevice);
  if (e != hipSuccess) return bail(set_error(SAPO_EHIP, "rotary table: %s", hipGetErrorString(e)));
  *out = tr;
  return SAPO_OK;
}

extern "C" size_t sapo_trainer_workspace_bytes(const sapo_trainer* tr, int S, int T) {
  if (!tr || S <= 0 || T < 2 || T > tr->cfg.max_seq) return 0;
  TrainPlan p;
  make_plan(tr->cfg, (size_t)S, (size_t)T, (size_t)S, nullptr, p);
  return p.bytes;
}

extern "C" size_t sapo_trainer_workspace_bytes_for(const sapo_trainer* tr, int S, int T, int S_micro) {
  if (!tr || S <= 0 || T < 2 || T > tr->cfg.max_seq || S_micro <= 0 || S_micro > S) return 0;
  TrainPlan p;
  make_plan(tr->cfg, (size_t)S_micro, (size_t)T, (size_t)S, nullptr, p);
  return p.bytes;
}

extern "C" int sapo_trainer_set_qkv_bias(sapo_trainer* tr, int layer, const float* bq, const float* bk, const float* bv,
                                         void* stream) {
  if (!tr || !bq || !bk || !bv) return set_error(SAPO_EINVAL, "NULL argument");
  if (layer < 0 || layer >= tr->cfg.n_layers) return set_error(SAPO_EINVAL, "layer %d out of range", layer);
  const Dims D(tr->cfg);
  float* dst = tr->theta + tr->off[tr->n_in + layer];
  hipStream_t st = (hipStream_t)stream;
  T_CK(hipMemcpyAsync(dst, bq, D.q * sizeof(float), hipMemcpyDeviceToDevice, st));
  T_CK(hipMemcpyAsync(dst + D.q, bk, D.kv * sizeof(float), hipMemcpyDeviceToDevice, st));
  T_CK(hipMemcpyAsync(dst + D.q + D.kv, bv, D.kv * sizeof(float), hipMemcpyDeviceToDevice, st));
  tr->use_bias = true;
  return SAPO_OK;
}

extern "C" int sapo_trainer_get_qkv_bias(const sapo_trainer* tr, int layer, float* bq, float* bk, float* bv, void* stream) {
  if (!tr || !bq || !bk || !bv) return set_error(SAPO_EINVAL, "NULL argument");
  if (layer < 0 || layer >= tr->cfg.n_layers) return set_error(SAPO_EINVAL, "layer %d out of range", layer);
  const Dims D(tr->cfg);
  const float* src = tr->theta + tr->off[tr->n_in + layer];
  hipStream_t st = (hipStream_t)stream;
  T_CK(hipMemcpyAsync(bq, src, D.q * sizeof(float), hipMemcpyDeviceToDevice, st));
  T_CK(hipMemcpyAsync(bk, src + D.q, D.kv * sizeof(float), hipMemcpyDeviceToDevice, st));
  T_CK(hipMemcpyAsync(bv, src + D.q + D.kv, D.kv * sizeof(float), hipMemcpyDeviceToDevice, st));
  return SAPO_OK;
}

extern "C" int sapo_trainer_steps(const sapo_trainer* tr) { return tr ? tr->t : -1; }

extern "C" int sapo_trainer_set_matmul_pieces(sapo_trainer* tr, int pieces) {
  if (!tr) return set_error(SAPO_EINVAL, "trainer is NULL");
  if (pieces < 1 || pieces > 3)
    return set_error(SAPO_EINVAL, "pieces must be 3 (fp32 accuracy), 2 (16 significant bits) or 1 (bf16 operands)");
  tr->pieces = pieces;
  return SAPO_OK;
}

extern "C" int sapo_trainer_read(const sapo_trainer* tr, int what, int tensor, float* out, size_t n, void* stream) {
  if (!tr || !out) return set_error(SAPO_EINVAL, "NULL argument");
  if (tensor < 0 || tensor >= (int)tr->len.size()) return set_error(SAPO_EINVAL, "tensor index %d out of range", tensor);
  if (n != tr->len[tensor]) return set_error(SAPO_EINVAL, "tensor %d has %zu elements, not %zu", tensor, tr->len[tensor], n);
  const float* src = what == 0 ? tr->theta : what == 1 ? tr->grad : what == 2 ? tr->m : what == 3 ? tr->v : nullptr;
  if (!src) return set_error(SAPO_EINVAL, "what must be 0 (parameters), 1 (gradient), 2 or 3 (Adam moments)");
  T_CK(hipMemcpyAsync(out, src + tr->off[tensor], n * sizeof(float), hipMemcpyDeviceToDevice, (hipStream_t)stream));
  return SAPO_OK;
}

extern "C" int sapo_trainer_export(const sapo_trainer* tr, void* const* tensors_out, int n_tensors, void* stream) {
  if (!tr || !tensors_out) return set_error(SAPO_EINVAL, "NULL argument");
  if (n_tensors != tr->n_in) return set_error(SAPO_EINVAL, "n_tensors is %d, expected %d", n_tensors, tr->n_in);
  for (int i = 0; i < n_tensors; ++i)
    if (!tensors_out[i]) return set_error(SAPO_EINVAL, "tensor %d is NULL", i);
  for (int i0 = 0; i0 < n_tensors; i0 += kExportTasks) {
    ExportTasks a;
    a.n = std::min(kExportTasks, n_tensors - i0);
    size_t blocks = 0;
    for (int k = 0; k < a.n; ++k) {
      const int i = i0 + k;
      a.t[k] = ExportTask{tr->theta + tr->off[i], tensors_out[i], tr->len[i], (unsigned)blocks,
                          tr->cfg.dtype == SAPO_DTYPE_F32 || gain_tensor(tr->cfg, i) ? 1u : 0u};
      blocks += (tr->len[i] + kExportBlock - 1) / kExportBlock;
    }
    T_CK(launch(KID_MISC, k_export, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, a));
  }
  return SAPO_OK;
}

// The rows of a micro-batch that the loss depends on.  Attention is causal and a row's gradient is zero behind its sequence's last
// masked token, so what lies behind it (answers that end before their row does) needs neither pass.  Sequence s goes on with
// lens[s].x positions, side by side with the others': row first[s] + t is token tokens[first[s] + t] at position t; rows: those that
// predict a masked token, token_rows: the same as indices into [S, T].
struct PackedUpdate {
  int2* lens = nullptr;
  int *first = nullptr, *pos = nullptr, *tokens = nullptr, *rows = nullptr, *token_rows = nullptr;
  // in buffers that are free until the backward pass through the layers (token_rows) or the embedding's gradient (lens)
  void init(const TrainPlan& p, int S, int n_rows) {
    lens = (int2*)p.eorder; first = p.first; pos = p.mpos; tokens = p.mpos + n_rows; rows = p.mrows; token_rows = (int*)p.dh_r;
  }
};
__global__ void __launch_bounds__(256) k_packed_update(const uint8_t* __restrict__ mask, const int32_t* __restrict__ tokens, int T, int S,
                                                       const int2* __restrict__ lens, int* __restrict__ first, int* __restrict__ pos,
                                                       int* __restrict__ row_tokens, int* __restrict__ rows, int* __restrict__ token_rows) {
  __shared__ int2 part[4];
  const int s = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int row0 = 0, out0 = 0;   // rows and listed ones of the sequences in front
  for (int i = threadIdx.x; i < s; i += 256) { row0 += lens[i].x; out0 += lens[i].y; }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) { row0 += __shfl_xor(row0, o, 64); out0 += __shfl_xor(out0, o, 64); }
  if (lane == 0) part[wave] = make_int2(row0, out0);
  __syncthreads();
  row0 = (part[0].x + part[1].x) + (part[2].x + part[3].x);
  out0 = (part[0].y + part[1].y) + (part[2].y + part[3].y);
  const int n = lens[s].x;
  if (threadIdx.x == 0) {
    first[s] = row0;
    if (s == S - 1) first[S] = row0 + n;
  }
  for (int t0 = 0; t0 <= n; t0 += 256) {
    const int t = t0 + threadIdx.x;
    if (t < n) { pos[row0 + t] = t; row_tokens[row0 + t] = tokens[(size_t)s * T + t]; }
    const bool on = t >= 1 && t <= n && mask[(size_t)s * T + t] != 0;
    const unsigned long long all = __ballot(on);
    __syncthreads();   // part is read
    if (lane == 0) part[wave].x = __popcll(all);
    __syncthreads();
    int o = out0 + __popcll(all & ((1ull << lane) - 1ull));
    for (int w = 0; w < wave; ++w) o += part[w].x;
    if (on) { rows[o] = row0 + t - 1; token_rows[o] = s * T + t - 1; }
    out0 += (part[0].x + part[1].x) + (part[2].x + part[3].x);
  }
}
__global__ void __launch_bounds__(256) k_packed_count(const int2* __restrict__ lens, int S, int* __restrict__ count) {
  __shared__ int part[4];
  int n = 0;
  for (int i = threadIdx.x; i < S; i += 256) n += lens[i].x;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = n;
  __syncthreads();
  if (threadIdx.x == 0) *count = (part[0] + part[1]) + (part[2] + part[3]);
}

// Forward, LM head and backward over one micro-batch of S_ sequences: gradients are written to tr->grad by the first one of
// an update (first) and added by the others (zeroing the buffer and adding to the zeros moved 6 GB at 0.5B: 21 x 301 tokens,
// one piece, 43.0 -> 42.0 ms), the log-probs go to logp_new [S_, T_].  p.n_masked holds the count of masked tokens of the whole training set and
// the LM head is packed (p.head_nt, p.head_t).  n_packed: rows that go on (PackedUpdate), 0: all as they lie.
static int update_rows(sapo_trainer* tr, const TrainPlan& p, const int32_t* tokens, const uint8_t* completion_mask,
                       const float* logp_old, const float* advantages, int S_, int T_, float eps_low, float eps_high,
                       float* logp_new, const int* rows, int n_rows, int n_packed, bool first, hipStream_t st) {
  const sapo_model_config& c = tr->cfg;
  const Dims D(c);
  const size_t S = S_, T = T_, M = n_packed > 0 ? (size_t)n_packed : S * T;
  PackedUpdate pk;
  if (n_packed > 0) {
    pk.init(p, S_, n_packed);
    T_CK(g_packed_lens(completion_mask, T_, 0, S_, false, pk.lens, st));
    T_CK(launch(KID_MISC, k_packed_update, dim3(S_), dim3(256), 0, st, completion_mask, tokens, T_, S_, (const int2*)pk.lens, pk.first, pk.pos,
                pk.tokens, pk.rows, pk.token_rows));
    rows = pk.rows;
  }
  const int32_t* row_tokens = n_packed > 0 ? pk.tokens : tokens;   // of each row
  const int* token_rows = n_packed > 0 ? pk.token_rows : rows;     // the listed rows as tokens of the batch
  const int d = (int)D.d, q = (int)D.q, kv = (int)D.kv, nqkv = (int)D.nqkv, F = (int)D.F, V = (int)D.V;
  const int hq = c.n_q_heads, hkv = c.n_kv_heads, hd = c.head_dim;
  const int Mi = (int)M;
  auto TH = [&](int tensor) { return tr->theta + tr->off[tensor]; };
  auto GR = [&](int tensor) { return tr->grad + tr->off[tensor]; };
  const float keep = first ? 0.f : 1.f;   // of the gradients there
  const int t_final = 1 + 9 * D.L, t_head = c.tied_embeddings ? 0 : t_final + 1;
  const int rep = hq / hkv;
  const float att_scale = 1.0f / sqrtf((float)hd);
  const bool fused_attn = fused_attention(c);
  const size_t n_sc = S * hq * T * T;
  const long TT = (long)(T * T), Trow = (long)(T * D.nqkv), Tq = (long)(T * D.q);
  Batch b_scores, b_pv, b_dp, b_dq, b_dk, b_dv;
  // per (sequence, query head): Q_h and the group's K -> scores
  b_scores.nh = hq; b_scores.bdiv = rep; b_scores.count = S_ * hq;
  b_scores.a1 = Trow; b_scores.a2 = hd; b_scores.b1 = Trow; b_scores.b2 = hd; b_scores.c1 = hq * TT; b_scores.c2 = TT;
  // P and the group's V -> the head's columns of the attention output
  b_pv = b_scores; b_pv.a1 = hq * TT; b_pv.a2 = TT; b_pv.c1 = Tq; b_pv.c2 = hd;
  // dO_h and the group's V -> dP
  b_dp = b_scores; b_dp.a1 = Tq; b_dp.a2 = hd;
  // dS and the group's K -> dQ_h
  b_dq = b_scores; b_dq.a1 = hq * TT; b_dq.a2 = TT; b_dq.c1 = Trow; b_dq.c2 = hd;
  // per (sequence, KV head), one query head of the group at a time: dS_h^T Q_h -> dK, P_h^T dO_h -> dV
  b_dk.nh = hkv; b_dk.bdiv = 1; b_dk.count = S_ * hkv;
  b_dk.a1 = hq * TT; b_dk.a2 = rep * TT; b_dk.b1 = Trow; b_dk.b2 = (long)rep * hd; b_dk.c1 = Trow; b_dk.c2 = hd;
  b_dv = b_dk; b_dv.b1 = Tq;
  b_scores.causal = 1; b_dp.causal = 1; b_pv.causal = 2; b_dq.causal = 2; b_dk.causal = 3; b_dv.causal = 3;

  // The projections and the LM head run on the packed GEMM (k_gemm_x3); forms as in sgemm<TA, TB>.
  const int NP = tr->pieces;
  const X3Bufs xh{p.packa, p.packb, p.packa_cap, p.packb_cap, NP, p.kparts, split_parts_floats(D), 0};   // of the LM head's products
  X3Bufs xb = xh;                                                                                       // of the layers'
  xb.left_out = (int)(S * T - M);
  // Forward products are split over K with three pieces only: with two and one a sequence's log-probs do not depend on the
  // batch around it (where operands are rounded to bf16 a last bit decides roundings downstream, about 1e-2 of a log-prob
  // after 24 layers).
  const bool split_fwd = NP == 3;
  struct Mat { const float* x; int ld; uint32_t *row_mx, *col_mx; };   // a matrix by rows, with its maxima
  auto mm_nt = [&](const Mat& X, const Mat& W, float* C, int ldc, int M_, int N_, int K_, float beta,
                   const float* Cin = nullptr, const X3Bufs* bufs = nullptr, const void* w_packed = nullptr) {   // C = beta Cin + X W^T
    return gemm_x3(X3Op{X.x, X.ld, M_, K_, false, X.row_mx, X.col_mx}, X3Op{W.x, W.ld, N_, K_, false, W.row_mx, W.col_mx}, C, Cin, ldc,
                   beta, bufs ? *bufs : xb, st, w_packed, split_fwd);
  };
  auto mm_nn = [&](const Mat& A_, const Mat& B_, float* C, int ldc, int M_, int N_, int K_, float beta,
                   const X3Bufs* bufs = nullptr, const void* b_packed = nullptr) {   // C = beta C + A B
    return gemm_x3(X3Op{A_.x, A_.ld, M_, K_, false, A_.row_mx, A_.col_mx}, X3Op{B_.x, B_.ld, N_, K_, true, B_.col_mx, nullptr}, C, C, ldc,
                   beta, bufs ? *bufs : xb, st, b_packed);
  };
  auto mm_tn = [&](const Mat& A_, const Mat& B_, float* C, int Mg, int Ng, int Kg, float beta, const X3Bufs* bufs = nullptr) {   // C = beta C + A^T B
    return gemm_x3_tn(A_.x, A_.ld, B_.x, B_.ld, C, Mg, Ng, Kg, beta, bufs ? *bufs : xb, st, A_.col_mx, B_.col_mx);
  };
  auto rows_max = [&](const float* x, int K_, uint32_t* out) { return NP == 3 ? row_max(x, Mi, K_, out, st) : hipSuccess; };
  if (NP == 3 && !first) T_CK(g_fill_f32((float*)p.mx_zero, 0.f, p.mx_zero_n, st));   // the first micro-batch: with head_c

  const int blocks64 = (Mi + 127) / 128 * 2;   // blocks of 64 tokens that a packed operand by rows of tokens holds
  // ---- forward, every activation kept
  float* h = p.layer[0].h;
  T_CK(launch(KID_EMBED, k_embed_rows, dim3(Mi), dim3(256), 0, st, row_tokens, (const float*)TH(0), h, d, V));
  for (int l = 0; l < D.L; ++l) {
    const LayerActs& a = p.layer[l];
    const LayerMax& mx = p.mx[l];
    const int t0 = 1 + 9 * l;   // attn_norm, wq, wk, wv, wo, ffn_norm, w_gate, w_up, w_down
    T_CK(rmsnorm_fwd(a.h, TH(t0), c.rms_eps, Mi, d, a.xn, a.r1, NP == 3 ? p.xn_r : nullptr, st));
    T_CK(mm_nt(Mat{a.xn, d, p.xn_r, mx.xn_c}, Mat{TH(t0 + 1), d, mx.wqkv_r, mx.wqkv_c}, a.qkv, nqkv, Mi, nqkv, d, 0.f));   // wq, wk, wv are adjacent
    if (tr->use_bias) T_CK(g_add_row_bias(a.qkv, TH(tr->n_in + l), Mi, nqkv, st));
    {
      const size_t total = M * (size_t)(hq + hkv) * (hd / 2);
      T_CK(launch(KID_ROPE_APPEND, k_rope, dim3(blocks256(total)), dim3(256), 0, st, a.qkv, (const float2*)tr->rope, (int)T,
                  (const int*)pk.pos, hq + hkv, hd, nqkv, 1.0f, total));
    }
    if (fused_attn) {
      const dim3 ag(hq, (unsigned)S, (unsigned)((T + 63) / 64));
      uint32_t* const ao_r = NP == 3 ? mx.ao_r : nullptr;
      auto fwd = [&](auto kernel) {
        return launch(KID_ATTN_GENERIC, kernel, ag, dim3(256), 0, st, (const float*)a.qkv, (int)T, (const int*)pk.first, hq, hkv, att_scale, a.ao,
                      a.lse, ao_r);
      };
      hipError_t e = hipErrorInvalidValue;
      if (hd == 16) e = NP == 3 ? fwd(k_tattn_fwd<16, 4>) : fwd(k_tattn_fwd<16, 1>);
      if (hd == 32) e = NP == 3 ? fwd(k_tattn_fwd<32, 4>) : fwd(k_tattn_fwd<32, 1>);
      if (hd == 64) e = NP == 3 ? fwd(k_tattn_fwd<64, 4>) : fwd(k_tattn_fwd<64, 1>);
      if (hd == 128) e = NP == 3 ? fwd(k_tattn_fwd<128, 4>) : fwd(k_tattn_fwd<128, 1>);
      T_CK(e);
    } else {
      T_CK((sgemm<0, 1>(a.qkv, nqkv, a.qkv + q, nqkv, p.prob, (int)T, (int)T, (int)T, hd, 0.f, st, b_scores)));
      T_CK(launch(KID_ATTN_GENERIC, k_softmax_causal, dim3((unsigned)(S * hq * T)), dim3(64), 0, st, p.prob, a.lse, (int)T,
                  att_scale));
      T_CK((sgemm<0, 0>(p.prob, (int)T, a.qkv + q + kv, nqkv, a.ao, q, (int)T, hd, (int)T, 0.f, st, b_pv)));
      T_CK(rows_max(a.ao, q, mx.ao_r));
    }
    T_CK(mm_nt(Mat{a.ao, q, mx.ao_r, mx.ao_c}, Mat{TH(t0 + 4), q, mx.wo_r, mx.wo_c}, a.h2, d, Mi, d, q, 1.f, a.h));
    T_CK(rmsnorm_fwd(a.h2, TH(t0 + 5), c.rms_eps, Mi, d, a.xn2, a.r2, NP == 3 ? p.xn_r : nullptr, st));
    T_CK(mm_nt(Mat{a.xn2, d, p.xn_r, mx.xn2_c}, Mat{TH(t0 + 6), d, mx.wgu_r, mx.wgu_c}, a.gu, 2 * F, Mi, 2 * F, d, 0.f));   // w_gate, w_up are adjacent
    float* h_next = (l + 1 < D.L) ? p.layer[l + 1].h : p.h_last;
    if (p.packed_ffn) {
      auto pack = [&](auto kernel, dim3 grid, int threads) {
        return launch(KID_SWIGLU, kernel, grid, dim3(threads), 0, st, (const float*)a.gu, Mi, F, x3_steps(F), (u32x4_t*)p.packa, mx.act_r);
      };
      const dim3 tiles(F / 64, blocks64);
      if (NP == 3) {
        const dim3 rows_grid(blocks64 * (64 / kActRows));
        T_CK(F <= 5 * kActStep ? pack(k_swiglu_fwd_pack_rows<5>, rows_grid, 512) : F <= 9 * kActStep ? pack(k_swiglu_fwd_pack_rows<9>, rows_grid, 512)
                                                                                             : pack(k_swiglu_fwd_pack_rows<0>, rows_grid, 512));
      } else {
        T_CK(NP == 2 ? pack(k_swiglu_fwd_pack<2>, tiles, 256) : pack(k_swiglu_fwd_pack<1>, tiles, 256));
      }
      T_CK(gemm_x3(X3Op{nullptr, 0, Mi, F, false, mx.act_r, nullptr}, X3Op{TH(t0 + 8), F, d, F, false, mx.wd_r, mx.wd_c}, h_next, a.h2, d, 1.f,
                   xb, st, nullptr, split_fwd, p.packa));
      continue;
    }
    if (F % 4 == 0 && M <= 65535) {
      T_CK(launch(KID_SWIGLU, k_swiglu_fwd4, dim3((F / 4 + 255) / 256, Mi), dim3(256), 0, st, (const float*)a.gu, a.act, F,
                  NP == 3 ? mx.act_r : nullptr));
    } else {
      T_CK(launch(KID_SWIGLU, k_swiglu_fwd, dim3(blocks256(M * D.F)), dim3(256), 0, st, (const float*)a.gu, a.act, F, M * D.F));
      T_CK(rows_max(a.act, F, mx.act_r));
    }
    T_CK(mm_nt(Mat{a.act, F, mx.act_r, mx.act_c}, Mat{TH(t0 + 8), F, mx.wd_r, mx.wd_c}, h_next, d, Mi, d, F, 1.f, a.h2));
  }
  T_CK(rmsnorm_fwd(p.h_last, TH(t_final), c.rms_eps, Mi, d, p.xf, p.rf, NP == 3 ? p.xn_r : nullptr, st));

  // ---- LM head, over the rows that predict a masked token only (the others have no log-prob to report and a zero
  // d logits row): their final-normed rows gathered, then chunks of them: logits, log-probs, d logits, d rows (into
  // p.dh, scattered to p.dx afterwards) and d head
  T_CK(g_fill_f32(logp_new, 0.f, S * T, st));
  T_CK(g_fill_f32(p.dx, 0.f, M * D.d, st));
  // the embedding's gradient is added up row by row, by the head's rows first where the two are one tensor
  if (first && t_head != 0) T_CK(g_fill_f32(GR(0), 0.f, D.V * D.d, st));
  if (first && n_rows == 0) T_CK(g_fill_f32(GR(t_head), 0.f, D.V * D.d, st));
  if (n_rows > 0) {
    T_CK(launch(KID_MISC, k_move_rows, dim3(n_rows), dim3(256), 0, st, (const float*)p.xf, rows, d, 0, p.xfc, (const uint32_t*)p.xn_r,
                p.xfc_r));
    for (size_t r0 = 0; r0 < (size_t)n_rows; r0 += p.chunk) {
      const int R = (int)(((size_t)n_rows - r0 < p.chunk) ? (size_t)n_rows - r0 : p.chunk);
      const Mat xfc{p.xfc + r0 * D.d, d, p.xfc_r + r0, p.xfc_c}, logits{p.logits, V, p.dl_r, p.dl_c}, head{TH(t_head), d, p.head_r, p.head_c};
      T_CK(mm_nt(xfc, head, p.logits, V, R, V, d, 0.f, nullptr, &xh, p.head_nt));
      T_CK(launch(KID_SCORE_ROWS, k_logp_dlogits, dim3(R), dim3(kLogpThreads), 0, st, p.logits, V, token_rows + r0, (int)T, tokens, completion_mask,
                  logp_old, advantages, eps_low, eps_high, (const long long*)p.n_masked, logp_new, p.dl_r));
      T_CK(mm_nn(logits, head, p.dh + r0 * D.d, d, R, d, V, 0.f, &xh, p.head_t));
      T_CK(mm_tn(logits, xfc, GR(t_head), V, d, R, r0 == 0 ? keep : 1.f, &xh));
    }
    T_CK(launch(KID_MISC, k_move_rows, dim3(n_rows), dim3(256), 0, st, (const float*)p.dh, rows, d, 1, p.dx, (const uint32_t*)nullptr,
                (uint32_t*)nullptr));
  }
  // ---- backward through the layers
  const int n_gpart = (Mi + 255) / 256;
  auto norm_bwd = [&](const float* dxn, const float* hin, const float* rstd, int gain_tensor_idx, int accumulate) -> hipError_t {
    if (norm_rows_vectorised(d)) {
      const int n_part = (Mi + kNormRows - 1) / kNormRows;
      const hipError_t e = with_norm_width(d, [&](auto nv) {
        constexpr int NV = decltype(nv)::value;
        return launch(KID_RMSNORM, NP == 3 ? k_rmsnorm_bwd_rows<NV, true> : k_rmsnorm_bwd_rows<NV, false>, dim3(n_part), dim3(256), 0, st, dxn,
                      hin, rstd, (const float*)TH(gain_tensor_idx), Mi, d, p.dh, accumulate, p.gpart, p.dh_r);
      });
      if (e != hipSuccess) return e;
      return launch(KID_MISC, k_gain_sum, dim3((d + 15) / 16), dim3(256), 0, st, (const float*)p.gpart, n_part, d, !first, GR(gain_tensor_idx));
    }
    hipError_t e = launch(KID_MISC, k_gain_grad_partial, dim3((d + 255) / 256, n_gpart), dim3(256), 0, st, dxn, hin, rstd, Mi, d,
                          p.gpart);
    if (e != hipSuccess) return e;
    e = launch(KID_MISC, k_gain_grad_finish, dim3((d + 255) / 256), dim3(256), 0, st, (const float*)p.gpart, n_gpart, d, !first,
               GR(gain_tensor_idx));
    if (e != hipSuccess) return e;
    e = launch(KID_RMSNORM, k_rmsnorm_bwd, dim3(Mi), dim3(256), 0, st, dxn, hin, rstd, (const float*)TH(gain_tensor_idx), d,
               p.dh, accumulate);
    return e != hipSuccess ? e : rows_max(p.dh, d, p.dh_r);
  };
  T_CK(norm_bwd(p.dx, p.h_last, p.rf, t_final, 0));
  for (int l = D.L - 1; l >= 0; --l) {
    const LayerActs& a = p.layer[l];
    const int t0 = 1 + 9 * l;
    const LayerMax& mx = p.mx[l];
    // down projection
    const Mat dh1{p.dh, d, p.dh_r, mx.dh1_c}, dh2{p.dh, d, p.dh_r, mx.dh2_c};   // the residual gradient before and after the FFN's norm
    T_CK(mm_nn(dh1, Mat{TH(t0 + 8), F, mx.wd_r, mx.wd_c}, p.dact, F, Mi, F, d, 0.f));
    if (p.packed_ffn) {
      const int KB_rows = x3_steps(2 * F), KB_cols = x3_steps(Mi);
      const SwigluMax maxima{mx.dgu_r, mx.dgu_c, mx.act_c};
      auto pack = [&](auto kernel) {
        return launch(KID_SWIGLU, kernel, dim3(F / 64, blocks64), dim3(256), 0, st, (const float*)p.dact, (const float*)a.gu, Mi, F, KB_rows,
                      (u32x4_t*)p.packa, KB_cols, (u32x4_t*)p.dgu, (u32x4_t*)p.act_cols, maxima);
      };
      if (NP == 3)
        T_CK(launch(KID_SWIGLU, k_swiglu_bwd_max, dim3(F / 64, (Mi + 255) / 256), dim3(256), 0, st, (const float*)p.dact, (const float*)a.gu, Mi, F,
                    maxima));
      T_CK(NP == 3 ? pack(k_swiglu_bwd_pack<3>) : NP == 2 ? pack(k_swiglu_bwd_pack<2>) : pack(k_swiglu_bwd_pack<1>));
      // gate / up projections, then the down projection's weights
      T_CK(gemm_x3(X3Op{nullptr, 0, Mi, 2 * F, false, mx.dgu_r, nullptr}, X3Op{TH(t0 + 6), d, d, 2 * F, true, mx.wgu_c, nullptr}, p.dx, p.dx, d,
                   0.f, xb, st, nullptr, true, p.packa));
      T_CK(gemm_x3(X3Op{nullptr, 0, 2 * F, Mi, true, mx.dgu_c, nullptr}, X3Op{a.xn2, d, d, Mi, true, mx.xn2_c, nullptr}, GR(t0 + 6), GR(t0 + 6), d,
                   keep, xb, st, nullptr, true, p.dgu, true));
      T_CK(gemm_x3(X3Op{p.dh, d, d, Mi, true, mx.dh1_c, nullptr}, X3Op{nullptr, 0, F, Mi, true, mx.act_c, nullptr}, GR(t0 + 8), GR(t0 + 8), F, keep,
                   xb, st, p.act_cols, true, nullptr, true));
    } else {
      T_CK(mm_tn(dh1, Mat{a.act, F, mx.act_r, mx.act_c}, GR(t0 + 8), d, F, Mi, keep));
      if (F % 4 == 0 && M <= 65535) {
        T_CK(launch(KID_SWIGLU, k_swiglu_bwd4, dim3((F / 4 + 255) / 256, Mi), dim3(256), 0, st, (const float*)p.dact,
                    (const float*)a.gu, p.dgu, F, NP == 3 ? mx.dgu_r : nullptr));
      } else {
        T_CK(launch(KID_SWIGLU, k_swiglu_bwd, dim3(blocks256(M * D.F)), dim3(256), 0, st, (const float*)p.dact, (const float*)a.gu,
                    p.dgu, F, M * D.F));
        T_CK(rows_max(p.dgu, 2 * F, mx.dgu_r));
      }
      const Mat dgu{p.dgu, 2 * F, mx.dgu_r, mx.dgu_c};
      T_CK(mm_nn(dgu, Mat{TH(t0 + 6), d, mx.wgu_r, mx.wgu_c}, p.dx, d, Mi, d, 2 * F, 0.f));
      T_CK(mm_tn(dgu, Mat{a.xn2, d, nullptr, mx.xn2_c}, GR(t0 + 6), 2 * F, d, Mi, keep));
    }
    T_CK(norm_bwd(p.dx, a.h2, a.r2, t0 + 5, 1));
    // output projection
    T_CK(mm_nn(dh2, Mat{TH(t0 + 4), q, mx.wo_r, mx.wo_c}, p.dao, q, Mi, q, d, 0.f));
    T_CK(mm_tn(dh2, Mat{a.ao, q, mx.ao_r, mx.ao_c}, GR(t0 + 4), d, q, Mi, keep));
    // attention and the rotary embedding; dgu is free here and takes the partial dk / dv
    float* kv_parts = fused_attn && rep > 1 && 2 * D.F >= 2 * D.q ? p.dgu : nullptr;
    if (fused_attn) {
      hipError_t e = hipErrorInvalidValue;
      auto bwd = [&](auto f) { return f(a.qkv, a.ao, p.dao, a.lse, S_, T_, pk.first, M, hq, hkv, att_scale, p.dqkv, p.delta, kv_parts, st); };
      if (hd == 16) e = NP == 3 ? bwd(tattn_bwd<16, 4>) : bwd(tattn_bwd<16, 1>);
      if (hd == 32) e = NP == 3 ? bwd(tattn_bwd<32, 4>) : bwd(tattn_bwd<32, 1>);
      if (hd == 64) e = NP == 3 ? bwd(tattn_bwd<64, 4>) : bwd(tattn_bwd<64, 1>);
      if (hd == 128) e = NP == 3 ? bwd(tattn_bwd<128, 4>) : bwd(tattn_bwd<128, 1>);
      T_CK(e);
    } else {
      T_CK((sgemm<0, 1>(a.qkv, nqkv, a.qkv + q, nqkv, p.prob, (int)T, (int)T, (int)T, hd, 0.f, st, b_scores)));
      T_CK(launch(KID_ATTN_GENERIC, k_probs_from_lse, dim3(blocks256(n_sc)), dim3(256), 0, st, p.prob, (const float*)a.lse, (int)T,
                  att_scale, n_sc));
      T_CK((sgemm<0, 1>(p.dao, q, a.qkv + q + kv, nqkv, p.dsc, (int)T, (int)T, (int)T, hd, 0.f, st, b_dp)));     // dP = dO V^T
      T_CK(launch(KID_ATTN_GENERIC, k_attn_delta, dim3((unsigned)(M * hq)), dim3(64), 0, st, (const float*)p.dao, (const float*)a.ao,
                  (int)T, hq, hd, p.delta));
      T_CK(launch(KID_ATTN_GENERIC, k_dscores, dim3(blocks256(n_sc)), dim3(256), 0, st, (const float*)p.prob, p.dsc,
                  (const float*)p.delta, (int)T, att_scale, n_sc));
      T_CK((sgemm<0, 0>(p.dsc, (int)T, a.qkv + q, nqkv, p.dqkv, nqkv, (int)T, hd, (int)T, 0.f, st, b_dq)));       // dQ = dS K
      const bool one_launch = T % 16 == 0 && hd % 4 == 0 && nqkv % 4 == 0 && q % 4 == 0 && (long)T * hd * S_ * hkv >= 128 * 128;
      if (one_launch) {   // the query heads of a group are segments of one contraction (added in head order)
        Batch kd = b_dk, vd = b_dv;
        kd.kseg = vd.kseg = (int)T;
        kd.sega = vd.sega = TT;
        kd.segb = vd.segb = hd;
        T_CK((sgemm<1, 0>(p.dsc, (int)T, a.qkv, nqkv, p.dqkv + q, nqkv, (int)T, hd, rep * (int)T, 0.f, st, kd)));        // dK = sum_h dS_h^T Q_h
        T_CK((sgemm<1, 0>(p.prob, (int)T, p.dao, q, p.dqkv + q + kv, nqkv, (int)T, hd, rep * (int)T, 0.f, st, vd)));     // dV = sum_h P_h^T dO_h
      }
      for (int hh = 0; hh < (one_launch ? 0 : rep); ++hh) {   // otherwise one launch per head of the group, in order
        const float beta = hh > 0 ? 1.f : 0.f;
        T_CK((sgemm<1, 0>(p.dsc + (size_t)hh * T * T, (int)T, a.qkv + (size_t)hh * hd, nqkv, p.dqkv + q, nqkv, (int)T, hd, (int)T,
                          beta, st, b_dk)));                                                                       // dK += dS^T Q
        T_CK((sgemm<1, 0>(p.prob + (size_t)hh * T * T, (int)T, p.dao + (size_t)hh * hd, q, p.dqkv + q + kv, nqkv, (int)T, hd,
                          (int)T, beta, st, b_dv)));                                                               // dV += P^T dO
      }
    }
    if (kv_parts) {
      T_CK(launch(KID_ROPE_APPEND, k_attn_bwd_finish, dim3(Mi), dim3(256), 0, st, p.dqkv, (const float*)kv_parts, rep,
                  M * 2 * D.kv, (const float2*)tr->rope, (int)T, (const int*)pk.pos, hq, hkv, hd, NP == 3 ? mx.dqkv_r : nullptr));
    } else {
      const size_t total = M * (size_t)(hq + hkv) * (hd / 2);
      T_CK(launch(KID_ROPE_APPEND, k_rope, dim3(blocks256(total)), dim3(256), 0, st, p.dqkv, (const float2*)tr->rope, (int)T,
                  (const int*)pk.pos, hq + hkv, hd, nqkv, -1.0f, total));
      T_CK(rows_max(p.dqkv, nqkv, mx.dqkv_r));
    }
    if (tr->use_bias) {   // the biases enter before the rotary embedding: their gradient is the column sum of dqkv here
      T_CK(launch(KID_MISC, k_colsum_partial, dim3((nqkv + 255) / 256, n_gpart), dim3(256), 0, st, (const float*)p.dqkv, Mi, nqkv,
                  p.gpart));
      T_CK(launch(KID_MISC, k_gain_grad_finish, dim3((nqkv + 255) / 256), dim3(256), 0, st, (const float*)p.gpart, n_gpart, nqkv,
                  !first, GR(tr->n_in + l)));
    }
    // query / key / value projections
    const Mat dqkv{p.dqkv, nqkv, mx.dqkv_r, mx.dqkv_c};
    T_CK(mm_nn(dqkv, Mat{TH(t0 + 1), d, mx.wqkv_r, mx.wqkv_c}, p.dx, d, Mi, d, nqkv, 0.f));
    T_CK(mm_tn(dqkv, Mat{a.xn, d, nullptr, mx.xn_c}, GR(t0 + 1), nqkv, d, Mi, keep));
    T_CK(norm_bwd(p.dx, a.h, a.r1, t0, 1));
  }
  T_CK(launch(KID_EMBED, k_embed_order, dim3((Mi + kEmbedChunk - 1) / kEmbedChunk), dim3(1024), 0, st, row_tokens, Mi, V, p.eorder));
  for (int m0 = 0; m0 < Mi; m0 += kEmbedChunk) {
    const int n = std::min(kEmbedChunk, Mi - m0);
    T_CK(launch(KID_EMBED, k_embed_add, dim3(n, (d + 255) / 256), dim3(64), 0, st, row_tokens + m0, (const int*)(p.eorder + m0), n,
                (const float*)(p.dh + (size_t)m0 * D.d), d, V, GR(0)));
  }

  return SAPO_OK;
}

extern "C" int sapo_policy_update(sapo_trainer* tr, const int32_t* tokens, const uint8_t* completion_mask,
                                  const float* logp_old, const float* advantages, int S_, int T_, float eps_low,
                                  float eps_high, float* out_loss, float* out_logp_new, void* workspace,
                                  size_t workspace_bytes, void* stream) {
  if (!tr || !tokens || !completion_mask || !logp_old || !advantages || !out_loss || !workspace)
    return set_error(SAPO_EINVAL, "NULL argument");
  if (S_ <= 0 || T_ < 2) return set_error(SAPO_EINVAL, "S must be positive and T at least 2");
  if (T_ > tr->cfg.max_seq) return set_error(SAPO_EINVAL, "T = %d exceeds max_seq = %d", T_, tr->cfg.max_seq);
  if (T_ > 8192) return set_error(SAPO_EINVAL, "at most 8192 tokens per sequence");
  if (!(eps_low >= 0.f && eps_low < 1.f) || !(eps_high >= 0.f)) return set_error(SAPO_EINVAL, "eps_low in [0, 1), eps_high >= 0");
  const sapo_model_config& c = tr->cfg;
  const Dims D(c);
  const size_t S = S_, T = T_, M = S * T;
  if (M >= ((size_t)1 << 30)) return set_error(SAPO_EINVAL, "batch too large");
  // Micro-batches: the largest number of sequences whose activations fit the workspace is pushed through forward
  // and backward at a time, the gradients adding up; the whole set at once when the workspace allows it.
  TrainPlan p;
  size_t S_mb = S;
  // grid limits: sequences per launch of the fused attention kernels, (sequence, query head) pairs of a batched GEMM
  const size_t most = fused_attention(c) ? (size_t)65535 : (size_t)65535 / c.n_q_heads;
  if (S_mb > most) S_mb = most;
  make_plan(c, S_mb, T, S, nullptr, p);
  if (workspace_bytes < p.bytes) {
    size_t lo = 0, hi = S_mb;   // plan(lo) fits (lo = 0: nothing known to fit), plan(hi) does not
    while (hi - lo > 1) {
      const size_t mid = (lo + hi) / 2;
      make_plan(c, mid, T, S, nullptr, p);
      if (p.bytes <= workspace_bytes) lo = mid; else hi = mid;
    }
    if (lo == 0) {
      make_plan(c, 1, T, S, nullptr, p);
      return set_error(SAPO_EWORKSPACE, "workspace is %zu bytes, at least %zu needed (one sequence at a time)", workspace_bytes,
                       p.bytes);
    }
    S_mb = lo;
  }
  make_plan(c, S_mb, T, S, (char*)workspace, p);
  hipStream_t st = (hipStream_t)stream;
  const int t_head = c.tied_embeddings ? 0 : 1 + 9 * c.n_layers + 1;
  const int d = (int)D.d, V = (int)D.V;
  T_CK(launch(KID_MISC, k_count_mask, dim3(1), dim3(256), 0, st, completion_mask, M, p.n_masked));
  const int NP = tr->pieces;
  const float* head = tr->theta + tr->off[t_head];
  if (NP == 3) {   // maxima of the weights' rows
    RowMaxTasks t;
    t.n = 0;
    unsigned blocks = 0;
    auto flush = [&]() {
      const hipError_t e = launch(KID_MISC, k_row_max, dim3(blocks), dim3(256), 0, st, t);
      t.n = 0;
      blocks = 0;
      return e;
    };
    auto add = [&](const float* src, size_t rows, size_t K, uint32_t* out) -> hipError_t {
      t.t[t.n++] = RowMaxTask{src, out, (int)rows, (int)K, blocks};
      blocks += (unsigned)((rows + 3) / 4);
      return t.n == kRowMaxTasks ? flush() : hipSuccess;
    };
    T_CK(add(head, D.V, D.d, p.head_r));
    for (int l = 0; l < D.L; ++l) {
      auto w = [&](int k) { return tr->theta + tr->off[1 + 9 * l + k]; };
      T_CK(add(w(1), D.nqkv, D.d, p.mx[l].wqkv_r));
      T_CK(add(w(4), D.d, D.q, p.mx[l].wo_r));
      T_CK(add(w(6), 2 * D.F, D.d, p.mx[l].wgu_r));
      T_CK(add(w(8), D.d, D.F, p.mx[l].wd_r));
    }
    if (t.n > 0) T_CK(flush());
    T_CK(g_fill_f32((float*)p.head_c, 0.f, (size_t)(p.mx_zero - p.head_c) + p.mx_zero_n, st));
  }
  T_CK(x3_pack(X3Op{head, d, V, d, false, p.head_r, p.head_c}, p.head_nt, p.head_cap, NP, st));        // rows = vocabulary
  T_CK(x3_pack(X3Op{head, d, d, V, true, p.head_c, nullptr}, p.head_t, p.head_t_cap, NP, st));       // rows = d
  // The rows that predict a masked token, per micro-batch (indices within it, ascending), and how many there are:
  // the host needs the numbers to size the LM head's GEMMs, so the call waits here once, before the forward passes
  // are enqueued, for these small kernels (and for whatever the stream held before).
  const size_t n_mb = (S + S_mb - 1) / S_mb;
  std::vector<int> counts(2 * n_mb, 0);
  const int *n_rows = counts.data(), *n_needed = n_rows + n_mb;
  for (size_t i = 0; i < n_mb; ++i) {
    const size_t s0 = i * S_mb;
    const int n = (int)(S - s0 < S_mb ? S - s0 : S_mb);
    T_CK(g_masked_rows(completion_mask + s0 * T, T_, 0, n, p.mpos, p.mrows + s0 * T, p.mcount + i, st));
    T_CK(g_packed_lens(completion_mask + s0 * T, T_, 0, n, false, (int2*)p.eorder, st));
    T_CK(launch(KID_MISC, k_packed_count, dim3(1), dim3(256), 0, st, (const int2*)p.eorder, n, p.mcount + n_mb + i));
  }
  T_CK(hipMemcpyAsync(counts.data(), p.mcount, 2 * n_mb * sizeof(int), hipMemcpyDeviceToHost, st));
  T_CK(hipStreamSynchronize(st));
  for (size_t i = 0; i < n_mb; ++i) {
    const size_t s0 = i * S_mb;
    const int n = (int)(S - s0 < S_mb ? S - s0 : S_mb);
    if (n_rows[i] < 0 || (size_t)n_rows[i] > (size_t)n * T || n_needed[i] < 0 || (size_t)n_needed[i] > (size_t)n * T)
      return set_error(SAPO_EHIP, "row count read back from the device is out of range");
    // without the rows that nothing depends on, where they are enough
    const bool packs = fused_attention(c) && leaves_rows_out((size_t)n * T, (size_t)n_needed[i], least_update_rows(tr->pieces));
    const int rc = update_rows(tr, p, tokens + s0 * T, completion_mask + s0 * T, logp_old + s0 * T, advantages + s0, n, T_,
                               eps_low, eps_high, p.logp_all + s0 * T, p.mrows + s0 * T, n_rows[i], packs ? n_needed[i] : 0, i == 0, st);
    if (rc != SAPO_OK) return rc;
  }
  // ---- the loss (the surrogate of sapo_clipped_surrogate on the log-probs just computed)
  T_CK(g_surrogate_loss(p.logp_all, logp_old, completion_mask, advantages, S_, T_, eps_low, eps_high, p.loss, nullptr, p.sur_ws,
                        st));
  T_CK(hipMemcpyAsync(out_loss, p.loss, sizeof(float), hipMemcpyDeviceToDevice, st));
  if (out_logp_new) T_CK(hipMemcpyAsync(out_logp_new, p.logp_all, M * sizeof(float), hipMemcpyDeviceToDevice, st));

  // ---- Adam
  tr->t += 1;
  const float c1 = (float)(1.0 - pow((double)tr->opt.beta1, (double)tr->t));
  const float c2 = (float)(1.0 - pow((double)tr->opt.beta2, (double)tr->t));
  T_CK(launch(KID_MISC, k_adam, dim3(blocks256(tr->n_params)), dim3(256), 0, st, tr->theta, (const float*)tr->grad, tr->m, tr->v,
              tr->n_params, tr->opt.lr, tr->opt.beta1, tr->opt.beta2, tr->opt.eps, c1, c2));
  return SAPO_OK;
}
