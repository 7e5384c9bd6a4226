// FFN of a decode step with 65 .. 256 rows: gate/up + SwiGLU, and the down projection split over K with the kernel that
// adds its parts to the residual.  Operands as in kernels_mfma.hip (X32 / W32 order, IEEE half).
//
// What bounds it is what a compute unit takes in: its loads return in the order they were asked for, whichever wave asked,
// so rows that lie in the L2 (150 GB/s on their own) queue behind weights that come from HBM, and the two times add up.
// A kernel that only reads 384 KB of weights and 768 KB of shared rows per workgroup takes 22 us on 140 compute units,
// as the 1.5B gate/up projection did on 140 tiles of 256 x 128 (23 us; 20 without its weights, 20 without its rows, 21.5
// without its MFMAs; deeper rings changed nothing).  So: workgroups of 128 rows x NB 32-feature blocks, NB such that they
// are just about as many as the compute units; no pass over the rows in front (the O projection leaves them normalised but
// for the scale, with their sums of squares); 8 parts over K instead of 16 .. 32 and the parts as they lie in the registers.
// us per step, tiles of 128 / 256 x 128 -> these kernels: 0.5B 1123 -> 925 (72 rows), 1196 -> 973 (128), 1358 -> 1106 (192),
// 1531 -> 1172 (256); 1.5B 1865 -> 1672 (96), 1960 -> 1777 (128), 2267 -> 2051 (192), 2472 -> 2162 (256).  Launches at 192
// rows, 0.5B: norm 5.0 + gate/up 11.6 -> 10.5, down 10.9 -> 7.0, adding the parts 5.6 -> 4.6; 1.5B at 256: 5.3 + 23.2 ->
// 22.1, 18.6 -> 14.9, 6.2 -> 5.2.
#include "tiles.h"
#include <type_traits>

namespace sapo {

// The k loop: 4 waves, each 32 rows x NB feature blocks, stages of 64 k.  A wave's rows go straight into its registers, the
// weights, which all four read, through an LDS ring; kAhead stages of both are requested ahead.  With one workgroup per
// compute unit nobody else covers a wave's waits, so the fragments of a 16-k step are read while the step before is
// multiplied, the first ones of a stage in front of the last step of the stage before.
template <int NB>
struct RowsLoop {
  static constexpr int H = 4, kAhead = 3, R = kAhead + 1, PER = NB + H;   // requests per wave and stage
  static constexpr int kStage = NB * H * 1024, kBytes = R * kStage;
  u32x4 x[kAhead][H];
  Frag w[2][NB];
  const char *wbase, *xbase;
  unsigned woff[NB];   // this wave's ring copies: fragments wave NB .. wave NB + NB - 1 of a stage, fragment = block H + step
  unsigned off, ring;
  int nst;

  // rows of block tblk (past the last one, n_tblk - 1: its results are not stored), feature blocks fblk0 .. (past n_fblk - 1
  // likewise), n_stages stages of 64 k from 16-k step ks0 on
  __device__ __forceinline__ void begin(const uint4* Xp, const uint4* Wp, int tblk, int n_tblk, int fblk0, int n_fblk, int KS, int ks0,
                                        int n_stages, const uint4* smem) {
    const int wave = wave_index(threadIdx.x);
    xbase = (const char*)(Xp + ((size_t)min(tblk, n_tblk - 1) * KS + ks0) * 64);
    wbase = (const char*)(Wp + ((size_t)fblk0 * KS + ks0) * 64);
#pragma unroll
    for (int c = 0; c < NB; ++c) {
      const int i = wave * NB + c;
      woff[c] = (unsigned)((min(fblk0 + i / H, n_fblk - 1) - fblk0) * KS + i % H) * 1024u;
    }
    ring = __builtin_amdgcn_readfirstlane(lds_addr(smem)) + (unsigned)(wave * NB * 1024);
    off = (threadIdx.x & 63) * 16;
    nst = n_stages;
    first(std::integral_constant<int, 0>());
    if (nst > 1) first(std::integral_constant<int, 1>());
    if (nst > 2) first(std::integral_constant<int, 2>());
  }
  template <int C> __device__ __forceinline__ void request_w(int st) {
    dma16(wbase + woff[C] + (size_t)st * (H * 1024), off, ring + (unsigned)((st % R) * kStage + C * 1024));
  }
  template <int HH, int P> __device__ __forceinline__ void request_x(int st) {
    reg16<HH * 1024>(x[P][HH], xbase + (size_t)st * (H * 1024), off);
  }
  template <typename P> __device__ __forceinline__ void first(P) {
    constexpr int st = P::value;
    request_w<0>(st); request_w<1>(st);
    if constexpr (NB > 2) request_w<2>(st);
    if constexpr (NB > 3) request_w<3>(st);
    if constexpr (NB > 4) request_w<4>(st);
    request_x<0, st>(st); request_x<1, st>(st); request_x<2, st>(st); request_x<3, st>(st);
  }
  // Stage st has landed for every wave, and nobody reads stage st - 1 any more (its fragments are in registers: lgkmcnt 0).
  // DONE: requests of stage st + kAhead - 1 issued so far.
  template <int P, int DONE> __device__ __forceinline__ void arrive(int st) {
    auto wait = [](auto n) {
      constexpr int N = decltype(n)::value;
      __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (0 << 8) | ((N >> 4) << 14));
    };
    const int behind = nst - 1 - st;   // stages behind this one
    if (behind >= kAhead - 1) wait(std::integral_constant<int, PER * (kAhead - 2) + DONE>());
    else if (behind == 1) wait(std::integral_constant<int, PER>());
    else wait(std::integral_constant<int, 0>());
#pragma unroll
    for (int h = 0; h < H; ++h) landed(x[P][h]);
    wg_barrier();
  }
  template <int S> __device__ __forceinline__ void fragments(int st, int h, const uint4* smem) {
    const uint4* buf = smem + (st % R) * (NB * H * 64) + (threadIdx.x & 63);
#pragma unroll
    for (int f = 0; f < NB; ++f) w[S][f].u = buf[(f * H + h) * 64];
  }
  template <int P> __device__ __forceinline__ void stage(int st, const uint4* smem, f32x16 (&acc)[NB]) {
    const bool more = st + kAhead < nst;
    auto step = [&](auto hc) {
      constexpr int h = decltype(hc)::value, S = h & 1;
      if constexpr (h + 1 < H) {
        fragments<S ^ 1>(st, h + 1, smem);
      } else if (st + 1 < nst) {
        arrive<(P + 1) % kAhead, PER - 1>(st + 1);   // all but this step's own request
        fragments<S ^ 1>(st + 1, 0, smem);
      }
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(1);
      auto feature = [&](auto fc) {
        constexpr int f = decltype(fc)::value;
        if constexpr (f < NB) {
          Frag xx; xx.n = x[P][h];
          acc[f] = mfma32(w[S][f], xx, acc[f]);
          if constexpr (h == 0) {   // the ring copies go out one after each MFMA of the first step
            __builtin_amdgcn_sched_barrier(0);
            if (more) request_w<f>(st + kAhead);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      };
      feature(std::integral_constant<int, 0>()); feature(std::integral_constant<int, 1>()); feature(std::integral_constant<int, 2>());
      feature(std::integral_constant<int, 3>()); feature(std::integral_constant<int, 4>());
      __builtin_amdgcn_s_setprio(0);
      __builtin_amdgcn_sched_barrier(0);
      if (more) request_x<h, P>(st + kAhead);
      __builtin_amdgcn_sched_barrier(0);
    };
    step(std::integral_constant<int, 0>()); step(std::integral_constant<int, 1>());
    step(std::integral_constant<int, 2>()); step(std::integral_constant<int, 3>());
  }
  __device__ __forceinline__ void run(const uint4* smem, f32x16 (&acc)[NB]) {
#pragma unroll
    for (int f = 0; f < NB; ++f)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[f][v] = 0.f;
    arrive<0, PER>(0);
    fragments<0>(0, 0, smem);
    int st = 0;
    for (; st + kAhead <= nst; st += kAhead) {
      stage<0>(st, smem, acc);
      stage<1>(st + 1, smem, acc);
      stage<2>(st + 2, smem, acc);
    }
    if (st < nst) stage<0>(st, smem, acc);
    if (st + 1 < nst) stage<1>(st + 1, smem, acc);
  }
};

// Sum of a row's sums of squares, parts [parts][s_pad]: lanes l and l + 32 hold the same row and ask for every other part each,
// the first 2 NL of them in front of the k loop; they are added behind it, with what is left (more than 48 parts).
template <int NL> struct RowParts {
  float v[NL];
  __device__ __forceinline__ void request(const float* __restrict__ ssq, int parts, int s_pad, int row) {
    const int half = (threadIdx.x >> 5) & 1;
#pragma unroll
    for (int i = 0; i < NL; ++i) v[i] = ssq[(size_t)min(2 * i + half, parts - 1) * s_pad + row];
  }
  __device__ __forceinline__ float sum(const float* __restrict__ ssq, int parts, int s_pad, int row) const {
    const int half = (threadIdx.x >> 5) & 1;
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NL; ++i) s += (2 * i + half < parts) ? v[i] : 0.f;
    for (int i = 2 * NL + half; i < parts; i += 2) s += ssq[(size_t)i * s_pad + row];
    return sum_xor32(s);
  }
};

// The product of a wave whose rows do not all fit half as they lie: the rows that do not (`refit`, per lane) from the residual,
// normalised first, their scale then 1; the others as before to the bit (same values, same order).  Straight from global
// memory: this is there for correctness.
template <int NB>
__device__ __forceinline__ void refit_rows(const float* __restrict__ h_row, const float* __restrict__ gain, float eps, bool refit,
                                           const uint4* __restrict__ Wp, int fblk0, int n_fblk, int K, f32x16 (&acc)[NB], float& scale) {
  const int lane = threadIdx.x & 63, KS = K >> 4;
  float sum = 0.f;
#pragma clang loop unroll(disable)
  for (int k = (lane >> 5) * 4; k < K; k += 8) sum += sum_squares4(*(const float4*)(h_row + k));
  const float row_scale = rsqrtf(sum_xor32(sum) / (float)K + eps);
#pragma unroll
  for (int f = 0; f < NB; ++f)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[f][v] = 0.f;
#pragma clang loop unroll(disable)
  for (int ks = 0; ks < KS; ++ks) {
    const int k = ks * 16 + (lane >> 5) * 8;
    Frag x;
#pragma unroll
    for (int e = 0; e < 8; ++e) x.h[e] = from_f32<f16>((refit ? h_row[k + e] * row_scale : h_row[k + e]) * gain[k + e]);
#pragma unroll
    for (int f = 0; f < NB; ++f) {
      Frag w;
      w.u = Wp[((size_t)min(fblk0 + f, n_fblk - 1) * KS + ks) * 64 + lane];
      acc[f] = mfma32(w, x, acc[f]);
    }
  }
  scale = refit ? 1.f : scale;
}

// act = silu(gate) * up, half, in X32 order over F = 16 n_fblk.  A 32-feature block of the weights holds 16 gate rows
// and the 16 matching up rows: accumulator entries 4 r + j and 4 (r + 2) + j of a lane are a pair.
template <int NB, int NL>
__global__ void __launch_bounds__(256, 2) k_rows_gate_up(const uint4* __restrict__ Xp, const uint4* __restrict__ Wp,
                                                         const float* __restrict__ ssq, int M, int n_fblk, int K, int parts, int s_pad,
                                                         float eps, f16* __restrict__ act, const float* __restrict__ h,
                                                         const float* __restrict__ gain) {
  extern __shared__ uint4 smem[];
  const int n_tblk = (M + 31) >> 5, token_tiles = (n_tblk + 3) >> 2;
  // the token tiles of a feature tile run on one XCD at the same time: its weights come from HBM once
  const int j = blockIdx.x >> 3, by = j % token_tiles, bx = (j / token_tiles) * 8 + (blockIdx.x & 7);
  if (bx * NB >= n_fblk) return;
  const int wave = wave_index(threadIdx.x), lane = threadIdx.x & 63;
  const int tblk = by * 4 + wave, tok = tblk * 32 + (lane & 31);
  f32x16 acc[NB];
  RowParts<NL> rp;
  {
    RowsLoop<NB> loop;
    loop.begin(Xp, Wp, tblk, n_tblk, bx * NB, n_fblk, K >> 4, 0, K >> 6, smem);
    rp.request(ssq, parts, s_pad, min(tok, M - 1));
    loop.run(smem, acc);
  }
  if (tblk >= n_tblk) return;
  // Xp holds half(h * gain), scaled here: what half cannot hold of a row as it lies, it may hold of the normalised row.  That
  // is, if a value was clamped (an infinite part), or if the row is so small that half's spacing below 2^-14 counts: at a
  // root mean square of 2^-10, 2^-25 is an eighth of the rounding of a value of that size.
  const float mean = rp.sum(ssq, parts, s_pad, min(tok, M - 1)) / (float)K;
  float scale = rsqrtf(mean + eps);
  const bool refit = mean < 0x1p-20f || mean == INFINITY;
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(refit) != 0, 0))
    refit_rows<NB>(h + (size_t)min(tok, M - 1) * K, gain, eps, refit, Wp, bx * NB, n_fblk, K, acc, scale);
  if (tok >= M) return;
  const int F = n_fblk * 16;
#pragma unroll
  for (int f = 0; f < NB; ++f) {
    if (bx * NB + f >= n_fblk) break;
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const int f0 = (bx * NB + f) * 16 + 8 * r + (lane >> 5) * 4;
      f16x4 o;
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = from_f32<f16>(silu_f(acc[f][4 * r + i] * scale) * (acc[f][4 * (r + 2) + i] * scale));
      *(f16x4*)(act + x32_chunk(tok, f0, F >> 4) * 8 + (f0 & 4)) = o;
    }
  }
}

// Down projection, part z of kRowSplits over K: the accumulators go out as they lie in the registers (a wave's store is one
// contiguous KiB: [part][row block][feature block][r][lane] of 4 floats).  XCD z runs part z of every tile, so the part's K
// range of the token operand sits in one L2.
template <int NB>
__global__ void __launch_bounds__(256, 2) k_rows_down(const uint4* __restrict__ Xp, const uint4* __restrict__ Wp, int M, int n_fblk, int K,
                                                      float4* __restrict__ partial, int main_blocks, Prefetch pf) {
  extern __shared__ uint4 smem[];
  if ((int)blockIdx.x >= main_blocks) {
    prefetch_role<4>(pf, blockIdx.x - main_blocks, (int)gridDim.x - main_blocks, smem);
    return;
  }
  const int n_tblk = (M + 31) >> 5, token_tiles = (n_tblk + 3) >> 2;
  const int z = blockIdx.x & 7, j = blockIdx.x >> 3, by = j % token_tiles, bx = j / token_tiles;
  const int wave = wave_index(threadIdx.x), lane = threadIdx.x & 63;
  const int tblk = by * 4 + wave, nst = K >> 6;
  const int st0 = z * nst / kRowSplits, st1 = (z + 1) * nst / kRowSplits;
  f32x16 acc[NB];
  if (st1 > st0) {
    RowsLoop<NB> loop;
    loop.begin(Xp, Wp, tblk, n_tblk, bx * NB, n_fblk, K >> 4, st0 * 4, st1 - st0, smem);
    loop.run(smem, acc);
  } else {   // fewer stages than parts
#pragma unroll
    for (int f = 0; f < NB; ++f)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[f][v] = 0.f;
  }
  if (tblk >= n_tblk) return;
#pragma unroll
  for (int f = 0; f < NB; ++f) {
    if (bx * NB + f >= n_fblk) break;
    float4* out = partial + (((size_t)z * n_tblk + tblk) * n_fblk + bx * NB + f) * 256 + lane;
#pragma unroll
    for (int r = 0; r < 4; ++r) out[r * 64] = make_float4(acc[f][4 * r], acc[f][4 * r + 1], acc[f][4 * r + 2], acc[f][4 * r + 3]);
  }
}

// h += the parts of k_rows_down in part order; half(h * gain) in X16 order; sums of squares, ssq[part][s_pad], a part per
// workgroup of `per` feature blocks.  A workgroup per (feature blocks, row block), wave r the features 8 r .. 8 r + 7 of a
// block: every read of the parts is a contiguous KiB, all eight in flight.
__global__ void __launch_bounds__(256) k_rows_finish(const float4* __restrict__ partial, float* __restrict__ h,
                                                     const float* __restrict__ gain, int M, int n_fblk, int per, int s_pad,
                                                     f16* __restrict__ xp, float* __restrict__ ssq) {
  __shared__ float part[4][32];
  const int tblk = blockIdx.y, n_tblk = gridDim.y, d = n_fblk * 32;
  const int r = wave_index(threadIdx.x), lane = threadIdx.x & 63, tok = tblk * 32 + (lane & 31);
  float s = 0.f;
  for (int fblk = blockIdx.x * per; fblk < min(n_fblk, (int)(blockIdx.x + 1) * per); ++fblk) {
    const int f0 = fblk * 32 + 8 * r + (lane >> 5) * 4;
    float4 v = *(const float4*)(h + (size_t)min(tok, M - 1) * d + f0);
    const float4 g = *(const float4*)(gain + f0);
    float4 p[kRowSplits];
#pragma unroll
    for (int z = 0; z < kRowSplits; ++z) p[z] = partial[(((size_t)z * n_tblk + tblk) * n_fblk + fblk) * 256 + r * 64 + lane];
#pragma unroll
    for (int z = 0; z < kRowSplits; ++z) { v.x += p[z].x; v.y += p[z].y; v.z += p[z].z; v.w += p[z].w; }
    if (tok < M) {
      *(float4*)(h + (size_t)tok * d + f0) = v;
      f16x4 o;
      o[0] = from_f32<f16>(v.x * g.x); o[1] = from_f32<f16>(v.y * g.y); o[2] = from_f32<f16>(v.z * g.z); o[3] = from_f32<f16>(v.w * g.w);
      *(f16x4*)(xp + x16_chunk(tok, f0, d >> 5) * 8 + (f0 & 4)) = o;
    }
    s += sum_xor32(sum_squares4(v));
  }
  if (lane < 32) part[r][lane] = s;
  __syncthreads();
  if (r == 0 && lane < 32 && tok < M)
    ssq[(size_t)blockIdx.x * s_pad + tok] = (part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]);
}
// feature blocks per part, so that the consumer finds at most 96 parts
static int finish_blocks(int d) { return (d / 32 + 95) / 96; }
int r_down_parts(int d) { return (d / 32 + finish_blocks(d) - 1) / finish_blocks(d); }

// Feature blocks per workgroup: rounds of workgroups (one per compute unit) x (blocks + a stage's fixed cost), the least.
// Named the fastest of 2 .. 5 blocks at 96, 128, 192 and 256 rows of both decoders (1.5B gate/up, 256 rows: 5 blocks 2154 us per
// step, 4 2346, 3 2253, 2 2367; 0.5B, 96 rows: 2 920, 3 953).
static int pick_blocks(int n_fblk, int per_tile) {
  const int cu = n_compute_units();
  int best = 2;
  double least = 1e30;
  for (int nb = 2; nb <= 5; ++nb) {
    const double cost = (double)(((n_fblk + nb - 1) / nb * per_tile + cu - 1) / cu) * (nb + 1);
    if (cost < least) { least = cost; best = nb; }
  }
  return best;
}
template <int NB, typename Kernel, typename... A>
static hipError_t launch_rows(Kernel kernel, bool& attr_done, int grid, hipStream_t st, A... args) {
  if (!attr_done) {
    const hipError_t e = hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, RowsLoop<NB>::kBytes);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  return launch(KID_GEMM_ROWS, kernel, dim3(grid), dim3(256), RowsLoop<NB>::kBytes, st, args...);
}
template <int NB, int NL>
static hipError_t gate_up(const void* Xp, const void* Wp, const float* ssq, int parts, int s_pad, int M, int n_fblk, int K, float eps,
                          const float* h, const float* gain, void* act, hipStream_t st) {
  static bool attr_done = false;
  const int grid = ((n_fblk + NB - 1) / NB + 7) / 8 * 8 * ((M + 127) / 128);
  return launch_rows<NB>(k_rows_gate_up<NB, NL>, attr_done, grid, st, (const uint4*)Xp, (const uint4*)Wp, ssq, M, n_fblk, K, parts, s_pad, eps,
                         (f16*)act, h, gain);
}
template <int NB>
static hipError_t down(const void* Xp, const void* Wp, int M, int n_fblk, int K, float* partial, const Prefetch& pf, hipStream_t st) {
  static bool attr_done = false;
  const int grid = kRowSplits * ((n_fblk + NB - 1) / NB) * ((M + 127) / 128);
  return launch_rows<NB>(k_rows_down<NB>, attr_done, grid + prefetch_blocks(pf, 4, kPrefetchKbRows), st, (const uint4*)Xp, (const uint4*)Wp, M, n_fblk, K,
                         (float4*)partial, grid, pf);
}

hipError_t r_gate_up(const void* Xp, const void* Wp, const float* ssq, int parts, int s_pad, int M, int F, int K, float eps, const float* h,
                     const float* gain, void* act, hipStream_t st) {
  if (M <= 0 || M > s_pad || F % 32 != 0 || K % 64 != 0 || parts < 1) return hipErrorInvalidValue;
  const int n_fblk = F / 16;
  auto go = [&](auto nl) {
    constexpr int NL = decltype(nl)::value;
    switch (pick_blocks(n_fblk, (M + 127) / 128)) {
      case 2: return gate_up<2, NL>(Xp, Wp, ssq, parts, s_pad, M, n_fblk, K, eps, h, gain, act, st);
      case 3: return gate_up<3, NL>(Xp, Wp, ssq, parts, s_pad, M, n_fblk, K, eps, h, gain, act, st);
      case 4: return gate_up<4, NL>(Xp, Wp, ssq, parts, s_pad, M, n_fblk, K, eps, h, gain, act, st);
      default: return gate_up<5, NL>(Xp, Wp, ssq, parts, s_pad, M, n_fblk, K, eps, h, gain, act, st);
    }
  };
  return parts <= 28 ? go(std::integral_constant<int, 14>()) : go(std::integral_constant<int, 24>());
}

size_t r_down_partial_floats(int M, int d) { return (size_t)kRowSplits * ((M + 31) / 32 * 32) * d; }
hipError_t r_down(const void* Xp, const void* Wp, int M, int d, int K, float* partial, float* h, const float* gain, int s_pad, void* xp,
                  float* ssq, const Prefetch& pf, hipStream_t st) {
  if (M <= 0 || M > s_pad || d % 32 != 0 || K <= 0 || K % 64 != 0) return hipErrorInvalidValue;
  const int n_fblk = d / 32;
  hipError_t e;
  switch (pick_blocks(n_fblk, kRowSplits * ((M + 127) / 128))) {
    case 2: e = down<2>(Xp, Wp, M, n_fblk, K, partial, pf, st); break;
    case 3: e = down<3>(Xp, Wp, M, n_fblk, K, partial, pf, st); break;
    case 4: e = down<4>(Xp, Wp, M, n_fblk, K, partial, pf, st); break;
    default: e = down<5>(Xp, Wp, M, n_fblk, K, partial, pf, st); break;
  }
  if (e != hipSuccess) return e;
  return launch(KID_MISC, k_rows_finish, dim3(r_down_parts(d), (M + 31) / 32), dim3(256), 0, st, (const float4*)partial, h, gain, M,
                n_fblk, finish_blocks(d), s_pad, (f16*)xp, ssq);
}

}  // namespace sapo
