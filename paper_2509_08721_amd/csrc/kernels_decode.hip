// Decode-side 16-bit MFMA kernels for gfx950 (one new token per sequence and step).  Operands are
// IEEE half: packed weights hold the model's bf16 values converted to half, activations are rounded
// to half (see the note at the top of kernels_mfma.hip).
//
// Every projection of a decode step is a "skinny" GEMM: few tokens (64 per block), all weights
// streamed once from HBM.  The kernels here are built around v_mfma_f32_16x16x32_f16 with both
// operands already in fragment order in global memory, so that a wave's operand load is one
// contiguous 1 KiB read that goes straight into registers:
//   weights  W16[((tile * KS + ks) * 64 + lane)]           (uint4 = 8 half)
//            = W[tile*16 + lane%16][ks*32 + (lane/16)*8 .. +7],                       KS = K / 32
//   tokens   X16[(((tok/64) * KS + ks) * 4 + (tok/16)%4) * 64 + tok%16 + 16*((k%32)/8)]
//            = x[tok][ks*32 + ((k%32)/8)*8 .. +7]
// D = W-fragment x X-fragment leaves lane l with features (l/16)*4 .. +3 of token l%16.
//
// RMSNorm never runs on its own: the kernel that produces the residual stream also writes
// half(h * gain) in X16 order plus per-tile sums of squares of h, and the GEMM that consumes it
// multiplies its accumulators by rsqrt(mean(h^2) + eps) (the scale is per token, so it commutes
// with the contraction).
#include <climits>

#include "common.h"
#include "coherent.h"

namespace sapo {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
union Frag16 {
  uint4 u;
  u32x4 n;
  bf16x8 v;
  f16x8 h;
};

__device__ __forceinline__ f32x4 mfma16(const Frag16& a, const Frag16& b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(a.h, b.h, c, 0, 0, 0);
}
__device__ __forceinline__ float silu_f(float x) { return x / (1.0f + __expf(-x)); }

// ---------------------------------------------------------------------------------------
// Sum of the ssq parts of one token, spread over the 8 waves of a workgroup: thread (grp, tok)
// loads parts grp, grp + 8, ... early (ssq_issue) and the sums meet in LDS later (ssq_publish, ssq_scale).
// ---------------------------------------------------------------------------------------
constexpr int kSsqPerThread = kMaxSsqParts / 8;

// ssq is not null and parts >= 1.  Every thread asks for all kSsqPerThread values, the bound of the buffer descriptor
// answering for a part past the end with zero: with a request under a branch each, the compiler waited for the first
// one on the spot - a memory round trip in front of the kernel's weight requests.
__device__ __forceinline__ void ssq_issue(const float* __restrict__ ssq, int parts, int stride, int tok0,
                                          float (&sq)[kSsqPerThread]) {
  const int tok = threadIdx.x & 63, grp = wave_index(threadIdx.x);
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)ssq, 0, parts * stride * 4, 0x00020000);
#pragma unroll
  for (int i = 0; i < kSsqPerThread; ++i)
    sq[i] = __uint_as_float(
        __builtin_amdgcn_raw_buffer_load_b32(r, (unsigned)((grp + 8 * i) * stride + tok0 + tok) * 4u, 0, 0));
}
// s_part: LDS [8][64].  Call before a __syncthreads(); ssq_scale() after it.
__device__ __forceinline__ void ssq_publish(const float (&sq)[kSsqPerThread], float* s_part) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < kSsqPerThread; ++i) s += sq[i];
  s_part[threadIdx.x] = s;
}
__device__ __forceinline__ float ssq_scale(const float* s_part, int tok_local, int norm_dim, float eps) {
  float s = 0.f;
#pragma unroll
  for (int g = 0; g < 8; ++g) s += s_part[g * 64 + tok_local];
  return 1.0f / sqrtf(s / (float)norm_dim + eps);
}

__device__ __forceinline__ void prefetch_behind(const SkinnyArgs& a, int first, void* lds_1k) {
  const int block = (int)blockIdx.x - first;
  if (block < 0) return;
  if (block < a.pf_blocks) prefetch_role<8>(a.pf, block, a.pf_blocks, lds_1k);
  else prefetch_role<8>(a.pf2, block - a.pf_blocks, (int)gridDim.x - first - a.pf_blocks, lds_1k);
}

// ---------------------------------------------------------------------------------------
// Skinny GEMM.  512 threads = 8 waves per workgroup.
// A workgroup owns NT 16-feature tiles x TG 16-token groups over the whole K; wave w takes the
// k steps w, w + 8, ... (the requests of R of them in flight), and the
// 8 partial results are summed through LDS in wave order, so results never depend on timing.
// Small per-workgroup operands matter more than the number of workgroups: a compute unit ingests
// roughly 100 GB/s, so a 64-token block is split into 4 / TG workgroups per tile, which re-read
// the tile's weights from the L2 they share (block ids are laid out so that they land on the
// same XCD: ids that differ by a multiple of 8).
// Epilogues:
//   STORE  : out_f32[tok][feat] = acc * scale(tok)
//   SWIGLU : tiles come in (gate, up) pairs; act = silu(gate * scale) * (up * scale) -> half, X16 order
//   RESID  : h[tok][feat] += acc;  xp_out = half(h * gain_next) in X16 order;  ssq_out[tile][tok] =
//            sum of h^2 over the tile's 16 features
//   RESID_X32 (more than 64 rows): as RESID, but X32 order, and sums of squares over all tiles of the workgroup,
//            infinite where some h * gain of theirs is beyond half's range and was clamped
// ---------------------------------------------------------------------------------------
// Bound of the operands' buffer descriptors: a lane offset with this bit set fetches nothing and arrives as zero.  A k step past the
// end is asked for that way, not left out under a branch: the number of requests in flight is then the same on every path,
// and a wave multiplies what has arrived instead of waiting, in front of its first product, for all of it.  The
// registers of a step that has been multiplied take the request for the step R rounds on at once.  0.5B, us per step
// of 32, 48 and 64 rows 619, 642, 665 -> 607, 621, 657; 128 and 256 rows 924, 1122 -> 919, 1111; 1.5B, 128 rows 1775 -> 1752.
constexpr unsigned kSkinnyRecords = 0x40000000u;

template <int NT, int TG, int TS, int R, int MODE>
// The first arguments are passed one by one (and once more inside the struct): the hardware preloads the first 14 dwords
// of a kernel's arguments into scalar registers when it starts a wave (-amdgpu-kernarg-preload-count), but not the
// members of a struct passed by value.  What the kernel needs before its first requests then costs no load:
// 0.5 us less from the start of a workgroup to its first weight request.
__global__ void __launch_bounds__(512) k_skinny16(const uint4* Wp_, const uint4* Xp_, const float* ssq_in_, float* h_,
                                                  const float* gain_next_, int N_, int K_, int n_rows_, int ssq_parts_,
                                                  SkinnyArgs a_rest) {
  constexpr bool RESID = MODE == SKM_RESID || MODE == SKM_RESID_X32;
  SkinnyArgs a = a_rest;
  a.Wp = Wp_; a.Xp = Xp_; a.ssq_in = ssq_in_; a.h = h_; a.gain_next = gain_next_;
  a.N = N_; a.K = K_; a.n_rows = n_rows_; a.ssq_parts = ssq_parts_;
  a.s_pad = (a.n_rows + 63) & ~63;
  const int n_units = (a.N >> 4) / NT;
  // the 8 partial results meet in LDS CH tiles at a time: [8 waves][CH * TG][64 lanes] float4 <= 128 KiB
  constexpr int CH = (NT * TG > 16) ? 16 / TG : NT;
  static_assert(NT % CH == 0 && (MODE != SKM_SWIGLU || CH % 2 == 0), "tile chunking");
  constexpr int RS = (CH * TG * 64 + 511) / 512;   // output slots per thread and chunk
  extern __shared__ float4 red[];
  __shared__ float s_part[512];
  const int tid = threadIdx.x, wave = wave_index(tid), lane = tid & 63;
  const int KS = a.K >> 5;
  // block id -> (unit, token block, token split).  Ids are dealt round-robin to the 8 XCDs; the workgroups
  // that read the same weight tiles (all token blocks and splits of a unit) sit 8 ids apart, so they run on
  // one XCD at about the same time and the tiles come from HBM once.
  const int nblk = (a.n_rows + 63) >> 6;
  const int j = blockIdx.x >> 3, inner = j % (TS * nblk);
  const int unit = (j / (TS * nblk)) * 8 + (blockIdx.x & 7);
  const int tb = inner / TS;
  const int tg0 = (inner % TS) * TG;
  if (unit >= n_units) {
    const int first = (n_units + 7) / 8 * 8 * TS * nblk;
    prefetch_behind(a_rest, first, red);
    return;
  }
  const int tile0 = unit * NT;
  f32x4 acc[NT][TG];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int g = 0; g < TG; ++g) acc[t][g] = f32x4{0.f, 0.f, 0.f, 0.f};
  float sq[kSsqPerThread];
  if (!RESID) ssq_issue(a.ssq_in, a.ssq_parts, a.s_pad, tb * 64, sq);
  // RESID, single chunk: this thread's residual / gain operands are requested up front
  float4 h_old[RS], g_next[RS];
  if (RESID && CH == NT) {
#pragma unroll
    for (int i = 0; i < RS; ++i) {
      const int slot = tid + 512 * i;
      h_old[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      g_next[i] = h_old[i];
      if (slot < NT * TG * 64) {
        const int t = slot / (TG * 64), g = (slot >> 6) % TG, l = slot & 63;
        const int tok = tb * 64 + (tg0 + g) * 16 + (l & 15);
        const int f0 = (tile0 + t) * 16 + (l >> 4) * 4;
        if (tok < a.n_rows) {
          h_old[i] = *(const float4*)(a.h + (size_t)tok * a.N + f0);
          g_next[i] = *(const float4*)(a.gain_next + f0);
        }
      }
    }
  }

  const __amdgpu_buffer_rsrc_t wr =
      __builtin_amdgcn_make_buffer_rsrc((void*)(a.Wp + (size_t)tile0 * KS * 64), 0, kSkinnyRecords, 0x00020000);
  const __amdgpu_buffer_rsrc_t xr =
      __builtin_amdgcn_make_buffer_rsrc((void*)(a.Xp + ((size_t)tb * KS * 4 + tg0) * 64), 0, kSkinnyRecords, 0x00020000);
  Frag16 wf[R][NT], xf[R][TG];
  auto request = [&](int i, int ks) {
    const unsigned off = lane * 16u | (ks < KS ? 0u : kSkinnyRecords);
#pragma unroll
    for (int t = 0; t < NT; ++t) wf[i][t].n = __builtin_amdgcn_raw_buffer_load_b128(wr, off, (t * KS + ks) * 1024, 2);
#pragma unroll
    for (int g = 0; g < TG; ++g) xf[i][g].n = __builtin_amdgcn_raw_buffer_load_b128(xr, off + g * 1024u, ks * 4096, 0);
  };
  auto multiply = [&](int i) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int g = 0; g < TG; ++g) acc[t][g] = mfma16(wf[i][t], xf[i][g], acc[t][g]);
  };
#pragma unroll
  for (int i = 0; i < R; ++i) request(i, wave + 8 * i);
  if (!RESID) ssq_publish(sq, s_part);   // while the weights are on their way
  int k0 = wave;
  for (; k0 + 8 * R < KS; k0 += 8 * R) {
#pragma unroll
    for (int i = 0; i < R; ++i) {
      multiply(i);
      request(i, k0 + 8 * (R + i));
    }
  }
#pragma unroll
  for (int i = 0; i < R; ++i) multiply(i);
  auto sum8 = [&](int tg, int l) -> float4 {   // tg = (t - chunk start) * TG + g
    float4 s = red[(size_t)tg * 64 + l];
#pragma unroll
    for (int w = 1; w < 8; ++w) {
      const float4 p = red[(size_t)(w * CH * TG + tg) * 64 + l];
      s.x += p.x; s.y += p.y; s.z += p.z; s.w += p.w;
    }
    return s;
  };
#pragma unroll
  for (int c0 = 0; c0 < NT; c0 += CH) {
    // cross-wave reduction of tiles c0 .. c0 + CH - 1
    if (c0 > 0) __syncthreads();
#pragma unroll
    for (int t = 0; t < CH; ++t)
#pragma unroll
      for (int g = 0; g < TG; ++g)
        red[(size_t)(wave * CH * TG + t * TG + g) * 64 + lane] =
            make_float4(acc[c0 + t][g][0], acc[c0 + t][g][1], acc[c0 + t][g][2], acc[c0 + t][g][3]);
    __syncthreads();
    if (MODE == SKM_SWIGLU) {
      const int KSo = (a.N >> 1) >> 5;   // act has F = N / 2 features
      for (int slot = tid; slot < (CH / 2) * TG * 64; slot += 512) {
        const int pp = slot / (TG * 64), g = (slot >> 6) % TG, l = slot & 63;
        const float4 gs = sum8((2 * pp) * TG + g, l), us = sum8((2 * pp + 1) * TG + g, l);
        const int tl = (tg0 + g) * 16 + (l & 15), tok = tb * 64 + tl;
        const int f0 = (((tile0 + c0) >> 1) + pp) * 16 + (l >> 4) * 4;
        f16x4 o;
        if (tok < a.n_rows) {
          const float sc = ssq_scale(s_part, tl, a.norm_dim, a.eps);
          o[0] = from_f32<f16>(silu_f(gs.x * sc) * (us.x * sc)); o[1] = from_f32<f16>(silu_f(gs.y * sc) * (us.y * sc));
          o[2] = from_f32<f16>(silu_f(gs.z * sc) * (us.z * sc)); o[3] = from_f32<f16>(silu_f(gs.w * sc) * (us.w * sc));
        } else {
          o[0] = o[1] = o[2] = o[3] = (f16)0.f;
        }
        *(f16x4*)((f16*)a.xp_out + x16_chunk(tok, f0, KSo) * 8 + (f0 & 4)) = o;
      }
    } else if (MODE == SKM_STORE) {
      for (int slot = tid; slot < CH * TG * 64; slot += 512) {
        const int t = slot / (TG * 64), g = (slot >> 6) % TG, l = slot & 63;
        const float4 s = sum8(t * TG + g, l);
        const int tl = (tg0 + g) * 16 + (l & 15), tok = tb * 64 + tl;
        const int f0 = (tile0 + c0 + t) * 16 + (l >> 4) * 4;
        if (tok < a.n_rows) {
          const float sc = ssq_scale(s_part, tl, a.norm_dim, a.eps);
          float4 o = make_float4(s.x * sc, s.y * sc, s.z * sc, s.w * sc);
          if (a.bias) {
            const float4 bb = *(const float4*)(a.bias + f0);
            o.x += bb.x; o.y += bb.y; o.z += bb.z; o.w += bb.w;
          }
          *(float4*)(a.out_f32 + (size_t)tok * a.ldc + f0) = o;
        }
      }
    } else {
      if (CH == NT) {
        // The operands requested up front are taken here, outside the branch on the row bound: otherwise the
        // compiler, which cannot see that they landed rounds ago, waits for every outstanding memory operation where
        // the branch rejoins - and that includes the residual store just issued, a full round trip in front of the
        // second store.
#pragma unroll
        for (int i = 0; i < RS; ++i)
          asm volatile("" ::"v"(h_old[i].x), "v"(h_old[i].y), "v"(h_old[i].z), "v"(h_old[i].w), "v"(g_next[i].x),
                       "v"(g_next[i].y), "v"(g_next[i].z), "v"(g_next[i].w));
      }
#pragma unroll
      for (int i = 0; i < RS; ++i) {
        const int slot = tid + 512 * i;
        if (slot >= CH * TG * 64) break;   // a whole wave leaves together (64 slots per wave)
        const int t = slot / (TG * 64), g = (slot >> 6) % TG, l = slot & 63;
        float4 s = sum8(t * TG + g, l);
        const int tok = tb * 64 + (tg0 + g) * 16 + (l & 15);
        const int f0 = (tile0 + c0 + t) * 16 + (l >> 4) * 4;
        f16x4 o;
        float q = 0.f;
        if (tok < a.n_rows) {
          float4 ho, gn;
          if (CH == NT) { ho = h_old[i]; gn = g_next[i]; }
          else { ho = *(const float4*)(a.h + (size_t)tok * a.N + f0); gn = *(const float4*)(a.gain_next + f0); }
          s.x += ho.x; s.y += ho.y; s.z += ho.z; s.w += ho.w;
          *(float4*)(a.h + (size_t)tok * a.N + f0) = s;
          o[0] = from_f32<f16>(s.x * gn.x); o[1] = from_f32<f16>(s.y * gn.y);
          o[2] = from_f32<f16>(s.z * gn.z); o[3] = from_f32<f16>(s.w * gn.w);
          q = sum_squares4(s);
          if (MODE == SKM_RESID_X32 &&
              !(fmaxf(fmaxf(fabsf(s.x * gn.x), fabsf(s.y * gn.y)), fmaxf(fabsf(s.z * gn.z), fabsf(s.w * gn.w))) <= 65504.f))
            q = INFINITY;
        } else {
          o[0] = o[1] = o[2] = o[3] = (f16)0.f;
        }
        const size_t chunk = MODE == SKM_RESID_X32 ? x32_chunk(tok, f0, a.N >> 4) : x16_chunk(tok, f0, a.N >> 5);
        *(f16x4*)((f16*)a.xp_out + chunk * 8 + (f0 & 4)) = o;
        q = sum_xor16(q);
        q = sum_xor32(q);
        if (l < 16) {
          if (MODE == SKM_RESID_X32) s_part[((c0 + t) * TG + g) * 16 + l] = q;
          else a.ssq_out[(size_t)(tile0 + c0 + t) * a.s_pad + tok] = q;
        }
      }
    }
  }
  if constexpr (MODE == SKM_RESID_X32) {   // one part per unit instead of one per tile
    static_assert(NT * TG * 16 <= 512, "parts of the unit's tiles");
    __syncthreads();
    if (tid < TG * 16) {
      float q = 0.f;
#pragma unroll
      for (int t = 0; t < NT; ++t) q += s_part[t * TG * 16 + tid];
      a.ssq_out[(size_t)unit * a.s_pad + tb * 64 + tg0 * 16 + tid] = q;
    }
  }
}

// TS: workgroups per (tile unit, token block); TG x TS covers the token groups of a block
template <int NT, int TG, int TS, int R, int MODE>
static hipError_t launch_skinny(SkinnyArgs a, hipStream_t st) {
  constexpr int CH = (NT * TG > 16) ? 16 / TG : NT;
  static bool attr_done = false;
  const size_t smem = (size_t)8 * CH * TG * 64 * sizeof(float4);
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute((const void*)k_skinny16<NT, TG, TS, R, MODE>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  if ((a.N / 16) % NT != 0) return hipErrorInvalidValue;
  const int units = a.N / 16 / NT;
  const int blocks = (a.n_rows + 63) / 64;
  if (TG * TS * 16 < 64 && (blocks > 1 || a.n_rows > TG * TS * 16)) return hipErrorInvalidValue;
  if (a.s_pad != blocks * 64) return hipErrorInvalidValue;
  // Blocks per wave that prefetches.  Beside O and down as many workgroups as compute units are left.  Beside gate/up 18 (14 to 18 the
  // same) - except where its own workgroups are more than the units: with up to 2 token groups two of them share a unit and 9 is
  // best (1.5B, 24 and 32 rows 1195, 1213 -> 1184, 1202 us per step), with 3 and 4 a unit holds one (150 registers and
  // more), the prefetching ones start behind the last, and few and long ones are best (28: 48 and 64 rows 1538, 1612 -> 1532, 1572).
  const int main = (units + 7) / 8 * 8 * TS * blocks, cu = n_compute_units();
  const int per = MODE != SKM_SWIGLU ? prefetch_per_wave(a.pf, a.pf2, 8, cu - main, 10, kPrefetchKb) : main <= cu ? 18 : TG <= 2 ? 9 : kPrefetchKb;
  a.pf_blocks = prefetch_blocks(a.pf, 8, per);
  const int gx = main + a.pf_blocks + prefetch_blocks(a.pf2, 8, per);
  return launch(KID_GEMM_SKINNY, k_skinny16<NT, TG, TS, R, MODE>, dim3(gx), dim3(512), smem, st, a.Wp, a.Xp, a.ssq_in, a.h, a.gain_next,
                a.N, a.K, a.n_rows, a.ssq_parts, a);
}

// One token block with 2 .. 4 groups of 16 rows: all groups in one workgroup, one group each, or two each.
template <int NT, int R, int MODE>
static hipError_t launch_groups(const SkinnyArgs& a, int groups, hipStream_t st) {
  if (groups == 2) return launch_skinny<NT, 2, 1, R, MODE>(a, st);
  if (groups == 3) return launch_skinny<NT, 3, 1, R, MODE>(a, st);
  return launch_skinny<NT, 4, 1, R, MODE>(a, st);
}
template <int R, int MODE>
static hipError_t launch_singles(const SkinnyArgs& a, int groups, hipStream_t st) {
  if (groups == 2) return launch_skinny<1, 1, 2, R, MODE>(a, st);
  if (groups == 3) return launch_skinny<1, 1, 3, R, MODE>(a, st);
  return launch_skinny<1, 1, 4, R, MODE>(a, st);
}
template <int R, int MODE>
static hipError_t launch_pairs(const SkinnyArgs& a, int groups, hipStream_t st) {
  if (groups == 2) return launch_skinny<1, 2, 1, R, MODE>(a, st);
  return launch_skinny<1, 2, 2, R, MODE>(a, st);
}

// ---------------------------------------------------------------------------------------
// Skinny GEMM for at most 16 rows (one token group): the same sums in the same order as k_skinny16 - wave w multiplies
// the k steps w, w + 8, ..., the 8 partial results are added through LDS in wave order - with the work cut along the
// features instead.  With one token group there are only N / 16 tiles: the 0.5B down projection was 56 workgroups of
// 155 KB of weights (and as much again of token operand, rows past the end included), the gate/up projection 152
// workgroups of 115 KB that multiplied the three token groups that do not exist as well.  A workgroup here takes one
// gate/up pair of tiles, or FR = 16 or 8 of a tile's 16 features, and lanes whose row of either operand does not
// exist are turned away by the buffer bounds instead of fetching.  0.5B decoder, one row: gate/up 9.8 -> 7.8 us, down
// 7.8 -> 6.7 us per launch with the weights cold, 5.5 and 5.0 us when they were prefetched.
// What follows the last product is a chain that nothing hides, so it is cut over four waves, one feature per thread (one wave with
// four features per thread: 0.5 to 1 us of a launch whose weights lie in the L2), and the rows' sums of squares are
// added up while the weights are on their way.  us per step, 0.5B, 1 and 16 rows 577, 590 -> 570, 578; 1.5B, 8 rows 1137 -> 1102.
// ssq_out is left per group of 4 features ([tile][4][16 rows], in the same N / 16 x 64 floats): a tile's features may lie
// in several workgroups.  The consumer adds the four in the order in which k_skinny16's producer adds them.
// ---------------------------------------------------------------------------------------

// Sums of squares for at most 16 rows: thread (wave, lane) asks for parts wave, wave + 8, ...; lane = group of 4 features
// x row.  parts == 1 (rows that come from an embedding gather): one value per row.  What does not exist arrives as zero.
__device__ __forceinline__ void ssq_issue_few(const float* __restrict__ ssq, int parts, float (&sq)[kSsqPerThread]) {
  const int wave = wave_index(threadIdx.x), lane = threadIdx.x & 63;
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void*)ssq, 0, parts > 1 ? parts * 256 : 64, 0x00020000);
#pragma unroll
  for (int i = 0; i < kSsqPerThread; ++i)
    sq[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, (unsigned)(wave + 8 * i) * 256u + lane * 4u, 0, 0));
}
// The four groups of a part are added as (0 + 1) + (2 + 3), then the wave's parts in their order: four parts at a time
// come together in one register, lane group q holding the sum of part q, and go round to all lanes again.
__device__ __forceinline__ void ssq_publish_few(const float (&sq)[kSsqPerThread], float* s_part) {
  static_assert(kSsqPerThread % 4 == 0, "four parts at a time");
  const auto swap16 = [](float a, float b, float& x, float& y) {   // odd rows of a against even rows of b
    const lane_u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    x = __uint_as_float(r[0]); y = __uint_as_float(r[1]);
  };
  const auto swap32 = [](float a, float b, float& x, float& y) {   // upper half of a against lower half of b
    const lane_u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    x = __uint_as_float(r[0]); y = __uint_as_float(r[1]);
  };
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < kSsqPerThread; i += 4) {
    float x, y, p01, p23, v[4];
    swap16(sq[i], sq[i + 1], x, y);
    p01 = x + y;
    swap16(sq[i + 2], sq[i + 3], x, y);
    p23 = x + y;
    swap32(p01, p23, x, y);
    const float all = x + y;   // lane group q: part i + q
    swap16(all, all, x, y);    // groups 0 0 2 2 and 1 1 3 3
    swap32(x, x, v[0], v[2]);
    swap32(y, y, v[1], v[3]);
    s += v[0]; s += v[1]; s += v[2]; s += v[3];
  }
  s_part[threadIdx.x] = s;
}

template <int FR, int R, int MODE>
__global__ void __launch_bounds__(512) k_skinny_few(const uint4* Wp_, const uint4* Xp_, const float* ssq_in_, float* h_,
                                                    const float* gain_next_, int N_, int K_, int n_rows_, int ssq_parts_,
                                                    SkinnyArgs a_rest) {
  SkinnyArgs a = a_rest;   // the leading arguments arrive preloaded (see k_skinny16)
  a.Wp = Wp_; a.Xp = Xp_; a.ssq_in = ssq_in_; a.h = h_; a.gain_next = gain_next_;
  a.N = N_; a.K = K_; a.n_rows = n_rows_; a.ssq_parts = ssq_parts_;
  const int n_units = a.N / (MODE == SKM_SWIGLU ? 32 : 16);
  static_assert(FR == 16 || (FR == 8 && MODE != SKM_SWIGLU), "whole tiles, or halves of them");
  constexpr int PT = 16 / FR;                       // workgroups per tile (SWIGLU: tile pair)
  constexpr int NA = MODE == SKM_SWIGLU ? 2 : 1;    // weight fragments per k step
  constexpr int EW = FR / 4;                        // waves of the epilogue: one per 4 features
  __shared__ float4 red[8 * NA * 64];
  __shared__ float s_part[512];
  const int tid = threadIdx.x, wave = wave_index(tid), lane = tid & 63;
  const int KS = a.K >> 5;
  // the parts of a tile sit 8 block ids apart: one XCD fetches the lines they share
  const int j = blockIdx.x >> 3, part = j % PT;
  const int unit = (j / PT) * 8 + (blockIdx.x & 7);
  if (unit >= n_units) {
    const int first = (n_units + 7) / 8 * 8 * PT;
    prefetch_behind(a_rest, first, red);
    return;
  }
  const int row = lane & 15, kg = lane >> 4;
  float sq[kSsqPerThread];
  if (MODE != SKM_RESID) ssq_issue_few(a.ssq_in, a.ssq_parts, sq);
  // epilogue coordinates of a thread of the first EW waves: row of the batch, its one feature; the 4 features of a group
  // lie in neighbouring lanes
  const int tok = lane >> 2, f = unit * 16 + part * FR + wave * 4 + (lane & 3);
  const bool live = tok < a.n_rows;
  // Of one or two rows the next operand's other rows are written as well, whatever they hold (nobody reads them): lines of which
  // 16 or 32 bytes in 256 were written leave the L2 slower than whole ones.  0.5B, us per step with 1 and 2 rows 551, 555 ->
  // 546, 548; from 3 rows on (535) no difference.
  const bool whole = a.n_rows <= 2;
  float h_old = 0.f, g_next = 0.f;
  if (MODE == SKM_RESID && wave < EW) {
    h_old = a.h[(size_t)min(tok, a.n_rows - 1) * a.N + f];   // clamped, so that the request sits under no lane mask
    g_next = a.gain_next[f];
  }
  unsigned woff[NA];
  woff[0] = row < FR ? (unsigned)(kg * 16 + part * FR + row) * 16u : kSkinnyRecords;
  if (NA == 2) woff[NA - 1] = (unsigned)KS * 1024u + lane * 16u;   // the up tile lies behind its gate tile
  const unsigned xoff = row < a.n_rows ? lane * 16u : kSkinnyRecords;
  const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(a.Wp + (size_t)unit * (MODE == SKM_SWIGLU ? 2 : 1) * KS * 64), 0, kSkinnyRecords, 0x00020000);
  const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc((void*)a.Xp, 0, kSkinnyRecords, 0x00020000);
  f32x4 acc[NA];
#pragma unroll
  for (int t = 0; t < NA; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  Frag16 wf[R][NA], xf[R];
  auto request = [&](int i, int ks) {
    const unsigned gone = ks < KS ? 0u : kSkinnyRecords;
#pragma unroll
    for (int t = 0; t < NA; ++t) wf[i][t].n = __builtin_amdgcn_raw_buffer_load_b128(wr, woff[t] | gone, ks * 1024, 2);
    xf[i].n = __builtin_amdgcn_raw_buffer_load_b128(xr, xoff | gone, ks * 4096, 0);
  };
  auto multiply = [&](int i) {
#pragma unroll
    for (int t = 0; t < NA; ++t) acc[t] = mfma16(wf[i][t], xf[i], acc[t]);
  };
#pragma unroll
  for (int i = 0; i < R; ++i) request(i, wave + 8 * i);
  float bias = 0.f;
  if (MODE == SKM_STORE && a.bias && wave < EW) bias = a.bias[f];
  if (MODE != SKM_RESID) ssq_publish_few(sq, s_part);   // requested first, here first
  __builtin_amdgcn_sched_barrier(0);   // nothing that waits for the weights moves up
  int k0 = wave;
  for (; k0 + 8 * R < KS; k0 += 8 * R) {
#pragma unroll
    for (int i = 0; i < R; ++i) {
      multiply(i);
      request(i, k0 + 8 * (R + i));
    }
  }
#pragma unroll
  for (int i = 0; i < R; ++i) multiply(i);
#pragma unroll
  for (int t = 0; t < NA; ++t) red[(wave * NA + t) * 64 + lane] = make_float4(acc[t][0], acc[t][1], acc[t][2], acc[t][3]);
  __syncthreads();
  if (wave >= EW) return;
  auto sum8 = [&](int t) -> float {
    const float* r = (const float*)red + t * 256 + tid;
    float s = r[0];
#pragma unroll
    for (int w = 1; w < 8; ++w) s += r[w * NA * 256];
    return s;
  };
  float s = sum8(0);
  if (MODE == SKM_SWIGLU) {
    const float us = sum8(NA - 1), sc = ssq_scale(s_part, tok, a.norm_dim, a.eps);
    if (live || whole) ((f16*)a.xp_out)[x16_chunk(tok, f, a.N >> 6) * 8 + (f & 7)] = from_f32<f16>(silu_f(s * sc) * (us * sc));
  } else if (MODE == SKM_STORE) {
#pragma clang fp contract(off)   // rounded before the bias is added, as with more rows
    float o = s * ssq_scale(s_part, tok, a.norm_dim, a.eps);
    if (a.bias) o += bias;
    if (live) a.out_f32[(size_t)tok * a.ldc + f] = o;
  } else {
    s += h_old;
    const float4 all = make_float4(dpp_quad<0>(s), dpp_quad<1>(s), dpp_quad<2>(s), dpp_quad<3>(s));
    if (live || whole) ((f16*)a.xp_out)[x16_chunk(tok, f, a.N >> 5) * 8 + (f & 7)] = from_f32<f16>(s * g_next);
    if (live) {
      a.h[(size_t)tok * a.N + f] = s;
      if ((lane & 3) == 0) a.ssq_out[unit * 64 + (part * EW + wave) * 16 + tok] = sum_squares4(all);
    }
  }
}

template <int FR> static int few_blocks(int units) { return (units + 7) / 8 * 8 * (16 / FR); }
// Blocks of 1 KiB per wave that prefetches, us per step: beside gate/up (0.5B 304 workgroups, 1.5B 560) 9 -> 6, 0.5B, 1 and 16
// rows 560, 566 -> 555, 561; 1.5B 1028, 1077 -> 1019, 1069 (4: 1014, 1060, but 578, 584 on the 0.5B decoder, where two workgroups
// per compute unit no longer hold them all).  Beside down as many workgroups as compute units are left, of 10 blocks at least: 18 ->
// 10 573, 575 -> 569, 571 (0.5B); 18 -> 24 1044, 1173 -> 1034, 1146 (1.5B, which takes half tiles then).
template <int FR, int R, int MODE>
static hipError_t launch_few(SkinnyArgs a, hipStream_t st) {
  const int units = a.N / (MODE == SKM_SWIGLU ? 32 : 16), main = few_blocks<FR>(units);
  const int per = MODE == SKM_SWIGLU ? kPrefetchKbFew : prefetch_per_wave(a.pf, a.pf2, 8, n_compute_units() - main, 10, kPrefetchKb);
  a.pf_blocks = prefetch_blocks(a.pf, 8, per);
  return launch(KID_GEMM_SKINNY, k_skinny_few<FR, R, MODE>, dim3(main + a.pf_blocks + prefetch_blocks(a.pf2, 8, per)), dim3(512), 0, st, a.Wp, a.Xp,
                a.ssq_in, a.h, a.gain_next, a.N, a.K, a.n_rows, a.ssq_parts, a);
}
template <int FR, int MODE>
static hipError_t launch_few_r(const SkinnyArgs& a, hipStream_t st) {
  const int per_wave = ((a.K >> 5) + 7) / 8;
  if (per_wave <= 4) return launch_few<FR, 4, MODE>(a, st);
  if (per_wave <= 6) return launch_few<FR, 6, MODE>(a, st);
  return launch_few<FR, 20, MODE>(a, st);
}

// Blocking (feature tiles x token groups) of a STORE or RESID launch with several token blocks.  With 4 x 4 a narrow output leaves
// compute units idle (1.5B QKV at 256 rows: 128 workgroups of 393 KB); two tiles per workgroup double the workgroups at
// 295 KB each.  Of these as few token groups as still give every workgroup a compute unit of its own: each takes in less.
// us per step with 4 groups, 2 and 1, 0.5B: O projection 72 rows (56, 112, 224 workgroups) 909, 886, 870; 192 rows (84, 168, 336)
// 1012, 993, 1005; 256 rows (112, 224, 448) 1076, 1056, 1072; QKV 72 rows (72, 144, 288) 909, 892, 900; 192 rows (108, 216)
// 1012, 997; 256 rows (144, 288) 1076, 1082.  1.5B: O 96 rows (96, 192, 384) 1598, 1555, 1584; 192 rows (144, 288) 1924, 1961; QKV
// 96 rows (128, 256, 512) 1598, 1557, 1613; 192 rows (192, 384) 1924, 1946.
// K above 2048 or a number of tiles that is no multiple of 4: 2 x 2 where the output is a residual.
enum WideTile { WIDE_1X1, WIDE_2X1, WIDE_2X2, WIDE_2X4, WIDE_4X4 };
static WideTile wide_tile(int n_rows, int mode, int N, int K) {
  const int tiles = N / 16, blocks = (n_rows + 63) / 64, cu = n_compute_units();
  if (tiles % 4 == 0 && (mode == SKM_STORE || K <= 2048)) {
    if (tiles / 4 * blocks >= 192) return WIDE_4X4;
    const int by_two = tiles / 2 * blocks;
    return 4 * by_two <= cu ? WIDE_2X1 : 2 * by_two <= cu ? WIDE_2X2 : WIDE_2X4;
  }
  return mode != SKM_STORE && tiles % 2 == 0 ? WIDE_2X2 : WIDE_1X1;
}
// Its launch.  R: with K up to 1024 all of a wave's k steps in one round.
template <int MODE>
static hipError_t launch_wide(WideTile wide, const SkinnyArgs& a, int per_wave, hipStream_t st) {
  switch (wide) {
    case WIDE_2X1: return per_wave <= 4 ? launch_skinny<2, 1, 4, 4, MODE>(a, st) : launch_skinny<2, 1, 4, 3, MODE>(a, st);
    case WIDE_2X2:
      return per_wave <= 4 ? launch_skinny<2, 2, 2, 4, MODE>(a, st) : per_wave <= 8 ? launch_skinny<2, 2, 2, 3, MODE>(a, st)
                                                                                     : launch_skinny<2, 2, 2, 9, MODE>(a, st);
    case WIDE_2X4: return launch_skinny<2, 4, 1, 3, MODE>(a, st);
    case WIDE_4X4: return launch_skinny<4, 4, 1, 3, MODE>(a, st);
    default: return hipErrorInvalidValue;
  }
}
// 16-feature tiles that a workgroup of the launch below reads, as a power of two: what the block numbering calls a unit.
static int skinny_unit_log2(int n_rows, int mode, int N, int K) {
  const int tiles = N / 16;
  if (n_rows <= kFewRows) return mode == SKM_SWIGLU ? 1 : 0;
  if (n_rows <= 64) return mode != SKM_SWIGLU ? 0 : K <= 1024 ? 2 : 1;
  if (mode == SKM_SWIGLU) return tiles % 8 == 0 ? 3 : K <= 1024 ? 2 : 1;
  const WideTile t = wide_tile(n_rows, mode, N, K);
  return t == WIDE_4X4 ? 2 : t == WIDE_1X1 ? 0 : 1;
}
int d_skinny_units(int n_rows, int mode, int N, int K) { return N / 16 >> skinny_unit_log2(n_rows, mode, N, K); }
// Prefetch of a skinny GEMM's weights by an earlier launch of a step of n_rows rows.
Prefetch d_prefetch_skinny(const void* w16, int n_rows, int mode, int N, int K) {
  return make_prefetch(w16, K / 32, N / 16, skinny_unit_log2(n_rows, mode, N, K));
}

// Blocking.  A workgroup reads NT weight tiles and TG token groups over the whole K, so what it must
// ingest is (NT + TG) * K * 32 bytes for NT * TG output tiles.  With one 64-token block the kernels
// are latency-bound and small workgroups win (1 x 1; the gate/up pairs 4 x 4); with several blocks
// the re-reads of the token operand dominate and the blocking goes towards square.
hipError_t d_gemm_skinny(const SkinnyArgs& a, int mode, hipStream_t st) {
  if (a.K % 32 != 0 || a.N % 16 != 0 || a.n_rows <= 0 || (mode == SKM_RESID_X32 && a.n_rows <= 64)) return hipErrorInvalidValue;
  if (mode != SKM_RESID && mode != SKM_RESID_X32 && (a.ssq_in == nullptr || a.ssq_parts < 1 || a.ssq_parts > kMaxSsqParts)) return hipErrorInvalidValue;
  const int per_wave = ((a.K >> 5) + 7) / 8;   // k steps per wave
  const int tiles = a.N / 16;
  const bool multi = a.n_rows > 64;
  if (a.n_rows <= kFewRows) {
    if (mode == SKM_SWIGLU) return a.N % 32 == 0 ? launch_few_r<16, SKM_SWIGLU>(a, st) : hipErrorInvalidValue;
    if (mode == SKM_STORE) return launch_few_r<16, SKM_STORE>(a, st);
    // Half tiles where twice the workgroups, with those that prefetch, still have a compute unit each, and a tile is long.
    // 24 layers, us per layer against whole tiles at 16 rows (1 .. 8 rows: within 0.1 either way): 56 tiles of 155 KB -0.24,
    // of 287 KB -0.52, 80 tiles of 287 KB -0.76 (160 + 56 workgroups).  96 tiles were +0.9 .. +1.8 as long as 72 prefetched beside
    // the 192; with the 64 that prefetch_per_wave leaves them (1.5B's down) a step of 1, 4, 8 and 16 rows takes 1027, 1038,
    // 1066, 1153 us, with whole tiles 1041, 1059, 1085, 1188.
    const int room = n_compute_units() - few_blocks<8>(tiles);
    return room >= 0 && prefetch_per_wave(a.pf, a.pf2, 8, room, 10, 0) > 0 && per_wave > 8 ? launch_few_r<8, SKM_RESID>(a, st) : launch_few_r<16, SKM_RESID>(a, st);
  }
  const int groups = multi ? 4 : (a.n_rows + 15) / 16;   // 16-token groups of a block that hold rows (2 .. 4)
  if (mode == SKM_SWIGLU) {
    if (a.N % 64 != 0) return hipErrorInvalidValue;
    if (multi && tiles % 8 == 0) return launch_skinny<8, 4, 1, 2, SKM_SWIGLU>(a, st);
    if (per_wave <= 4) return launch_groups<4, 4, SKM_SWIGLU>(a, groups, st);
    return launch_groups<2, 6, SKM_SWIGLU>(a, groups, st);
  }
  const WideTile wide = multi ? wide_tile(a.n_rows, mode, a.N, a.K) : WIDE_1X1;
  if (mode == SKM_RESID_X32) return launch_wide<SKM_RESID_X32>(wide, a, per_wave, st);
  // one token block, more 16-token workgroups than compute units (0.5B QKV: 72 tiles x 4 = 288): some compute
  // units would get two workgroups and ingest twice; 32-token workgroups (144 of them, 86 KB each) keep it one each
  const bool tg2 = !multi && tiles * groups > 256;
  if (mode == SKM_STORE) {
    if (wide != WIDE_1X1) return launch_wide<SKM_STORE>(wide, a, per_wave, st);
    if (tg2) return per_wave <= 4 ? launch_pairs<4, SKM_STORE>(a, groups, st) : launch_pairs<8, SKM_STORE>(a, groups, st);
    return per_wave <= 4 ? launch_singles<4, SKM_STORE>(a, groups, st) : launch_singles<8, SKM_STORE>(a, groups, st);
  }
  if (wide != WIDE_1X1) return launch_wide<SKM_RESID>(wide, a, per_wave, st);
  if (tg2 && per_wave <= 4) return launch_pairs<4, SKM_RESID>(a, groups, st);
  if (tg2 && per_wave <= 8) return launch_pairs<8, SKM_RESID>(a, groups, st);
  if (per_wave <= 4) return launch_singles<4, SKM_RESID>(a, groups, st);
  if (per_wave <= 8) return launch_singles<8, SKM_RESID>(a, groups, st);
  return launch_singles<20, SKM_RESID>(a, groups, st);
}

// ---------------------------------------------------------------------------------------
// Rows of the residual stream -> X16 order: xp = half(h * gain), ssq[row] = sum h^2 (one part).
// One workgroup of 128 threads per row; thread i handles the 8 features 8 i .. 8 i + 7 (+1024 j).
// ---------------------------------------------------------------------------------------
__device__ __forceinline__ void row_to_x16(const float (&v)[8], const float* __restrict__ gain, int k, int row, int KS,
                                           uint4* __restrict__ xp) {
  Frag16 f;
#pragma unroll
  for (int e = 0; e < 8; ++e) f.h[e] = from_f32<f16>(v[e] * gain[k + e]);
  xp[x16_chunk(row, k, KS)] = f.u;
}
__device__ __forceinline__ float block128_sum(float s, float* red) {
  s = wave_reduce_sum(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  return red[0] + red[1];
}

__global__ void __launch_bounds__(128) k_pack_rows_x16(const float* __restrict__ h, const float* __restrict__ gain, int d,
                                                       uint4* __restrict__ xp, float* __restrict__ ssq) {
  __shared__ float red[2];
  const int row = blockIdx.x;
  float ss = 0.f;
  for (int k = threadIdx.x * 8; k < d; k += 1024) {
    float v[8];
    const float4 a = *(const float4*)(h + (size_t)row * d + k), b = *(const float4*)(h + (size_t)row * d + k + 4);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w; v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
#pragma unroll
    for (int e = 0; e < 8; ++e) ss += v[e] * v[e];
    row_to_x16(v, gain, k, row, d >> 5, xp);
  }
  ss = block128_sum(ss, red);
  if (threadIdx.x == 0) ssq[row] = ss;
}
hipError_t d_pack_rows_x16(const float* h, const float* gain, int M, int d, void* xp, float* ssq, hipStream_t st) {
  return launch(KID_MISC, k_pack_rows_x16, dim3(M), dim3(128), 0, st, h, gain, d, (uint4*)xp, ssq);
}

// Embedding row of token id `tok` -> h[row] (fp32), X16 half(h * gain), ssq[row].  128 threads.
__device__ __forceinline__ void embed_row_x16(const bf16* __restrict__ embed, int tok, int row, int d,
                                              const float* __restrict__ gain, float* __restrict__ h,
                                              uint4* __restrict__ xp, float* __restrict__ ssq, float* red) {
  float ss = 0.f;
  for (int k = threadIdx.x * 8; k < d; k += 1024) {
    Frag16 e; e.u = *(const uint4*)(embed + (size_t)tok * d + k);
    float v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) { v[i] = (float)e.v[i]; ss += v[i] * v[i]; }
    *(float4*)(h + (size_t)row * d + k) = make_float4(v[0], v[1], v[2], v[3]);
    *(float4*)(h + (size_t)row * d + k + 4) = make_float4(v[4], v[5], v[6], v[7]);
    row_to_x16(v, gain, k, row, d >> 5, xp);
  }
  ss = block128_sum(ss, red);
  if (threadIdx.x == 0) ssq[row] = ss;
}

// Decode-side embedding gather of the token sampled at the previous step.
__global__ void __launch_bounds__(128) k_embed_x16(const int32_t* __restrict__ tokens, int tok_stride, const int* step,
                                                   const bf16* __restrict__ embed, int d, const float* __restrict__ gain,
                                                   float* __restrict__ h, uint4* __restrict__ xp, float* __restrict__ ssq,
                                                   const int* __restrict__ slot_seq) {
  __shared__ float red[2];
  const int row = blockIdx.x;
  const int seq = slot_seq ? slot_seq[row] : row;
  int tok = tokens[(size_t)seq * tok_stride + (*step - 1)];
  if (tok < 0) tok = 0;   // a step that reported a fault left -1 behind: never an index
  embed_row_x16(embed, tok, row, d, gain, h, xp, ssq, red);
}
hipError_t d_embed_x16(const int32_t* tokens, int tok_stride, const int* step, const void* embed, int M, int d,
                       const float* gain, float* h, void* xp, float* ssq, const int* slot_seq, hipStream_t st) {
  return launch(KID_EMBED, k_embed_x16, dim3(M), dim3(128), 0, st, tokens, tok_stride, step, (const bf16*)embed, d, gain, h,
                (uint4*)xp, ssq, slot_seq);
}

// ---------------------------------------------------------------------------------------
// LM head for decode: logits tile -> online log-sum-exp + Gumbel-max; logits are never stored.
// 512 threads = 8 waves; X (64 tokens x K, X16 order) is staged once into LDS and every wave owns
// whole 16-vocabulary tiles over the full K: tile = global wave index + j * (number of waves), its
// weights streamed in groups of U k steps with the next group in flight while the current one is
// multiplied.  A lane keeps, for its token of each 16-token group, the running (max, sum exp) and
// the best perturbed score; lanes, waves and workgroups are merged in a fixed order.
// partials: [n_wg][64][5] (max, sum exp, best y, its logit, its id).
// ---------------------------------------------------------------------------------------
struct LaneState {
  float m[4], l[4], by[4], bz[4];
  int bid[4];
};

// global -> LDS copy of one wave-wide 1 KiB block (lane l's 16 bytes land at lds + 16 l); completion is awaited with
// wait_vmcnt_d (requests complete in order)
__device__ __forceinline__ unsigned lds_addr16(const void* p) {
  return (unsigned)(size_t)(const __attribute__((address_space(3))) void*)p;
}
__device__ __forceinline__ void dma16_lds(const void* g, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(g) : "memory");
}
template <int N> __device__ __forceinline__ void wait_vmcnt_d() {
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));
}

template <int U>
__global__ void __launch_bounds__(512) k_lmhead_sample16(const uint4* __restrict__ Wp, const uint4* __restrict__ Xp, int KS,
                                                         int n_tiles, const float* __restrict__ ssq, int ssq_parts,
                                                         bool ssq_quarters, int s_pad, int norm_dim, float eps, int n_rows, int seq0,
                                                         SampleParams sp, float* __restrict__ partials) {
  extern __shared__ uint4 xs[];   // [KS][4][64]
  __shared__ float s_part[512];
  __shared__ float s_scale[64];
  const int tid = threadIdx.x, wave = wave_index(tid), lane = tid & 63;
  // The wave's first weight group is requested before anything else, and the token operand goes to LDS without
  // passing through registers (copied through registers, every 16 bytes were one load, wait, LDS store - a
  // dependent round trip per loop pass, KS / 2 of them in front of the first weight request).
  int tile = blockIdx.x * 8 + wave;
  Frag16 cur[U], nxt[U];
  if (tile < n_tiles) {
    const uint4* wb = Wp + (size_t)tile * KS * 64 + lane;
#pragma unroll
    for (int i = 0; i < U; ++i) cur[i].n = __builtin_nontemporal_load((const u32x4*)(wb + (size_t)i * 64));
  }
  float sq[kSsqPerThread];
  if (ssq_quarters) ssq_issue_few(ssq, ssq_parts, sq);
  else ssq_issue(ssq, ssq_parts, s_pad, 0, sq);
  // the sampling parameters too (behind the copy below they would be read through the vector path, one more round trip)
  resolve_sample_params(sp);
  const int step = *sp.step;
  const bool noisy = sp.temperature != 0.f;
  const float inv_t = noisy ? 1.0f / sp.temperature : 1.0f;
  const int fq = lane >> 4, tl = lane & 15;
  uint32_t seq_id[4];   // the noise is keyed on the sequence, which need not be the row
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int row = g * 16 + tl;
    seq_id[g] = (uint32_t)((sp.slot_seq && row < n_rows) ? sp.slot_seq[row] : seq0 + row);
  }
  {
    const unsigned xs0 = __builtin_amdgcn_readfirstlane(lds_addr16(xs));
    for (int b = wave * 64; b < KS * 256; b += 512) dma16_lds(Xp + b + lane, xs0 + (unsigned)b * 16u);
  }
  if (ssq_quarters) ssq_publish_few(sq, s_part);
  else ssq_publish(sq, s_part);
  wait_vmcnt_d<0>();   // this wave's blocks of the operand have landed ...
  __syncthreads();     // ... and everybody's
  if (tid < 64) s_scale[tid] = ssq_scale(s_part, tid, norm_dim, eps);
  __syncthreads();
  float scale[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) scale[g] = s_scale[g * 16 + tl];
  LaneState stt;
#pragma unroll
  for (int g = 0; g < 4; ++g) { stt.m[g] = -INFINITY; stt.l[g] = 0.f; stt.by[g] = -INFINITY; stt.bz[g] = 0.f; stt.bid[g] = 0x7fffffff; }

  const int n_waves = gridDim.x * 8;
  const int groups_per_tile = KS / U;
  f32x4 acc[4];
#pragma unroll
  for (int g = 0; g < 4; ++g) acc[g] = f32x4{0.f, 0.f, 0.f, 0.f};
  int grp = 0;
  while (tile < n_tiles) {
    // prefetch the next group (of this tile, or the first of the wave's next tile)
    int ntile = tile, ngrp = grp + 1;
    if (ngrp == groups_per_tile) { ngrp = 0; ntile = tile + n_waves; }
    if (ntile < n_tiles) {
      const uint4* wb = Wp + ((size_t)ntile * KS + (size_t)ngrp * U) * 64 + lane;
#pragma unroll
      for (int i = 0; i < U; ++i) nxt[i].n = __builtin_nontemporal_load((const u32x4*)(wb + (size_t)i * 64));
    }
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const int ks = grp * U + i;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        Frag16 x; x.u = xs[(ks * 4 + g) * 64 + lane];
        acc[g] = mfma16(cur[i], x, acc[g]);
      }
    }
    if (grp == groups_per_tile - 1) {
      const int v0 = tile * 16 + fq * 4;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        float z[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) z[j] = acc[g][j] * scale[g];
        const float mt = fmaxf(fmaxf(z[0], z[1]), fmaxf(z[2], z[3]));
        const float mn = fmaxf(stt.m[g], mt);
        stt.l[g] = stt.l[g] * __expf(stt.m[g] - mn) + ((__expf(z[0] - mn) + __expf(z[1] - mn)) + (__expf(z[2] - mn) + __expf(z[3] - mn)));
        stt.m[g] = mn;
        float gn[4] = {0.f, 0.f, 0.f, 0.f};
        if (noisy) gumbel4(sp.seed_lo, sp.seed_hi, seq_id[g], (uint32_t)step, (uint32_t)(v0 >> 2), gn);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float y = noisy ? z[j] * inv_t + gn[j] : z[j];
          if (y > stt.by[g]) { stt.by[g] = y; stt.bz[g] = z[j]; stt.bid[g] = v0 + j; }   // ids ascend: ties keep the lower id
        }
        acc[g] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }
#pragma unroll
    for (int i = 0; i < U; ++i) cur[i] = nxt[i];
    tile = ntile; grp = ngrp;
  }
  // merge the 4 lanes that share a token (fixed order), then the 8 waves, one row of partials per token
  __syncthreads();          // everybody is done reading xs: reuse it
  float* sm = (float*)xs;   // [8 waves][64 tokens][5]
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    LseAcc a; a.m = stt.m[g]; a.l = stt.l[g];
    BestAcc b; b.y = stt.by[g]; b.z = stt.bz[g]; b.id = stt.bid[g];
#pragma unroll
    for (int o = 16; o <= 32; o <<= 1) {
      a.merge(__shfl_xor(a.m, o, 64), __shfl_xor(a.l, o, 64));
      b.add(__shfl_xor(b.y, o, 64), __shfl_xor(b.z, o, 64), __shfl_xor(b.id, o, 64));
    }
    if (fq == 0) {
      float* p = sm + ((size_t)wave * 64 + g * 16 + tl) * 5;
      p[0] = a.m; p[1] = a.l; p[2] = b.y; p[3] = b.z; ((int*)p)[4] = b.id;
    }
  }
  __syncthreads();
  if (tid < 64) {
    LseAcc a; a.init();
    BestAcc b; b.init();
    for (int w = 0; w < 8; ++w) {
      const float* p = sm + ((size_t)w * 64 + tid) * 5;
      a.merge(p[0], p[1]);
      b.add(p[2], p[3], ((const int*)p)[4]);
    }
    float* p = partials + ((size_t)blockIdx.x * 64 + tid) * 5;
    p[0] = a.m; p[1] = a.l; p[2] = b.y; p[3] = b.z; ((int*)p)[4] = b.id;
  }
}

// Merge the per-workgroup partials of one sequence, write its token and log-prob, and gather the
// token's embedding row as the input of the next decode step (residual row, X16 row for the first
// layer's norm gain, sum of squares).  One workgroup of 128 threads per sequence.
__global__ void __launch_bounds__(128) k_lmhead_merge_embed(const float* __restrict__ partials, int n_wg, int row_stride,
                                                            int seq0, SampleParams sp, const bf16* __restrict__ embed, int d,
                                                            const float* __restrict__ gain, float* __restrict__ h,
                                                            uint4* __restrict__ xp, float* __restrict__ ssq) {
  __shared__ float red[2];
  __shared__ int s_tok;
  const int r = blockIdx.x, lane = threadIdx.x & 63;
  if (threadIdx.x < 64) {
    LseAcc a; a.init();
    BestAcc b; b.init();
    resolve_outputs(sp);
    constexpr int NB = 4;   // a lane's next partials, in flight together (256 workgroups of k_lmhead_sample16: all of them)
    for (int w0 = lane; w0 < n_wg; w0 += 64 * NB) {
      float v[NB][5];
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        const float* p = partials + ((size_t)min(w0 + 64 * u, n_wg - 1) * row_stride + r) * 5;
#pragma unroll
        for (int k = 0; k < 5; ++k) v[u][k] = p[k];
      }
#pragma unroll
      for (int u = 0; u < NB; ++u)
        if (w0 + 64 * u < n_wg) {
          a.merge(v[u][0], v[u][1]);
          b.add(v[u][2], v[u][3], __float_as_int(v[u][4]));
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      a.merge(__shfl_xor(a.m, o, 64), __shfl_xor(a.l, o, 64));
      b.add(__shfl_xor(b.y, o, 64), __shfl_xor(b.z, o, 64), __shfl_xor(b.id, o, 64));
    }
    if (lane == 0) {
      const int step = *sp.step;
      s_tok = emit_token(sp, sp.slot_seq ? sp.slot_seq[r] : seq0 + r, step, b.id, b.z - (a.m + logf(a.l)));
      // every workgroup has used the step index before it arrives here: the last one to arrive moves it on
      if (sp.arrivals && atomicAdd(sp.arrivals, 1) == (int)gridDim.x - 1) {
        *sp.arrivals = 0;
        *const_cast<int*>(sp.step) = step + 1;
      }
    }
  }
  __syncthreads();
  embed_row_x16(embed, s_tok, seq0 + r, d, gain, h, xp, ssq, red);
}

size_t d_lmhead_sample_partial_floats() { return (size_t)256 * 64 * 5; }

template <int U>
static hipError_t launch_lmhead(const uint4* Wp, const uint4* Xp, int KS, int n_tiles, const float* ssq, int ssq_parts,
                                bool ssq_quarters, int s_pad, int norm_dim, float eps, int n_rows, int seq0, SampleParams sp, float* partials,
                                int n_wg, hipStream_t st) {
  static bool attr_done = false;
  const size_t smem = (size_t)KS * 256 * sizeof(uint4) < 8 * 64 * 5 * 4 ? 8 * 64 * 5 * 4 : (size_t)KS * 256 * sizeof(uint4);
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute((const void*)k_lmhead_sample16<U>, hipFuncAttributeMaxDynamicSharedMemorySize, 131072);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  return launch(KID_LMHEAD_SAMPLE, k_lmhead_sample16<U>, dim3(n_wg), dim3(512), smem, st, Wp, Xp, KS, n_tiles, ssq, ssq_parts, ssq_quarters, s_pad, norm_dim, eps, n_rows, seq0, sp,
                                                partials);
}

bool d_lmhead_sample_supported(int K, int n_rows) { return n_rows <= 64 && K % 32 == 0 && (size_t)K * 128 <= 131072; }

hipError_t d_lmhead_sample(const void* Wp, const void* Xp, int K, int V, const float* ssq, int ssq_parts, bool ssq_quarters, int s_pad,
                           float eps, int n_rows, SampleParams sp, float* partials, const void* embed,
                           const float* gain_first, float* h, void* xp_first, float* ssq_first, hipStream_t st) {
  if (!d_lmhead_sample_supported(K, n_rows) || V % 16 != 0 || ssq == nullptr || ssq_parts < 1 || ssq_parts > kMaxSsqParts)
    return hipErrorInvalidValue;
  const int KS = K / 32, n_tiles = V / 16;
  int n_wg = 256;
  if (n_wg > (n_tiles + 7) / 8) n_wg = (n_tiles + 7) / 8;
  hipError_t e;
  {
    if (KS % 7 == 0)
      e = launch_lmhead<7>((const uint4*)Wp, (const uint4*)Xp, KS, n_tiles, ssq, ssq_parts, ssq_quarters, s_pad, K, eps, n_rows, 0, sp, partials, n_wg, st);
    else if (KS % 4 == 0)
      e = launch_lmhead<4>((const uint4*)Wp, (const uint4*)Xp, KS, n_tiles, ssq, ssq_parts, ssq_quarters, s_pad, K, eps, n_rows, 0, sp, partials, n_wg, st);
    else
      e = launch_lmhead<1>((const uint4*)Wp, (const uint4*)Xp, KS, n_tiles, ssq, ssq_parts, ssq_quarters, s_pad, K, eps, n_rows, 0, sp, partials, n_wg, st);
  }
  if (e != hipSuccess) return e;
  return d_lmhead_merge_embed(partials, n_wg, 64, n_rows, sp, embed, K, gain_first, h, xp_first, ssq_first, st);
}

hipError_t d_lmhead_merge_embed(const float* partials, int n_parts, int row_stride, int n_rows, SampleParams sp,
                                const void* embed, int d, const float* gain_first, float* h, void* xp_first,
                                float* ssq_first, hipStream_t st) {
  return launch(KID_LMHEAD_SAMPLE_MERGE, k_lmhead_merge_embed, dim3(n_rows), dim3(128), 0, st, partials, n_parts, row_stride,
                0, sp, (const bf16*)embed, d, gain_first, h, (uint4*)xp_first, ssq_first);
}

// =======================================================================================
// Decode attention over the paged KV cache, fused with rotary + KV append of the new token.
// One workgroup (NW waves) per (sequence, KV head); all query heads of the group ride together as
// the 16 columns of 16x16x32 MFMAs.  S^T = K Q^T (tokens x queries) so that each lane owns one
// query column: the running max / sum are per-lane scalars plus two cross-lane shuffles, and the
// probabilities a lane produces are exactly its operand of O^T = V^T P^T.  Token rows are permuted
// inside a 32-token page pair so that a lane's 8 probabilities are 8 consecutive tokens, which is
// what a lane gets from a V page in one 16-byte load (v_page_at).  Waves take page pairs round-robin, PD
// pairs at a time with all their K/V fragments in flight at once; the first chunk is requested
// before the query rows are even read (K/V addresses depend on the page table only), so a step
// pays one memory round trip, not one per dependent stage.  Waves are merged through LDS.
// Queries, keys, values and probabilities are IEEE half (the cache's type on this path); the
// output goes out as half in X16 order (the O projection's operand).
// ---------------------------------------------------------------------------------------
// The prefix workgroup of the shared-prompt variant (see ShareArgs): block (prompt p, KV head kvh) walks the page
// pairs 0 .. prefix_pairs - 1 of the prompt once, with the query heads of all G siblings as columns of up to four
// 16-column MFMA tiles (column c = sibling c / rep, head c % rep), and leaves per column the merged, unnormalised
// (max, sum, weighted values) of its waves in sh.pre, stored write-through; then it publishes the launch number.
template <int HD, int NW>
__device__ __forceinline__ void attention_prefix_role(const float* __restrict__ qkv, const float2* __restrict__ rope,
                                                      const RowMap& rm, const KVCache& kv, int n_q_heads,
                                                      const ShareArgs& sh, float* sm_o, f16* qs64, float (*sm_m)[16],
                                                      float (*sm_l)[16]) {
  constexpr int KK = HD / 32, DT = HD / 16, NT = kSharePrefixMaxColumns / 16;
  const int tid = threadIdx.x, wave = wave_index(tid), lane = tid & 63;
  const int qcol = lane & 15, grp = lane >> 4;
  const int hkv = kv.n_kv_heads, rep = n_q_heads / hkv;
  const int p = blockIdx.x / hkv, kvh = blockIdx.x % hkv;
  const int row0 = p * sh.G;
  const int ncols = sh.G * rep;
  int seq, pos;
  rm.get(row0, seq, pos);             // every sibling is at this position; the shared pages are the same for all
  const int* pt = kv.page_table + (size_t)seq * kv.pages_per_seq;
  const f16* kpool = (const f16*)kv.k;
  const f16* vpool = (const f16*)kv.v;
  const size_t page_elems = (size_t)hkv * kPageTokens * HD;
  auto load_pair = [&](int pp, Frag16 (&kf)[2][KK], Frag16 (&vf)[DT]) {
    const int pa = pt[2 * pp], pb = pt[2 * pp + 1];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const f16* kp = kpool + (size_t)((lane & 15) < 8 ? pa : pb) * page_elems + (size_t)kvh * kPageTokens * HD;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) kf[t][kk].u = *(const uint4*)(kp + k_frag_at(t, kk, lane));
    }
    const f16* vp = vpool + (size_t)(grp < 2 ? pa : pb) * page_elems + (size_t)kvh * HD * kPageTokens;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) vf[dt].u = *(const uint4*)(vp + v_frag_at(dt, lane));
  };
  Frag16 kf[2][2][KK], vf[2][DT];
#pragma unroll
  for (int j = 0; j < 2; ++j)
    if (wave + NW * j < sh.prefix_pairs) load_pair(wave + NW * j, kf[j], vf[j]);
  // rotated queries of every column (zero rows for the columns past G x rep)
  {
    const int half = HD / 2;
    const size_t row_floats = (size_t)(n_q_heads + 2 * hkv) * HD;
    for (int idx = tid; idx < NT * 16 * half; idx += NW * 64) {
      const int cc = idx / half, i = idx % half;
      float r1 = 0.f, r2 = 0.f;
      if (cc < ncols) {
        const float* x = qkv + (size_t)(row0 + cc / rep) * row_floats + (size_t)(kvh * rep + cc % rep) * HD;
        const float2 cs = rope[(size_t)pos * half + i];
        r1 = rot_first(x[i], x[i + half], cs.x, cs.y);
        r2 = rot_second(x[i], x[i + half], cs.x, cs.y);
      }
      qs64[cc * HD + i] = from_f32<f16>(r1);
      qs64[cc * HD + i + half] = from_f32<f16>(r2);
    }
  }
  __syncthreads();
  const float scale = 1.0f / sqrtf((float)HD);
  float m_run[NT], l_run[NT];
  f32x4 o[NT][DT];
#pragma unroll
  for (int jt = 0; jt < NT; ++jt) {
    m_run[jt] = -INFINITY; l_run[jt] = 0.f;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[jt][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  for (int c0 = 0; wave + NW * c0 < sh.prefix_pairs; c0 += 2) {
    if (c0 > 0) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
        if (wave + NW * (c0 + j) < sh.prefix_pairs) load_pair(wave + NW * (c0 + j), kf[j], vf[j]);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if (wave + NW * (c0 + j) >= sh.prefix_pairs) break;
#pragma unroll
      for (int jt = 0; jt < NT; ++jt) {
        Frag16 qf[KK];
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) qf[kk].u = *(const uint4*)(qs64 + (jt * 16 + qcol) * HD + kk * 32 + grp * 8);
        f32x4 sc[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          sc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int kk = 0; kk < KK; ++kk) sc[t] = mfma16(kf[j][t][kk], qf[kk], sc[t]);
        }
        // every token of a shared pair lies inside every sibling's context: nothing to mask
        float pv[8];
        float m_loc = -INFINITY;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          pv[e] = sc[e >> 2][e & 3] * scale;
          m_loc = fmaxf(m_loc, pv[e]);
        }
        m_loc = max_xor16(m_loc);
        m_loc = max_xor32(m_loc);
        const float m_new = fmaxf(m_run[jt], m_loc);
        const float alpha = __expf(m_run[jt] - m_new);
        float psum = 0.f;
        Frag16 pf;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float pe = __expf(pv[e] - m_new);
          psum += pe;
          pf.h[e] = (f16)pe;
        }
        l_run[jt] = l_run[jt] * alpha + psum;
        m_run[jt] = m_new;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
#pragma unroll
          for (int i = 0; i < 4; ++i) o[jt][dt][i] *= alpha;
          o[jt][dt] = mfma16(vf[j][dt], pf, o[jt][dt]);
        }
      }
    }
  }
  // merge the waves tile by tile; a wave without a pair carries (-inf, 0, 0) and drops out (wave 0 always has pair 0)
#pragma unroll
  for (int jt = 0; jt < NT; ++jt) {
    float l = l_run[jt];
    l = sum_xor16(l);
    l = sum_xor32(l);
    if (jt > 0) __syncthreads();   // the previous tile's sums have been read
    if (grp == 0) { sm_m[wave][qcol] = m_run[jt]; sm_l[wave][qcol] = l; }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int i = 0; i < 4; ++i) sm_o[((size_t)wave * HD + dt * 16 + grp * 4 + i) * 16 + qcol] = o[jt][dt][i];
    __syncthreads();
    for (int idx = tid; idx < 16 * (HD / 8); idx += NW * 64) {
      const int q = idx / (HD / 8), d0 = (idx % (HD / 8)) * 8;
      const int cc = jt * 16 + q;
      if (cc >= ncols) continue;
      float mx = -INFINITY;
#pragma unroll
      for (int w = 0; w < NW; ++w) mx = fmaxf(mx, sm_m[w][q]);
      float den = 0.f, wgt[NW];
#pragma unroll
      for (int w = 0; w < NW; ++w) { wgt[w] = __expf(sm_m[w][q] - mx); den += wgt[w] * sm_l[w][q]; }
      float num[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        num[e] = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) num[e] += wgt[w] * sm_o[((size_t)w * HD + d0 + e) * 16 + q];
      }
      const size_t base = ((size_t)(row0 + cc / rep) * n_q_heads + kvh * rep + cc % rep) * (HD + 4);
      st_f4<true>(sh.pre, (base + 4 + d0) * sizeof(float), make_float4(num[0], num[1], num[2], num[3]));
      st_f4<true>(sh.pre, (base + 8 + d0) * sizeof(float), make_float4(num[4], num[5], num[6], num[7]));
      if (d0 == 0) {
        st_f32<true>(sh.pre, base * sizeof(float), mx);
        st_f32<true>(sh.pre, (base + 1) * sizeof(float), den);
      }
    }
  }
  coh_drain();        // this thread's write-through stores have completed ...
  __syncthreads();    // ... and everybody's
  if (tid == 0) {
    const unsigned launch_no = (unsigned)(*rm.step) * (unsigned)sh.n_layers + (unsigned)sh.layer + 1u;
    (void)__hip_atomic_exchange(&sh.flags[blockIdx.x], launch_no, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// LDS = true is the measured alternative to the register-direct K/V reads: the same requests go global -> LDS
// (one 1 KiB block per fragment, lane l's 16 bytes at 16 l, so the read back is conflict-free) into PD slots per
// wave and are read into registers pair by pair; the requests in flight and the order of the arithmetic are the
// same, the results bit-identical.
// SHARE = true: the shared-prompt variant (ShareArgs): the first sh.n_prefix blocks are prefix workgroups, the others
// cover page pairs sh.prefix_pairs .. of their row and fold the prefix workgroup's partial result into the merge.
template <int HD, int NW, int PD, bool LDS, bool SHARE>
__global__ void __launch_bounds__(NW * 64) k_decode_attention16(const float* __restrict__ qkv,
                                                               const float2* __restrict__ rope, const int* step_,
                                                               const int* page_table_, int lp_pages_, int rows_,
                                                               int heads_, int n_main, void* kpool_, RowMap rm,
                                                               KVCache kv, uint4* __restrict__ out, ShareArgs sh, Prefetch pf) {
  extern __shared__ float sm_o[];   // [NW][HD][16]; LDS: [NW][PD][NFRAG] KiB of staged pairs, a wave's output over its slot 0
  if ((int)blockIdx.x >= n_main) {   // uniform over the workgroup
    const int first = (n_main + 7) & ~7;
    if ((int)blockIdx.x >= first) prefetch_role<NW>(pf, blockIdx.x - first, (int)gridDim.x - first, sm_o);
    return;
  }
  // What leads from the start of the kernel to its first requests arrives preloaded (see k_skinny16): 14 dwords.  What they point
  // to - step counter, page table - is read through the scalar cache, all at once: behind one another and through the
  // vector path, where the wait for the counter held the row's own values back as well, these reads were 1 us of a
  // launch at any context.  us per step, with the last pair's handling below: 0.5B, 64 rows, contexts of 150 663 -> 648,
  // 1 row, 1060 716 -> 682; 1.5B, 1 row, 160 1080 -> 1037.
  const int step = load_uniform(step_);
  kv.page_table = page_table_; kv.pages_per_seq = lp_pages_ >> 16; kv.n_kv_heads = heads_ & 0xffff; kv.k = kpool_;
  const int rep = (heads_ >> 16) & 0xff, n_q_heads = rep * kv.n_kv_heads;
  const int per_rep = (65536 + rep - 1) / rep;
  constexpr int KK = HD / 32;   // k steps of S^T = K Q^T
  constexpr int DT = HD / 16;   // 16-row tiles of O^T
  constexpr int NFRAG = 2 * KK + DT;                        // 1 KiB fragments of one page pair
  constexpr size_t kOStride = LDS ? (size_t)PD * NFRAG * 256 : (size_t)HD * 16;   // floats between two waves' outputs
  __shared__ __attribute__((aligned(16))) f16 qs[16 * HD];
  __shared__ __attribute__((aligned(16))) f16 knew[HD];
  __shared__ __attribute__((aligned(16))) f16 vnew[HD];
  __shared__ float sm_m[NW][16], sm_l[NW][16];
  if constexpr (SHARE) {
    static_assert(!LDS, "the shared-prompt variant reads K/V register-direct");
    if ((int)blockIdx.x < sh.n_prefix) {   // uniform over the workgroup
      rm.step = step_; rm.Lp = lp_pages_ & 0xffff;
      attention_prefix_role<HD, NW>(qkv, rope, rm, kv, n_q_heads, sh, sm_o, (f16*)(sm_o + (size_t)NW * HD * 16), sm_m, sm_l);
      return;
    }
  }
  const int tid = threadIdx.x, wave = wave_index(tid), lane = tid & 63;
  const int qcol = lane & 15, grp = lane >> 4;
  const int hkv = kv.n_kv_heads;
  // Siblings read the same prompt pages: the rows of a group (consecutive rows, one KV head) run on one XCD, whose L2 fetches
  // them once.  Block ids are dealt round-robin to the XCDs.
  int s, kvh;
  if constexpr (SHARE) {
    const int bid = (int)blockIdx.x - sh.n_prefix;
    s = bid / hkv; kvh = bid % hkv;
  } else {
    const int group_log2 = (heads_ >> 24) & 7, j = (int)blockIdx.x >> 3, g = (j >> group_log2) * 8 + ((int)blockIdx.x & 7), p = g / hkv;
    s = (p << group_log2) + (j & ((1 << group_log2) - 1)); kvh = g - p * hkv;
    if (s >= rows_) return;
  }
  const int pp0 = SHARE ? sh.prefix_pairs : 0;   // first page pair this workgroup covers
  // The row's sequence and prompt length.  Rows that are the sequences in order, all with one prompt length, are marked by the
  // sign bit: the other arguments, a load each before what they point to can be asked for, are not touched for them.
  int seq = s, pos = (lp_pages_ & 0xffff) + step - 1;
  if (heads_ >= 0) {
    if (rm.slot_seq) seq = load_uniform(rm.slot_seq + s);
    if (rm.lens) pos = load_uniform(rm.lens + seq / rm.G) + step - 1;
  }
  const int* pt = kv.page_table + (size_t)seq * kv.pages_per_seq;
  // Entries of the wave's first pairs, asked for beside the step counter: clamped to the sequence's entries instead of its pages,
  // which the counter decides.  A pair that does not exist is not requested below.
  int first_pa[PD], first_pb[PD];
#pragma unroll
  for (int j = 0; j < PD; ++j) {
    const int e = 2 * (pp0 + wave + NW * j);
    first_pa[j] = load_uniform(pt + min(e, kv.pages_per_seq - 1));
    first_pb[j] = load_uniform(pt + min(e + 1, kv.pages_per_seq - 1));
  }
  const int new_page = load_uniform(pt + pos / kPageTokens), new_slot = pos % kPageTokens;
  const int ctx = pos + 1;
  f16* kpool = (f16*)kv.k;
  f16* vpool = (f16*)kv.v;
  const size_t page_elems = (size_t)hkv * kPageTokens * HD;
  const int npairs = (ctx + 31) / 32;
  const int last_page = (ctx - 1) / kPageTokens;

  // K rows of the two score tiles and the V tile of page pair pp: tile t row r is pair-token
  // 8 (r / 4) + 4 t + r % 4; the lane's V chunk holds pair-tokens 8 grp .. 8 grp + 7
  auto load_pages = [&](int pa, int pb, Frag16 (&kf)[2][KK], Frag16 (&vf)[DT]) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const f16* kp = kpool + (size_t)((lane & 15) < 8 ? pa : pb) * page_elems + (size_t)kvh * kPageTokens * HD;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) kf[t][kk].u = *(const uint4*)(kp + k_frag_at(t, kk, lane));
    }
    const f16* vp = vpool + (size_t)(grp < 2 ? pa : pb) * page_elems + (size_t)kvh * HD * kPageTokens;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) vf[dt].u = *(const uint4*)(vp + v_frag_at(dt, lane));
  };
  auto load_pair = [&](int pp, Frag16 (&kf)[2][KK], Frag16 (&vf)[DT]) {
    load_pages(load_uniform(pt + 2 * pp), load_uniform(pt + min(2 * pp + 1, last_page)), kf, vf);
  };
  // the same requests into slot j of this wave's staging area
  const unsigned stage0 = LDS ? __builtin_amdgcn_readfirstlane(lds_addr16(sm_o) + (unsigned)wave * PD * NFRAG * 1024u) : 0u;
  auto stage_pages = [&](int pa, int pb, int j) {
    const unsigned dst = stage0 + (unsigned)j * NFRAG * 1024u;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const f16* kp = kpool + (size_t)((lane & 15) < 8 ? pa : pb) * page_elems + (size_t)kvh * kPageTokens * HD;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) dma16_lds(kp + k_frag_at(t, kk, lane), dst + (unsigned)(t * KK + kk) * 1024u);
    }
    const f16* vp = vpool + (size_t)(grp < 2 ? pa : pb) * page_elems + (size_t)kvh * HD * kPageTokens;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) dma16_lds(vp + v_frag_at(dt, lane), dst + (unsigned)(2 * KK + dt) * 1024u);
  };
  auto stage_pair = [&](int pp, int j) { stage_pages(load_uniform(pt + 2 * pp), load_uniform(pt + min(2 * pp + 1, last_page)), j); };
  auto read_pair = [&](int j, Frag16 (&kf)[2][KK], Frag16 (&vf)[DT]) {
    const uint4* src = (const uint4*)sm_o + ((size_t)(wave * PD + j) * NFRAG) * 64 + lane;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) kf[t][kk].u = src[(t * KK + kk) * 64];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) vf[dt].u = src[(2 * KK + dt) * 64];
  };
  // The row's own q / k / v values and rotary pairs are requested before the cached pages: loads complete in the
  // order they were issued, so behind the pages they would be waited for together with every page in flight, and
  // behind the appended key's stores together with those stores' acknowledgements.
  constexpr int half = HD / 2;
  constexpr int NQ = 16 * half / (NW * 64);   // query elements per thread
  static_assert(NQ * NW * 64 == 16 * half && half <= NW * 64 && HD <= NW * 64, "whole passes over the 16 query rows");
  const float* row = qkv + (size_t)s * (n_q_heads + 2 * hkv) * HD;
  // every thread asks (clamped to a valid row or element) so that nothing here sits under a branch
  float qx1[NQ], qx2[NQ];
  float2 qcs[NQ];
#pragma unroll
  for (int n = 0; n < NQ; ++n) {
    const int idx = tid + n * NW * 64, r = min(idx / half, rep - 1), i = idx % half;
    const float* x = row + (size_t)(kvh * rep + r) * HD;
    qx1[n] = x[i];
    qx2[n] = x[i + half];
  }
  const int ki = min(tid, half - 1), vi = min(tid, HD - 1);
  float kx1 = row[(size_t)(n_q_heads + kvh) * HD + ki], kx2 = row[(size_t)(n_q_heads + kvh) * HD + ki + half];
  float vx = row[(size_t)(n_q_heads + hkv + kvh) * HD + vi];
  // ... the rotary pairs behind them: they need the position, which is a load away (the step counter)
#pragma unroll
  for (int n = 0; n < NQ; ++n) qcs[n] = rope[(size_t)pos * half + (tid + n * NW * 64) % half];
  float2 kcs = rope[(size_t)pos * half + ki];
  __builtin_amdgcn_sched_barrier(0);   // ... and these requests stay in front of the pages'

  constexpr int PR = LDS ? 1 : PD;   // register sets of fragments
  Frag16 kf[PR][2][KK], vf[PR][DT];
  // ---- the first page pairs are requested; rotary on the group's queries and the new key; append key / value ----
  // The number of pairs a wave requests (0 .. PD, wave-uniform) selects one of PD + 1 copies of the code: within a
  // copy the compiler knows how many requests stand behind the row's own values and waits for those alone, while
  // the pages are still on their way.  (Requests under a branch each would leave it a wait for everything; asking
  // for a page again in place of a missing pair costs more than it saves: a compute unit's ingest is the bound.)
  auto first_pairs_and_rotary = [&](auto n_c) {
    constexpr int n_req = decltype(n_c)::value;
#pragma unroll
    for (int j = 0; j < n_req; ++j) {
      // a last pair of one page: that page for both
      const int pa = first_pa[j], pb = 2 * (pp0 + wave + NW * j) < last_page ? first_pb[j] : pa;
      if constexpr (LDS) stage_pages(pa, pb, j);
      else load_pages(pa, pb, kf[j], vf[j]);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int n = 0; n < NQ; ++n) {
      const int idx = tid + n * NW * 64, r = idx / half, i = idx % half;
      const bool live = r < rep;   // columns past the group's heads are zero
      qs[r * HD + i] = from_f32<f16>(live ? rot_first(qx1[n], qx2[n], qcs[n].x, qcs[n].y) : 0.f);
      qs[r * HD + i + half] = from_f32<f16>(live ? rot_second(qx1[n], qx2[n], qcs[n].x, qcs[n].y) : 0.f);
    }
    if (tid < half) {
      f16* kp = kpool + (size_t)new_page * page_elems + (size_t)kvh * kPageTokens * HD;
      const f16 k1 = from_f32<f16>(rot_first(kx1, kx2, kcs.x, kcs.y)), k2 = from_f32<f16>(rot_second(kx1, kx2, kcs.x, kcs.y));
      kp[k_page_at(new_slot, tid)] = k1; kp[k_page_at(new_slot, tid + half)] = k2;
      knew[tid] = k1; knew[tid + half] = k2;
    }
    if (tid < HD) {
      const f16 vv = from_f32<f16>(vx);
      vpool[(size_t)new_page * page_elems + (size_t)kvh * HD * kPageTokens + v_page_at(new_slot, tid)] = vv;
      vnew[tid] = vv;
    }
  };
  {
    static_assert(PD <= 3, "one copy per number of requested pairs");
    const int mine = npairs - pp0 - wave;                                // pairs wave, wave + NW, ... below it
    const int n_req = mine <= 0 ? 0 : min((mine + NW - 1) / NW, PD);
    if (n_req == 0) first_pairs_and_rotary(std::integral_constant<int, 0>());
    else if (n_req == 1 || PD == 1) first_pairs_and_rotary(std::integral_constant<int, 1>());
    else if (n_req == 2 || PD == 2) first_pairs_and_rotary(std::integral_constant<int, (PD >= 2 ? 2 : 1)>());
    else first_pairs_and_rotary(std::integral_constant<int, PD>());
  }
  __syncthreads();
  Frag16 qf[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) qf[kk].u = *(const uint4*)(qs + qcol * HD + kk * 32 + grp * 8);
  const float scale = 1.0f / sqrtf((float)HD);
  float m_run = -INFINITY, l_run = 0.f;
  f32x4 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (int c0 = 0; pp0 + wave + NW * c0 < npairs; c0 += PD) {
    if (c0 > 0) {
#pragma unroll
      for (int j = 0; j < PD; ++j)
        if (pp0 + wave + NW * (c0 + j) < npairs) {
          if constexpr (LDS) stage_pair(pp0 + wave + NW * (c0 + j), j);   // every slot has been read into registers and used
          else load_pair(pp0 + wave + NW * (c0 + j), kf[j], vf[j]);
        }
    }
    // pairs of this chunk that exist for this wave (LDS: requests issued above, in slot order)
    const int n_chunk = min(PD, (npairs - (pp0 + wave + NW * c0) + NW - 1) / NW);
#pragma unroll
    for (int jj = 0; jj < PD; ++jj) {
      const int pp = pp0 + wave + NW * (c0 + jj);
      if (pp >= npairs) break;
      constexpr int kSetStride = LDS ? 0 : 1;
      const int j = jj * kSetStride;          // register set: the pair's own, or the single one of the LDS variant
      if constexpr (LDS) {
        // slot jj has landed once at most the later slots' requests are outstanding (requests complete in order)
        const int newer = n_chunk - 1 - jj;
        if (newer >= 3) wait_vmcnt_d<3 * NFRAG>();
        else if (newer == 2) wait_vmcnt_d<2 * NFRAG>();
        else if (newer == 1) wait_vmcnt_d<NFRAG>();
        else wait_vmcnt_d<0>();
        asm volatile("" ::: "memory");
        read_pair(jj, kf[0], vf[0]);
      }
      // The pair with the token that this workgroup appends, which comes from LDS and not from the global copy written above.
      // Tokens past it may hold anything in V (even NaN bit patterns): zero.  Both on whole dwords under masks - as
      // 16-bit elements under a running index this was 150 instructions of the wave that ends last.
      if (pp == pos / 32) {
        const int at = pos & 31;
        uint4 kn[KK];
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) kn[kk] = *(const uint4*)(knew + kk * 32 + grp * 8);
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const int r = lane & 15;
          const bool mine = 8 * (r >> 2) + 4 * t + (r & 3) == at;
#pragma unroll
          for (int kk = 0; kk < KK; ++kk) {
            kf[j][t][kk].u.x = mine ? kn[kk].x : kf[j][t][kk].u.x;
            kf[j][t][kk].u.y = mine ? kn[kk].y : kf[j][t][kk].u.y;
            kf[j][t][kk].u.z = mine ? kn[kk].z : kf[j][t][kk].u.z;
            kf[j][t][kk].u.w = mine ? kn[kk].w : kf[j][t][kk].u.w;
          }
        }
        unsigned keep[4], put[4];   // of the lane's tokens 8 grp + 2 d, + 1: those before the new one, and it
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const int n = at - (8 * grp + 2 * d);
          keep[d] = n >= 2 ? 0xffffffffu : n == 1 ? 0x0000ffffu : 0u;
          put[d] = n == 1 ? 0xffff0000u : n == 0 ? 0x0000ffffu : 0u;
        }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          const unsigned v = ((const unsigned short*)vnew)[dt * 16 + (lane & 15)], vv = v | v << 16;
#pragma unroll
          for (int d = 0; d < 4; ++d) vf[j][dt].n[d] = (vf[j][dt].n[d] & keep[d]) | (vv & put[d]);
        }
      }
      f32x4 sc[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        sc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) sc[t] = mfma16(kf[j][t][kk], qf[kk], sc[t]);
      }
      // lane (query qcol, group grp) now holds pair-tokens 8 grp + e, e = 4 t + i
      float p[8];
      float m_loc = -INFINITY;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int n = pp * 32 + 8 * grp + e;
        const float sv = sc[e >> 2][e & 3] * scale;
        p[e] = (n < ctx) ? sv : -INFINITY;
        m_loc = fmaxf(m_loc, p[e]);
      }
      m_loc = max_xor16(m_loc);
      m_loc = max_xor32(m_loc);
      const float m_new = fmaxf(m_run, m_loc);
      const float alpha = __expf(m_run - m_new);
      float psum = 0.f;
      Frag16 pf;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float pe = __expf(p[e] - m_new);
        psum += pe;
        pf.h[e] = (f16)pe;
      }
      l_run = l_run * alpha + psum;
      m_run = m_new;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
#pragma unroll
        for (int i = 0; i < 4; ++i) o[dt][i] *= alpha;
        o[dt] = mfma16(vf[j][dt], pf, o[dt]);
      }
    }
  }
  l_run = sum_xor16(l_run);
  l_run = sum_xor32(l_run);
  if (grp == 0) { sm_m[wave][qcol] = m_run; sm_l[wave][qcol] = l_run; }
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int i = 0; i < 4; ++i) sm_o[(size_t)wave * kOStride + (size_t)(dt * 16 + grp * 4 + i) * 16 + qcol] = o[dt][i];
  if constexpr (SHARE) {
    // the prompt's part of this row comes from the prefix workgroup (prompt s / G, this KV head): wait, bounded by the
    // wall clock, until its flag shows this launch's number; a wait that gives up sets the fault word, which makes the
    // sampler emit -1 for the step
    if (tid == 0) {
      const unsigned launch_no = (unsigned)step * (unsigned)sh.n_layers + (unsigned)sh.layer + 1u;
      const unsigned* flag = sh.flags + (size_t)(s / sh.G) * hkv + kvh;
      const unsigned long long t0 = wall_clock64();
      while ((int)(__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - launch_no) < 0) {
        if (wall_clock64() - t0 > sh.spin_ticks) {
          atomicOr(sh.fault, 2u);
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
    }
  }
  __syncthreads();
  // thread -> (query head q, head dim d): one half of the X16 output (the query heads run fastest over the lanes: their
  // LDS columns are adjacent).  With one thread per 16-byte chunk only rep x HD / 8 threads - one wave - did the
  // whole merge, 80 dependent LDS reads each: 0.8 us at the end of a 4.5 us kernel.  Waves that had no page pair
  // carry (m = -inf, l = 0, o = 0) and drop out of the merge.
  const int KSo = (n_q_heads * HD) >> 5;
  static_assert(16 * HD * 16 < 65536, "idx / rep by a multiplication: idx times the remainder of 65536 stays below 65536");
  for (int idx = tid; idx < rep * HD; idx += NW * 64) {
    const int d = idx * per_rep >> 16, q = idx - d * rep;
    float mx = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) mx = fmaxf(mx, sm_m[w][q]);
    // the prefix part (shared-prompt variant): read past the L2, it was written by another workgroup of this launch
    float m_p = -INFINITY, l_p = 0.f, o_p = 0.f;
    if constexpr (SHARE) {
      const size_t base = ((size_t)s * n_q_heads + kvh * rep + q) * (HD + 4);
      m_p = ld_f32<true>(sh.pre, base * sizeof(float));
      l_p = ld_f32<true>(sh.pre, (base + 1) * sizeof(float));
      o_p = ld_f32<true>(sh.pre, (base + 4 + d) * sizeof(float));
      mx = fmaxf(mx, m_p);
    }
    const float w_p = SHARE ? __expf(m_p - mx) : 0.f;
    float den = w_p * l_p, wgt[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) { wgt[w] = __expf(sm_m[w][q] - mx); den += wgt[w] * sm_l[w][q]; }
    const float inv = 1.0f / den;
    float num = w_p * o_p;
#pragma unroll
    for (int w = 0; w < NW; ++w) num += wgt[w] * sm_o[(size_t)w * kOStride + (size_t)d * 16 + q];
    ((f16*)out)[x16_chunk(s, (kvh * rep + q) * HD + (d & ~7), KSo) * 8 + (d & 7)] = from_f32<f16>(num * inv);
  }
}

// Rows of one KV head that run on one XCD, as a power of two: the siblings of a prompt, at most 8 (the rows of a larger group
// would crowd one XCD).  us per step, rows dealt one by one -> in groups: 0.5B, 64 rows, contexts of 1050 795 -> 781, of 240 667 ->
// 661; 1.5B, 256 rows, contexts of 710 2324 -> 2279.
static int sibling_group_log2(int G) { return G >= 8 ? 3 : G >= 4 ? 2 : G >= 2 ? 1 : 0; }

template <int HD, int NW, int PD, bool LDS = false, bool SHARE = false>
static hipError_t launch_decode_attention(const float* qkv, const float2* rope, RowMap rm, KVCache kv, void* out, int S,
                                          int n_q_heads, hipStream_t st, const Prefetch& pf, const ShareArgs& sh = ShareArgs()) {
  static bool attr_done = false;
  static_assert(PD <= 4, "the LDS variant's waits cover up to 4 slots");
  const size_t smem = LDS ? (size_t)NW * PD * (HD / 8) * 1024
                          : (size_t)NW * HD * 16 * sizeof(float) + (SHARE ? (size_t)kSharePrefixMaxColumns * HD * sizeof(f16) : 0);
  if (!attr_done) {
    hipError_t e = hipFuncSetAttribute((const void*)k_decode_attention16<HD, NW, PD, LDS, SHARE>,
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e != hipSuccess) return e;
    attr_done = true;
  }
  const int group_log2 = sibling_group_log2(rm.G), group = 1 << group_log2;
  const int n_main = SHARE ? sh.n_prefix + S * kv.n_kv_heads : ((S + group - 1) / group * kv.n_kv_heads + 7) / 8 * 8 * group;
  // Prefetching workgroups: at most 5 / 8 of the compute units, more of them only held up the few that attend (us per step with
  // 120, 136, 152, 168, 200, 240 of them: 0.5B, 1 row 573, 568, 566, 568, 576, 584; 1.5B, 1 row 128, 152, 176, 200, 224: 1053, 1038,
  // 1035, 1044, 1051), and as many as these leave.
  const int room = std::min(n_compute_units() * 5 / 8, n_compute_units() - n_main);
  const int n_pf = prefetch_blocks(pf, NW, prefetch_per_wave(pf, Prefetch(), NW, room, 8, 18));
  const int blocks = n_pf > 0 ? ((n_main + 7) & ~7) + n_pf : n_main;
  // fields of the packed arguments (max_seq is at most 3584, 16 query heads per KV head: both checked when the handle is made)
  if (kv.n_kv_heads > 0xffff || n_q_heads / kv.n_kv_heads > 16 || rm.Lp > 0xffff || kv.pages_per_seq > 0x7fff) return hipErrorInvalidValue;
  return launch(SHARE ? KID_DECODE_ATTN_SHARED : KID_DECODE_ATTN, k_decode_attention16<HD, NW, PD, LDS, SHARE>, dim3(blocks),
                dim3(NW * 64), smem, st, qkv, rope, rm.step, kv.page_table, rm.Lp | (kv.pages_per_seq << 16), S,
                kv.n_kv_heads | (n_q_heads / kv.n_kv_heads << 16) | (group_log2 << 24) | (rm.slot_seq || rm.lens ? 0 : INT_MIN), n_main, kv.k, rm, kv, (uint4*)out, sh, pf);
}

hipError_t d_decode_attention(const float* qkv, const float2* rope, RowMap rm, KVCache kv, void* out, int S, int n_q_heads,
                              const ShareArgs* share, const Prefetch& pf, hipStream_t st) {
  if (!rm.decode) return hipErrorInvalidValue;
  if (share && share->prefix_pairs > 0) {
    // what the two-role launch assumes: rows are P x G sequences in order, all at one position, with their own
    // page-table rows; the columns of all siblings fit the prefix workgroup's four MFMA tiles
    const int rep = n_q_heads / kv.n_kv_heads;
    if (kv.head_dim != 64 || !rm.decode || rm.lens || rm.slot_seq || share->G < 1 || S % share->G != 0 ||
        share->G * rep > kSharePrefixMaxColumns || share->n_prefix != (S / share->G) * kv.n_kv_heads || !share->pre ||
        !share->flags || !share->fault || share->prefix_pairs * 32 > rm.Lp)
      return hipErrorInvalidValue;
    return launch_decode_attention<64, 8, 3, false, true>(qkv, rope, rm, kv, out, S, n_q_heads, st, pf, *share);
  }
  // SAPO_ATTN_LDS=1 in the environment: the LDS-staged variant, kept as the measured alternative (0.5B-class decoder,
  // 64 sequences, same waves and pairs in flight: 6.6 against 5.8 us per launch at contexts 128..383, 12.5 against
  // 11.4 us at 512..1535).  Two slots of 8 KiB per wave are what 8 waves fit into the 160 KiB.  Read per call, so
  // that a test can switch it; a captured decode step keeps the variant it was captured with.
  const char* lds_env = getenv("SAPO_ATTN_LDS");
  if (kv.head_dim == 64) {
    if (lds_env && lds_env[0] == '1') return launch_decode_attention<64, 8, 2, true>(qkv, rope, rm, kv, out, S, n_q_heads, st, pf);
    // more workgroups than compute units: with two page pairs in flight per wave two workgroups fit a unit (0.5B, 192 rows:
    // a step of 1112 us with three pairs, 1048 with two, 1051 with one, 1060 with four waves of three)
    if (S * kv.n_kv_heads > n_compute_units()) return launch_decode_attention<64, 8, 2>(qkv, rope, rm, kv, out, S, n_q_heads, st, pf);
    return launch_decode_attention<64, 8, 3>(qkv, rope, rm, kv, out, S, n_q_heads, st, pf);
  }
  if (kv.head_dim == 128) {
    // more workgroups than compute units: 4-wave workgroups with one page pair in flight per wave leave room for
    // two per compute unit, so the whole grid is resident at once (1.5B, 256 sequences: 24.7 us against 29.8)
    if (S * kv.n_kv_heads > n_compute_units()) return launch_decode_attention<128, 4, 1>(qkv, rope, rm, kv, out, S, n_q_heads, st, pf);
    return launch_decode_attention<128, 8, 2>(qkv, rope, rm, kv, out, S, n_q_heads, st, pf);
  }
  return hipErrorInvalidValue;
}

}  // namespace sapo
